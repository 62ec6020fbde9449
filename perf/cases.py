"""The work whose speed this library is judged by, as a user's program calls it.

Every case is one call (or one replay) of a public entry point of
``paper_2608_15764_amd.ilpsweep`` on resident device memory:

cell     one plain K-load cell (``sweep_plain``, ``sweep_plain_noalloc``)
sweep    a K sweep, ascending then reversed: back to back (``sweep_run``),
         captured once and replayed (``sweep_graph_launch``), or captured,
         launched and destroyed in one call (``sweep_batched``)
batch    many points of different sizes as one fused graph
paths    LDS-direct against matched register cells (``sweep_run``)
streams  two co-resident streams (``sweep_two_stream_kind``, ``_split``)
sum      the compensated streaming sum (``sweep_reduce_fp``)
fill     the seeded fill (``sweep_fill_u32``)
xcd      the read by chosen XCDs (``sweep_xcd_subset``, ``sweep_xcd_split``)

The pointer chases are left out: their time is hops times the latency of one
dependent load, which is what they are called to measure.

A case returns every number of the results but the clock readings (and the
rates made of them) and the kernels' register counts.  The bytes of a cell
are its issued logical loads: the fixed-work control makes them the work,
also where a small buffer is read many times.
"""
import math

import numpy as np
import torch

from paper_2608_15764_amd import ilpsweep as isw

KIB, MIB, GIB = 1 << 10, 1 << 20, 1 << 30
EXACT = ("sum32", "xor32", "issued_loads", "issued_bytes", "target_loads", "mismatch")
KEYS = EXACT + ("waves", "iters_min", "iters_max")
TYPES = (np.uint32, np.uint32, np.uint64, np.uint64, np.uint64, np.float64)
SUM_TYPES = {"f32": (isw.F32, torch.float32, 4), "bf16": (isw.BF16, torch.bfloat16, 2),
             "fp8_e4m3": (isw.FP8_E4M3, torch.float8_e4m3fn, 1)}


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest call: the quick check of an installation
        dict(name="cell 4 MiB", kind="cell", entry="plain", bytes=4 * MIB, K=4, V=16, waves=8,
             passes=1.0, policy=isw.CACHE_DEFAULT, order=isw.ORDER_ROUND_ROBIN, lanes=False),
        # the plumbing configuration: 256 workgroups, 4-byte loads, per-thread sinks
        dict(name="cell 64 MiB, 4 B, lane sinks", kind="cell", entry="plain", bytes=64 * MIB,
             K=8, V=4, waves=4, passes=1.0, policy=isw.CACHE_DEFAULT,
             order=isw.ORDER_ROUND_ROBIN, lanes=True),
        # a ragged cell at the largest occupancy, called where nothing may be allocated
        dict(name="cell 16.3 MiB, 8 B, no alloc", kind="cell", entry="noalloc",
             bytes=33333 * 512, K=3, V=8, waves=32, passes=1.0, policy=isw.CACHE_BYPASS_L1_NT,
             order=isw.ORDER_ROUND_ROBIN, lanes=False),
        # one curve of the regime map on its L2 backend: 1 GiB read per cell
        dict(name="sweep 4 MiB, 4 B, run", kind="sweep", entry="run", bytes=4 * MIB, V=4,
             waves=16, max_K=16, passes=256.0, policy=isw.CACHE_BYPASS_L1_NT,
             order=isw.ORDER_ROUND_ROBIN),
        # one curve of the address-order experiment inside the last-level cache
        dict(name="sweep 16 MiB, blocked, graph", kind="sweep", entry="graph", bytes=16 * MIB,
             V=16, waves=16, max_K=8, passes=1.0, policy=isw.CACHE_BYPASS_L1_NT,
             order=isw.ORDER_BLOCKED),
        # the timed K sweep at one occupancy
        dict(name="sweep 1 GiB, graph", kind="sweep", entry="graph", bytes=GIB, V=16, waves=8,
             max_K=16, passes=1.0, policy=isw.CACHE_BYPASS_L1_NT, order=isw.ORDER_ROUND_ROBIN),
        # the batched sweep: 64 points of 1 MiB to 2 GiB, 17.5 GiB, one fused launch
        dict(name="batch 64 points, fused", kind="batch", points=64, lo=MIB, hi=2 * GIB, K=8,
             V=16, waves=4, policy=isw.CACHE_NT),
        # the path comparison at two depths
        dict(name="paths 2 GiB", kind="paths", bytes=2 * GIB, depths=2, depth=8, waves=4,
             policy=isw.CACHE_BYPASS_L1_NT),
        # two streams in one workgroup
        dict(name="streams 2 GiB", kind="streams", entry="kind", bytes=2 * GIB, depth=8,
             waves_a=4, waves_b=4, b="lds_async", policy=isw.CACHE_BYPASS_L1_NT),
        # a short ragged payload at the default occupancy
        dict(name="sum f32, 1000003", kind="sum", dtype="f32", n=1000003, waves=32),
        # the precision row's payload
        dict(name="sum bf16, 4 GiB", kind="sum", dtype="bf16", n=2 * GIB, waves=32),
        # a K sweep's buffer
        dict(name="fill 1 GiB", kind="fill", bytes=GIB),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("cell", "cell", "sweep", "sweep", "batch", "paths", "streams", "sum",
                       "sum", "fill", "xcd"))
    policy = rng.randrange(4)
    if kind == "cell":
        V = rng.choice((4, 8, 16))
        lanes = rng.random() < 0.3
        entry = rng.choice(("plain", "plain", "noalloc"))
        top = 64 * MIB if lanes else 512 * MIB if V == 4 else GIB
        # K up to 14: 16-byte loads with K above that do not reach 32 waves per CU
        return dict(kind=kind, entry=entry, bytes=_log(rng, 256 * KIB, top) // (64 * V) * 64 * V,
                    K=rng.randint(1, 14), V=V, waves=4 * rng.randint(1, 8),
                    passes=rng.choice((1.0, 1.0, 1.37, 2.0)), policy=policy,
                    order=rng.randrange(3), lanes=lanes)
    if kind == "sweep":
        V = rng.choice((4, 8, 16))
        size = _log(rng, MIB, 128 * MIB if V == 4 else 512 * MIB) // (64 * V) * 64 * V
        return dict(kind=kind, entry=rng.choice(("run", "graph", "graph", "batched")), bytes=size,
                    V=V, waves=4 * rng.randint(1, 8), max_K=rng.randint(3, 14),
                    passes=1.0 if size > 32 * MIB else float(rng.choice((1, 2, 8))),
                    policy=policy, order=rng.randrange(3))
    if kind == "batch":
        lo = _log(rng, 64 * KIB, 4 * MIB)
        return dict(kind=kind, points=rng.randint(5, 64), lo=lo,
                    hi=lo * _log(rng, 4, 256), K=rng.randint(2, 14), V=rng.choice((8, 16)),
                    waves=4 * rng.randint(1, 6), policy=policy)
    if kind == "paths":
        return dict(kind=kind, bytes=_log(rng, 16 * MIB, 2 * GIB) // 1024 * 1024, depths=1,
                    depth=rng.randint(3, 16), waves=rng.choice((2, 4, 8)), policy=policy)
    if kind == "streams":
        return dict(kind=kind, entry=rng.choice(("kind", "split")),
                    bytes=_log(rng, 16 * MIB, 2 * GIB) // 2048 * 2048, depth=rng.randint(3, 16),
                    waves_a=rng.randint(2, 8), waves_b=rng.randint(2, 8),
                    b=rng.choice(("plain", "lds_async")), policy=policy)
    if kind == "sum":
        dtype = rng.choice(tuple(SUM_TYPES))
        return dict(kind=kind, dtype=dtype, waves=4 * rng.randint(1, 8),
                    n=_log(rng, 1000, 4 * GIB // SUM_TYPES[dtype][2]))
    if kind == "fill":
        return dict(kind=kind, bytes=4 * _log(rng, MIB, GIB))
    # two to eight XCDs, or every XCD with the even ones' share up to a quarter larger
    if rng.random() < 0.5:
        mask = 0
        while bin(mask).count("1") < 2:
            mask = rng.randrange(1, 256)
        return dict(kind="xcd", entry="subset", bytes=_log(rng, 64 * MIB, GIB) // 1024 * 1024,
                    waves=rng.choice((4, 8)), mask=mask, policy=policy)
    return dict(kind="xcd", entry="split", bytes=_log(rng, 64 * MIB, GIB) // 1024 * 1024,
                waves=rng.choice((4, 8, 16)), even=round(rng.uniform(1.0, 1.25), 3),
                policy=policy)


# -------------------------------------------------------- inputs, plans, calls
def _cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _words(nbytes, seed):
    """Uniform random words, as the seeded fill gives them."""
    buf = torch.empty(nbytes // 4, dtype=torch.int32, device="cuda")
    g = _generator(seed)
    for part in buf.split(1 << 28):
        part.random_(-(1 << 31), 1 << 31, generator=g)
    return buf


def _payload(dtype, n, seed):
    """N(0, 1) values in the payload's type."""
    t = SUM_TYPES[dtype][1]
    out = torch.empty(n, dtype=t, device="cuda")
    g = _generator(seed)
    for part in out.split(1 << 27):
        part.copy_(torch.randn(part.numel(), device="cuda", generator=g))
    return out


def _loads(case):
    return int(case["bytes"] // case["V"] * case["passes"])


def _sweep_Ks(case):
    up = list(range(1, case["max_K"] + 1))
    return up + up[::-1]


def _points(case):
    """Log-spaced point sizes in whole 64-KiB steps, laid out back to back."""
    n, out, at = case["points"], [], 0
    for i in range(n):
        size = case["lo"] * (case["hi"] / case["lo"]) ** (i / max(1, n - 1))
        size = max(1, round(size / (64 * KIB))) * 64 * KIB
        out.append((at, size))
        at += size
    return out, at


def _path_cells(case):
    ds = [case["depth"] >> i for i in range(case["depths"])]
    return [(d, kind) for d in ds for kind in (isw.KIND_LDS_ASYNC, isw.KIND_LDS_MATCHED)]


def _weights(case):
    return [case["even"], 1.0] * 4


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": dict(case)}
    if kind == "fill":
        s["buf"] = torch.empty(case["bytes"] // 4, dtype=torch.int32, device="cuda")
        s["seed"] = seed
        return s
    if kind == "sum":
        s["buf"] = _payload(case["dtype"], case["n"], seed)
        return s
    if kind == "batch":
        points, total = _points(case)
        s["buf"] = _words(total, seed)
        base, V = s["buf"].data_ptr(), case["V"]
        cells = [isw.make_cell(base + at, size, case["K"], V, case["waves"], size // V,
                               cache_policy=case["policy"]) for at, size in points]
        s["graph"] = isw.sweep_graph_create(cells, isw.make_opts(fuse=True))
        return s
    s["buf"] = buf = _words(case["bytes"], seed)
    n = case["bytes"]
    if kind == "cell":
        lane_out = None
        if case["lanes"]:
            lane_out = s["lanes"] = torch.zeros((_cus() * case["waves"] * 64, 2),
                                                dtype=torch.int32, device="cuda")
        s["opts"] = isw.make_opts(cache_policy=case["policy"], order=case["order"],
                                  lane_out=lane_out)
    elif kind == "sweep":
        s["cells"] = isw.cell_array([
            isw.make_cell(buf, n, K, case["V"], case["waves"], _loads(case),
                          cache_policy=case["policy"], order=case["order"])
            for K in _sweep_Ks(case)])
        if case["entry"] == "graph":
            s["graph"] = isw.sweep_graph_create(s["cells"])
    elif kind == "paths":
        s["cells"] = isw.cell_array([
            isw.make_cell(buf, n, d, 16, case["waves"], n // 16, kind=k,
                          cache_policy=case["policy"]) for d, k in _path_cells(case)])
    else:
        s["opts"] = isw.make_opts(cache_policy=case["policy"])
    return s


def _told(result):
    return {k: result[k] for k in KEYS}


def _told_all(raw):
    """The same fields of a raw result array, one array per field."""
    a = np.frombuffer(raw, dtype=np.dtype(isw.sweep_result_t))
    return {k: a[k].copy() for k in KEYS}


def run(state):
    c, buf = state["case"], state["buf"]
    kind = c["kind"]
    if kind == "cell":
        call = isw.sweep_plain if c["entry"] == "plain" else isw.sweep_plain_noalloc
        out = _told(call(buf, c["bytes"], c["K"], c["V"], c["waves"], _loads(c), state["opts"]))
        if c["lanes"]:
            out["lanes"] = state["lanes"]
        return out
    if kind == "sweep" and c["entry"] == "run" or kind == "paths":
        return _told_all(isw.sweep_run(state["cells"], raw=True))
    if kind == "sweep" and c["entry"] == "batched":
        return _told_all(isw.sweep_batched(state["cells"], raw=True)[0])
    if kind in ("sweep", "batch"):
        return _told_all(isw.sweep_graph_launch(state["graph"], raw=True)[0])
    if kind == "streams":
        call = (isw.sweep_two_stream_split if c["entry"] == "split"
                else isw.sweep_two_stream_kind)
        kind_b = isw.KIND_PLAIN if c["b"] == "plain" else isw.KIND_LDS_ASYNC
        return [_told(r) for r in call(buf, c["bytes"], c["depth"], c["waves_a"], c["waves_b"],
                                       kind_b, c["bytes"] // 16, state["opts"])]
    if kind == "sum":
        total, r = isw.sweep_reduce_fp(buf, c["n"], SUM_TYPES[c["dtype"]][0], c["waves"])
        return {"sum": total, **_told(r)}
    if kind == "fill":
        isw.sweep_fill_u32(buf, c["bytes"], state["seed"])
        return buf
    if c["entry"] == "subset":
        return _told(isw.sweep_xcd_subset(buf, c["bytes"], c["waves"], c["mask"], state["opts"]))
    return _told(isw.sweep_xcd_split(buf, c["bytes"], c["waves"], _weights(c), state["opts"]))


# --------------------------------------------------------------- work and truth
def _issued(loads, K):
    return 64 * K * (loads // (64 * K))


def _xcd_vectors(case):
    """16-byte vectors an XCD read covers, from the start of the buffer."""
    n_vec, waves = case["bytes"] // 16, _cus() * case["waves"]
    if case["entry"] == "subset":
        act = waves // 8 * bin(case["mask"]).count("1")
        return n_vec // (act * 512) * act * 512
    w = _weights(case)
    total = n_vec // 512
    return sum(int(total * (x / sum(w))) for x in w) * 512


def work(case):
    kind = case["kind"]
    if kind == "cell":
        b = _issued(_loads(case), case["K"]) * case["V"]
        if case["lanes"]:
            b += _cus() * case["waves"] * 64 * 8
    elif kind == "sweep":
        b = sum(_issued(_loads(case), K) for K in _sweep_Ks(case)) * case["V"]
    elif kind == "batch":
        b = sum(_issued(size // case["V"], case["K"]) for _, size in _points(case)[0]) * case["V"]
    elif kind == "paths":
        b = sum(_issued(case["bytes"] // 16, d) for d, _ in _path_cells(case)) * 16
    elif kind == "streams":
        b = 2 * _issued(case["bytes"] // 32, case["depth"]) * 16
    elif kind == "sum":
        return {"bytes": case["n"] * SUM_TYPES[case["dtype"]][2], "flops": case["n"]}
    elif kind == "fill":
        b = case["bytes"]
    else:
        b = _xcd_vectors(case) * 16
    return {"bytes": b, "flops": b // 2}      # an add and an xor per word


def _xor(words):
    """XOR of all words of an integer tensor."""
    out = 0
    for part in words.split(1 << 28):
        while part.numel() > 4096:
            half = part.numel() // 2
            rest = part[2 * half:]
            part = torch.cat((part[:half] ^ part[half:2 * half], rest))
        out ^= int(np.bitwise_xor.reduce(part.cpu().numpy()))
    return out & 0xFFFFFFFF


def _sinks(words, n):
    """(sum32, xor32) of the first n words of the buffer read round and round."""
    turns, rest = divmod(n, words.numel())
    s, x = 0, 0
    if turns:
        s = turns * int(words.sum(dtype=torch.int64))
        x = _xor(words) if turns % 2 else 0
    if rest:
        s += int(words[:rest].sum(dtype=torch.int64))
        x ^= _xor(words[:rest])
    return s & 0xFFFFFFFF, x


def _result(words, loads, V, target):
    out = dict.fromkeys(KEYS)
    out["sum32"], out["xor32"] = _sinks(words, loads * V // 4)
    out["issued_loads"], out["issued_bytes"] = loads, loads * V
    out["target_loads"], out["mismatch"] = target, (target - loads) / target
    return out


def _columns(each):
    """Results of several cells, one array per field."""
    out = dict.fromkeys(KEYS)
    for k, t in zip(EXACT, TYPES):
        out[k] = np.array([r[k] for r in each], dtype=t)
    return out


def _cells(words, Ks, V, target):
    known = {K: _result(words, _issued(target, K), V, target) for K in set(Ks)}
    return _columns([known[K] for K in Ks])


def _lane_sinks(case, words):
    """(sum32, xor32) of every thread of a cell in its work-group order."""
    K, V, n_waves = case["K"], case["V"], _cus() * case["waves"]
    n_vec, Q = case["bytes"] // V, _loads(case) // (64 * K)
    G = -(-Q // n_waves)
    q = torch.arange(G * n_waves, device="cuda")
    q = q.view(n_waves, G) if case["order"] == isw.ORDER_BLOCKED else q.view(G, n_waves).T
    s = torch.zeros((n_waves, 64), dtype=torch.int64, device="cuda")
    x = torch.zeros((n_waves, 64), dtype=torch.int32, device="cuda")
    lane = torch.arange(64, device="cuda")
    rows = words.view(n_vec, V // 4)
    for i in range(G):
        live = (q[:, i] < Q)[:, None]
        for j in range(K):
            seg = j * Q + q[:, i] if case["order"] == isw.ORDER_STRIDED else q[:, i] * K + j
            v = rows[(seg[:, None] * 64 + lane) % n_vec]
            for k in range(V // 4):
                w = torch.where(live, v[..., k], 0)
                s += w
                x ^= w
    s = (s & 0xFFFFFFFF).to(torch.int64)
    s = torch.where(s >= 1 << 31, s - (1 << 32), s).to(torch.int32)
    return torch.stack((s, x), dim=-1).view(-1, 2)


def _splitmix(n, seed):
    """The low halves of the first n SplitMix64 outputs (Steele, Lea, Flood, 2014)."""
    out = torch.empty(n, dtype=torch.int32, device="cuda")
    wrap = lambda v: (v + (1 << 63)) % (1 << 64) - (1 << 63)  # noqa: E731
    for at in range(0, n, 1 << 26):
        i = torch.arange(at + 1, min(n, at + (1 << 26)) + 1, dtype=torch.int64, device="cuda")
        z = i * wrap(0x9E3779B97F4A7C15) + wrap(seed)
        for shift, mul in ((30, 0xBF58476D1CE4E5B9), (27, 0x94D049BB133111EB), (31, 1)):
            z = (z ^ ((z >> shift) & ((1 << (64 - shift)) - 1))) * wrap(mul)
        z = z & 0xFFFFFFFF
        out[at:at + z.numel()] = torch.where(z >= 1 << 31, z - (1 << 32), z).to(torch.int32)
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "fill":
        return _splitmix(case["bytes"] // 4, seed)
    if kind == "sum":
        parts = []
        for part in _payload(case["dtype"], case["n"], seed).split(1 << 26):
            d = part.double()
            whole = d.numel() // 4096 * 4096
            parts += d[:whole].view(-1, 4096).sum(dim=1).tolist() + d[whole:].tolist()
        out = dict.fromkeys(("sum",) + KEYS)
        out["sum"] = math.fsum(parts)
        return out
    if kind == "batch":
        points, total = _points(case)
        buf, V = _words(total, seed), case["V"]
        return _columns([_result(buf[at // 4:(at + size) // 4], _issued(size // V, case["K"]),
                                 V, size // V) for at, size in points])
    buf = _words(case["bytes"], seed)
    if kind == "cell":
        out = _result(buf, _issued(_loads(case), case["K"]), case["V"], _loads(case))
        if case["lanes"]:
            out["lanes"] = _lane_sinks(case, buf)
        return out
    if kind == "sweep":
        return _cells(buf, _sweep_Ks(case), case["V"], _loads(case))
    if kind == "paths":
        return _cells(buf, [d for d, _ in _path_cells(case)], 16, case["bytes"] // 16)
    if kind == "streams":
        half, target = case["bytes"] // 8, case["bytes"] // 32
        n = _issued(target, case["depth"])
        return [_result(buf[:half], n, 16, target), _result(buf[half:], n, 16, target)]
    return _result(buf, _xcd_vectors(case), 16, _xcd_vectors(case))
