"""Kernels at the sizes where their split of the work changes: edges of
chunks and batches, remainders, the smallest and the largest."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import numpy as np

from gpu_util import decode_recs, dev_bytes, host_words, recs
from oracle import splitmix
from paper_2608_15764_amd import ilpsweep as isw

SEED = 0x1D5EED00 + 33
FILL_CHUNK = 4 << 10            # bytes one wave of the fill writes


@pytest.mark.parametrize("nbytes", [8, FILL_CHUNK - 16, FILL_CHUNK - 4, FILL_CHUNK,
                                    FILL_CHUNK + 4, FILL_CHUNK + 16, 7 * FILL_CHUNK - 12,
                                    4099 * FILL_CHUNK + 4092 * 4])
def test_fill_at_chunk_edges(nbytes):
    print("fill", nbytes, flush=True)
    buf = dev_bytes((nbytes + 15) // 16 * 16 + 4096).zero_()
    isw.sweep_fill_u32(buf, nbytes, SEED)
    torch.cuda.synchronize()
    assert np.array_equal(host_words(buf)[:nbytes // 4], splitmix.words(SEED, 0, nbytes // 4))
    assert not buf[nbytes:].any()


@pytest.mark.parametrize("wgs", [1, 255, 256, 1023, 1024, 1025, 2048, 2049, 4096])
def test_finish_folds_every_record(wgs):
    """The cell result is the fold of its wave records, at the edges of the
    finishing kernel's batches (4096 records) and of its threads."""
    nbytes, waves = 1 << 20, 4 * wgs
    buf = dev_bytes(nbytes)
    isw.sweep_fill_u32(buf, nbytes, SEED + 1)
    out = recs(waves)
    L = 64 * waves + 64 * 3                  # an uneven deal, wrapping
    print("finish", waves, "records", flush=True)
    r = isw.sweep_plain(buf, nbytes, 1, 4, 4, L, isw.make_opts(grid_wgs=wgs, wave_out=out))
    h = decode_recs(out)
    assert r["waves"] == waves
    assert r["sum32"] == int(h["sum32"].sum(dtype=np.uint64) & 0xFFFFFFFF)
    assert r["xor32"] == int(np.bitwise_xor.reduce(h["xor32"]))
    assert r["window_ticks"] == int(h["t1"].max() - h["t0"].min())


@pytest.mark.parametrize("n", [1, 4, 5, 64, 65])
def test_cells_of_one_call_keep_apart(n):
    """Up to 64 cells carry their record offsets in the finishing launch, more
    read them from memory; up to four launches of a graph are replayed as
    launches.  The results are those of single calls every way, on every
    replay."""
    nbytes = 2 << 20
    buf = dev_bytes(nbytes)
    isw.sweep_fill_u32(buf, nbytes, SEED + 2)
    cells = [isw.make_cell(buf, nbytes, 1 + i % 9, 16, 4 * (1 + i % 3), nbytes // 16 + 4096 * i)
             for i in range(n)]
    ones = [isw.sweep_plain(buf, nbytes, c.K, 16, c.waves_per_cu, c.total_logical_loads)
            for c in cells]
    want = [(r["sum32"], r["xor32"]) for r in ones]
    print("cells", n, flush=True)
    got = [isw.sweep_run(cells), isw.sweep_batched(cells)[0]]
    stream = torch.cuda.Stream()
    with isw.sweep_graph_create(cells) as g:
        for s in (None, stream, None):
            got.append(isw.sweep_graph_launch(g, stream=s)[0])
            torch.zeros(1000, device="cuda").add_(1)
            torch.cuda.synchronize()
    for rs in got:
        assert [(r["sum32"], r["xor32"]) for r in rs] == want
        assert all(r["window_ticks"] > 0 for r in rs)


@pytest.mark.parametrize("runs", [1, 4, 5])
def test_fused_runs_replay_after_each_other(runs):
    """Fused launches, few enough to be replayed as launches and one too
    many, of two points each."""
    nbytes = 1 << 20
    buf = dev_bytes(4 * nbytes)
    isw.sweep_fill_u32(buf, 4 * nbytes, SEED + 6)
    cells = [isw.make_cell(buf.data_ptr() + nbytes * (i % 4), nbytes, 2 + i // 2, 16, 8,
                           nbytes // 16 + 640 * i) for i in range(2 * runs)]
    want = [(r["sum32"], r["xor32"]) for r in isw.sweep_run(cells)]
    print("fused runs", runs, flush=True)
    with isw.sweep_graph_create(cells, isw.make_opts(fuse=True)) as g:
        for _ in range(3):
            rs, ms = isw.sweep_graph_launch(g)
            assert [(r["sum32"], r["xor32"]) for r in rs] == want and ms > 0
            torch.zeros(1000, device="cuda").add_(1)
            torch.cuda.synchronize()


def _prefix_sinks(words, n):
    """(sum32, xor32) of the first n of `words` (a device int32 tensor)."""
    s, x = int(words[:n].sum(dtype=torch.int64)) & 0xFFFFFFFF, 0
    part = words[:n]
    while part.numel() > 1024:
        half = part.numel() // 2
        part = torch.cat((part[:half] ^ part[half:2 * half], part[2 * half:]))
    for w in part.tolist():
        x ^= w & 0xFFFFFFFF
    return s, x


@pytest.mark.parametrize("order", [0, 1, 2])
@pytest.mark.parametrize("policy", [0, 1, 2, 3])
@pytest.mark.parametrize("nbytes", [(1 << 31) - 3072, (1 << 31) + 3072, (1 << 32) - 3072, 1 << 32,
                                    (1 << 32) + 3072])
def test_plain_at_the_32_bit_edges(nbytes, policy, order):
    """Buffers around 2 and 4 GiB, where byte offsets fill 31 and 32 bits
    and the 64-bit walk takes over; a pass and a bit, so that groups wrap."""
    buf = dev_bytes(nbytes)
    isw.sweep_fill_u32(buf, nbytes, SEED + 3)
    n_vec, K = nbytes // 16, 5
    L = n_vec + 64 * 1000 + 77
    print("plain", nbytes, "policy", policy, "order", order, flush=True)
    r = isw.sweep_plain(buf, nbytes, K, 16, 16, L,
                        isw.make_opts(cache_policy=policy, order=order))
    issued = 64 * K * (L // (64 * K))
    words = buf.view(torch.int32)
    s, x = _prefix_sinks(words, nbytes // 4)
    more, morex = _prefix_sinks(words, (issued - n_vec) * 4)
    assert r["issued_loads"] == issued
    assert (r["sum32"], r["xor32"]) == ((s + more) & 0xFFFFFFFF, x ^ morex)


@pytest.mark.parametrize("policy", [0, 1, 2, 3])
@pytest.mark.parametrize("kind", [isw.KIND_LDS_ASYNC, isw.KIND_LDS_MATCHED])
@pytest.mark.parametrize("nbytes,D", [(6144, 16), (1024, 1), ((1 << 32) - 3072, 5),
                                      ((1 << 32) + 3072, 5)])
def test_rings_at_the_edges_of_their_walks(nbytes, D, kind, policy):
    """The LDS rings over buffers smaller than one group and on both sides of
    4 GiB; waves with no, one and several groups."""
    buf = dev_bytes(nbytes)
    isw.sweep_fill_u32(buf, nbytes, SEED + 4)
    n_vec = nbytes // 16
    L = n_vec + 64 * 1000 + 77
    print("ring", kind, nbytes, "policy", policy, flush=True)
    call = isw.sweep_lds_async if kind == isw.KIND_LDS_ASYNC else isw.sweep_lds_matched_plain
    r = call(buf, nbytes, D, 16, 3, L, isw.make_opts(cache_policy=policy))
    issued = 64 * D * (L // (64 * D))
    words = buf.view(torch.int32)
    turns, rest = divmod(issued, n_vec)
    s, x = _prefix_sinks(words, nbytes // 4)
    more, morex = _prefix_sinks(words, rest * 4)
    assert r["issued_loads"] == issued
    assert (r["sum32"], r["xor32"]) == ((turns * s + more) & 0xFFFFFFFF,
                                        (x if turns % 2 else 0) ^ morex)


@pytest.mark.parametrize("kind_b", [isw.KIND_PLAIN, isw.KIND_LDS_ASYNC])
@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("nbytes", [(1 << 33) - 4096, (1 << 33) + 4096])
def test_two_streams_around_4_gib_each(nbytes, split, kind_b):
    buf = dev_bytes(nbytes)
    isw.sweep_fill_u32(buf, nbytes, SEED + 5)
    half, D = nbytes // 32, 7                     # vectors of a stream's region
    L = 2 * (half + 64 * 500 + 5)
    print("two streams", nbytes, "split", split, "kind_b", kind_b, flush=True)
    call = isw.sweep_two_stream_split if split else isw.sweep_two_stream_kind
    rs = call(buf, nbytes, D, 4, 2, kind_b, L, isw.make_opts(cache_policy=3))
    issued = 64 * D * (L // 2 // (64 * D))
    words = buf.view(torch.int32)
    for r, part in zip(rs, (words[:half * 4], words[half * 4:])):
        s, x = _prefix_sinks(part, half * 4)
        more, morex = _prefix_sinks(part, (issued - half) * 4)
        assert r["issued_loads"] == issued
        assert (r["sum32"], r["xor32"]) == ((s + more) & 0xFFFFFFFF, x ^ morex)


@pytest.mark.parametrize("wgs", [1, 2, 255, 256, 257, 2047, 2048, 2049, 5000])
def test_reduce_finish_takes_every_pair_and_record(wgs):
    """The final combine at the edges of its 256 threads and of their batches
    of eight pairs, on integers whose sums FP32 holds exactly."""
    n = 64 * 4 * 4 * 4 * wgs + 999          # a full group per wave, and a rest
    g = torch.Generator(device="cuda").manual_seed(wgs)
    p = torch.randint(-8, 9, (n,), device="cuda", generator=g).float()
    print("reduce", wgs, "workgroups", flush=True)
    total, r = isw.sweep_reduce_fp(p, n, isw.F32, 8, isw.make_opts(grid_wgs=wgs))
    assert total == float(p.double().sum())
    assert r["waves"] == 4 * wgs and r["window_ticks"] > 0


@pytest.mark.parametrize("policy", [0, 1, 2, 3])
@pytest.mark.parametrize("V,K,w", [(4, 1, 4), (8, 5, 4), (16, 6, 4), (16, 7, 4), (16, 3, 8),
                                   (16, 4, 8), (4, 14, 8)])
def test_fused_forms_match_single_cells(V, K, w, policy):
    """Both forms of the fused loop, on the sides of the 6 MiB in flight where
    the choice changes: points of one segment, of less than a group per
    wave, of a ragged last group and read more than once."""
    seg = 64 * V
    sizes = [seg, 3 * seg, 700 * seg, 4099 * seg, 20000 * seg]
    buf = dev_bytes(sum(sizes))
    isw.sweep_fill_u32(buf, sum(sizes), SEED + 7)
    cells, at = [], 0
    for i, n in enumerate(sizes):
        loads = (1 + 2 * (i % 3)) * (n // V) + 64 * K + 77 * i
        cells.append(isw.make_cell(buf.data_ptr() + at, n, K, V, w, loads, cache_policy=policy))
        at += n
    print("fused form", V, K, w, "policy", policy, flush=True)
    want = [(r["issued_loads"], r["sum32"], r["xor32"]) for r in isw.sweep_run(cells)]
    with isw.sweep_graph_create(cells, isw.make_opts(fuse=True)) as g:
        for _ in range(2):
            rs, _ = isw.sweep_graph_launch(g)
            assert [(r["issued_loads"], r["sum32"], r["xor32"]) for r in rs] == want


@pytest.mark.parametrize("w", [4, 8, 12])
@pytest.mark.parametrize("groups", [0, 1, 2, 3, 7])
@pytest.mark.parametrize("rest", [0, 1, 8, 511])
def test_bf16_sum_by_groups_per_wave(groups, rest, w):
    """The BF16 sum where a wave has no, one, two and more groups (the ring's
    start, its first turn and its drain), on integers: the sums are exact."""
    loads = 8 if w == 4 else 4
    waves = 8 * 4
    n = (groups * waves + (groups + 1) // 2) * loads * 64 * 8 + rest
    if n == 0:
        n = 8
    g = torch.Generator(device="cuda").manual_seed(n)
    p = torch.randint(-8, 9, (n,), device="cuda", generator=g).to(torch.bfloat16)
    print("bf16 sum", n, "waves per CU", w, flush=True)
    total, r = isw.sweep_reduce_fp(p, n, isw.BF16, w, isw.make_opts(grid_wgs=8))
    assert total == float(p.double().sum())
    assert r["waves"] == waves and r["issued_bytes"] == 2 * n


def _wrapped_sinks(words, n_vec, issued):
    """Sinks of `issued` 16-byte loads that walk `n_vec` vectors round."""
    turns, rest = divmod(issued, n_vec)
    s, x = _prefix_sinks(words, n_vec * 4)
    more, morex = _prefix_sinks(words, rest * 4)
    return (turns * s + more) & 0xFFFFFFFF, (x if turns & 1 else 0) ^ morex


@pytest.mark.parametrize("order", [0, 1, 2])
@pytest.mark.parametrize("nbytes", [(128 << 20), (128 << 20) + 1024, (1 << 32) - 1024,
                                    (1 << 32) + 1024])
@pytest.mark.parametrize("K,w", [(5, 4), (15, 4), (16, 4), (4, 8), (5, 8), (16, 8), (2, 16),
                                 (3, 16), (13, 32)])
def test_plain_forms_at_the_lines_between_them(K, w, nbytes, order):
    """The plain loop's two forms at the lines where the choice changes: 8 MiB
    in flight, 16 KiB groups of few waves, 128 MiB; both walks; a pass and a
    bit, so that groups wrap."""
    buf = dev_bytes(nbytes)
    isw.sweep_fill_u32(buf, nbytes, SEED + 8)
    n_vec = nbytes // 16
    L = n_vec + 64 * K * 1000 + 77
    print("plain form", K, w, nbytes, "order", order, flush=True)
    r = isw.sweep_plain(buf, nbytes, K, 16, w, L, isw.make_opts(cache_policy=3, order=order))
    issued = 64 * K * (L // (64 * K))
    assert r["issued_loads"] == issued
    assert (r["sum32"], r["xor32"]) == _wrapped_sinks(buf.view(torch.int32), n_vec, issued)


def test_points_of_both_plain_forms_fuse():
    """A fused batch of points whose single cells take different plain kernels
    (below and above 128 MiB and 4 GiB) gives what the cells give."""
    sizes = [96 << 20, 160 << 20, (1 << 32) + 1024]
    buf = dev_bytes(sizes[-1])
    isw.sweep_fill_u32(buf, sizes[-1], SEED + 9)
    cells = [isw.make_cell(buf, n, 8, 16, 16, n // 16, cache_policy=3) for n in sizes]
    want = [(r["issued_loads"], r["sum32"], r["xor32"]) for r in isw.sweep_run(cells)]
    print("fused points of", sizes, flush=True)
    with isw.sweep_graph_create(cells, isw.make_opts(fuse=True)) as g:
        rs, _ = isw.sweep_graph_launch(g)
    assert [(r["issued_loads"], r["sum32"], r["xor32"]) for r in rs] == want


@pytest.mark.parametrize("dtype", ["f32", "bf16", "fp8"])
@pytest.mark.parametrize("w,mib", [(12, 256), (12, 257), (16, 257), (20, 300), (24, 257),
                                   (28, 300), (32, 512), (32, 513)])
def test_sum_with_fewer_loads_at_a_time(w, mib, dtype):
    """The sum over more than 256 MiB by many waves asks for one or two loads
    at a time: on integers every form gives the exact sum, with a ragged last
    group and trailing elements."""
    dt, td, eb = {"f32": (isw.F32, torch.float32, 4), "bf16": (isw.BF16, torch.bfloat16, 2),
                  "fp8": (isw.FP8_E4M3, torch.float8_e4m3fn, 1)}[dtype]
    n = (mib << 20) // eb + 64 * 4 * 5 * 16 + 16 // eb - 1
    g = torch.Generator(device="cuda").manual_seed(w * 1000 + mib)
    ints = torch.randint(-8, 9, (n,), device="cuda", generator=g, dtype=torch.int8)
    p = ints.to(td)
    print("sum", dtype, n, "waves per CU", w, flush=True)
    total, r = isw.sweep_reduce_fp(p, n, dt, w)
    assert total == float(ints.sum(dtype=torch.int64))
    assert r["issued_bytes"] == n * eb
    # a grid of eight workgroups stays with four loads at a time
    small, _ = isw.sweep_reduce_fp(p[:n // 16 * 16], n // 16 * 16, dt, w, isw.make_opts(grid_wgs=8))
    assert small == float(ints[:n // 16 * 16].sum(dtype=torch.int64))


@pytest.mark.parametrize("nbytes", [(64 << 20) - 1024, 64 << 20])
@pytest.mark.parametrize("V,K,w", [(4, 8, 16), (4, 9, 16), (4, 14, 16), (4, 15, 16), (4, 14, 12),
                                   (8, 8, 8), (8, 9, 8), (8, 14, 8), (8, 15, 8), (8, 3, 28),
                                   (8, 16, 4)])
def test_plain_forms_of_narrow_loads(V, K, w, nbytes):
    """The same for 4- and 8-byte loads, whose paced form lies between 8 and 14
    MiB in flight: the same words as 16-byte loads of a like number of bytes."""
    buf = dev_bytes(nbytes)
    isw.sweep_fill_u32(buf, nbytes, SEED + 10)
    n_vec = nbytes // V
    L = n_vec + 64 * K * 1000 + 77
    print("plain form", V, K, w, nbytes, flush=True)
    r = isw.sweep_plain(buf, nbytes, K, V, w, L, isw.make_opts(cache_policy=3))
    issued = 64 * K * (L // (64 * K))
    assert r["issued_loads"] == issued
    words = buf.view(torch.int32)
    turns, rest = divmod(issued, n_vec)
    s, x = _prefix_sinks(words, nbytes // 4)
    more, morex = _prefix_sinks(words, rest * V // 4)
    assert (r["sum32"], r["xor32"]) == ((turns * s + more) & 0xFFFFFFFF,
                                        (x if turns & 1 else 0) ^ morex)


@pytest.mark.parametrize("policy", [0, 2, 3])
@pytest.mark.parametrize("nbytes,K,w", [(4 << 20, 14, 4), (4 << 20, 15, 4), (4 << 20, 16, 8),
                                        (64 << 20, 8, 4), ((64 << 20) - 1024, 8, 4)])
def test_strided_plain_forms(nbytes, K, w, policy):
    """Strided cells on both sides of their own line, over whole turns of the
    buffer: each turn's loads cover every segment once in some order."""
    buf = dev_bytes(nbytes)
    isw.sweep_fill_u32(buf, nbytes, SEED + 11)
    words = buf.view(torch.int32)
    segs = nbytes // 1024
    L = 64 * K * segs                      # Q = segs: every load j of a group is turn j
    print("strided form", nbytes, K, w, "policy", policy, flush=True)
    r = isw.sweep_plain(buf, nbytes, K, 16, w, L, isw.make_opts(cache_policy=policy, order=2))
    s, x = _prefix_sinks(words, nbytes // 4)
    assert r["issued_loads"] == L
    assert (r["sum32"], r["xor32"]) == ((K * s) & 0xFFFFFFFF, x if K & 1 else 0)


@pytest.mark.parametrize("entry", ["plain", "lds", "streams", "subset", "sum"])
def test_event_time_of_a_single_call_holds_no_host_time(entry):
    """The event time of a call's only dispatch is its clock window and the
    start and end of a dispatch, which take about 1 us of a kernel longer than
    the 4.2 us floor; the host needs 4 us more from a marker to a launch."""
    nbytes = 256 << 20
    buf = dev_bytes(nbytes)
    isw.sweep_fill_u32(buf, nbytes, SEED + 12)
    n = nbytes // 16
    call = {"plain": lambda: [isw.sweep_plain(buf, nbytes, 4, 16, 16, n)],
            "lds": lambda: [isw.sweep_lds_async(buf, nbytes, 8, 16, 4, n)],
            "streams": lambda: isw.sweep_two_stream(buf, nbytes, 8, 4, 4, n),
            "subset": lambda: [isw.sweep_xcd_subset(buf, nbytes, 8, 0xFF)],
            "sum": lambda: [isw.sweep_reduce_fp(buf.zero_(), nbytes // 4, isw.F32, 16)[1]]}[entry]
    print("event time", entry, flush=True)
    over = []
    for _ in range(40):
        rs = call()
        over.append(rs[0]["event_ms"] * 1e3 - max(r["window_ns"] for r in rs) * 1e-3)
    assert 0 < float(np.median(over[8:])) < 2.5, sorted(over)


@pytest.mark.parametrize("policy", [0, 1, 2, 3])
@pytest.mark.parametrize("V,order,w,nbytes", [
    (16, 0, 8, (128 << 20) + 1024), (16, 0, 12, 128 << 20), (16, 1, 12, (128 << 20) + 1024),
    (16, 2, 8, 4 << 20), (16, 2, 12, 4 << 20), (16, 2, 28, (4 << 20) + 1024),
    (16, 2, 16, (64 << 20) - 1024), (8, 2, 28, 256 << 20), (8, 2, 32, 256 << 20),
    (4, 2, 32, (256 << 20) - 512), (4, 2, 32, 256 << 20),
    (4, 2, 32, (1 << 32) + 512), (8, 2, 32, (1 << 32) + 1024), (16, 1, 32, (1 << 32) + 1024)])
def test_plain_forms_on_both_sides_of_every_line(V, order, w, nbytes, policy):
    """The forms of the plain loop at the lines in waves, order and size where
    the choice changes, under every policy and both walks, at a small and a
    large K: a pass and a bit, so that groups wrap, and in strided cells a step
    between the loads of a group that is no whole turn of the buffer."""
    buf = dev_bytes(nbytes)
    isw.sweep_fill_u32(buf, nbytes, SEED + 13)
    words = buf.view(torch.int32)
    whole = _prefix_sinks(words, nbytes // 4)
    n_vec = nbytes // V
    for K in (2, 13):
        L = n_vec + 64 * K * 1000 + 77
        Q = L // (64 * K)
        assert Q * 64 % n_vec                       # the strided step between two loads
        print("plain form", V, "order", order, w, nbytes, "policy", policy, "K", K, flush=True)
        r = isw.sweep_plain(buf, nbytes, K, V, w, L,
                            isw.make_opts(cache_policy=policy, order=order))
        turns, rest = divmod(64 * K * Q, n_vec)
        more = _prefix_sinks(words, rest * V // 4)
        assert r["issued_loads"] == 64 * K * Q
        assert (r["sum32"], r["xor32"]) == ((turns * whole[0] + more[0]) & 0xFFFFFFFF,
                                            (whole[1] if turns & 1 else 0) ^ more[1])


@pytest.mark.parametrize("policy", [0, 1, 2, 3])
@pytest.mark.parametrize("nbytes,K,w", [(4 << 20, 8, 8), (4 << 20, 15, 8), (4 << 20, 16, 16),
                                        (1 << 20, 16, 24), ((4 << 20) + 1024, 16, 24)])
def test_strided_groups_that_wrap_between_their_loads(nbytes, K, w, policy):
    """Strided 16-byte cells that read a small buffer many times, with a step
    between the loads of a group that wraps and is no whole turn."""
    buf = dev_bytes(nbytes)
    isw.sweep_fill_u32(buf, nbytes, SEED + 14)
    segs = nbytes // 1024
    Q = segs + segs // 3 + 1
    print("strided wrap", nbytes, K, w, "policy", policy, flush=True)
    r = isw.sweep_plain(buf, nbytes, K, 16, w, 64 * K * Q,
                        isw.make_opts(cache_policy=policy, order=2))
    assert Q % segs and r["issued_loads"] == 64 * K * Q
    assert (r["sum32"], r["xor32"]) == _wrapped_sinks(buf.view(torch.int32), nbytes // 16,
                                                      64 * K * Q)
