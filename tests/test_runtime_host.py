"""The host runtime of the built library on a HIP runtime without a device
(fake_hip.cpp): what it launches, with which pointers, and what it does when
memory runs out."""
import json
import os
import shutil
import subprocess
import sys

import pytest

from conftest import ROOT

ROCM = "/opt/rocm/include"

# loaded first, the stand-in serves the library's dependency of the same name
PRELUDE = """
import ctypes as C, json, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
fake.fake_limit_pinned.argtypes = [C.c_size_t]
fake.fake_kernel.restype = C.c_char_p
fake.fake_arg.restype = C.c_uint64
from paper_2608_15764_amd import ilpsweep as isw
buf = 1 << 40
out = {}
def launched():
    return [fake.fake_kernel(i).decode() for i in range(fake.fake_launches())]
def refused(call):
    fake.fake_reset()
    try:
        call()
    except isw.SweepError as e:
        return e.code
    return 0
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    from paper_2608_15764_amd import build
    if not shutil.which("g++") or not os.path.exists(os.path.join(ROCM, "hip")):
        pytest.skip("no g++ or HIP headers")
    if not os.path.exists(build.LIB):
        pytest.skip("the library is not built")
    fake = str(tmp_path_factory.mktemp("fake") / "libamdhip64.so.7")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-Wl,-soname,libamdhip64.so.7", "-I", ROCM,
                    os.path.join(ROOT, "tests", "fake_hip.cpp"), "-o", fake],
                   check=True, stderr=subprocess.DEVNULL)

    def run(body):
        r = subprocess.run([sys.executable, "-c", PRELUDE + body + "\nprint(json.dumps(out))", fake],
                           capture_output=True, text=True, cwd=ROOT, timeout=120)
        assert r.returncode == 0, r.stderr
        return json.loads(r.stdout.strip().split("\n")[-1])
    return run


def test_calls_after_a_failed_growth_have_their_results_to_write_to(host):
    """A long sweep that cannot have pinned memory for its results gives up the
    shorter block it had; the calls after it get one of their own, or fail too:
    no kernel is handed an address near 0."""
    got = host("""
cells = isw.cell_array([isw.make_cell(buf, 1 << 20, 1, 16, 4, 1 << 16)] * 3000)
calls = {
    "subset": lambda: isw.sweep_xcd_subset(buf, 64 << 20, 4, 0x0F),
    "split": lambda: isw.sweep_xcd_split(buf, 64 << 20, 4, [1.0] * 8),
    "streams": lambda: isw.sweep_two_stream(buf, 64 << 20, 4, 2, 2, 1 << 22),
    "sum": lambda: isw.sweep_reduce_fp(buf, 1 << 20, isw.F32, 8),
    "cell": lambda: isw.sweep_plain(buf, 1 << 20, 1, 16, 4, 1 << 16),
}
for name, call in calls.items():
    for limit in (1 << 20, 8):
        isw.sweep_shutdown()
        fake.fake_limit_pinned(4096)
        isw.sweep_init(0)
        long = refused(lambda: isw.sweep_run(cells))
        fake.fake_limit_pinned(limit)
        code = refused(call)
        args = [[fake.fake_arg(i, k) for k in range(6)] for i in range(fake.fake_launches())
                if b"finish_" in fake.fake_kernel(i)]
        out[f"{name} {limit}"] = [long, code, launched(), args]
""")
    to = {"finish_xcd": (2, 3), "finish_cells": (2,), "finish_reduce": (2, 5)}
    for name, (long, code, kernels, args) in got.items():
        assert long == -5, name
        if name.endswith(" 8"):
            assert code == -5 and not kernels, (name, code, kernels)
        else:
            last = next(k for k in to if k in kernels[-1])
            assert len(args) == 1 and all(args[0][k] > 4096 for k in to[last]), (name, args)


def test_timed_dispatches_run_from_the_end_of_the_one_before(host):
    """The first timed dispatch of a call is timed from the end of a gate that
    waits for its submission, the next ones from each other; the gate's flag is
    up when the call returns, also where the dispatch fails to launch."""
    got = host("""
cells = isw.cell_array([isw.make_cell(buf, 1 << 20, K, 16, 4, 1 << 16) for K in (1, 2, 3)])
calls = {
    "run": lambda: isw.sweep_run(cells),
    "plain": lambda: isw.sweep_plain(buf, 1 << 20, 1, 16, 4, 1 << 16),
    "subset": lambda: isw.sweep_xcd_subset(buf, 64 << 20, 4, 0x0F),
    "split": lambda: isw.sweep_xcd_split(buf, 64 << 20, 4, [1.0] * 8),
    "streams": lambda: isw.sweep_two_stream(buf, 64 << 20, 4, 2, 2, 1 << 22),
    "sum": lambda: isw.sweep_reduce_fp(buf, 1 << 20, isw.F32, 8),
}
isw.sweep_init(0)
def gate():
    at = [i for i, k in enumerate(launched()) if "gate" in k]
    i = at[0]
    flag = C.c_uint32.from_address(fake.fake_arg(i, 0)).value
    return at, flag, fake.fake_arg(i, 1) & 0xFFFFFFFF, fake.fake_arg(i, 1) >> 32
for name, call in calls.items():
    code = refused(call)
    at, flag, ticket, ticks = gate()
    n = {"run": 3, "subset": 0, "split": 0}.get(name, 1)
    froms = [fake.fake_interval_from(i) for i in range(n)]
    fake.fake_reset()
    fake.fake_fail_launch(at[0] + 1)
    try:
        call()
        failed = 0
    except isw.SweepError as e:
        failed = e.code
    out[name] = [code, at, flag, ticket, ticks, froms, failed, gate()]
""")
    for name, (code, at, flag, ticket, ticks, froms, failed, after) in got.items():
        g = at[0]
        # (an XCD read finds no record of the wave it looks for, and says so)
        assert code == (0 if froms else -6), (name, code)
        assert len(at) == 1 and flag == ticket > 0, name
        assert froms == [g, g + 1, g + 2][:len(froms)], (name, froms)
        assert 0 < ticks <= 100_000, (name, ticks)          # 1 ms of the 100 MHz clock at most
        assert failed == -4 and after[1] == after[2] == ticket + 1, (name, failed, after)


def test_the_plain_loop_is_one_along_a_K_curve(host):
    """Which form of the plain loop runs depends on nothing that a K curve
    varies: the cells of a curve run one kernel but for its K (of one load the
    forms are the same).  A grid of several turns takes the form of one."""
    got = host("""
MIB = 1 << 20
for V in (4, 8, 16):
    for w in range(4, 33, 4):
        for mib in (1, 4, 5, 64, 65, 128, 129, 256, 1024, 5120):
            for order in range(3):
                for policy in range(4):
                    def cells(turns):
                        wgs = 256 * w // 4 * turns if turns else 0
                        return [isw.make_cell(buf, mib * MIB, K, V, w, mib * MIB // V * 16,
                                              cache_policy=policy, order=order, grid_wgs=wgs)
                                for K in range(1, 17)]
                    for turns in (0, 3):
                        fake.fake_reset()
                        isw.sweep_run(cells(turns))
                        ran = [k for k in launched() if "plain_kload" in k]
                        forms = [k[:k.index("ILi")] for k in ran]
                        out[f"{V} {w} {mib} {order} {policy} {turns}"] = [
                            len(ran), sorted(set(forms[1:])), forms[0]]
""")
    spaced = 0
    for case, (n, forms, first) in got.items():
        assert n == 16 and len(forms) == 1, (case, forms)
        assert "spaced" not in first and ("far" in first) == (" 5120 " in case), (case, first)
        assert ("far" in first) == ("far" in forms[0]), (case, first, forms)
        assert got[case[:-1] + "0"][1] == forms, case
        spaced += "spaced" in forms[0]
    assert 0 < spaced < len(got)


def test_a_fused_batch_of_several_turns_takes_the_form_of_one(host):
    """The fused loop's form goes by the bytes in flight: a grid of more
    workgroups than the CUs hold has no more of them."""
    got = host("""
for K, w in ((3, 8), (6, 4), (7, 4), (4, 8)):
    for turns in (1, 2, 8):
        cells = [isw.make_cell(buf + (i << 20), 1 << 20, K, 16, w, 1 << 20,
                               grid_wgs=256 * w // 4 * turns) for i in range(3)]
        fake.fake_reset()
        with isw.sweep_graph_create(cells, isw.make_opts(fuse=True)) as g:
            isw.sweep_graph_launch(g)
        out[f"{K} {w} {turns}"] = [k[:k.index("ILi")] for k in launched() if "fused" in k]
""")
    for case, ran in got.items():
        K, w, _ = map(int, case.split())
        back_to_back = K * w <= 24                    # 256 CUs x w waves x K KiB up to 6 MiB
        assert len(ran) == 1 and ("ahead" in ran[0]) == back_to_back, (case, ran)
