"""A partial range searched in parts, on the host: the library's split and
tables (split_range, stage_parts) driven through the kernels' per-lane code
must score every mapping of [lo, hi) exactly once, nothing outside it, and
with the oracle's makespan.  Ranges start and end inside blocks, on their
edges, and at the ends of the space; spaces have three modes per tool, mixed
radices and fixed tools; both contention readings.  And a batch's replica on the
kernel for more tools than it has (lay_replica): every mapping scored once and
as the oracle has it, with and without shared prefixes, fan-outs included."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from workloads import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
N = 12


@pytest.fixture(scope="module")
def host_range(tmp_path_factory):
    cc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    cc = cc if os.path.exists(cc) else shutil.which("hipcc")
    if cc is None:
        pytest.skip("hipcc not available")
    tmp = tmp_path_factory.mktemp("host_range")
    exe, out = str(tmp / "host_range"), str(tmp / "out.bin")
    subprocess.check_call([cc, "-O2", "-std=c++17", "-x", "hip", "--offload-arch=gfx950",
                           "--cuda-host-only", f"-DHOST_RANGE_N={N}",
                           "-I" + os.path.join(ROOT, "include"),
                           "-I" + os.path.join(ROOT, "paper_2607_22242_amd", "csrc"),
                           os.path.join(ROOT, "tests", "host_search", "host_range.cpp"),
                           "-o", exe], stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)

    def run(inst, allowed, lo, hi, share):
        text = [f"{len(allowed)} {lo} {hi} {int(share)} {len(inst['edges'])} {len(inst['contention_q16'])} "
                f"{inst['vram_budget_mib']}"]
        text += [" ".join(map(str, t)) + f" {a}" for t, a in zip(inst["tools"], allowed)]
        text += [f"{u} {v}" for u, v in inst["edges"]]
        text.append(" ".join(map(str, inst["contention_q16"])))
        parts = int(subprocess.run([exe, out], input="\n".join(text) + "\n", capture_output=True,
                                   text=True, check=True, timeout=300).stdout)
        times, ms = np.fromfile(out, dtype=np.uint32).reshape(2, -1)
        return parts, times, ms.astype(np.int64)
    return run


def check(oracle_mod, inst, allowed, share, got, lo, hi):
    parts, times, ms = got
    space = oracle_mod.Space(allowed)
    assert parts >= 1
    want_times = np.zeros(space.size(), dtype=np.uint32)
    want_times[lo:hi] = 1
    assert (times == want_times).all()
    Q = oracle_mod.Problem.from_instance(inst, sharing=share)
    want = Q.eval_many(space.base3(np.arange(lo, hi, dtype=np.uint64)))
    want = np.where(want == oracle_mod.INFEASIBLE, 0xFFFFFFFF, want)
    np.testing.assert_array_equal(ms[lo:hi], want)


@pytest.mark.parametrize("shape,tight,masked,share,lo,hi", [
    ("random", True, False, False, 1, 531440),            # all but the first and last mapping
    ("random", False, False, False, 19683, 531441),       # the start on a block's edge
    ("chain", True, False, False, 12345, 98765),          # blocks of the smallest level only
    ("permuted", True, False, False, 19682, 39367),       # one block, one mapping each side
    ("permuted", False, True, False, 777, 0.93),          # mixed radices
    ("random", True, True, False, 0, 0.5),
    ("random", True, False, True, 100_001, 500_003),
    ("permuted", True, True, True, 4_321, 0.9)])
def test_parts_cover_the_range_once(host_range, oracle_mod, shape, tight, masked, share, lo, hi):
    seed = 9100 + lo % 97
    inst = synth.random_instance(seed, N, shape, tight=tight)
    allowed = [(7, 7, 7, 7, 7, 6, 7, 7, 7, 3, 7, 2)[(v + seed) % N] for v in range(N)] if masked \
        else [7] * N
    total = oracle_mod.Space(allowed).size()
    hi = int(hi * total) if isinstance(hi, float) else hi
    check(oracle_mod, inst, allowed, share, host_range(inst, allowed, lo, hi, share), lo, hi)


# work: mappings of the launch (1: a mapping per lane; 10^10: six inner digits,
# or shared prefixes where the problem has them)
@pytest.mark.parametrize("n,shape,fits,share,work", [
    (1, "chain", False, False, 1), (4, "permuted", False, False, 1),
    (9, "random", False, False, 10**10), (11, "permuted", False, True, 10**10),
    (8, "random", False, True, 1), (7, "fanout", True, False, 10**10),
    (12, "random", False, False, 10**10), (12, "fanout", True, False, 1)])
def test_replica_on_a_wider_kernel(host_range, oracle_mod, n, shape, fits, share, work):
    inst = synth.random_instance(9150 + n, n, shape, tight=not fits)
    if fits:
        inst["vram_budget_mib"] = sum(t[4] for t in inst["tools"])
    allowed = [(7, 5, 7, 3, 7, 2)[v % 6] if n == 9 else 7 for v in range(n)]
    got = host_range(inst, allowed, work, 0, share)
    check(oracle_mod, inst, allowed, share, got, 0, oracle_mod.Space(allowed).size())
