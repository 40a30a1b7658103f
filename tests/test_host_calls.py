"""The host side of the library's calls, on the CPU: tests/host_search/host_calls.cpp
runs api.cpp on a stand-in for the HIP runtime whose streams do their work
when they are waited for."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from workloads import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def build(tmp_path_factory, *flags):
    cc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    cc = cc if os.path.exists(cc) else shutil.which("hipcc")
    if cc is None:
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("host_calls") / "host_calls")
    subprocess.check_call([cc, "-O2", "-std=c++17", "-pthread", "-x", "hip", "--offload-arch=gfx950",
                           "--cuda-host-only",
                           "-I" + os.path.join(ROOT, "include"),
                           "-I" + os.path.join(ROOT, "paper_2607_22242_amd", "csrc"),
                           os.path.join(ROOT, "tests", "host_search", "host_calls.cpp"),
                           "-o", exe, *flags], stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)

    def run(what, *problems):
        text = []
        for inst, allowed, share in problems:
            allowed = allowed or [7] * len(inst["tools"])
            text.append(f"{len(allowed)} {int(share)} {len(inst['edges'])} "
                        f"{len(inst['contention_q16'])} {inst['vram_budget_mib']}")
            text += [" ".join(map(str, t)) + f" {a}" for t, a in zip(inst["tools"], allowed)]
            text += [f"{u} {v}" for u, v in inst["edges"]]
            text.append(" ".join(map(str, inst["contention_q16"])))
        r = subprocess.run([exe, what], input="\n".join(text) + "\n", capture_output=True, text=True,
                           timeout=300)
        assert r.returncode == 0, (r.returncode, r.stderr[-2000:])
        assert r.stdout.endswith("ok\n")
        return r.stdout.split("\n")[:-2]
    return run


@pytest.fixture(scope="module")
def host_calls(tmp_path_factory):
    return build(tmp_path_factory)


@pytest.fixture(scope="module")
def host_calls_small_chunks(tmp_path_factory):
    return build(tmp_path_factory, "-DHOST_CALLS_N=15", "-DDEVMAP_CHUNK_PREFIXES=8")


@pytest.mark.parametrize("n,levels", [(15, 4), (19, 19)])
def test_range_in_parts_needs_little_stack(host_calls, n, levels):
    host_calls("stack", (synth.random_instance(9900 + n, n, "random", levels=levels), None, False))


@pytest.mark.parametrize("n,shape,masks,shared", [
    (13, "random", [7] * 13, 1),                # shared prefixes in thin waves
    (21, "chain", [3] * 21, 0),                 # closed form, in a space that has prefixes enough
    (21, "permuted", [3] * 21, 1),              # shared prefixes in full waves
    (12, "random", [7] * 12, 0)])               # too few prefixes
def test_counters_of_a_space_searched_whole(host_calls, n, shape, masks, shared):
    inst = synth.random_instance(9920 + n, n, shape)
    inst["tools"] = [[max(1, x // 20) for x in t[:4]] + [t[4]] for t in inst["tools"]]
    assert host_calls("stats", (inst, masks, False)) == [str(shared)]


def small_problems():
    """Four problems of 6 and 10 tools: both contention readings, a chain, a
    fan-out that fits its budget, restricted modes."""
    fan = synth.random_instance(9942, 6, "fanout")
    fan["vram_budget_mib"] = sum(t[4] for t in fan["tools"])
    return [(synth.random_instance(9940, 6, "random", tight=True), None, False),
            (synth.random_instance(9941, 6, "chain"), None, True), (fan, None, False),
            (synth.random_instance(9943, 10, "permuted"), [3, 7, 1, 5, 3, 7, 2, 3, 6, 3], False)]


def test_calls_without_a_slot(host_calls):
    host_calls("slots", *small_problems())


def test_batches_around_a_full_slot(host_calls):
    host_calls("replicas", (synth.random_instance(9950, 6, "permuted", tight=True),
                            [3, 7, 1, 5, 3, 2], False))


# 3^40 mappings: two replicas hold more than 64 bits count
@pytest.mark.parametrize("shape", ["random", "chain"])
def test_blocks_of_the_largest_batches(host_calls, shape):
    inst = synth.random_instance(9960, 40, shape)
    inst["tools"] = [[1 + t[0] % 99, 1 + t[1] % 99, t[2] % 99, t[3] % 9, t[4]] for t in inst["tools"]]
    host_calls("blocks", (inst, None, False))


def test_workspaces_of_fewer_bytes(host_calls):
    host_calls("room", (synth.random_instance(9970, 15, "random", tight=True), None, False))


# 15 tools, by chunks of eight prefixes; 34 tools (2^12 * 3^7 mappings, 64-bit masks); and 15 tools
# of which one outlasts the others whatever they do, so that no child is ruled out: its prefixes
# are searched, at once and shared
@pytest.mark.parametrize("n,share,long,chunks", [(15, False, False, True), (15, True, False, True),
                                                 (34, False, False, False), (15, False, True, False)])
def test_children_are_scored_once(request, oracle_mod, n, share, long, chunks):
    run = request.getfixturevalue("host_calls_small_chunks" if chunks else "host_calls")
    inst = synth.random_instance(9980 + n, n, "permuted", tight=True, small_values=True)
    allowed = [7] * n
    if n == 34:
        allowed = [1] * n
        for k in range(19):
            allowed[7 * k % n] = 7 if k % 8 in (1, 4, 6) else (3, 5)[k % 2]
    if long:
        inst["tools"][6][:2] = [100_000, 100_000]
        inst["edges"] = [e for e in inst["edges"] if 6 not in e]
        allowed[6] = 3
    x, ms, launches, shared, children, prefixes = map(int, run("children", (inst, allowed, share))[0].split())
    assert launches >= (2 if chunks else 1) and (shared > 0) == long
    assert (children > 0) != long and (prefixes > 0) == long
    Q, space = oracle_mod.Problem.from_instance(inst, sharing=share), oracle_mod.Space(allowed)
    assert int(Q.eval_many(space.base3(np.array([x], dtype=np.uint64)))[0]) == ms


def test_closed_forms_where_they_gain(host_calls):
    """A fan-out's last labels have to hold combinations: with tools of one
    mode there, it is scored one by one."""
    def fan(n, allowed, shape="fanout"):
        inst = synth.random_instance(9990 + n, n, shape)
        inst["tools"] = [[max(1, x // 20) for x in t[:4]] + [t[4]] for t in inst["tools"]]
        inst["vram_budget_mib"] = sum(t[4] for t in inst["tools"])
        return inst, allowed, False

    got = host_calls("closed",
                     fan(14, [7] * 14),                       # 3^14: 3 labels, 27 combinations
                     fan(24, [3] * 19 + [1] * 5),             # 2^19: 2 labels, 1 combination
                     fan(29, [3] * 24 + [1] * 5),             # 2^24: 5 labels, 1 combination
                     fan(28, [3] * 23 + [1, 1, 1, 1, 3]),     # 5 labels, 2 combinations
                     fan(24, [3] * 20 + [1] * 4),             # 2^20: 2 labels, 1 combination
                     fan(25, [3] * 20 + [1, 1, 1, 1, 7]),     # 3 labels, 3 combinations
                     fan(28, [3] * 22 + [1, 1, 7, 1, 1, 1]),  # 4 labels, 3 combinations
                     fan(29, [3] * 24 + [1] * 5, "chain"))
    assert got == ["3 5", "2 0", "0 0", "0 0", "0 0", "3 5", "4 5", "5 5"]
    # work for two labels in all, which need hold no more than one combination
    assert host_calls("closed", fan(24, [3] * 19 + [1] * 5), fan(10, [7] * 10)) == ["2 2", "0 2"]
    # more work, too little of it in fan-outs that gain
    assert host_calls("closed", fan(29, [3] * 24 + [1] * 5), fan(10, [7] * 10)) == ["0 0", "0 0"]
    # three labels' work, of which two gain from it
    assert host_calls("closed", fan(25, [3] * 20 + [1, 1, 1, 1, 7]), fan(13, [7] * 11 + [1, 3]),
                      fan(15, [3] * 12 + [1] * 3)) == ["3 3", "2 3", "0 0"]


def test_ranges_in_parts_where_they_gain(host_calls):
    """Problems without edges need three times as many mappings, and a tool of
    three modes."""
    def tight(n, shape, allowed):
        return synth.random_instance(10000 + n, n, shape, tight=True), allowed, False

    lanes = 9 << 19
    assert host_calls("parts", tight(16, "random", [7] * 16), tight(24, "random", [3] * 24),
                      tight(16, "fanout", [7] * 16), tight(24, "fanout", [3] * 23 + [7]),
                      tight(24, "fanout", [3] * 24), tight(14, "fanout", [7] * 14)) == \
        [str(lanes), str(lanes), str(3 * lanes), str(3 * lanes), "0", "0"]


@pytest.mark.parametrize("what", ["allocations", "runtime"])
def test_failures(host_calls, what):
    big = synth.random_instance(9945, 15, "random", tight=True, small_values=True)
    wide = synth.random_instance(9946, 34, "random", levels=34, small_values=True)
    host_calls(what, *small_problems(), (big, None, False), (wide, [1] * 22 + [3] * 12, False))
