"""Batches whose replicas of different tool counts share a launch (smaller
problems laid out for the kernel of the largest), against single searches."""
import pytest
import torch  # (before the library: one HIP runtime in the process)

import paper_2607_22242_amd as S
from workloads import synth

pytestmark = pytest.mark.gpu
assert torch.version.hip


# (tools, shape, sharing, two modes per tool from this tool on)
@pytest.mark.parametrize("name,problems", [
    ("one tool to twelve", [(n, ("chain", "fanout", "permuted", "random")[n % 4], False, n)
                            for n in range(1, 13)]),
    ("both readings", [(5, "random", False, 5), (8, "permuted", True, 8), (3, "chain", True, 3),
                       (8, "fanout", False, 8), (11, "random", True, 11)]),
    ("onto a kernel without prefixes for them", [(6, "random", False, 6), (33, "random", False, 3),
                                                 (13, "permuted", False, 13)]),
    ("onto 64-bit indices", [(4, "fanout", False, 4), (9, "random", True, 9),
                             (24, "permuted", False, 4), (22, "random", True, 2)])])
def test_mixed_launch_matches_single_searches(name, problems):
    handles, want, rp, lat = [], [], [], []
    keep = []
    for k, (n, shape, sharing, three) in enumerate(problems):
        inst = synth.random_instance(9300 + k, n, shape, tight=k % 2 == 0)
        allowed = [7 if v < three else (1, 2, 3, 1)[v % 4] for v in range(n)]
        for rep in range(3):
            new = synth.perturb(inst["tools"], 10 * k + rep)
            measured = dict(inst, tools=[r + [t[4]] for r, t in zip(new, inst["tools"])])
            P = S.Problem.from_instance(measured, allowed, sharing=sharing)
            want.append(S.sched_bruteforce_argmin(P.handle, 0, P.n_mappings, S.workspace([P.handle])))
            rp.append(k)
            lat.append(new)
        keep.append(S.Problem.from_instance(inst, allowed, sharing=sharing))
        handles.append(keep[-1].handle)
    order = sorted(range(len(rp)), key=lambda i: (i * 7) % len(rp))  # replicas in no order
    print(f"batch {name}: {len(rp)} replicas", flush=True)
    got = S.sched_eval_batch(handles, [rp[i] for i in order], [lat[i] for i in order],
                             S.workspace(handles, len(rp)))
    assert got == [want[i] for i in order]


def test_mixed_fan_outs_in_closed_form(oracle_mod):
    """Fan-outs of several tool counts, masks and contention levels in one
    launch of their closed form, against the oracle over each whole space."""
    import numpy as np
    handles, keep, rp, lat, want = [], [], [], [], []
    for k, (n, levels, masked) in enumerate([(12, 4, False), (13, 1, True), (15, 3, True), (14, 2, True),
                                             (5, 4, False)]):
        inst = synth.random_instance(9350 + k, n, "fanout", levels=levels)
        inst["vram_budget_mib"] = sum(t[4] for t in inst["tools"])
        allowed = [(3, 7, 6, 7, 7, 2, 7, 5)[(v + k) % 8] if masked else 7 for v in range(n)]
        keep.append(S.Problem.from_instance(inst, allowed))
        handles.append(keep[-1].handle)
        space = oracle_mod.Space(allowed)
        idx = space.base3(np.arange(space.size(), dtype=np.uint64))
        for rep in range(2):
            new = synth.perturb(inst["tools"], 10 * k + rep)
            Q = oracle_mod.Problem.from_instance(
                dict(inst, tools=[r + [t[4]] for r, t in zip(new, inst["tools"])]))
            ms = Q.eval_many(idx)
            want.append((int(ms.argmin()), int(ms.min())))
            rp.append(k)
            lat.append(new)
    order = sorted(range(len(rp)), key=lambda i: (i * 7) % len(rp))
    print(f"batch of fan-outs: {len(rp)} replicas", flush=True)
    got = S.sched_eval_batch(handles, [rp[i] for i in order], [lat[i] for i in order],
                             S.workspace(handles, len(rp)))
    assert got == [want[i] for i in order]
