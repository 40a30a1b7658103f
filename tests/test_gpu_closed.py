"""Closed-form searches (serial chains; fan-outs that fit the budget together):
every mapping they record against the oracle (all of a small space, a sample
of a large one), and their winner against the record."""
import numpy as np
import pytest
import torch  # (before the library: one HIP runtime in the process)

import paper_2607_22242_amd as S
from workloads import synth

pytestmark = pytest.mark.gpu
assert torch.version.hip

# tools whose modes are restricted, some to one mode, the last labels among them
MIXED = (7, 3, 6, 5, 7, 2, 3, 5, 4, 6, 3, 1)


# chains of 5 to 16 tools: 1 to 5 labels walked per lane, fan-outs of 12 to 16: 2 to 5; levels 1 to 4
@pytest.mark.parametrize("shape,n,levels,masked,tight", [
    ("chain", 5, 2, False, True), ("chain", 12, 4, False, False), ("fanout", 12, 2, False, False),
    ("chain", 13, 1, False, True), ("chain", 14, 4, False, False), ("chain", 15, 2, False, True),
    ("chain", 16, 3, False, False), ("chain", 24, 4, True, True), ("chain", 29, 2, True, False),
    ("fanout", 13, 4, False, False), ("fanout", 14, 3, False, False),
    ("fanout", 15, 2, False, False), ("fanout", 16, 1, False, False),
    ("fanout", 16, 4, False, False), ("fanout", 25, 4, True, False),
    ("fanout", 32, 3, True, False)])
def test_closed_forms_every_mapping(oracle_mod, shape, n, levels, masked, tight):
    inst = synth.random_instance(9400 + n, n, shape, tight=tight, levels=levels)
    if shape == "fanout":
        inst["vram_budget_mib"] = sum(t[4] for t in inst["tools"])
    allowed = [MIXED[(v * 5 + n) % 12] if v >= n - (16 if n == 29 else 22) else 1 << (v % 3) for v in range(n)] \
        if masked else [7] * n
    if shape == "chain" and n == 29:  # a budget that some tools never fit
        inst["vram_budget_mib"] = 12000
        allowed = [a | 1 for a in allowed]
    P, space = S.Problem.from_instance(inst, allowed), oracle_mod.Space(allowed)
    assert shape == "chain" or P.n_mappings >= 9 << 15
    out = torch.full((P.n_mappings,), 0x7FFFFFFE, dtype=torch.int32, device="cuda")
    ws = S.workspace([P.handle])
    print(f"{shape} of {n} tools, {levels} levels, {P.n_mappings} mappings", flush=True)
    best = S.sched_bruteforce_record(P.handle, ws, out)
    got = out.cpu().numpy().view(np.uint32).astype(np.int64)
    assert (got != 0x7FFFFFFE).all()
    idx = np.arange(P.n_mappings, dtype=np.uint64)
    if P.n_mappings > 2_000_000:
        idx = np.random.default_rng(n).choice(idx, 300_000, replace=False)
    want = oracle_mod.Problem.from_instance(inst).eval_many(space.base3(idx))
    want = np.where(want == oracle_mod.INFEASIBLE, 0xFFFFFFFF, want)
    np.testing.assert_array_equal(got[idx.astype(np.int64)], want)
    k = int(got.argmin())
    assert best == (k, int(got[k])) == S.sched_bruteforce_argmin(P.handle, 0, P.n_mappings, ws)
