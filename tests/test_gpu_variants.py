"""Shared-prefix searches of spaces without gpu_queue (the evaluator's variants
with and without a VRAM budget that binds), 21 to 32 tools: a sample of the
recorded mappings against the oracle, the winner against the record, and the
pruned search's subspaces on the same kernels."""
import numpy as np
import pytest
import torch  # (before the library: one HIP runtime in the process)

import paper_2607_22242_amd as S
from workloads import synth

pytestmark = pytest.mark.gpu
assert torch.version.hip


# fixed: tools with one mode (cpu or gpu_now), so that the record stays small
@pytest.mark.parametrize("n,budget,fixed", [
    (21, "all", 0), (22, "most", 0), (23, "quarter", 0), (26, "all", 3), (26, "quarter", 3),
    (27, "all", 4), (28, "quarter", 5), (32, "all", 8), (32, "quarter", 8)])
def test_spaces_without_queue(oracle_mod, n, budget, fixed):
    inst = synth.random_instance(9500 + n, n, "permuted")
    total = sum(t[4] for t in inst["tools"])
    inst["vram_budget_mib"] = {"all": total, "most": total - 1, "quarter": total // 4}[budget]
    allowed = [3] * n
    for k in range(fixed):
        allowed[(7 * k + 3) % n] = 1 + k % 2
    P, space = S.Problem.from_instance(inst, allowed), oracle_mod.Space(allowed)
    out = torch.full((P.n_mappings,), 0x7FFFFFFE, dtype=torch.int32, device="cuda")
    ws = S.workspace([P.handle])
    print(f"{n} tools, {fixed} fixed, budget {budget}: {P.n_mappings} mappings", flush=True)
    best = S.sched_bruteforce_record(P.handle, ws, out)
    got = out.cpu().numpy().view(np.uint32).astype(np.int64)
    assert (got != 0x7FFFFFFE).all()
    k = int(got.argmin())
    assert best == (k, int(got[k])) if got[k] != 0xFFFFFFFF else best == (S.NO_INDEX, S.INFEASIBLE)
    idx = np.random.default_rng(n).integers(0, P.n_mappings, 200_000, dtype=np.uint64)
    want = oracle_mod.Problem.from_instance(inst).eval_many(space.base3(idx))
    want = np.where(want == oracle_mod.INFEASIBLE, 0xFFFFFFFF, want)
    np.testing.assert_array_equal(got[idx.astype(np.int64)], want)
    assert S.sched_pruned_argmin(P.handle, S.pruned_workspace(P.handle))[:2] == best
