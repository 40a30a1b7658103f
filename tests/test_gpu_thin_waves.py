"""Shared prefixes in waves that are not full (spaces of 2^17 to 2^19 prefixes):
every mapping of the search against the oracle."""
import numpy as np
import pytest
import torch  # (before the library: one HIP runtime in the process)

import paper_2607_22242_amd as S
from workloads import synth

pytestmark = pytest.mark.gpu
assert torch.version.hip


# nine combinations (28 prefixes a wave) and six (42); the fewest prefixes;
# inner tools that stop a prefix early and such that do not
@pytest.mark.parametrize("n,shape,tight,masks,share", [
    (13, "random", True, {}, False), (13, "permuted", False, {}, False),
    (13, "permuted", True, {}, True), (14, "random", True, {0: 3, 13: 5}, False),
    (14, "permuted", False, {v: 3 for v in range(4)}, False),
    (21, "permuted", True, {v: 1 + v % 2 for v in range(8)}, False)])
def test_thin_waves_every_mapping(oracle_mod, n, shape, tight, masks, share):
    inst = synth.random_instance(9700 + n, n, shape, tight=tight)
    allowed = [masks.get(v, 7) for v in range(n)]
    P, space = S.Problem.from_instance(inst, allowed, sharing=share), oracle_mod.Space(allowed)
    out = torch.full((P.n_mappings,), 0x7FFFFFFE, dtype=torch.int32, device="cuda")
    print(f"thin waves, {n} tools: {P.n_mappings} mappings", flush=True)
    best = S.sched_bruteforce_record(P.handle, S.workspace([P.handle]), out)
    got = out.cpu().numpy().view(np.uint32).astype(np.int64)
    want = oracle_mod.Problem.from_instance(inst, sharing=share).eval_many(
        space.base3(np.arange(P.n_mappings, dtype=np.uint64)))
    want = np.where(want == oracle_mod.INFEASIBLE, 0xFFFFFFFF, want)
    np.testing.assert_array_equal(got, want)
    k = int(want.argmin())
    assert best == (k, int(want[k]))
