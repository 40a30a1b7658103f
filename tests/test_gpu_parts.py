"""Partial ranges large enough to be searched in parts (aligned blocks with
their low tools enumerated deepest first on the shared-prefix kernel)."""
import numpy as np
import pytest
import torch  # (before the library: one HIP runtime in the process)

import paper_2607_22242_amd as S
from workloads import synth

pytestmark = pytest.mark.gpu
assert torch.version.hip


def test_part_ranges_match_oracle(oracle_mod):
    inst = synth.load(2)
    P, Q = S.Problem.from_instance(inst), oracle_mod.Problem.from_instance(inst)
    ws = S.workspace([P.handle])
    for lo, hi in [(1, 4_718_593), (14_348_907, 19_131_876), (P.n_mappings - 5_000_001, P.n_mappings - 1)]:
        print(f"parts [{lo}, {hi})", flush=True)
        got = S.sched_bruteforce_argmin(P.handle, lo, hi, ws)
        assert got == Q.argmin(lo, hi)
        assert S.sched_bruteforce_argmin_noalloc(P.handle, lo, hi) == got


# 26 tools: the most the parts serve; 64-bit indices from 21 tools on
@pytest.mark.parametrize("n,binary,share,tight", [
    (17, False, False, True), (19, False, False, False), (16, False, True, True),
    (23, True, True, False), (26, True, False, True)])
def test_parts_add_up_to_the_full_search(n, binary, share, tight):
    inst = synth.random_instance(9200 + n, n, "permuted", tight=tight)
    allowed = [(3, 5, 3, 6)[v % 4] for v in range(n)] if binary else None
    P = S.Problem.from_instance(inst, allowed, sharing=share)
    ws = S.workspace([P.handle])
    full = S.sched_bruteforce_argmin(P.handle, 0, P.n_mappings, ws)
    rng = np.random.default_rng(n)
    cuts = sorted({0, P.n_mappings, *(int(rng.integers(1, P.n_mappings)) for _ in range(3))})
    best = (S.NO_INDEX, S.INFEASIBLE)
    for lo, hi in zip(cuts, cuts[1:]):
        print(f"{n} tools parts [{lo}, {hi})", flush=True)
        x, ms = S.sched_bruteforce_argmin(P.handle, lo, hi, ws)
        assert ms == S.INFEASIBLE or lo <= x < hi
        best = min(best, (x, ms), key=lambda r: (r[1], r[0]))
    assert best == full
