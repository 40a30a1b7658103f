"""The pruned search's second level of bounds, against the exhaustive search:
spaces whose prefixes survive in several chunks (small latencies, many ties),
spaces with few tools left for the extension, and restricted ones."""
import pytest
import torch  # (before the library: one HIP runtime in the process)

import paper_2607_22242_amd as S
from workloads import synth

pytestmark = pytest.mark.gpu
assert torch.version.hip


@pytest.mark.parametrize("n,shape,small,masked,share", [
    (14, "random", True, False, False), (17, "random", True, False, False),
    (17, "fanout", True, False, False), (18, "permuted", True, False, False),
    (16, "permuted", True, False, True), (24, "permuted", False, True, False),
    (30, "permuted", False, True, False)])
def test_children_match_exhaustive(n, shape, small, masked, share):
    inst = synth.random_instance(9600 + n, n, shape, tight=shape != "fanout", small_values=small)
    allowed = [(3, 7, 6, 1, 5, 3, 2, 3)[v % 8] for v in range(n)] if masked else None
    P = S.Problem.from_instance(inst, allowed, sharing=share)
    print(f"pruned {n} tools, {shape}: {P.n_mappings} mappings", flush=True)
    x, ms, st = S.sched_pruned_argmin(P.handle, S.pruned_workspace(P.handle))
    assert (x, ms) == S.sched_bruteforce_argmin(P.handle, 0, P.n_mappings, S.workspace([P.handle]))
    print(st, flush=True)
    assert st["launches"] >= 1 and st["mappings_searched"] <= P.n_mappings


# 64-bit masks: the children's list walked without shared prefixes, up to six inner digits
@pytest.mark.parametrize("n,share", [(33, False), (36, True), (40, False)])
def test_children_of_wide_problems(n, share):
    inst = synth.random_instance(9650 + n, n, "permuted", tight=True)
    # 2^12 * 3^7 mappings: 12 tools with two modes, 7 with three, spread over the labels
    allowed = [1] * n
    for k in range(19):
        allowed[(7 * k) % n] = 7 if k % 8 in (1, 4, 6) else (3, 5)[k % 2]
    P = S.Problem.from_instance(inst, allowed, sharing=share)
    print(f"pruned {n} tools: {P.n_mappings} mappings", flush=True)
    assert 1 << 22 <= P.n_mappings <= 1 << 25
    x, ms, st = S.sched_pruned_argmin(P.handle, S.pruned_workspace(P.handle))
    assert (x, ms) == S.sched_bruteforce_argmin(P.handle, 0, P.n_mappings, S.workspace([P.handle]))
    assert st["prefix_tools"] >= 1 and st["launches"] >= 1 and st["shared_prefix_launches"] == 0
