"""Calls that overlap: host threads with a stream and a workspace each, more of
them than there are page-locked slots, mixing searches, ranges, probes, scores
and batches; every answer equals the one that the same call gave alone."""
import threading

import numpy as np
import pytest
import torch  # (before the library: one HIP runtime in the process)

import paper_2607_22242_amd as S
from workloads import synth

pytestmark = pytest.mark.gpu
assert torch.version.hip

THREADS, ROUNDS = 12, 6  # (8 slots)


def test_threads_with_streams_of_their_own():
    kinds = [(5, "random", False), (9, "permuted", True), (12, "random", False), (14, "chain", False),
             (15, "permuted", False)]
    insts = [synth.random_instance(9800 + n, n, shape, tight=n != 14) for n, shape, _ in kinds]
    problems = [S.Problem.from_instance(i, sharing=k[2]) for i, k in zip(insts, kinds)]
    handles = [p.handle for p in problems]
    small = [0, 1]
    rp = [small[r % 2] for r in range(40)]
    lat = [synth.perturb(insts[i]["tools"], 50 + r) for r, i in enumerate(rp)]
    # 700 indices go through a slot, 5,000 do not
    idx = [np.random.default_rng(p.n).integers(0, p.n_mappings, m, dtype=np.uint64)
           for p in problems for m in (700, 5000)]

    def call(k, ws, stream):
        p = problems[k % 5]
        what = k // 5 % 5
        if what == 0:
            return S.sched_bruteforce_argmin(p.handle, 0, p.n_mappings, ws, stream)
        if what == 1:
            return S.sched_bruteforce_argmin(p.handle, 1, p.n_mappings - 1, ws, stream)
        if what == 2:
            return S.sched_eval_reprobes(p.handle, k * 97 % p.n_mappings, ws, stream=stream)
        if what == 3:
            return [S.sched_eval_mappings(p.handle, idx[2 * (k % 5) + j], ws, stream).tolist()
                    for j in range(2)]
        return S.sched_eval_batch([handles[i] for i in small], rp, lat, ws, stream)

    ws = S.workspace(handles, len(rp))
    want = [call(k, ws, None) for k in range(25)]
    # (workspaces and streams are made here: the threads only call)
    spaces = [S.workspace(handles, len(rp)) for _ in range(THREADS)]
    streams = [torch.cuda.Stream() for _ in range(THREADS)]
    torch.cuda.synchronize()
    wrong, failed, start = [], [], threading.Barrier(THREADS)

    def work(t):
        try:
            start.wait(timeout=60)
            for r in range(ROUNDS):
                for j in range(25):
                    k = (j * 7 + t * 3 + r) % 25
                    if call(k, spaces[t], streams[t]) != want[k]:
                        wrong.append((t, r, k))
        except Exception as e:  # (reported below, on the test's own thread)
            failed.append((t, repr(e)))

    print(f"{THREADS} threads, {ROUNDS} rounds of 25 calls", flush=True)
    threads = [threading.Thread(target=work, args=(t,)) for t in range(THREADS)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed and not wrong, (failed[:3], wrong[:10])


def test_batch_of_more_replicas_than_a_slot_holds():
    inst = synth.random_instance(9820, 6, "permuted", tight=True)
    P = S.Problem.from_instance(inst)
    R = 2500  # (2,048 results fit a slot)
    lat = [synth.perturb(inst["tools"], r % 61) for r in range(R)]
    ws = S.workspace([P.handle], R)
    print(f"batch of {R} replicas", flush=True)
    got = S.sched_eval_batch([P.handle], [0] * R, lat, ws)
    want = []
    for r in range(61):
        Q = S.Problem.from_instance(dict(inst, tools=[x + [t[4]] for x, t in zip(lat[r], inst["tools"])]))
        want.append(S.sched_bruteforce_argmin(Q.handle, 0, Q.n_mappings, ws))
    assert got == [want[r % 61] for r in range(R)]
