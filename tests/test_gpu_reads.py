"""Reads of fields through the pinned staging buffers: sizes that leave a last word and a short chunk, sizes
for one and for several copying threads, several threads reading at once, and reads behind queued steps on
streams of the caller's."""

import threading

import numpy as np
import pytest

from paper_1902_09813_amd import btrt, btrt3
from paper_1902_09813_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [(1, 1), (3, 5), (257, 255), (511, 511), (513, 513), (1021, 1027), (1500, 1999)], ids=lambda s: f"{s[0]}x{s[1]}")
def test_field_at_step_zero_is_phi0(size):
    # At step 0 phi is phi0 exactly (k0 = K2 = 1 in FP64), so the read itself is checked.
    print(f"[gpu] read {size}", flush=True)
    w = W.c3().scaled(*size, 0)
    phi0 = np.random.default_rng(3).random((size[1], size[0]))
    with btrt.Solver(btrt.problem_from_workload(w), phi0) as s:
        for _ in range(3):
            assert np.array_equal(s.field(), phi0)


def test_concurrent_reads():
    rng = np.random.default_rng(4)
    w = W.c3().scaled(1024, 1536, 0)
    phi0 = [rng.random((1536, 1024)) for _ in range(4)]
    bad = []

    def work(k):
        with btrt.Solver(btrt.problem_from_workload(w), phi0[k]) as s:
            for _ in range(8):
                if not np.array_equal(s.field(), phi0[k]):
                    bad.append(k)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad


PER_THREAD = 2  # hipStreamPerThread: another stream in each thread


def _on(stream, problem):
    problem.grid.stream = stream
    return problem


@pytest.mark.parametrize("stream", ["per_thread", "torch"])
def test_reads_behind_queued_steps_on_a_callers_stream(stream):
    # Fields of 2 MB and more are read by several threads: every share must come after the steps and the
    # gather that the calling thread has just queued. The buffer they pass through holds another field
    # (of an earlier read), so a share that runs ahead shows.
    import torch

    print(f"[gpu] reads on a caller's stream: {stream}", flush=True)
    own = torch.cuda.Stream()
    handle = PER_THREAD if stream == "per_thread" else own.cuda_stream
    w = W.c3().scaled(1200, 1100, 0)
    want = []
    with btrt.Solver(btrt.problem_from_workload(w), w.phi0()) as s:
        for _ in range(3):
            want.append(s.step(200).field())
    with btrt.Solver(_on(handle, btrt.problem_from_workload(w)), w.phi0()) as s:
        for v in want:
            assert np.array_equal(s.step(200).field(), v)
    with btrt.Batch([(btrt.problem_from_workload(w), w.phi0())], stream=handle) as b:
        for v in want:
            assert np.array_equal(b.step(200).field(0), v)
    w3 = W.d3_nonlinear(96, 80, 70)
    with btrt3.Solver3(btrt3.problem_from_workload3(w3), w3.phi0()) as s:
        want3 = [s.step(60).field() for _ in range(2)]
    with btrt3.Solver3(_on(handle, btrt3.problem_from_workload3(w3)), w3.phi0()) as s:
        for v in want3:
            assert np.array_equal(s.step(60).field(), v)
