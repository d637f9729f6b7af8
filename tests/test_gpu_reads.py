"""Reads of fields through the pinned staging buffers: sizes that leave a last word and a short chunk, sizes
for one and for several copying threads, and several threads reading at once."""

import threading

import numpy as np
import pytest

from paper_1902_09813_amd import btrt
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
