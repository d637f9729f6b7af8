"""One D3Q19 step per launch against the oracle, at the widths where the lanes of a row change.

A row takes whole 128-byte lines of lanes (16 nodes in FP64, 32 in FP32), a wavefront covers several rows
of a narrow box, and its last workgroup of a plane is ragged; faces on none, some and all sides, so a
wavefront holds interior, wrapped and bounced links at once. The automatic shape of a large box with
faces takes the same launches, also for odd counts.
"""
import numpy as np
import pytest

from paper_1902_09813_amd import btrt, btrt3
from paper_1902_09813_amd import workloads as W
from tests._cases import normwise, run_oracle3

pytestmark = pytest.mark.gpu

SIZES = [(1, 1, 1), (1, 9, 2), (15, 5, 3), (16, 17, 2), (17, 16, 3), (31, 3, 5), (33, 8, 4), (65, 5, 2), (129, 3, 3)]
FACES = [(0,) * 6, (1, 1, 0, 0, 0, 0), (0, 0, 1, 1, 0, 0), (0, 0, 0, 0, 1, 1), (1,) * 6]


def _box(size, bc, steps):
    nx, ny, nz = size
    rng = np.random.default_rng(nx + 7 * ny + 31 * nz)
    return W.Workload3("step", nx, ny, nz, steps, flux_a=(0.02, -0.03, 0.01), flux_b=(0.01, 0.0, 0.02),
                       A0=(0.04, 0.005, 0.0, 0.03, -0.004, 0.05), beta=0.3, bc_type=bc,
                       source=1e-3 * rng.standard_normal((nz, ny, nx)),
                       bc_value=(0.3, 0.1, 0.7, 0.2, 0.5, 0.4), k2=1.1, k0=0.9, phi0_array=rng.random((nz, ny, nx)))


# 12 steps of some 100 operations: 1e-12 in FP64 leaves a thousand roundings, 1e-5 in FP32 a hundred.
@pytest.mark.parametrize("precision,tol", [(btrt.F64, 1e-12), (btrt.F32, 1e-5)])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "x".join(map(str, s)))
def test_step_against_the_oracle(size, precision, tol):
    for bc in FACES:
        w = _box(size, bc, 12)
        with btrt3.Solver3(btrt3.problem_from_workload3(w, precision=precision), w.phi0()) as s:
            s.step(w.steps)
            f, phi = s.populations(), s.field()
        o = run_oracle3(w)
        assert normwise(phi, o.phi()) <= tol and normwise(f, o.f) <= tol, bc


@pytest.mark.parametrize("precision", [btrt.F64, btrt.F32])
def test_automatic_shape_with_faces_keeps_the_bits(precision):
    w = _box((131, 127, 129), (1, 1, 0, 0, 1, 1), 5)
    out = []
    for shape in ((0, 0, 0), (1, 0, 0), (2, 0, 0)):
        with btrt3.Solver3(btrt3.problem_from_workload3(w, precision=precision), w.phi0()) as s:
            s.set_launch(*shape)
            s.step(2).step(3)
            out.append((s.populations(), s.field()))
    for f, phi in out[1:]:
        assert np.array_equal(f, out[0][0]) and np.array_equal(phi, out[0][1])
