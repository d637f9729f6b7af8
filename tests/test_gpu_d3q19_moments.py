"""The moment form of the D3Q19 sweep (k0 = 1, K2 = 1): against the oracle (FP64, 1e-12 normwise) and
bit for bit between one and two steps per launch and chunk heights, around the tile sizes (62 x 6
output columns with one step per launch, 60 x 12 with two), for boxes thinner than a tile, on every
kind of boundary (edges and corners of the box with unequal face values), with and without a source.
"""
import dataclasses
import sys

import numpy as np
import pytest

from paper_1902_09813_amd import btrt, btrt3
from paper_1902_09813_amd import workloads as W
from tests._cases import normwise, run_oracle3
from tests._paper3 import C3

pytestmark = pytest.mark.gpu

BCS = [(0, 0, 0, 0, 0, 0), (1, 1, 1, 1, 1, 1), (1, 1, 0, 0, 0, 0), (0, 0, 1, 1, 0, 0), (0, 0, 0, 0, 1, 1)]
SIZES = [(1, 1, 1), (2, 7, 3), (60, 12, 4), (61, 13, 5), (63, 6, 2), (124, 5, 9)]


def box(nx, ny, nz, bc, source, beta):
    rng = np.random.default_rng(nx + 3 * ny + 5 * nz)
    return W.Workload3(f"mom3_{nx}x{ny}x{nz}", nx, ny, nz, 9, flux_a=(0.02, -0.01, 0.015), flux_b=(0.03, 0.01, -0.02),
                       A0=(0.05, 0.01, 0.005, 0.04, -0.008, 0.03), beta=beta,
                       source=1e-3 * rng.standard_normal((nz, ny, nx)) if source else None, bc_type=bc,
                       bc_value=tuple(0.15 * (f + 1) * t for f, t in enumerate(bc)), phi0_array=rng.random((nz, ny, nx)))


@pytest.mark.parametrize("bc", BCS, ids=lambda b: "".join(map(str, b)))
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "x".join(map(str, s)))
def test_shapes_against_one_step_and_the_oracle(size, bc):
    for source, beta in [(False, 0.0), (True, 0.6)]:
        w = box(*size, bc, source, beta)
        print(f"[gpu] d3q19 moments {w.name} bc={bc} source={source}", flush=True)
        sys.stdout.flush()
        o = run_oracle3(w)
        for precision in (btrt.F64, btrt.F32):
            want = None
            for shape in [(1, 0, 0), (0, 0, 0), (2, 0, 0), (2, 1, 2), (2, 3, 4)]:
                with btrt3.Solver3(btrt3.problem_from_workload3(w, precision=precision), w.phi0()) as s:
                    s.set_launch(*shape)
                    f0 = s.populations()
                    s.step(w.steps)
                    got = (f0, s.populations(), s.field())
                if want is None:
                    want = got
                    if precision == btrt.F64:
                        assert normwise(got[0], run_oracle3(w, 0).f) <= 1e-15
                        assert normwise(got[1], o.f) <= 1e-12 and normwise(got[2], o.phi()) <= 1e-12
                assert all(np.array_equal(x, y) for x, y in zip(got, want)), (shape, precision)


@pytest.mark.parametrize("precision,u", [(btrt.F32, 2.0 ** -24), (btrt.F64, 2.0 ** -53)])
def test_initial_state_is_rounded_once(precision, u):
    # As in two dimensions (flux coefficients that FP32 holds exactly).
    c = np.rint(C3).astype(int)
    rng = np.random.default_rng(2)
    phi0 = rng.random((30, 31, 33))
    a, b = (0.03125, -0.015625, 0.0078125), (0.0625, 0.03125, -0.046875)
    with btrt3.Solver3(btrt3.Problem3(33, 31, 30, flux_a=a, flux_b=b, A0=(0.05, 0.01, 0.005, 0.04, -0.008, 0.03),
                                      precision=precision), phi0) as s:
        phi, f = s.field(), s.populations()
    assert np.array_equal(phi, phi0 if precision == btrt.F64 else phi0.astype(np.float32).astype(np.float64))
    p = phi0.astype(np.longdouble)
    B = [p * (a[k] + 0.5 * b[k] * p) for k in range(3)]
    ops = 8 if precision == btrt.F64 else 1.0001
    for i in range(19):
        wt = np.longdouble(1) / (3, 18, 36)[int(np.sum(np.abs(c[i])))]
        feq = wt * (p + 3 * sum(int(c[i][k]) * B[k] for k in range(3)))
        bound = ops * u * (wt * (np.abs(p) + 3 * sum(np.abs(c[i][k] * B[k]) for k in range(3))) + np.abs(feq))
        assert np.all(np.abs(f[i] - feq) <= bound), (i, precision)


@pytest.mark.parametrize("precision,scale,tol", [(btrt.F32, 1e14, 1e-5), (btrt.F64, 1e104, 1e-12)])
def test_determinant_beyond_the_range(precision, scale, tol):
    # det M overflows (3e38, 1.8e308) while M and its cofactors do not: 1/det M is 0 as a division gives it.
    # The oracle runs the diffusion tensor scaled down by what keeps K1 below one rounding of everything else.
    def run(factor):
        w = box(33, 20, 9, (0,) * 6, False, 0.5)
        w.A0 = tuple(factor * v for v in w.A0)
        return w
    want = run_oracle3(run(min(scale, 1e80))).phi()
    w = run(scale)
    for shape in [(1, 0, 0), (2, 0, 0)]:
        with btrt3.Solver3(btrt3.problem_from_workload3(w, precision=precision), w.phi0()) as s:
            s.set_launch(*shape)
            phi = s.step(w.steps).field()
        assert normwise(phi, want) <= tol, shape


def test_reported_shape_is_the_one_that_runs():
    # A shape read from one handle and set on another is the shape the first one runs: two steps per launch
    # only where the automatic choice takes them.
    for w, k in [(W.d3_nonlinear(104, 104, 100, steps=5), 2), (W.d3_nonlinear(60, 60, 60, steps=5), 1),
                 (box(128, 128, 128, (1,) * 6, False, 0.0), 1), (dataclasses.replace(box(128, 128, 128, (0, 0, 1, 1, 0, 0),
                                                                                   False, 0.0), k2=1.1), 1),
                 (dataclasses.replace(W.d3_nonlinear(128, 128, 128, steps=5), k2=1.1), 2),
                 (dataclasses.replace(W.d3_nonlinear(104, 104, 100, steps=5), k2=1.1), 1)]:
        with btrt3.Solver3(btrt3.problem_from_workload3(w), w.phi0()) as s:
            shape = s.launch()
            assert shape[0] == k, (w.name, shape)
            want = s.step(5).populations()
        with btrt3.Solver3(btrt3.problem_from_workload3(w), w.phi0()) as s:
            s.set_launch(*shape)
            assert s.launch() == shape
            assert np.array_equal(s.step(5).populations(), want)
