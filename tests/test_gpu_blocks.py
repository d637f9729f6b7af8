"""Automatic shapes on small grids (several steps per launch on regions of one node per thread): the bits
of one step per launch in the population form, at sizes around the output tiles, for every kind of
boundary, source and A, every storage format and the general node model, with step counts that end in a
shorter launch. (The moment form's automatic shapes are compared in test_gpu_moments.py.)
"""
import dataclasses
import sys

import numpy as np
import pytest

from paper_1902_09813_amd import btrt
from paper_1902_09813_amd import workloads as W

pytestmark = pytest.mark.gpu

BCS = [(0, 0, 0, 0), (1, 1, 1, 1), (0, 0, 1, 1), (1, 1, 0, 0)]
SIZES = [(1, 1), (3, 9), (4, 40), (17, 16), (64, 64), (131, 97), (401, 300)]


def case(nx, ny, bc, k0, k2, **kw):
    return W.Workload(f"block_{nx}x{ny}", nx, ny, 0, flux_a=(0.03, -0.02), flux_b=(0.04, 0.01), A0=(0.02, 0.006, 0.012),
                      bc_type=bc, bc_value=tuple(0.2 * (q + 1) * t for q, t in enumerate(bc)), k0=k0, k2=k2, seed=5,
                      phi0_kind="uniform", **kw)


def compare(w, precision, steps, walls=None):
    out = []
    for shape in [(1, 4, 0, 0), (0, 0, 0, 0)]:
        with btrt.Solver(btrt.problem_from_workload(w, precision=precision), w.phi0()) as s:
            if walls is not None:
                s.set_walls(walls)
            s.set_launch(*shape)
            if shape[0] == 0:
                assert s.launch() == (1, 4, 0, 0)  # the nearest the public shapes have
                sweep = s.sweep()
                assert sweep["kernel"] == btrt.SWEEP_BLOCKS and sweep["steps_per_launch"] > 1
                assert sweep["moments"] == (w.k0 == 1.0 and w.k2 == 1.0)
            s.step(steps - 4).step(4)
            out.append((s.populations(), s.field()))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1]), (w.name, precision)


@pytest.mark.parametrize("bc", BCS, ids=lambda b: "".join(map(str, b)))
@pytest.mark.parametrize("size", SIZES, ids=lambda s: f"{s[0]}x{s[1]}")
def test_automatic_small_grids_bitwise(size, bc):
    print(f"[gpu] blocks {size} bc={bc}", flush=True)
    sys.stdout.flush()
    nx, ny = size
    rng = np.random.default_rng(nx + ny)
    rates = (0.8, 1.3, 0.5, 1.2)
    for precision in (btrt.F64, btrt.F32, btrt.F16DEV):
        compare(case(nx, ny, bc, 1.0, rates, source=("sin", 0.003, 1, 2)), precision, 24)
        compare(case(nx, ny, bc, 0.9, rates, beta=0.7), precision, 23)
    field = np.zeros((ny, nx, 3))
    field[..., 0], field[..., 2] = rng.uniform(0.01, 0.05, (2, ny, nx))
    S = 1e-3 * rng.standard_normal((ny, nx))
    compare(case(nx, ny, bc, 1.0, rates, source=("field", S, -1e-3), A0_field=field), btrt.F64, 25)


@pytest.mark.parametrize("k2", [1.0, "hbb"])
def test_general_model_small_grids_bitwise(k2):
    for n in (5, 13, 40):
        w = dataclasses.replace(W.bfe(n=n), k2=k2)
        print(f"[gpu] blocks, general model {w.nx}x{w.ny} k2={k2}", flush=True)
        for precision in (btrt.F64, btrt.F32):
            compare(w, precision, 23, btrt.wall_schedule(w, 0, 23))
