"""Automatic shapes above 10^5 nodes: several steps per launch on regions of 64 columns by R rows a wavefront.

Every launch shape gives the same bits, so the automatic one is held against one step per launch: grids
whose last region is nearly empty or full (widths around 64 - 2 k and 64, heights around the regions'), grids
narrower or lower than a region between walls, walls on one axis, a source, an A0 field, phi-dependent
diffusion and both 16-bit formats' FP32 moments; odd counts and calls that leave a remainder.
"""
import numpy as np
import pytest

from paper_1902_09813_amd import btrt

pytestmark = pytest.mark.gpu

PER, DIR = btrt.PERIODIC, btrt.DIRICHLET
SIDES = [(DIR,) * 4, (PER,) * 4, (DIR, DIR, PER, PER), (PER, PER, DIR, DIR)]
SIZES = [(317, 331), (64, 1700), (50, 2200), (65, 1601), (2500, 41), (20000, 6), (1030, 995), (402, 1120)]


def _run(nx, ny, bc, kind, precision, launch):
    rng = np.random.default_rng(nx + 3 * ny)
    kw = dict(flux_a=(0.02, -0.01), A0=(0.02, 0.003, 0.01))
    if bc != (PER,) * 4:
        kw.update(bc_type=bc, bc_value=(0.1, 0.4, 0.2, 0.3))
    if kind == "source":
        kw.update(source=("sin", 1e-3, 1, 2))
    if kind == "beta":
        kw.update(flux_b=(0.05, 0.02), beta=1.0)
    if kind == "field":
        a0 = np.zeros((ny, nx, 3))
        a0[..., 0] = 0.01 + 0.005 * rng.random((ny, nx))
        a0[..., 2] = 0.01
        kw.update(A0_field=a0, source=("field", 1e-4 * rng.random((ny, nx)), 1.0))
        del kw["A0"]
    p = btrt.Problem(nx, ny, precision=precision, **kw)
    with btrt.Solver(p, rng.random((ny, nx))) as s:
        s.set_launch(*launch)
        assert s.sweep()["kernel"] == (btrt.SWEEP_STEP if launch[0] else btrt.SWEEP_REGIONS)
        s.step(1).step(9).step(14)
        return s.field(), s.populations()


@pytest.mark.parametrize("precision", [btrt.F64, btrt.F32])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: f"{s[0]}x{s[1]}")
def test_regions_keep_the_bits(size, precision):
    for n, bc in enumerate(SIDES):
        kind = ("plain", "source", "beta", "field")[(n + size[0]) % 4]
        a = _run(*size, bc, kind, precision, (0,))
        b = _run(*size, bc, kind, precision, (1,))
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]), (bc, kind)


@pytest.mark.parametrize("precision", [btrt.F16DEV, btrt.BF16DEV])
def test_regions_of_the_16_bit_formats(precision):
    a = _run(701, 353, SIDES[0], "source", precision, (0,))
    b = _run(701, 353, SIDES[0], "source", precision, (1,))
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
