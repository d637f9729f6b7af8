"""Batches on regions (strip_rows 0): the bits of the same instances solved one step at a time.

Instances smaller than a region on one or both axes, of a region's size and a little more, with walls on
both, one or no axis, with and without a source and phi-dependent diffusion, beside an instance with
K2 != 1 (populations, a launch of its own); every step count per launch, a persistent grid, graph replays
and a remainder.
"""
import numpy as np
import pytest

from paper_1902_09813_amd import btrt

pytestmark = pytest.mark.gpu

PER, DIR = btrt.PERIODIC, btrt.DIRICHLET
SIDES = [(DIR,) * 4, (PER,) * 4, (DIR, DIR, PER, PER), (PER, PER, DIR, DIR)]
SIZES = [(1, 1), (1, 70), (70, 1), (33, 20), (64, 32), (65, 33), (50, 50), (63, 130), (128, 97), (257, 200)]


def _problems(precision, mixed):
    out = []
    for i, (nx, ny) in enumerate(SIZES * 2):
        rng = np.random.default_rng(i)
        kw = dict(flux_a=(0.02, -0.01), A0=(0.02, 0.003, 0.01), precision=precision)
        bc = SIDES[(i + i // len(SIZES)) % 4]
        if bc != (PER,) * 4:
            kw.update(bc_type=bc, bc_value=(0.1, 0.4, 0.2, 0.3))
        if i % 2:
            kw.update(source=("sin", 1e-3, 1, 2))
        if i % 3 == 0:
            kw.update(flux_b=(0.05, 0.02), beta=1.0)
        if mixed and i == 5:
            kw.update(k2=1.1)
        out.append((btrt.Problem(nx, ny, **kw), rng.random((ny, nx))))
    return out


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("precision", [btrt.F64, btrt.F32])
def test_batch_regions_keep_the_bits(precision, mixed):
    probs = _problems(precision, mixed)
    want = []
    for p, phi0 in probs:
        with btrt.Solver(p, phi0) as s:
            s.set_launch(1)
            s.step(40)
            want.append(s.field())
    for config in ((2, 0, 0, 0), (4, 0, 0, 0), (6, 0, 2, 0), (7, 1, 0, 0), (7, 0, 2, 0)):
        with btrt.Batch(probs) as b:
            b.set_config(*config)
            b.step(3).step(1).step(36)
            for i, w in enumerate(want):
                assert np.array_equal(b.field(i), w), (config, i)
