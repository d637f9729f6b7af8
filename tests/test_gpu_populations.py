"""The population kernels (any rates but k0 = K2 = 1, whose state is kept as moments) on the benchmark
workloads' sizes, with the rates K2 = (1.1, 0.9, 0.9, 1.2) in their place:

* grids of 2^20 nodes and more: the automatic and the single-round FP64 strips, the non-temporal one-step
  and two-step tile kernels of single grids and of batches, against each other bit for bit and against the
  oracle (FP64, 1e-12 normwise);
* an A0 field with a growing source through every walker against the oracle;
* batches whose members all hold populations, with separable and without sources, walls and K1 per node, at
  every step count per launch, persistent and replayed from graphs, against each instance alone;
* FP32 populations and the 16-bit encodings within stated bounds of the oracle, and the full 4096^2 and 1024^2
  workloads against the stored oracle results (FP64) and within the bounds stated for the formats there;
* checkpoints, wall schedules set on a plain problem, a caller's memory and stream beyond the cache;
* the two-step D3Q19 population kernel at its automatic shape, and a cyclic shift of its periodic box.
"""
import dataclasses
import sys

import numpy as np
import pytest

from paper_1902_09813_amd import btrt, btrt3
from paper_1902_09813_amd import workloads as W
from tests._cases import normwise, run_oracle
from tests.test_gpu_full_length import BOUNDS, NAMES, errors, load
from tests.test_gpu_lowprec import ERROR_CASES, FMT_ID, FORMATS, initial_bound
from tests.test_gpu_parity import FP32_CASES
from tests.test_gpu_variants import CASES as FIELD_CASES

pytestmark = pytest.mark.gpu

RATES = (1.1, 0.9, 0.9, 1.2)


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def with_rates(w):
    return dataclasses.replace(w, name=w.name + "_rates", k2=RATES)


def solver(w, precision=btrt.F64, **kw):
    return btrt.Solver(btrt.problem_from_workload(w, precision=precision), w.phi0(), **kw)


def walled(n):
    c3 = W.c3()
    return W.Workload(f"walled_{n}", n, n, 0, flux_b=c3.flux_b, A0=c3.A0, beta=c3.beta, bc_type=(1, 1, 1, 1),
                      bc_value=(0.2, -0.1, 0.5, 0.3), seed=11, phi0_kind="uniform")


@pytest.mark.parametrize("walls", [False, True], ids=["periodic", "walled"])
def test_large_grid_strips_bitwise_and_oracle(walls):
    w = with_rates(walled(2048) if walls else W.c3().scaled(2048, 2048, 0))
    steps = 15
    say(f"[gpu] populations {w.name} {w.nx}x{w.ny}, {steps} steps")
    with solver(w, torch_memory=True) as s:
        want = s.set_launch(1, 4, 1, 0).step(steps).populations()
    o = run_oracle(w, steps)
    assert normwise(want, o.f) <= 1e-12
    for shape in [(0, 0, 0, 0), (6, 0, 0, 0), (7, 0, 0, 0), (2, 0, 0, 1), (4, 32, 4, 0)]:
        with solver(w, torch_memory=True) as s:
            s.set_launch(*shape)
            if shape[0] >= 6:
                assert s.launch()[1] >= 64 and s.launch()[2] == 1, s.launch()  # one round over the resident slots
            assert np.array_equal(s.step(steps).populations(), want), shape


@pytest.mark.parametrize("precision", [btrt.F64, btrt.F32, btrt.F16DEV], ids=lambda p: NAMES[p])
def test_beyond_the_cache_shapes_agree(precision):
    # 168 to 671 MB in two copies of the state: above 256 MB the one-step and tile kernels store non-temporally.
    w = with_rates(W.c3().scaled(4096, 1024, 0))
    want = None
    for shape in [(1, 4, 0, 0), (1, 16, 0, 0), (2, 0, 0, 1), (4, 32, 4, 0), (7, 64, 1, 0), (0, 0, 0, 0)]:
        say(f"[gpu] populations beyond the cache {NAMES[precision]} {shape}")
        with solver(w, precision, torch_memory=True) as s:
            f = s.set_launch(*shape).step(9).populations()
        want = f if want is None else want
        assert np.array_equal(f, want), shape


def test_batch_beyond_the_cache():
    ws = [with_rates(dataclasses.replace(W.c3().scaled(1536, 1536, 0), seed=100 + k)) for k in range(4)]
    steps = 7
    alone = []
    for w in ws:
        with solver(w, btrt.F32) as s:
            alone.append(s.set_fusion(1).step(steps).field())
    for cfg in [(1, 0, 0), (2, 0, 0), (4, 0, 0), (7, 0, 0)]:
        say(f"[gpu] population batch of 4 x 1536^2 FP32, config {cfg}")
        with btrt.Batch([(btrt.problem_from_workload(w, precision=btrt.F32), w.phi0()) for w in ws]) as b:
            b.set_config(*cfg).step(steps)
            for i in range(b.n):
                assert np.array_equal(b.field(i), alone[i]), (cfg, i)


@pytest.mark.parametrize("w", FIELD_CASES, ids=lambda w: w.name)
def test_a0_field_walkers_against_the_oracle(w):
    w = with_rates(w)
    steps = 31
    say(f"[gpu] populations, A0 field {w.name} {w.nx}x{w.ny}")
    o = run_oracle(w, steps)
    for precision in (btrt.F64, btrt.F32, btrt.F16DEV):
        want = None
        for shape in [(1, 4, 0, 0), (0, 0, 0, 0), (2, 0, 0, 1)] + [(k, 16, 1, 0) for k in (2, 3, 4, 5, 6, 7)]:
            with solver(w, precision) as s:
                f = s.set_launch(*shape).step(steps).populations()
            if want is None:
                want = f
                if precision == btrt.F64:
                    assert normwise(f, o.f) <= 1e-12
            assert np.array_equal(f, want), (shape, precision)


@pytest.mark.parametrize("precision", [btrt.F64, btrt.F32], ids=["f64", "f32"])
def test_population_batches_equal_each_instance_alone(precision):
    ws = W.c4(count=14, seed=43, steps=0, side_range=(8, 150))
    ws[1].nx, ws[2].ny = max(1, ws[1].nx // 3), 1
    ws = [dataclasses.replace(w, k2=RATES, k0=1.0 if i % 3 else 0.9, beta=0.5 * (i % 2),
                              source=w.source if i % 4 else None) for i, w in enumerate(ws)]
    probs = [(btrt.problem_from_workload(w, precision=precision), w.phi0()) for w in ws]
    steps = 37
    alone = []
    for w in ws:
        with solver(w, precision) as s:
            alone.append(s.set_fusion(1).step(steps).field())
        if precision == btrt.F64:
            assert normwise(alone[-1], run_oracle(w, steps).phi()) <= 1e-12, w.name
    for cfg in [(1, 0, 0, 0), (2, 0, 0, 0), (2, 2, 4, 0), (4, 0, 0, 16), (4, 2, 4, 5), (6, 0, 2, 32), (7, 4, 0, 8),
                (7, 0, 2, 0)]:
        say(f"[gpu] population batch {cfg} precision {precision}")
        with btrt.Batch(probs) as b:
            b.set_config(*cfg).step(16)
            b.residual()
            b.step(steps - 16)
            for i in range(b.n):
                assert np.array_equal(b.field(i), alone[i]), (cfg, i)


# Stated FP32 and 16-bit bounds as for unit rates: the arithmetic and the encodings are the same.
@pytest.mark.parametrize("w,bound", FP32_CASES, ids=lambda v: getattr(v, "name", ""))
def test_fp32_populations_against_the_oracle(w, bound):
    for k2 in (RATES, "hbb") if w.A0[0] == w.A0[2] else (RATES,):
        v = dataclasses.replace(w, k2=k2)
        with solver(v, btrt.F32) as s:
            phi = s.step(v.steps).field()
        ref = run_oracle(v).phi()
        e = normwise(phi, ref), float(np.sqrt(np.sum((phi - ref) ** 2) / np.sum(ref ** 2)))
        say(f"[gpu] FP32 populations {w.name} k2={k2}: max {e[0]:.3e} l2 {e[1]:.3e}, bound {bound:.0e}")
        assert max(e) <= bound


@pytest.mark.parametrize("precision", FORMATS, ids=lambda p: FMT_ID[p])
@pytest.mark.parametrize("w,bounds", ERROR_CASES, ids=lambda v: getattr(v, "name", ""))
def test_16_bit_encoding_against_the_oracle(w, bounds, precision):
    v = with_rates(w)
    with solver(v, precision) as s:
        f0 = s.populations()
        phi = s.step(v.steps).field()
    if v.bc_type == (0,) * 4:  # f(0) = f_eq(phi0), encoded
        feq = run_oracle(v, 0).f
        assert np.all(np.abs(f0 - feq) <= initial_bound(feq, precision))
    ref = run_oracle(v).phi()
    e = normwise(phi, ref), float(np.sqrt(np.sum((phi - ref) ** 2) / np.sum(ref ** 2)))
    say(f"[gpu] {FMT_ID[precision]} {v.name}: max {e[0]:.3e} l2 {e[1]:.3e}, bound {bounds[precision]:.0e}")
    assert max(e) <= bounds[precision]
    with solver(v, precision) as s:  # splits and fused launches keep the encoded state's bits
        for k in (1, 0, 100, 56):
            s.step(k)
        split = s.populations()
    with solver(v, precision) as s:
        assert np.array_equal(s.set_fusion(1).step(157).populations(), split)


@pytest.mark.parametrize("name", ["c3", "c2"])
def test_full_length(name):
    # Rates a rounding away from 1 keep the populations and change nothing else: 3e-14 of the second moments in
    # FP64, nothing in the other formats. So the stored oracle results and the formats' stated bounds are those
    # of the unit rates.
    w = dataclasses.replace({"c3": W.c3, "c2": W.c2}[name](), k2=1.0 + 2.0 ** -45)
    say(f"[gpu] population full length {w.name} f64")
    _, z = load(w)
    st = int(z["stride"])
    with solver(w, torch_memory=True) as s:
        ref = s.step(w.steps).field()
    e = np.max(np.abs(ref[::st, ::st] - z["phi_sub"])) / np.max(np.abs(z["phi_sub"]))
    say(f"    f64 against the oracle, every {st}th node: normwise {e:.3e}")
    assert e <= 1e-12
    for (n, precision), bound in BOUNDS.items():
        if n != name:
            continue
        with solver(w, precision, torch_memory=True) as s:
            e = errors(s.step(w.steps).field(), ref)
        say(f"    {NAMES[precision]}: max {e[0]:.3e} L2 {e[1]:.3e} GRE {e[2]:.3e}; bounds {bound}")
        assert all(x <= b for x, b in zip(e, bound)), (precision, e)


@pytest.mark.parametrize("bc", [(0,) * 6, (1,) * 6], ids=["periodic", "faces"])
def test_two_step_d3q19_populations_at_the_automatic_shape(bc):
    w = W.d3_nonlinear(128, 128, 128, steps=5)
    w = dataclasses.replace(w, k2=1.1, bc_type=bc, bc_value=tuple(0.1 * (f + 1) * t for f, t in enumerate(bc)))
    want = None
    for shape in [(1, 0, 0), (0, 0, 0), (2, 0, 0)]:
        with btrt3.Solver3(btrt3.problem_from_workload3(w), w.phi0()) as s:
            s.set_launch(*shape)
            f = s.step(w.steps).populations()
        want = f if want is None else want
        assert np.array_equal(f, want), shape


@pytest.mark.parametrize("precision", [btrt.F64, btrt.F32] + FORMATS, ids=lambda p: NAMES[p])
def test_checkpoints_resume_bitwise(precision):
    w = W.Workload("ck_rates", 131, 70, 0, A0=(0.03, 0.006, 0.02), beta=0.5, flux_a=(0.03, -0.02), flux_b=(0.02, 0.0),
                   source=("sin", 2e-3, 1, 1), bc_type=(1, 1, 1, 1), bc_value=(0.2, 0.6, 0.4, 0.1), seed=21, k2=RATES)
    for n1 in (0, 37):
        with solver(w, precision) as a, solver(w, precision) as b, solver(w, precision) as ref:
            r = [s.set_launch(4, 16, 4, 0).step(n1).residual() for s in (a, ref)]
            b.set_launch(6, 32, 1, 0).restore(a.checkpoint())
            assert r[0] == r[1] and b.info().step == n1
            want = ref.step(53).populations()
            assert np.array_equal(b.step(53).populations(), want) and b.residual() == ref.residual()
    with solver(dataclasses.replace(w, k2=1.0), precision) as m, solver(w, precision) as p:  # the other form's state
        for x, y in ((m, p), (p, m)):
            with pytest.raises(btrt.BtrtError) as e:
                x.restore(y.checkpoint())
            assert e.value.code == btrt.E_INVAL


@pytest.mark.parametrize("precision", [btrt.F64, btrt.F32], ids=lambda p: NAMES[p])
def test_wall_schedules_on_a_plain_problem(precision):
    # A schedule turns a plain population problem to the general node model; split, resumed and in every shape.
    w = W.Workload("walls_table", 140, 90, 0, A0=(0.03, 0.0, 0.02), flux_a=(0.02, 0.01), bc_type=(1, 1, 0, 0),
                   bc_value=(0.1, 0.2, 0.0, 0.0), seed=3, k2=RATES)
    rows = np.random.default_rng(1).uniform(0.0, 1.0, (30, 4 * (140 + 90) + 4))
    w.walls = lambda k: rows[k]
    o = run_oracle(w, 30)
    want = None
    for shape in [(1, 0, 0, 0), (0, 0, 0, 0), (2, 0, 0, 1), (4, 16, 1, 0), (7, 8, 1, 0)]:
        with solver(w, precision) as s:
            s.set_launch(*shape).set_walls(rows[:12]).step(12)
            data = s.checkpoint()
        with solver(w, precision) as s:
            f = s.set_launch(*shape).restore(data).set_walls(rows[12:]).step(18).populations()
        if want is None:
            want = f
            if precision == btrt.F64:
                assert normwise(f, o.f) <= 1e-12
        assert np.array_equal(f, want), shape


def test_callers_memory_and_stream_beyond_the_cache():
    w = with_rates(W.c2().scaled(1400, 1300, 41))
    with solver(w) as a, solver(w, torch_memory=True) as b:
        assert np.array_equal(a.step(w.steps).field(), b.step(w.steps).field())


def test_shift_invariance_d3q19_populations():
    w = dataclasses.replace(W.d3_nonlinear(24, 19, 13, steps=9), k2=1.1)
    shift = (5, 11, 7)
    ws = dataclasses.replace(w, phi0_array=np.roll(w.phi0(), shift, axis=(0, 1, 2)))
    for launch in [(1, 0, 0), (2, 3, 1), (2, 0, 3), (2, 5, 4)]:
        with btrt3.Solver3(btrt3.problem_from_workload3(w), w.phi0()) as a, \
                btrt3.Solver3(btrt3.problem_from_workload3(ws), ws.phi0()) as b:
            fa = a.set_launch(*launch).step(w.steps).populations()
            fb = b.set_launch(*launch).step(w.steps).populations()
        assert np.array_equal(np.roll(fa, shift, axis=(1, 2, 3)), fb), launch
