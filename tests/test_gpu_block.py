"""Block kernels (several steps per launch of lattices held on the chip, the
default of small handles) against single steps, bit for bit: every step is
rounded as a stored one is and computed by the same functions, so the fields
must be equal, and the check records equal up to the order of their FP64
summation (1e-12, as for the fused kernel)."""
import numpy as np
import pytest

import workloads as W
from paper_2010_01847_amd import Lattice, instance_from_case
from parity_util import log

pytestmark = pytest.mark.gpu

# calls ending after 1, 3, 10 (a check step), 19 (the snapshot step before
# one), 20 (the lone check step) and 61 steps
STEPS = (1, 2, 7, 9, 1, 41)
WALLS = dict(bc_x="isothermal", t_wall=(1.004, 0.997, 0, 0))
CHANNEL = dict(bc_x="gradient", bc_y="diffuse", grad_x=2e-3)
FLUX = dict(bc_y="heatflux", q_wall=(0, 0, 1e-3, -4e-4))
SQUARE = dict(bc_x="isothermal", bc_y="isothermal", wall_bc=(0, 0, 0, "heatflux"), t_wall=(1.0, 1.0, 1.0, 0.0),
              q_wall=(0, 0, 0, 1e-3))
# whole lattices (one and two nodes per thread, and one node too many for
# each), windows in LDS, tiles in registers (chosen by size), and the largest
# handles that run in them; sides off every window edge
CASES = [
    (2, 2, {}, "f32", "nearest"), (64, 16, WALLS, "f32", "nearest"), (41, 25, SQUARE, "f32", "nearest"),
    (1024, 2, {}, "f16", "stochastic"), (683, 3, FLUX, "f16_split", "nearest"),
    (40, 33, CHANNEL, "bf16", "stochastic"), (2, 1025, CHANNEL, "f32", "nearest"),
    (131, 67, {}, "f32", "stochastic"), (129, 65, CHANNEL, "f32", "nearest"), (75, 103, SQUARE, "bf16", "nearest"),
    (98, 90, FLUX, "bf16_split", "nearest"), (20, 700, WALLS, "f16", "nearest"),
    (401, 301, CHANNEL, "f32", "nearest"), (333, 290, SQUARE, "f32", "nearest"), (700, 257, {}, "f16", "stochastic"),
    (1031, 259, FLUX, "f16_split", "stochastic"), (801, 777, WALLS, "f32", "nearest"), (1500, 1101, CHANNEL, "f32", "nearest"),
]


def _run(cases, fields, storage, rounding, single, schedule=None, steps=STEPS, check=10):
    lat = Lattice([instance_from_case(c, 2.0 ** -19 if storage.startswith("f16") else 0.0) for c in cases],
                  storage=storage, check_interval=check, rounding=rounding, seed=9)
    if single:
        lat.set_step_fusion(1)
    if schedule:
        lat.set_schedule(schedule)
    for k, (c, f) in enumerate(zip(cases, fields)):
        lat.init(k, *f)
        for w in range(4):
            if c.q_wall[w]:
                lat.set_wall_flux(k, w, c.q_wall[w])
    out, done = [], 0
    for n in steps:
        lat.step(n)
        done += n
        out.append([lat.moments(k) + ((lat.last_check(k) if done >= check else None), lat.totals(k))
                    for k in range(len(cases))])
    lat.close()
    return out


def _same(a, b, what):
    for x, y in zip(a, b):
        for (u, v) in zip(x, y):
            assert all(np.array_equal(p, q) for p, q in zip(u[:3], v[:3])), what
            assert np.allclose(u[4], v[4], rtol=1e-12, atol=1e-12), what
            if v[3] is not None:
                assert u[3]["step"] == v[3]["step"]
                assert u[3]["residual"] == pytest.approx(v[3]["residual"], rel=1e-12, abs=1e-300), what
                assert u[3]["totals"] == pytest.approx(v[3]["totals"], rel=1e-12, abs=1e-13), what


def _field(nx, ny, kw, seed):
    ramp = kw.get("grad_x", 0.0) * np.arange(nx)[None, :]
    return (W.random_field(nx, ny, 0.01, 1.0, seed) - ramp,) + tuple(W.random_flux(nx, ny, 1e-3, seed + 1))


@pytest.mark.parametrize("nx,ny,kw,storage,rounding", CASES, ids=[f"{c[0]}x{c[1]}-{c[3]}-{c[4]}" for c in CASES])
def test_block_kernels_bitwise(nx, ny, kw, storage, rounding):
    case = W.Case("block", nx, ny, 0.6, 7.0, **kw)
    T = [_field(nx, ny, kw, 71)]
    ref = _run([case], T, storage, rounding, True)
    _same(_run([case], T, storage, rounding, False), ref, "eager")
    _same(_run([case], T, storage, rounding, False, "graph"), ref, "graph")
    log(f"block kernels {nx}x{ny} {storage} {rounding}: same bits")


@pytest.mark.parametrize("side_lo,side_hi", [(5, 40), (30, 150)])
def test_block_kernels_batched(side_lo, side_hi):
    """Instances of uneven sides in one handle, on two streams and in graphs
    replayed several times; check steps off as well."""
    cases = W.knudsen_sweep(n_inst=7, seed=3, side_lo=side_lo, side_hi=side_hi)
    T = [_field(c.nx, c.ny, dict(grad_x=c.grad_x), 80 + k) for k, c in enumerate(cases)]
    ref = _run(cases, T, "f32", "stochastic", True)
    _same(_run(cases, T, "f32", "stochastic", False), ref, "eager")
    _same(_run(cases, T, "f32", "stochastic", False, "graph"), ref, "graph")
    a, b = (_run_unchecked(cases, T, single) for single in (True, False))
    for u, v in zip(a, b):
        assert all(np.array_equal(p, q) for p, q in zip(u, v))


def _run_unchecked(cases, fields, single):
    lat = Lattice([instance_from_case(c) for c in cases], check_interval=-1)
    if single:
        lat.set_step_fusion(1)
    for k, f in enumerate(fields):
        lat.init(k, *f)
    lat.step(29)
    out = [lat.moments(k) for k in range(len(cases))]
    lat.close()
    return out


def test_wall_flux_after_a_block_launch():
    """A heat-flux change after a call applies to later steps only; readouts of
    the current time keep the flux its last step ran with."""
    case = W.Case("flux", 131, 37, 0.6, 7.0, **FLUX)
    T = _field(131, 37, {}, 5)
    outs = []
    for single in (True, False):
        lat = Lattice([instance_from_case(case)], check_interval=10)
        if single:
            lat.set_step_fusion(1)
        lat.init(0, *T)
        got = []
        for n, q in ((7, 2e-3), (11, -1e-3), (5, 5e-4), (6, 0.0)):
            lat.step(n)
            lat.set_wall_flux(0, 2, q)
            got.append(lat.moments(0))
        lat.close()
        outs.append(got)
    for a, b in zip(*outs):
        assert all(np.array_equal(u, v) for u, v in zip(a, b))
