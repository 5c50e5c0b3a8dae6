"""Handles in the block kernels around the rules that choose a launch: few steps
and check steps by the marching kernel or single steps, states before the last
step stored or replayed by a readout, every window shape and layout.  Whatever
is chosen, the fields equal single steps bit for bit."""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2010_01847_amd import Lattice, instance_from_case
from parity_util import log

pytestmark = pytest.mark.gpu

WALLS = dict(bc_x="isothermal", t_wall=(1.004, 0.997, 0, 0))
CHANNEL = dict(bc_x="gradient", bc_y="diffuse", grad_x=2e-3)
FLUX = dict(bc_y="heatflux", q_wall=(0, 0, 1e-3, -4e-4))
# calls that end on steps 1, 3, 10 (a check step), 19 (the snapshot step before
# one), 20, 22, 25, 29 (a snapshot step again), 30 and 61
STEPS = (1, 2, 7, 9, 1, 2, 3, 4, 1, 31)
# (nx, ny, walls, storage, rounding, every step, layout)
CASES = [
    # with the marching kernel beside the block kernels, the state before a
    # call's last step stored (first two) and not
    (1500, 1400, CHANNEL, "f32", "nearest", False, "auto"), (1500, 1100, FLUX, "f16", "stochastic", True, "auto"),
    (2048, 2000, FLUX, "f32", "stochastic", False, "auto"), (2000, 2051, WALLS, "f32", "nearest", False, "auto"),
    (2100, 2040, {}, "bf16_split", "nearest", True, "auto"), (1999, 2003, CHANNEL, "f16", "nearest", True, "auto"),
    # single steps up to a check step
    (1000, 1003, FLUX, "f32", "stochastic", False, "auto"),
    # the planes layout: whole lattice, window in LDS, tile
    (30, 20, CHANNEL, "f32", "nearest", False, "planes"), (131, 67, FLUX, "bf16", "stochastic", False, "planes"),
    (401, 301, WALLS, "f16", "nearest", False, "planes"), (801, 777, {}, "f32", "stochastic", False, "planes"),
    # the largest whole lattice of one node per thread (of two: test_many_small_lattices)
    (32, 32, WALLS, "f32", "nearest", False, "auto"),
    # windows of 28 x 28, 32 x 24 and 24 x 24
    (1189, 4, CHANNEL, "f32", "nearest", False, "auto"), (13, 9651, {}, "f16", "stochastic", False, "auto"),
    (4758, 4, WALLS, "f32", "stochastic", False, "auto"), (9, 16408, FLUX, "f32", "nearest", False, "auto"),
]


def _start(case, seed):
    ramp = case.grad_x * np.arange(case.nx)[None, :]
    T = W.random_field(case.nx, case.ny, 0.01, 1.0, seed) - ramp
    return tuple(torch.from_numpy(np.ascontiguousarray(a)).cuda()
                 for a in (T, *W.random_flux(case.nx, case.ny, 1e-3, seed + 1)))


def _run(cases, fields, single, storage, rounding, every, layout, schedule, shown, check=10, steps=STEPS):
    lat = Lattice([instance_from_case(c, 2.0 ** -19 if storage.startswith("f16") else 0.0) for c in cases],
                  storage=storage, check_interval=check, rounding=rounding, seed=9, layout=layout,
                  every_step=every)
    if single:
        lat.set_step_fusion(1)
    if schedule:
        lat.set_schedule(schedule)
    for k, (c, f) in enumerate(zip(cases, fields)):
        lat.init(k, *f)
        for w in range(4):
            if c.q_wall[w]:
                lat.set_wall_flux(k, w, c.q_wall[w])
    out = []
    for n in steps:
        lat.step(n)
        for k in shown:
            fields_k, again = lat.moments_device(k), lat.moments_device(k)
            assert all(torch.equal(a, b) for a, b in zip(fields_k, again))
            out.append((fields_k, lat.last_check(k) if check > 0 and lat.steps >= check else None))
    lat.close()
    return out


def _same(a, b, what):
    for (u, c), (v, d) in zip(a, b):
        assert all(torch.equal(p, q) for p, q in zip(u, v)), what
        if c is not None:
            # up to the order of their FP64 summation
            assert c["step"] == d["step"], what
            assert c["residual"] == pytest.approx(d["residual"], rel=1e-12, abs=1e-300), what
            assert c["totals"] == pytest.approx(d["totals"], rel=1e-12, abs=1e-10), what


@pytest.mark.parametrize("nx,ny,kw,storage,rounding,every,layout", CASES,
                         ids=[f"{c[0]}x{c[1]}-{c[3]}-{c[4]}-{c[6]}" for c in CASES])
def test_routes_bitwise(nx, ny, kw, storage, rounding, every, layout):
    cases = [W.Case("routes", nx, ny, 0.6, 7.0, **kw)]
    fields = [_start(cases[0], 31)]
    args = (storage, rounding, every, layout)
    ref = _run(cases, fields, True, *args, None, [0])
    _same(_run(cases, fields, False, *args, None, [0]), ref, "eager")
    _same(_run(cases, fields, False, *args, "graph", [0]), ref, "graph")
    log(f"routes of {nx}x{ny} {storage} {rounding} {layout}: same bits")


@pytest.mark.parametrize("n,nx,ny", [(2500, 20, 20), (600, 64, 32)])
def test_many_small_lattices(n, nx, ny):
    """Whole lattices of one and two nodes per thread: states of short launches
    replayed (of the first handle), of long ones stored; on two streams."""
    cases = [W.Case("many", nx - k % 3, ny - k % 4, 0.6, 7.0, **(FLUX if k % 2 else {})) for k in range(n)]
    base = {}
    fields = [base.setdefault((c.nx, c.ny), _start(c, 41)) for c in cases]
    args = ("f32", "nearest", False, "auto", None, [0, 1, n // 2 - 1, n // 2, n - 1])
    for check, steps in ((10, (7, 13, 2, 4, 40)), (-1, (7, 5, 60))):
        _same(_run(cases, fields, False, *args, check=check, steps=steps),
              _run(cases, fields, True, *args, check=check, steps=steps), f"check {check}")
