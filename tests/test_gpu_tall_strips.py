"""Large 16-bit handles march strips of 64 rows instead of 32, small ones of 16:
the split of the work changes no field bits.  A lattice of many strips whose field repeats along
y must stay equal, period by period, to one period of it."""
import pytest
import torch

import workloads as W
from paper_2010_01847_amd import Lattice, instance_from_case
from parity_util import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f16", "bf16", "f16_split"])
@pytest.mark.parametrize("kw", [{}, dict(bc_x="isothermal", t_wall=(1.004, 0.997, 0, 0))])
def test_periods_of_a_tall_lattice(storage, kw):
    # 2 strips x 7688 chunks of 64 rows (the last one half full); one period of
    # 1000 rows ends inside a chunk of either kind
    nx, ny, m = 59, 1000, 492
    T = torch.from_numpy(W.random_field(nx, ny, 1e-3, 1.0, 7)).cuda()
    got = []
    for reps in (1, 40, 44, m):     # 126, 5000 and 5500 strips of 16 rows: 16, 16 and 32 rows
        c = W.Case("tall", nx, ny * reps, 0.6, 7.0, **kw)
        lat = Lattice([instance_from_case(c, 2.0 ** -19)], storage=storage, check_interval=0)
        lat.set_step_fusion(6)
        lat.init(0, T.repeat(reps, 1))
        out = []
        for n in (6, 5, 13, 2):
            lat.step(n)
            out.append([t.view(reps, ny, nx) for t in lat.moments_device(0)])
        lat.close()
        got.append(out)
    for other in got[1:]:
        for one, many in zip(got[0], other):
            assert all(torch.equal(a.expand_as(b), b) for a, b in zip(one, many))
    log(f"{m} periods in {storage}: equal to one")


@pytest.mark.parametrize("order", [(6, 2, 6), (3, 6, 4)])
def test_changing_the_steps_per_launch(order):
    # fewer steps per launch go back to strips of 32 rows, between calls and
    # with a readout of the launch before pending; rounding to nearest, FP32
    # between, so a run is fixed by its launches alone
    nx, ny, m = 59, 1000, 492
    T = torch.from_numpy(W.random_field(nx, ny, 1e-3, 1.0, 8)).cuda()
    got = []
    for reps in (1, m):
        lat = Lattice([instance_from_case(W.Case("tall", nx, ny * reps, 0.6, 7.0), 2.0 ** -19)], storage="f16",
                      check_interval=0)
        lat.init(0, T.repeat(reps, 1))
        out = []
        for k in order:
            lat.set_step_fusion(k)
            lat.step(12)
            lat.set_step_fusion(5)
            out.append([t.view(reps, ny, nx) for t in lat.moments_device(0)])
        lat.close()
        got.append(out)
    for one, many in zip(*got):
        assert all(torch.equal(a.expand_as(b), b) for a, b in zip(one, many))


@pytest.mark.parametrize("storage", ["f16", "bf16_split"])
def test_strips_of_24_rows(storage):
    # 2 strips x 1875 chunks of 24 rows; one period runs in strips of 16
    nx, ny, m = 59, 1000, 45
    T = torch.from_numpy(W.random_field(nx, ny, 1e-3, 1.0, 9)).cuda()
    got = []
    for reps in (1, m, m + 40):     # 126, 5626 and 10626 strips of 16 rows: 16, 24 and 32 rows
        lat = Lattice([instance_from_case(W.Case("mid", nx, ny * reps, 0.6, 7.0), 2.0 ** -19)], storage=storage,
                      check_interval=0)
        lat.set_step_fusion(6)
        lat.init(0, T.repeat(reps, 1))
        out = []
        for n in (6, 5, 13, 2):
            lat.step(n)
            out.append([t.view(reps, ny, nx) for t in lat.moments_device(0)])
        lat.close()
        got.append(out)
    for other in got[1:]:
        for one, many in zip(got[0], other):
            assert all(torch.equal(a.expand_as(b), b) for a, b in zip(one, many))
