"""Two streams (the default of several instances) against one, for calls that
start on a lone check step and go on through further ones: their fields and
check records must agree."""
import numpy as np
import pytest

import workloads as W
from paper_2010_01847_amd import Lattice, instance_from_case
from parity_util import log

pytestmark = pytest.mark.gpu

CHANNEL = dict(bc_x="gradient", bc_y="diffuse", grad_x=2e-3)


@pytest.mark.parametrize("storage,rounding", [("f32", "nearest"), ("f16", "stochastic")])
@pytest.mark.parametrize("sizes", [((300, 200), (310, 150), (64, 64)), ((20, 20), (31, 9), (25, 33), (5, 7)),
                                   ((1500, 1100), (900, 1000))])
@pytest.mark.parametrize("check,calls", [(2, (1, 8, 7, 9, 1, 6)), (5, (4, 11, 4, 16))])
def test_two_streams_match_one(storage, rounding, sizes, check, calls):
    cases = [W.Case("streams", nx, ny, 0.6, 7.0, **(CHANNEL if k % 2 else {})) for k, (nx, ny) in enumerate(sizes)]
    fields = [W.random_field(c.nx, c.ny, 0.01, 1.0, 5 + k) - c.grad_x * np.arange(c.nx)[None, :]
              for k, c in enumerate(cases)]
    got = []
    for streams in (1, 2):
        lat = Lattice([instance_from_case(c, 2.0 ** -19 if storage == "f16" else 0.0) for c in cases], storage=storage,
                      rounding=rounding, check_interval=check, seed=3)
        lat.set_streams(streams)
        for k, f in enumerate(fields):
            lat.init(k, f)
        out = []
        for n in calls:
            lat.step(n)
            for k in range(len(cases)):
                out.append(lat.moments(k))
                if lat.steps >= check:
                    r = lat.last_check(k)
                    out.append((r["step"], r["residual"], r["totals"]))
        lat.close()
        got.append(out)
    # the streams launch the same kernels on the same tiles: the same bits
    for a, b in zip(*got):
        assert all(np.array_equal(u, v) for u, v in zip(a, b))
    log(f"{len(sizes)} instances, {storage}, check {check}: two streams equal one")
