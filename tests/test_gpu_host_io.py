"""Host fields of small instances go through pinned memory that the kernels
access, larger ones through device staging, and device fields through neither:
all must give the same bits.  So must the first FP64 readout of 16-bit storage
after a fused launch, which the replaying launch itself writes."""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2010_01847_amd import Lattice, instance_from_case
from paper_2010_01847_amd.lbm import lbm_moments_f64
from parity_util import log

pytestmark = pytest.mark.gpu

FLUX = dict(bc_y="heatflux", q_wall=(0, 0, 1e-3, -4e-4))
# three FP64 fields of 43 690 nodes are the largest below the line of 1 MiB
SIZES = [((2, 2), (401, 3)), ((257, 170), (210, 209)), ((300, 301), (17, 9))]


@pytest.mark.parametrize("sizes", SIZES)
@pytest.mark.parametrize("storage", ["f32", "f16"])
def test_host_fields_match_device_fields(sizes, storage):
    cases = [W.Case("io", nx, ny, 0.6, 7.0, **(FLUX if k else {})) for k, (nx, ny) in enumerate(sizes)]
    fields = [tuple(W.random_field(c.nx, c.ny, 1e-3, t0, 5 + k + 10 * i) for i, t0 in enumerate((1.0, 0.0, 0.0)))
              for k, c in enumerate(cases)]
    got = []
    for device in (False, True):
        lat = Lattice([instance_from_case(c, 2.0 ** -19) for c in cases], storage=storage, check_interval=5)
        out = []
        # the second pass re-initialises used instances, after a flux change
        for flux in (None, 2e-3):
            for k, f in enumerate(fields):
                if flux is not None:
                    lat.set_wall_flux(1, 2, flux)
                lat.init(k, *(tuple(torch.from_numpy(a).cuda() for a in f) if device else f))
            for n in (0, 5, 6):
                lat.step(n)
                for k in range(len(cases)):
                    dev = tuple(t.cpu().numpy() for t in lat.moments_device(k))
                    host = lat.moments_noalloc(k) if device else lat.moments(k)
                    assert all(np.array_equal(a, b) for a, b in zip(dev, host)), (sizes, storage, n, k)
                    out.append(host + lat.moments_f32(k) + (lat.totals(k),))
                    if n:
                        out.append(tuple(np.float64(v) for v in np.hstack(list(lat.last_check(k).values()))))
        lat.close()
        got.append(out)
    assert len(got[0]) == len(got[1])
    for a, b in zip(*got):
        assert all(np.array_equal(x, y) for x, y in zip(a, b))
    log(f"host and device fields of {sizes} in {storage}: {len(got[0])} records equal")


@pytest.mark.parametrize("storage", ["f16", "bf16_split"])
@pytest.mark.parametrize("steps", [2, 5, 11])
def test_first_16_bit_readout_matches_later_ones(storage, steps):
    # the first FP64 readout after a fused launch writes the caller's arrays in
    # the replay itself, later ones (and all others) copy from the readout buffer
    cases = [W.Case("r0", 131, 67, 0.6, 7.0), W.Case("r1", 53, 140, 0.55, 20.0, **FLUX), W.Case("r2", 7, 9, 0.7, 3.0)]
    lat = Lattice([instance_from_case(c, 2.0 ** -19) for c in cases], storage=storage, rounding="stochastic", seed=3)
    lat.set_step_fusion(6)
    for k, c in enumerate(cases):
        lat.init(k, W.random_field(c.nx, c.ny, 1e-3, 1.0, 5 + k))
    for first in (1, 0, 2):
        lat.step(steps)
        a = lat.moments_device(first)
        later = [lat.moments_device(k) for k in range(len(cases))]
        assert all(torch.equal(x, y) for x, y in zip(a, later[first])), (storage, steps, first)
        for k in range(len(cases)):
            host = lat.moments(k)
            assert all(np.array_equal(x.cpu().numpy(), y) for x, y in zip(later[k], host)), (storage, steps, first, k)
    # only the arrays asked for are written
    lat.step(steps)
    c = cases[1]
    out = [torch.full((c.ny, c.nx), -3.0, dtype=torch.float64, device="cuda") for _ in range(3)]
    lbm_moments_f64(lat.h, 1, out[0].data_ptr(), 0, out[2].data_ptr(), 1)
    full = lat.moments_device(1)
    assert torch.equal(out[0], full[0]) and torch.equal(out[2], full[2]) and bool((out[1] == -3.0).all())
    lat.close()
    log(f"first readouts of {storage} after {steps} steps: equal to later ones")
