"""Work split of the D3Q14 several-step kernels: it changes no bits."""
import numpy as np
import pytest

from test_gpu_d3q14 import _gpu, _random_start

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz,storage", [(301, 211, 163, "bf16"), (130, 500, 41, "f32"), (61, 13, 7, "f32")])
def test_default_z_ranges(nx, ny, nz, storage):
    """A new handle's z ranges (filling the last round of blocks) change only
    the work split: the same bits as a set range of 32 planes."""
    T0, q = _random_start(nx, ny, nz, 103)
    a = _gpu(nx, ny, nz, 0.7, 3.0, T0, q, 4, storage=storage, stochastic=storage != "f32", seed=5, fuse=2)
    b = _gpu(nx, ny, nz, 0.7, 3.0, T0, q, 4, storage=storage, stochastic=storage != "f32", seed=5, fuse=2,
             shape=dict(rows_per_tile=4, xcd_remap=0, nontemporal=0, tile_waves=1, zchunk=32))
    for u, v in zip(a, b):
        assert np.array_equal(u, v)
