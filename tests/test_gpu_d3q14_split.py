"""Work split of the D3Q14 several-step kernels: it changes no bits."""
import numpy as np
import pytest

from paper_2010_01847_amd.d3q14 import Box
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


# boxes that new FP32 handles advance three steps per launch: one and several
# z ranges, sides off and on the 58 x 18 tiles, a column wrapped into one tile
@pytest.mark.parametrize("nx,ny,nz", [(144, 260, 186), (498, 109, 118), (102, 394, 285), (47, 800, 171)])
@pytest.mark.parametrize("stochastic,layout", [(False, "chunked"), (True, "chunked"), (False, "planes"), (True, "planes")])
def test_three_steps_per_launch(nx, ny, nz, stochastic, layout):
    """Three steps per launch give the bits of single steps, whatever the
    split of the calls (1, 2, 3, 4 = 2 + 2, 5 = 3 + 2 and 7 = 3 + 2 + 2)."""
    T0, q = _random_start(nx, ny, nz, 107)
    got = []
    for fuse in (None, 1):
        box = Box(nx, ny, nz, 0.6, 5.0, storage="f32", stochastic=stochastic, seed=5, layout=layout)
        assert box.step_fusion() == 2
        if fuse:
            box.set_step_fusion(fuse)
        box.init(T0, q)
        for n in (3, 1, 4, 2, 5, 7):
            box.step(n)
            got.append(box.moments())
        box.close()
    for a, b in zip(got[:6], got[6:]):
        assert all(np.array_equal(u, v) for u, v in zip(a, b))
