"""The rasterizer at the grid sizes where a tile's cells halve (two workgroups
per CU) and its wavefronts share shapes, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_1810_02612_amd import lbl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,order", [(64, 504, 0), (64, 512, 0), (256, 248, 0), (256, 256, 0), (64, 2048, 0), (328, 344, 0),
                                         (512, 504, 0), (512, 512, 0), (128, 128, 1), (256, 256, 1), (512, 512, 1)])
def test_every_split_matches_the_oracle(nx, ny, order):
    rng = np.random.default_rng([nx, ny, order])
    n_props, n = 21, 600
    shapes = lbl.shapes_array(rng.integers(0, 2, n), rng.integers(0, n_props, n), rng.uniform(-5, 0.3 * nx + 5, n),
                              rng.uniform(-5, 0.3 * ny + 5, n), rng.uniform(0, 6, n), rng.uniform(0, 6, n))
    O = torch.full((nx * ny, n_props), 7, dtype=torch.uint8, device="cuda")
    print("raster split", nx, ny, order, flush=True)
    lbl.raster_frame(nx, ny, 0.3, shapes, n_props, O, cell_order=lbl.MORTON if order else lbl.ROW_MAJOR)
    torch.cuda.synchronize()
    got = O.cpu().numpy()
    if order:
        c = np.arange(nx * ny)
        z = np.zeros_like(c)
        for b in range(10):
            z |= ((c // nx >> b) & 1) << (2 * b) | ((c % nx >> b) & 1) << (2 * b + 1)
        got = got[z]
    want = oracle.raster_shapes(shapes["kind"], shapes["prop"], shapes["cx"], shapes["cy"], shapes["a"], shapes["b"],
                                nx, ny, 0.3, n_props)
    assert np.array_equal(got, want), int((got != want).sum())
