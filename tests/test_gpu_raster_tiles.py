"""The rasterizer at the edges of its tiles (64 x 8 cells, or 512 z-order ids)
and of its shape list (512 at a time), against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_1810_02612_amd import lbl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,n_props,n_shapes,order,offset", [
    (8, 8, 3, 1, lbl.ROW_MAJOR, 0), (8, 8, 3, 5, lbl.MORTON, 1), (64, 8, 64, 511, lbl.ROW_MAJOR, 0),
    (72, 40, 37, 512, lbl.ROW_MAJOR, 0), (200, 136, 48, 513, lbl.ROW_MAJOR, 0), (128, 16, 16, 1500, lbl.ROW_MAJOR, 3),
    (16, 16, 5, 40, lbl.MORTON, 0), (32, 32, 64, 1025, lbl.MORTON, 0), (256, 256, 33, 300, lbl.MORTON, 0)])
def test_tiles_match_the_oracle(nx, ny, n_props, n_shapes, order, offset):
    rng = np.random.default_rng([nx, ny, n_shapes])
    kind, prop = rng.integers(0, 2, n_shapes), rng.integers(0, n_props, n_shapes)
    cx, cy = rng.uniform(-5, 0.3 * nx + 5, n_shapes), rng.uniform(-5, 0.3 * ny + 5, n_shapes)
    a, b = rng.uniform(0, 3, n_shapes), rng.uniform(0, 3, n_shapes)
    shapes = lbl.shapes_array(kind, prop, cx, cy, a, b)
    buf = torch.full((offset + nx * ny * n_props + 16,), 7, dtype=torch.uint8, device="cuda")
    print("raster", nx, ny, n_props, n_shapes, order, offset, flush=True)
    lbl.raster_frame(nx, ny, 0.3, shapes, n_props, buf.data_ptr() + offset, cell_order=order)
    torch.cuda.synchronize()
    got = buf.cpu().numpy()
    assert (got[:offset] == 7).all() and (got[offset + nx * ny * n_props:] == 7).all()
    got = got[offset:offset + nx * ny * n_props].reshape(nx * ny, n_props)
    want = oracle.raster_shapes(shapes["kind"], shapes["prop"], shapes["cx"], shapes["cy"], shapes["a"], shapes["b"],
                                nx, ny, 0.3, n_props)
    if order == lbl.MORTON:
        ids = [w * 64 + q for w, q in (lbl.cell_position(nx, ny, c) for c in range(nx * ny))]
        got = got[ids]
    assert np.array_equal(got, want), int((got != want).sum())
