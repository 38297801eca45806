"""Frames read at any address and proposition count, one frame and in a batch:
every width of byte_mask's pieces and of a batch's 16-byte units, with O at
offsets that put runs of cells across the ends of units."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_1810_02612_amd import lbl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,order", [(24, 40, lbl.ROW_MAJOR), (8, 8, lbl.ROW_MAJOR), (32, 32, lbl.MORTON)])
def test_every_width_and_offset(nx, ny, order):
    rng = np.random.default_rng([nx, ny])
    n, n_traj = nx * ny, 200
    counts = rng.integers(0, 30, n_traj)
    row_ptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.uint64)
    col = rng.integers(0, n, int(row_ptr[-1])).astype(np.uint32)
    h = lbl.load_abstraction(nx, ny, row_ptr, col, cell_order=order)
    try:
        for P in list(range(1, 20)) + [23, 31, 32, 33, 47, 48, 49, 63, 64]:
            O = ((rng.random((n, P)) < 0.05) * rng.integers(1, 256, (n, P))).astype(np.uint8)
            want = oracle.label_csr(row_ptr, col, n, O)
            print("pack", nx, ny, order, P, flush=True)
            jobs = []
            for off in (0, 1, 5, 8, 15):
                buf = torch.full((n * P + 32,), 255, dtype=torch.uint8, device="cuda")
                Od = buf[off:off + n * P]
                Od.copy_(torch.from_numpy(O.reshape(-1)))
                L = torch.full((n_traj, P), 9, dtype=torch.uint8, device="cuda")
                lbl.label_frame(h, Od, P, L, flags=lbl.KERNEL_SPARSE)
                jobs.append((h, Od, P, torch.full((n_traj, P), 9, dtype=torch.uint8, device="cuda")))
                assert np.array_equal(L.cpu().numpy(), want), off
            lbl.label_batch(jobs)
            torch.cuda.synchronize()
            for j in jobs:
                assert np.array_equal(j[3].cpu().numpy(), want)
    finally:
        lbl.free_abstraction(h)
