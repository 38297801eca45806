"""Run kernels that form the cell masks from O: every width of a cell's pieces,
O aligned and not, on layouts of one tile round and of several row blocks, and
one with too many segments (the pack kernel runs, as the profile counts say)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_1810_02612_amd import lbl

pytestmark = pytest.mark.gpu


def blocks(rng, n_traj, nx, ny):
    """CSR rows of one block of up to 12 x 12 consecutive cells each; some empty."""
    w, h = rng.integers(1, 13, n_traj), rng.integers(1, 13, n_traj)
    w[rng.random(n_traj) < 0.05] = 0
    x0, y0 = rng.integers(0, nx, n_traj), rng.integers(0, ny, n_traj)
    k = np.arange(144)
    dx, dy = k % 12, k // 12
    x, y = x0[:, None] + dx, y0[:, None] + dy
    on = (dx < w[:, None]) & (dy < h[:, None]) & (x < nx) & (y < ny)
    return np.concatenate([[0], np.cumsum(on.sum(1))]).astype(np.uint64), (y * nx + x)[on].astype(np.uint32)


@pytest.mark.parametrize("n_traj,nx,ny,order", [(50, 8, 8, 0), (700, 72, 40, 0), (2000, 64, 64, 1), (9000, 64, 64, 1), (20000, 72, 40, 0), (70000, 256, 256, 0)])
def test_masks_from_the_frame(n_traj, nx, ny, order):
    rng = np.random.default_rng([n_traj, nx])
    row_ptr, col = blocks(rng, n_traj, nx, ny)
    n = nx * ny
    ids = np.arange(n, dtype=np.uint32)
    if order:
        w = [lbl.cell_position(nx, ny, int(c)) for c in ids]
        ids = np.array([a * 64 + b for a, b in w], np.uint32)
    h = lbl.load_abstraction(nx, ny, row_ptr, ids[col], cell_order=lbl.MORTON if order else lbl.ROW_MAJOR)
    n_seg = len(np.unique(np.repeat(np.arange(n_traj), np.diff(row_ptr.astype(np.int64))) // 8192 * n +
                          (col // nx // 8) * (nx // 8) + col % nx // 8))
    try:
        for P, off in ((5, 0), (7, 1), (8, 0), (12, 2), (15, 0), (16, 0), (17, 0), (31, 3), (32, 0), (33, 0), (48, 4), (49, 0), (64, 0), (64, 1)):
            O = ((rng.random((n, P)) < 0.02) * rng.integers(1, 256, (n, P))).astype(np.uint8)
            buf = torch.full((n * P + 32,), 255, dtype=torch.uint8, device="cuda")
            Od = buf[off:off + n * P]
            Oc = np.empty_like(O)
            Oc[ids] = O
            Od.copy_(torch.from_numpy(Oc.reshape(-1)))
            L = torch.full((n_traj, P), 9, dtype=torch.uint8, device="cuda")
            print("frame cells", n_traj, nx, ny, order, P, off, flush=True)
            lbl.profile_enable(True)
            lbl.label_frame(h, Od, P, L, flags=lbl.KERNEL_SPARSE)
            torch.cuda.synchronize()
            prof = lbl.profile_read()
            packs = prof["pack_launches"]
            if n_traj <= 2000 and P < 16:  # one launch: no combine either
                assert prof["emit_launches"] == (0 if packs == 0 else 1)
            lbl.profile_enable(False)
            pieces = 2 if P < 16 else -(-P // 16)
            aligned = P % 4 == 0 and (buf.data_ptr() + off) % 4 == 0
            assert packs == (0 if n_seg * pieces * (1 if aligned else 16) <= 50000 else 1), (n_seg, P, off)
            assert np.array_equal(L.cpu().numpy(), oracle.label_csr(row_ptr, col, n, O, threads=8))
    finally:
        lbl.free_abstraction(h)
