"""Frames of at most 4 propositions labeled by row tiles against the oracle, at
the row counts where a tile, a row block and the tile size's steps end."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_1810_02612_amd import lbl

pytestmark = pytest.mark.gpu


def rows(rng, n_traj, n):
    """CSR rows of blocks that move slowly over an n x n grid, so that
    neighbouring rows meet the same words; every 7th row is empty."""
    t = np.arange(n_traj)
    w, h = rng.integers(1, 15, n_traj), rng.integers(1, 11, n_traj)
    x0, y0 = (t // 61) % (n - 14), (t // 251) % (n - 10)
    w[t % 7 == 3] = 0
    k = np.arange(14 * 10)
    dx, dy = k % 14, k // 14
    on = (dx < w[:, None]) & (dy < h[:, None])
    cells = (y0[:, None] + dy) * n + x0[:, None] + dx
    ptr = np.concatenate([[0], np.cumsum(on.sum(1))]).astype(np.uint64)
    return ptr, cells[on].astype(np.uint32)


@pytest.mark.parametrize("n_traj", [63, 64, 65, 8191, 8193, 65535, 65537, 131073, 262143, 262273])
@pytest.mark.parametrize("order", [lbl.ROW_MAJOR, lbl.MORTON])
def test_row_tiles_match_the_oracle(n_traj, order):
    n = 64
    rng = np.random.default_rng([n_traj, order])
    row_ptr, col = rows(rng, n_traj, n)
    ids = np.arange(n * n, dtype=np.uint32)
    if order == lbl.MORTON:
        w = [lbl.cell_position(n, n, int(c)) for c in ids]
        ids = np.array([a * 64 + b for a, b in w], np.uint32)
    h = lbl.load_abstraction(n, n, row_ptr, ids[col], lbl.LOAD_SPARSE_ONLY, cell_order=order)
    try:
        per = 512 if n_traj >= 1 << 18 else 256 if n_traj >= 1 << 17 else 128 if n_traj >= 1 << 16 else 64
        assert lbl.abstraction_info(h)["sparse_tiles_direct"] == -(-n_traj // per)
        for P in (1, 2, 3, 4):
            O = ((rng.random((n * n, P)) < 0.02) * rng.integers(1, 256, (n * n, P))).astype(np.uint8)
            Oc = np.empty_like(O)
            Oc[ids] = O
            # O and L one byte into their buffers; bytes around L stay
            Od = torch.zeros(n * n * P + 8, dtype=torch.uint8, device="cuda")
            Od[1:1 + n * n * P] = torch.from_numpy(Oc.reshape(-1)).cuda()
            buf = torch.full((n_traj * P + 8,), 9, dtype=torch.uint8, device="cuda")
            print("row tiles", n_traj, order, P, flush=True)
            lbl.label_frame(h, Od[1:1 + n * n * P], P, buf[1:1 + n_traj * P])
            torch.cuda.synchronize()
            got = buf.cpu().numpy()
            assert (got[:1] == 9).all() and (got[1 + n_traj * P:] == 9).all()
            want = oracle.label_csr(row_ptr, col, n * n, O, threads=8)
            assert np.array_equal(got[1:1 + n_traj * P].reshape(n_traj, P), want)
    finally:
        lbl.free_abstraction(h)
