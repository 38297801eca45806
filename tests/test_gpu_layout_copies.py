"""Layouts that could not make the faster copies of their words label the same
frames: a failure is injected after the copies are made."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_1810_02612_amd import lbl

pytestmark = pytest.mark.gpu


def blocks(rng, n_traj, nx, ny, slow):
    """CSR rows of one block of consecutive cells each, at random or moving slowly."""
    t = np.arange(n_traj)
    w, h = rng.integers(1, 13, n_traj), rng.integers(1, 13, n_traj)
    x0 = t // 61 % (nx - 12) if slow else rng.integers(0, nx - 12, n_traj)
    y0 = t // 251 % (ny - 12) if slow else rng.integers(0, ny - 12, n_traj)
    k = np.arange(144)
    on = (k % 12 < w[:, None]) & (k // 12 < h[:, None])
    cells = (y0[:, None] + k // 12) * nx + x0[:, None] + k % 12
    return np.concatenate([[0], np.cumsum(on.sum(1))]).astype(np.uint64), cells[on].astype(np.uint32)


@pytest.mark.parametrize("n_traj,nx,ny,slow,flags", [(3000, 72, 40, False, 0), (20000, 64, 64, True, lbl.LOAD_SPARSE_ONLY),
                                                      (70000, 512, 512, False, lbl.LOAD_SPARSE_ONLY)])
def test_layout_without_copies(n_traj, nx, ny, slow, flags, monkeypatch):
    rng = np.random.default_rng([n_traj, nx])
    ptr, col = blocks(rng, n_traj, nx, ny, slow)
    full = lbl.load_abstraction(nx, ny, ptr, col, flags)
    monkeypatch.setenv("LBL_FAULT_LAYOUT", "1")
    plain = lbl.load_abstraction(nx, ny, ptr, col, flags)
    monkeypatch.delenv("LBL_FAULT_LAYOUT")
    try:
        a, b = lbl.abstraction_info(full), lbl.abstraction_info(plain)
        assert a["sparse_entries"] == b["sparse_entries"]
        assert b["sparse_frame_bytes"] >= 10 * b["sparse_entries"]  # the words themselves
        assert a["sparse_frame_bytes"] < b["sparse_frame_bytes"] and a["sparse_bytes"] > b["sparse_bytes"]
        for P in (1, 2, 3, 4, 8, 33, 64):
            O = ((rng.random((nx * ny, P)) < 0.02) * rng.integers(1, 256, (nx * ny, P))).astype(np.uint8)
            want = oracle.label_csr(ptr, col, nx * ny, O, threads=8)
            Od = torch.from_numpy(O).cuda()
            L = [torch.full((n_traj, P), 9, dtype=torch.uint8, device="cuda") for _ in range(5)]
            print("without copies", n_traj, nx, ny, slow, P, flush=True)
            lbl.label_frame(plain, Od, P, L[0], flags=lbl.KERNEL_SPARSE)
            lbl.label_frame_noalloc(plain, Od, P, L[1])
            lbl.label_batch([(plain, Od, P, L[2]), (full, Od, P, L[3])])
            lbl.label_frame(full, Od, P, L[4], flags=lbl.KERNEL_SPARSE)
            torch.cuda.synchronize()
            for x in L:
                assert np.array_equal(x.cpu().numpy(), want), P
    finally:
        lbl.free_abstraction(plain)
        lbl.free_abstraction(full)
