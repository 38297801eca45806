"""Frames of 1 to 4 propositions on the layouts that row tiles decline: by the
direct-mask kernels, with frames and labels at odd offsets, and by the run
kernels where a part's masks do not fit the direct kernel either; and row tiles
where only they hold a tile's masks.  The profile
counts say which kernels ran (row tiles: no pack)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_1810_02612_amd import lbl

pytestmark = pytest.mark.gpu


def profiled(h, O, P, L):
    lbl.profile_enable(True)
    lbl.label_frame(h, O, P, L, flags=lbl.KERNEL_SPARSE)
    torch.cuda.synchronize()
    p = lbl.profile_read()
    lbl.profile_enable(False)
    return p["pack_launches"], p["label_launches"], p["emit_launches"]


@pytest.mark.parametrize("n_traj,per", [(700, 60), (20011, 30)])
@pytest.mark.parametrize("P", [1, 2, 3, 4])
def test_direct_masks_at_odd_offsets(n_traj, per, P):
    n = 512
    rng = np.random.default_rng([n_traj, P])
    ptr = np.arange(n_traj + 1, dtype=np.uint64) * per
    col = rng.integers(0, n * n, n_traj * per).astype(np.uint32)  # over 384 words to any 64 rows
    h = lbl.load_abstraction(n, n, ptr, col, lbl.LOAD_SPARSE_ONLY)
    try:
        O = ((rng.random((n * n, P)) < 0.02) * rng.integers(1, 256, (n * n, P))).astype(np.uint8)
        want = oracle.label_csr(ptr, col, n * n, O, threads=8)
        for o_off, l_off in ((0, 0), (1, 0), (2, 3), (3, 1), (0, 15), (4, 2)):
            ob = torch.full((O.size + 16,), 255, dtype=torch.uint8, device="cuda")
            ob[o_off:o_off + O.size] = torch.from_numpy(O.reshape(-1)).cuda()
            lb = torch.full((n_traj * P + 32,), 0xA5, dtype=torch.uint8, device="cuda")
            print("direct masks", n_traj, P, o_off, l_off, flush=True)
            ran = profiled(h, ob[o_off:o_off + O.size], P, lb[l_off:l_off + n_traj * P])
            assert ran == (1, 1, 0)
            got = lb.cpu().numpy()
            assert (got[:l_off] == 0xA5).all() and (got[l_off + n_traj * P:] == 0xA5).all()
            assert np.array_equal(got[l_off:l_off + n_traj * P].reshape(n_traj, P), want)
    finally:
        lbl.free_abstraction(h)


def test_run_kernels_below_four_propositions():
    """400 row blocks of 16,384 single cells in some 10,300 words of 1024^2: a
    part of the direct split has more than the 6,144 segments whose masks fit
    for one proposition."""
    n, n_traj = 1024, 400 * 8192
    rng = np.random.default_rng(6)
    ptr = np.arange(n_traj + 1, dtype=np.uint64) * 2
    col = rng.integers(0, n * n, 2 * n_traj).astype(np.uint32)
    h = lbl.load_abstraction(n, n, ptr, col, lbl.LOAD_SPARSE_ONLY)
    try:
        for P, off in ((1, 0), (2, 1), (3, 2), (3, 0), (4, 1)):
            O = ((rng.random((n * n, P)) < 0.3) * rng.integers(1, 256, (n * n, P))).astype(np.uint8)
            ob = torch.full((O.size + 8,), 255, dtype=torch.uint8, device="cuda")
            ob[off:off + O.size] = torch.from_numpy(O.reshape(-1)).cuda()
            L = torch.full((n_traj, P), 9, dtype=torch.uint8, device="cuda")
            print("run kernels", P, off, flush=True)
            assert profiled(h, ob[off:off + O.size], P, L) == (1, 1, 1)
            assert np.array_equal(L.cpu().numpy(), oracle.label_csr(ptr, col, n * n, O, threads=8))
    finally:
        lbl.free_abstraction(h)


def test_row_tiles_where_direct_masks_do_not_fit():
    """3.2 million rows of 12 words that move slowly over 1024^2: 512 rows meet
    some 140 words, a part of the direct split over 1,536."""
    n, n_traj, per = 1024, 400 * 8192, 12
    rng = np.random.default_rng(7)
    ptr = np.arange(n_traj + 1, dtype=np.uint64) * per
    w = (np.arange(n_traj) * 2000 // 8192)[:, None] % (n * n // 64 - per) + np.arange(per)
    z = rng.integers(0, 64, w.shape)
    col = ((w // (n // 8) * 8 + z // 8) * n + w % (n // 8) * 8 + z % 8).astype(np.uint32).reshape(-1)
    h = lbl.load_abstraction(n, n, ptr, col, lbl.LOAD_SPARSE_ONLY)
    try:
        assert lbl.abstraction_info(h)["sparse_tiles_direct"] == -(-n_traj // 512)
        for P in (1, 4):
            O = (rng.random((n * n, P)) < 0.05).astype(np.uint8)
            L = torch.full((n_traj, P), 9, dtype=torch.uint8, device="cuda")
            print("row tiles beyond the direct split", P, flush=True)
            assert profiled(h, torch.from_numpy(O).cuda(), P, L) == (0, 1, 0)
            assert np.array_equal(L.cpu().numpy(), oracle.label_csr(ptr, col, n * n, O, threads=8))
    finally:
        lbl.free_abstraction(h)
