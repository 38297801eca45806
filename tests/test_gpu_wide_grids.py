"""Batches on a grid so wide that seven grid rows of a frame pass 2^32 bytes:
labels equal the definition, one frame's and its batch's alike."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1810_02612_amd import lbl

pytestmark = pytest.mark.gpu

NX, NY = 10_200_000, 8


@pytest.mark.parametrize("P,off", [(64, 0), (61, 3)])
def test_batch_of_a_wide_frame(P, off):
    assert 7 * NX * P > 1 << 32
    rng = np.random.default_rng(P)
    n_traj = 60
    x0 = np.concatenate([[0, 4, NX - 8], rng.integers(0, NX - 8, n_traj - 3)])
    x0[10] = 8 * (x0[10] // 8) + 5  # two words
    cells = (np.arange(8)[None, :, None] * NX + x0[:, None, None] + np.arange(6)[None, None, :]).reshape(n_traj, -1)
    cells = cells[:, rng.permutation(48)[:40]]
    row_ptr = np.arange(n_traj + 1, dtype=np.uint64) * 40
    h = lbl.load_abstraction(NX, NY, row_ptr, cells.astype(np.uint32).reshape(-1), lbl.LOAD_SPARSE_ONLY)
    try:
        buf = torch.zeros(NX * NY * P + off, dtype=torch.uint8, device="cuda")
        O = buf[off:].view(NX * NY, P)
        # a few propositions at a few of each trajectory's cells, in the first
        # and in the last grid row among them, and others all over the frame
        t = np.repeat(np.arange(n_traj), 3)
        at = torch.from_numpy(cells[t, rng.integers(0, 40, len(t))]).cuda()
        O[at, torch.from_numpy(rng.integers(0, P, len(t))).cuda()] = 1
        O[torch.from_numpy(7 * NX + x0).cuda(), torch.from_numpy(rng.integers(0, P, n_traj)).cuda()] = 255
        far = torch.from_numpy(rng.integers(0, NX * NY, 200_000)).cuda()
        O[far, torch.from_numpy(rng.integers(0, P, len(far))).cuda()] = 2
        want = (O[torch.from_numpy(cells).cuda().reshape(-1)].view(n_traj, 40, P) != 0).any(1).to(torch.uint8)
        L = torch.full((n_traj, P), 9, dtype=torch.uint8, device="cuda")
        B = torch.full((n_traj, P), 9, dtype=torch.uint8, device="cuda")
        print("wide frame", NX, P, off, flush=True)
        lbl.label_frame(h, buf[off:], P, L)
        lbl.label_batch([(h, buf[off:], P, B)])
        torch.cuda.synchronize()
        assert torch.equal(L, want), int((L != want).sum())
        assert torch.equal(B, want), int((B != want).sum())
    finally:
        lbl.free_abstraction(h)
