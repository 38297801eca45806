"""GPU labels from run entries against the oracle, at the sizes where rounds,
segments and row blocks end, and where a layout changes to nibble entries."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_1810_02612_amd import lbl

pytestmark = pytest.mark.gpu


def rows(rng, n_traj, nx, ny, split):
    """CSR rows of a few blocks of consecutive cells, one per grid row; with
    probability `split` a block also gets a second run in the same words."""
    ptr, col, n = [0], [np.zeros(0, np.uint32)], 0
    for t in range(n_traj):
        for _ in range(rng.integers(0, 4)):
            x0, y0, w, h = rng.integers(0, nx), rng.integers(0, ny), rng.integers(1, 20), rng.integers(1, 9)
            xs = np.arange(x0, min(nx, x0 + w))
            if rng.random() < split:
                xs = xs[(xs - x0) % 3 != 2]
            for y in range(y0, min(ny, y0 + h)):
                col.append(y * nx + xs)
                n += len(xs)
        ptr.append(n)
    return np.array(ptr, np.uint64), np.concatenate(col).astype(np.uint32)


@pytest.mark.parametrize("n_traj,nx,ny,split", [(1, 8, 8, 0.0), (65, 24, 40, 0.0), (8192, 64, 64, 0.1), (8193, 64, 64, 0.1),
                                                 (8257, 200, 136, 0.05), (3000, 64, 64, 1.0)])
@pytest.mark.parametrize("order", [lbl.ROW_MAJOR, lbl.MORTON])
def test_run_entries_match_the_oracle(n_traj, nx, ny, split, order):
    if order == lbl.MORTON and nx != ny or order == lbl.MORTON and nx & (nx - 1):
        pytest.skip("z-order ids need a square grid of a power of two")
    rng = np.random.default_rng([n_traj, nx])
    row_ptr, col = rows(rng, n_traj, nx, ny, split)
    ids = np.arange(nx * ny, dtype=np.uint32)
    if order == lbl.MORTON:
        w = [lbl.cell_position(nx, ny, int(c)) for c in ids]
        ids = np.array([a * 64 + b for a, b in w], np.uint32)
    h = lbl.load_abstraction(nx, ny, row_ptr, ids[col], cell_order=order)
    try:
        info = lbl.abstraction_info(h)
        if split <= 0.1 and info["sparse_entries"]:  # run entries are 8 bytes, nibble entries 10
            assert info["sparse_bytes"] >= 18 * info["sparse_entries"]
        for P in (5, 16, 17, 32, 33, 48, 64):
            O = ((rng.random((nx * ny, P)) < 0.03) * rng.integers(1, 256, (nx * ny, P))).astype(np.uint8)
            Oc = np.empty_like(O)
            Oc[ids] = O
            want = oracle.label_csr(row_ptr, col, nx * ny, O)
            Od = torch.from_numpy(Oc).cuda()
            L = torch.full((n_traj, P), 9, dtype=torch.uint8, device="cuda")
            print("runs", n_traj, nx, ny, split, order, P, flush=True)
            lbl.label_frame(h, Od, P, L, flags=lbl.KERNEL_SPARSE)
            B = [torch.full((n_traj, P), 9, dtype=torch.uint8, device="cuda") for _ in range(3)]
            lbl.label_batch([(h, Od, P, b) for b in B])
            torch.cuda.synchronize()
            for got in [L] + B:
                assert np.array_equal(got.cpu().numpy(), want), (P, int((got.cpu().numpy() != want).sum()))
    finally:
        lbl.free_abstraction(h)
