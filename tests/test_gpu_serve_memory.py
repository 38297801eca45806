"""The server's accounting: what a request on a run layout is admitted against."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_1810_02612_amd import lbl

pytestmark = pytest.mark.gpu

N, ROWS = 512, 2000


@pytest.fixture(scope="module")
def run_layout():
    """Blocks of consecutive cells on 512^2 (4096 words): run entries."""
    rng = np.random.default_rng(5)
    x0, y0 = rng.integers(0, N - 20, ROWS), rng.integers(0, N - 10, ROWS)
    cells = ((y0[:, None, None] + np.arange(10)[None, :, None]) * N + x0[:, None, None] + np.arange(20)).reshape(-1)
    ptr = np.arange(ROWS + 1, dtype=np.uint64) * 200
    h = lbl.load_abstraction(N, N, ptr, cells.astype(np.uint32), lbl.LOAD_SPARSE_ONLY)
    yield ptr, cells.astype(np.uint32), h
    lbl.free_abstraction(h)


def requests(run_layout, n, props):
    ptr, col, h = run_layout
    rng = np.random.default_rng([n, props])
    out = []
    for _ in range(n):
        O = (rng.random((N * N, props)) < 0.001).astype(np.uint8)
        L = torch.full((ROWS, props), 9, dtype=torch.uint8, device="cuda")
        out.append((torch.from_numpy(O).cuda(), L, oracle.label_csr(ptr, col, N * N, O, threads=8)))
    torch.cuda.synchronize()
    return out


def high_water(run_layout, req, props):
    s = lbl.serve_start(hbm_budget_bytes=1 << 30, max_batch_frames=1, n_streams=1)
    try:
        assert lbl.serve_wait(s, lbl.serve_submit(s, run_layout[2], req[0], props, req[1])) == lbl.OK
        assert np.array_equal(req[1].cpu().numpy(), req[2])
        return lbl.serve_stats(s)["budget_high_water"]
    finally:
        lbl.serve_stop(s)


@pytest.mark.parametrize("props", [16, 64])
def test_a_run_layout_needs_a_mask_per_cell(run_layout, props):
    mask = 4 if props <= 32 else 8
    need = high_water(run_layout, requests(run_layout, 1, props)[0], props)
    assert N * N * mask <= need < 2 * N * N * mask  # nibble tables would take four times as much
