"""The server's accounting: what a request on a run layout is admitted against,
batches that do not fit a slot in one piece, and the queue's bound while a
batch is being planned."""
import threading
import time

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


def test_a_batch_that_does_not_fit_a_slot_is_split(run_layout):
    reqs = requests(run_layout, 14, 64)
    need = high_water(run_layout, reqs[0], 64)
    s = lbl.serve_start(hbm_budget_bytes=4 * need, max_batch_frames=16, max_wait_us=0, n_streams=1)
    try:
        tickets = [lbl.serve_submit(s, run_layout[2], O, 64, L) for O, L, _ in reqs]
        for t, (_, L, want) in zip(tickets, reqs):
            assert lbl.serve_wait(s, t) == lbl.OK
            assert np.array_equal(L.cpu().numpy(), want)
        st = lbl.serve_stats(s)
        assert st["completed"] == 14 and st["failed"] == 0
        assert st["batches"] >= 4 and st["max_in_flight"] <= 5 and st["budget_high_water"] <= 4 * need, st
    finally:
        lbl.serve_stop(s)


def test_the_queue_counts_requests_being_planned(run_layout):
    """One batch in flight and a queue of 4: whatever is being planned counts
    with the queue, so never more than 8 requests are unfinished."""
    reqs = requests(run_layout, 6, 40)
    s = lbl.serve_start(hbm_budget_bytes=1 << 30, max_batch_frames=4, max_wait_us=0, max_queue=4, n_streams=1)
    accepted, busy, errors, most, stop = [0] * 6, [0] * 6, [], [0], threading.Event()

    def client(i):
        O, L, want = reqs[i]
        for _ in range(150):
            try:
                t = lbl.serve_submit(s, run_layout[2], O, 40, L)
            except lbl.LblError as e:
                if e.status != lbl.EBUSY:
                    errors.append(str(e))
                busy[i] += 1
                time.sleep(20e-6)
                continue
            accepted[i] += 1
            tickets[i].append(t)
            if len(tickets[i]) > 3 and lbl.serve_wait(s, tickets[i].pop(0)) != lbl.OK:
                errors.append(lbl.last_error())

    def watch():
        while not stop.is_set():
            st = lbl.serve_stats(s)
            most[0] = max(most[0], st["submitted"] - st["completed"] - st["failed"])

    tickets = [[] for _ in range(6)]
    try:
        w = threading.Thread(target=watch)
        w.start()
        th = [threading.Thread(target=client, args=(i,)) for i in range(6)]
        for t in th:
            t.start()
        for t in th:
            t.join()
        for q in tickets:
            for t in q:
                assert lbl.serve_wait(s, t) == lbl.OK
        stop.set()
        w.join()
        st = lbl.serve_stats(s)
        print("queue of 4: accepted", sum(accepted), "busy", sum(busy), "most unfinished", most[0], flush=True)
        assert not errors, errors[:3]
        assert st["completed"] == sum(accepted) > 0 and st["rejected"] == sum(busy) > 0 and st["failed"] == 0, st
        assert most[0] <= 8
        for _, L, want in reqs:
            assert np.array_equal(L.cpu().numpy(), want)
    finally:
        stop.set()
        lbl.serve_stop(s)
