"""Batches recorded into a graph keep their buffers: replays after many other
batches were laid out equal the oracle, and what is kept is bounded."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_1810_02612_amd import lbl

pytestmark = pytest.mark.gpu

N, ROWS = 64, 500


def load(seed):
    rng = np.random.default_rng(seed)
    ptr = np.arange(ROWS + 1, dtype=np.uint64) * 20
    col = rng.integers(0, N * N, ROWS * 20).astype(np.uint32)
    return ptr, col, lbl.load_abstraction(N, N, ptr, col)


def frame(rng, P):
    return (rng.random((N * N, P)) < 0.02).astype(np.uint8)


def jobs_of(h, O):
    return [(h, o, o.shape[1], torch.full((ROWS, o.shape[1]), 9, dtype=torch.uint8, device="cuda")) for o in O]


def recorded(jobs, stream):
    lbl.label_batch(jobs, stream=stream)  # laid out
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        lbl.label_batch(jobs, stream=stream)
    return g


def test_replays_after_other_batches():
    ptr, col, h = load(1)
    try:
        rng = np.random.default_rng(2)
        s = torch.cuda.Stream()
        O = [torch.from_numpy(frame(rng, P)).cuda() for P in (5, 37, 64)]
        jobs = jobs_of(h, O)
        torch.cuda.synchronize()
        g = recorded(jobs, s)
        for rep in range(4):
            # more batches than are kept, each in buffers of its own, and
            # memory taken and written in between
            others = [jobs_of(h, [O[k % 3]] * (1 + k % 2)) for k in range(12)]
            torch.cuda.synchronize()
            for other in others:
                lbl.label_batch(other, stream=s)
            junk = [torch.full((1 << 18,), 255, dtype=torch.uint8, device="cuda") for _ in range(64)]
            new = [frame(rng, o.shape[1]) for o in O]
            for o, x in zip(O, new):
                o.copy_(torch.from_numpy(x))
            for _, _, _, L in jobs:
                L.fill_(7)
            torch.cuda.synchronize()
            print("replay", rep, flush=True)
            with torch.cuda.stream(s):
                g.replay()
            torch.cuda.synchronize()
            for (_, _, _, L), x in zip(jobs, new):
                assert np.array_equal(L.cpu().numpy(), oracle.label_csr(ptr, col, N * N, x)), rep
            del junk
    finally:
        torch.cuda.synchronize()
        lbl.free_abstraction(h)


def test_recorded_batches_are_bounded_and_given_back():
    rng = np.random.default_rng(3)
    s = torch.cuda.Stream()
    O = [torch.from_numpy(frame(rng, 9)).cuda()]
    for turn in range(2):  # released with the abstraction: as many again
        ptr, col, h = load(10 + turn)
        try:
            kept = [jobs_of(h, O) for _ in range(8)]
            torch.cuda.synchronize()
            graphs = [recorded(j, s) for j in kept]
            one_more = jobs_of(h, O)
            lbl.label_batch(one_more, stream=s)
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                with pytest.raises(lbl.LblError) as e:
                    lbl.label_batch(one_more, stream=s)
                kept[0][0][3].fill_(5)  # the capture goes on
            assert e.value.status == lbl.EINVAL
            want = oracle.label_csr(ptr, col, N * N, O[0].cpu().numpy())
            for j in kept:
                j[0][3].fill_(7)
            torch.cuda.synchronize()
            with torch.cuda.stream(s):
                for x in graphs:
                    x.replay()
            torch.cuda.synchronize()
            assert all(np.array_equal(j[0][3].cpu().numpy(), want) for j in kept)
        finally:
            torch.cuda.synchronize()
            lbl.free_abstraction(h)
