"""Planner sweeps that look at an edge's source again, against the oracle: long
chains, grids and edges sorted by source, at the spans of sources (1 KiB of
distances) where a wavefront starts to look once only."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_1810_02612_amd import lbl

pytestmark = pytest.mark.gpu


def graph(rng, kind, n):
    """(vertices, src, dst) by ascending source."""
    if kind == "chain":
        return n, np.arange(n - 1), np.arange(1, n)
    if kind == "grid":
        i = np.arange(n * n).reshape(n, n)
        s = np.concatenate([i[:, :-1].ravel(), i[:-1].ravel(), i[:, 1:].ravel()])
        d = np.concatenate([i[:, 1:].ravel(), i[1:].ravel(), i[:, :-1].ravel()])
    else:  # "fan": every vertex has 8 edges to later ones, most of them to the last
        s = np.repeat(np.arange(n - 1), 8)
        d = np.minimum(s + rng.integers(1, 60, len(s)), n - 1)
        d[rng.random(len(s)) < 0.6] = n - 1
        return n, s, d
    o = np.argsort(s, kind="stable")
    return n * n, s[o], d[o]


@pytest.mark.parametrize("kind,n", [("chain", 64), ("chain", 1000), ("grid", 70), ("fan", 3000)])
@pytest.mark.parametrize("states", [1, 2, 3, 8])
def test_looks_match_the_oracle(kind, n, states):
    rng = np.random.default_rng([n, states])
    n_v, src, dst = graph(rng, kind, n)
    src, dst = src.astype(np.uint32), dst.astype(np.uint32)
    cost = rng.integers(1, 50, len(src)).astype(np.uint32)
    L = (rng.random((len(src), 2)) < 0.3).astype(np.uint8)
    delta = rng.integers(0, states, states << 2).astype(np.uint8)
    want_d, want_p = oracle.product_paths(n_v, src, dst, cost, L, delta, 0, 0)
    print("looks", kind, n, states, flush=True)
    dev = [torch.from_numpy(x.view(np.int32)).cuda() for x in (src, dst, cost)]
    dist = torch.zeros(n_v * states, dtype=torch.int32, device="cuda")
    pred = torch.zeros_like(dist)
    for _ in range(3):
        lbl.product_shortest_paths(n_v, *dev, torch.from_numpy(L).cuda(), 2, delta, 0, 0, dist, pred)
        assert np.array_equal(dist.cpu().numpy().view(np.uint32), want_d)
        assert np.array_equal(pred.cpu().numpy().view(np.uint32), want_p)
