"""Planner calls on either side of the edge count from which sweeps take their
large form, with edges in random order and by source, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_1810_02612_amd import lbl

pytestmark = pytest.mark.gpu

LINE = 3 << 18


@pytest.mark.parametrize("n_e", [LINE, LINE + 1, LINE + 300_001])
@pytest.mark.parametrize("by_source", [False, True])
@pytest.mark.parametrize("n_v,states", [(200_000, 1), (60_000, 3)])
def test_large_graphs_match_the_oracle(n_e, by_source, n_v, states):
    rng = np.random.default_rng([n_e, n_v, by_source])
    src = rng.integers(0, n_v, n_e).astype(np.uint32)
    if by_source:
        src.sort()
    dst = rng.integers(0, n_v, n_e).astype(np.uint32)
    dst[rng.random(n_e) < 0.1] = n_v - 1  # many ends in one vertex
    cost = rng.integers(1, 1000, n_e).astype(np.uint32)
    L = (rng.random((n_e, 2)) < 0.3).astype(np.uint8)
    delta = rng.integers(0, states, states << 2).astype(np.uint8)
    print("large graph", n_e, by_source, n_v, states, flush=True)
    want_d, want_p = oracle.product_paths(n_v, src, dst, cost, L, delta, 3, 0)
    dev = [torch.from_numpy(x.view(np.int32)).cuda() for x in (src, dst, cost)]
    dist = torch.zeros(n_v * states, dtype=torch.int32, device="cuda")
    pred = torch.zeros_like(dist)
    lbl.product_shortest_paths(n_v, *dev, torch.from_numpy(L).cuda(), 2, delta, 3, 0, dist, pred)
    assert np.array_equal(dist.cpu().numpy().view(np.uint32), want_d)
    assert np.array_equal(pred.cpu().numpy().view(np.uint32), want_p)
