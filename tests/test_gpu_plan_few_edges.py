"""Planner calls on graphs of many vertices and few edges, down to none: every
output is written."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1810_02612_amd import lbl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_v,n_e,states", [(1, 0, 1), (4097, 1, 3), (70001, 0, 2), (1500001, 9, 2), (3000000, 257, 1)])
def test_every_output_is_written(n_v, n_e, states):
    # a path 0, k, 2k, ... of n_e edges with costs 1, 2, ...
    k = max(1, (n_v - 1) // max(1, n_e))
    at = np.arange(n_e + 1) * k % n_v
    cost = np.arange(1, n_e + 1, dtype=np.int32)
    dev = [torch.from_numpy(x.astype(np.int32)).cuda() for x in (at[:-1], at[1:], cost)]
    L = torch.zeros((max(1, n_e), 1), dtype=torch.uint8, device="cuda")
    delta = np.repeat(np.arange(states), 2).astype(np.uint8)
    dist = torch.full((n_v * states,), 7, dtype=torch.int32, device="cuda")
    pred = torch.full_like(dist, 7)
    print("few edges", n_v, n_e, states, flush=True)
    lbl.product_shortest_paths(n_v, *dev, L, 1, delta, 0, states - 1, dist, pred)
    want_d, want_p = np.full(n_v * states, -1, np.int32), np.full(n_v * states, -1, np.int32)
    want_d[at * states + states - 1] = np.concatenate([[0], np.cumsum(cost)])
    want_p[at[1:] * states + states - 1] = np.arange(n_e) * states + states - 1
    assert np.array_equal(dist.cpu().numpy(), want_d)
    assert np.array_equal(pred.cpu().numpy(), want_p)
