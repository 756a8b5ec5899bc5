"""The key sort at the edges of its tiles and merges (tiles of 4096 keys, 2, 4
or 8 runs merged at once, fan-in 8 up to 2^18 keys), through the id-order
layout of requests too long to be ordered one by one: each request's chunks
must come out ascending; and through the popularity order, whose keys repeat
their high half."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_13692_amd import mpt
from paper_2609_13692_amd import workloads as wl

pytestmark = pytest.mark.gpu

T = 4096
SIZES = [600, T - 1, T, T + 1, 2 * T, 2 * T + 1, 3 * T + 7, 4 * T, 4 * T + 1, 8 * T, 8 * T + 1, 9 * T - 1, 64 * T - 1,
         64 * T, 64 * T + 1, 65 * T + 3, 257 * T + 11]


@pytest.mark.parametrize("n", SIZES)
def test_id_order_of_long_requests(n):
    rng = np.random.default_rng(n)
    u = 2 * n
    first = rng.choice(u, size=n - 5, replace=False)
    inst = wl.Instance(u, np.ones(u, dtype=np.int64), np.array([0, 3, n - 2, n - 2, n]),
                       np.concatenate([[9, 2, 7], first, [5, 1]]).astype(np.int32))
    print(f"[gpu] key sort n={n}", flush=True)
    got = mpt.Layouts(inst).global_order(mpt.MPT_ORDER_ID).cpu().numpy()
    assert np.array_equal(got, np.concatenate([[2, 7, 9], np.sort(first), [1, 5]]))


@pytest.mark.parametrize("u", [700, T, 5 * T + 1, 70 * T])
def test_popularity_order(u):
    inst = wl.random_small(m=30, u=u, kmin=520, kmax=690, wmax=3, seed=u)
    print(f"[gpu] popularity order u={u}", flush=True)
    got = mpt.Layouts(inst).global_order(mpt.MPT_ORDER_POPULARITY).cpu().numpy()
    assert np.array_equal(got, oracle.global_order_layout(inst, oracle.popularity_rank(inst)))
