"""Where one route hands over to another, the call does not get slower: each
test times a call just inside a route against the same call on the route
beyond its limit (or on inputs that the route should not notice). The best of
many passes, and bounds well above what runs differ by."""
import time

import numpy as np
import pytest
import torch

from paper_2609_13692_amd import mpt
from paper_2609_13692_amd import workloads as wl

pytestmark = pytest.mark.gpu


def best(call, passes=30):
    for _ in range(3):
        call()
    torch.cuda.synchronize()
    took = []
    for _ in range(passes):
        t = time.perf_counter()
        call()
        torch.cuda.synchronize()
        took.append(time.perf_counter() - t)
    return min(took) * 1e6


def uniform(lens, u, seed=0):
    rng = np.random.default_rng(seed)
    return wl.from_sets([rng.choice(u, size=k, replace=False).tolist() for k in lens],
                        rng.integers(1, 300, size=u).tolist(), u)


@pytest.mark.parametrize("m", [10, 100, 600])
def test_layouts_of_requests_up_to_the_rank_limit(m):
    """512 chunks per request: ranks; 513: the key sort."""
    took = {}
    for k in (512, 513):
        L = mpt.Layouts(uniform([k] * m, 5000, m))
        took[k] = best(lambda: L.global_order(mpt.MPT_ORDER_ID))
    print(f"[gpu] layouts m={m}: 512 chunks {took[512]:.0f} us, 513 {took[513]:.0f} us", flush=True)
    assert took[512] < 1.3 * took[513]


@pytest.mark.parametrize("m", [1, 2])
def test_orders_of_long_requests_up_to_the_slot_limit(m):
    """4096 slots: one launch; 4097: keys, their sort and the copy out."""
    took = {}
    for nnz in (4096, 4097):
        p = mpt.Problem(uniform([nnz - (m - 1) * (4096 // m)] + [4096 // m] * (m - 1), 5000, m))
        p.run()
        took[nnz] = best(p.extract)
    print(f"[gpu] orders m={m}: 4096 slots {took[4096]:.0f} us, 4097 {took[4097]:.0f} us", flush=True)
    assert took[4096] < 1.2 * took[4097]


@pytest.mark.parametrize("m", [10, 12])
def test_small_solves_of_large_totals(m):
    """sum_i w(R_i) of 2^49 (64-bit keys) and of 2^55 ((cost, part) pairs)."""
    took = {}
    for total in (1 << 49, 1 << 55):
        n = 1 << m
        f = np.zeros(n, dtype=np.int64)
        f[1 << np.arange(m)] = total // (2 * m)
        f[np.random.default_rng(m).integers(1, n, size=3 * m)] += total // (6 * m * m)
        for b in range(m):
            v = f.reshape(-1, 2, 1 << b)
            v[:, 0] += v[:, 1]
        W, ws = torch.as_tensor(f).cuda(), mpt.alloc_workspace(m, 0)
        C, S = torch.empty(n, dtype=torch.int64, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda")
        took[total] = best(lambda: mpt.mpt_solve_exact(m, W, C, S, ws))
    print(f"[gpu] small solves m={m}: {took[1 << 49]:.0f} us, large totals {took[1 << 55]:.0f} us", flush=True)
    assert took[1 << 55] < 2.2 * took[1 << 49]


def test_lists_of_long_requests_with_popular_chunks():
    """4000 requests of 30 chunks and one of 600, whose lists a key sort puts in
    order: four of the chunks held by everyone, or none by more than a few. The
    pair weights differ (their work is the demand), the lists must not."""
    took = {}
    rng = np.random.default_rng(1)
    for popular in (0, 4):
        u = 60000
        sets = [np.concatenate([np.arange(popular), popular + rng.choice(u - popular, size=k - popular, replace=False)])
                for k in [30] * 4000 + [600]]
        g = mpt.Greedy(wl.from_sets([s.tolist() for s in sets], rng.integers(1, 300, size=u).tolist(), u))
        g.pair_weights()
        spent = []
        for _ in range(10):
            mpt.profile_begin()
            g.pair_weights()
            spent.append(mpt.profile_end()["g_sort"]["total_ms"])
        took[popular] = min(spent) * 1e3
    print(f"[gpu] lists: {took[0]:.0f} us, with popular chunks {took[4]:.0f} us", flush=True)
    assert took[4] < 1.5 * took[0]


@pytest.mark.parametrize("k", [500, 2000])
def test_hierarchies_of_long_requests(k):
    """200 requests, few enough for one workgroup's rounds if they were short,
    and 230, which start on the whole chip."""
    took = {}
    for m in (200, 230):
        g = mpt.Greedy(uniform([k] * m, 2 * k, 3))
        took[m] = best(g.hierarchy, passes=8)
    print(f"[gpu] hierarchies k={k}: m=200 {took[200]:.0f} us, m=230 {took[230]:.0f} us", flush=True)
    assert took[200] < 1.4 * took[230]
