"""The greedy's remaining rounds in one workgroup, where it takes over: at once
for few short requests (m = 1 .. 222, either side of the rule at 221), after some
rounds of the whole chip, and never (a family whose clusters stay many); lists
of more than 64 chunks in its merges, on either side of the rule for long ones;
demand lists that keep their gaps (universes of more than 2^20 chunks); ties
everywhere. Against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_13692_amd import mpt
from paper_2609_13692_amd import workloads as wl

pytestmark = pytest.mark.gpu


def check(inst):
    print(f"[gpu] greedy tail {inst.name} m={inst.m}", flush=True)
    g = mpt.Greedy(inst)
    got = g.run()
    got.update(g.host())
    ref = oracle.greedy_solve(inst)
    for k in ("merge_a", "merge_b", "gain", "parent", "orders"):
        assert np.array_equal(got[k], ref[k]), k
    assert got["savings"] == ref["savings"] and got["mst"] == ref["mst"]


@pytest.mark.parametrize("m", [1, 2, 3, 63, 64, 65, 129, 220, 221, 222, 223, 300])
@pytest.mark.parametrize("wmax", [1, 500])
def test_sizes(m, wmax):
    check(wl.random_small(m=m, u=2 * m + 3, kmin=0, kmax=min(2 * m + 3, 14), wmax=wmax, seed=m))


@pytest.mark.parametrize("m,k", [(40, 65), (40, 200), (40, 800), (40, 900), (100, 140), (100, 150), (200, 500), (250, 130),
                                 (500, 64)])
def test_long_lists(m, k):
    check(wl.random_small(m=m, u=2 * k, kmin=k // 2, kmax=k, wmax=7, seed=k))


def test_many_clusters_left():
    """2500 pairs of equal requests that share nothing else: the first round
    leaves 2500 clusters, more than the tail holds, and no pair."""
    rng = np.random.default_rng(0)
    sets = [[2 * (i // 2), 2 * (i // 2) + 1] for i in range(5000)]
    order = rng.permutation(5000)
    check(wl.from_sets([sets[i] for i in order], [1] * 5000, 5000, "pairs"))


@pytest.mark.parametrize("m,k", [(300, 9), (500, 70)])
def test_demand_lists_with_gaps(m, k):
    """After rounds of the chip the tail walks demand lists in which merged
    clusters have left gaps: they are not closed for universes this large."""
    u = (1 << 20) + 4321
    small = wl.random_small(m=m, u=3 * k, kmin=k // 2, kmax=k, wmax=9, seed=m)
    place = np.random.default_rng(m).choice(u, size=3 * k, replace=False)
    w = np.ones(u, dtype=np.int64)
    w[place] = small.weights
    check(wl.Instance(u, w, small.req_off, place[small.req_chunks].astype(np.int32), "gaps"))


def test_chain_of_single_merges():
    """Nested requests with falling overlaps: one merge per round."""
    n = 260
    check(wl.from_sets([list(range(0, n - i)) for i in range(200)], [1] * n, n, "nested"))
