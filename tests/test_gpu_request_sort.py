"""The lexicographic request sort on either side of its rule (ranks up to 4096
requests, tiles of 256 merged eight at a time above) and at the edges of tiles
and merges: equal sequences, proper prefixes, sequences that agree on their
first 8 chunks and differ later, empty ones. DFS order and trie cost against
Python's sort and the oracle; layouts of requests of 64 to 513 chunks (wave,
workgroup and key-sort orders, in place too); refusals leave no output."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_13692_amd import mpt
from paper_2609_13692_amd import workloads as wl

pytestmark = pytest.mark.gpu


def family(m, seed):
    """Sequences over few chunks: many ties at every depth."""
    rng = np.random.default_rng([m, seed])
    stems = [rng.permutation(40)[:9].tolist() for _ in range(6)]
    seqs = []
    for i in range(m):
        kind = int(rng.integers(5))
        if kind == 0:
            s = []
        elif kind == 1:
            s = stems[int(rng.integers(6))][:int(rng.integers(1, 10))]
        elif kind == 2:      # agrees on 9 chunks, then differs (or not)
            s = stems[int(rng.integers(6))] + (40 + rng.permutation(5)[:int(rng.integers(0, 4))]).tolist()
        else:
            s = rng.permutation(60)[:int(rng.integers(1, 5))].tolist()
        seqs.append([int(c) for c in s])
    return seqs


@pytest.mark.parametrize("m", [1, 255, 256, 257, 4095, 4096, 4097, 4352, 6000, 16384, 16385, 16641])
def test_dfs_order(m):
    seqs = family(m, 1)
    inst = wl.from_sets(seqs, np.arange(1, 61).tolist(), 60)
    print(f"[gpu] request sort m={m}", flush=True)
    L = mpt.Layouts(inst)
    cost = L.cost(L.seqs(inst.req_chunks))
    want = sorted(range(m), key=lambda i: (seqs[i], i))
    assert np.array_equal(L.dfs.cpu().numpy(), want)
    seen = {tuple(s[:j + 1]) for s in seqs for j in range(len(s))}
    assert cost == sum(int(inst.weights[t[-1]]) for t in seen)


def test_order_of_many_requests():
    """131073 short sequences: four merges, the last run one request long."""
    rng = np.random.default_rng(5)
    m = 131073
    lens = rng.integers(0, 4, size=m)
    off = np.zeros(m + 1, dtype=np.int64)
    np.cumsum(lens, out=off[1:])
    base = rng.integers(0, 300, size=m)
    flat = np.concatenate([(b + 300 * np.arange(k)) for b, k in zip(base, lens)]).astype(np.int32)
    inst = wl.Instance(1200, rng.integers(1, 9, size=1200), off, flat)
    print("[gpu] request sort m=131073", flush=True)
    L = mpt.Layouts(inst)
    L.cost(L.seqs(flat))
    key = np.where(lens > 0, base, -1)
    want = np.lexsort((np.arange(m), lens, key))
    assert np.array_equal(L.dfs.cpu().numpy(), want)


@pytest.mark.parametrize("m", [4096, 5000])
def test_cache_grid(m):
    inst = wl.gen_retrieval(m=m, u=3 * m, topics=m // 32, k=6, seed=3)
    lay = oracle.global_order_layout(inst, oracle.popularity_rank(inst))
    mx = max(int(inst.weights[inst.req_chunks[inst.req_off[i]:inst.req_off[i + 1]]].sum()) for i in range(m))
    # capacities below one request, of many, of all: distances that stop the
    # search early, at block edges and never
    win, cap = zip(*[(w, c) for w in (1, 7, 300, 0, m) for c in (0, mx // 2, mx, 9 * mx, 100 * mx, 10 ** 12)])
    print(f"[gpu] cache grid m={m}", flush=True)
    L = mpt.Layouts(inst, n_configs=len(win))
    got, unbounded = L.simulate(L.seqs(lay), win, cap)
    assert unbounded == oracle.trie_cost(inst, lay)
    assert got == [oracle.lru_cache_cost(inst, lay, oracle.window_schedule(inst, lay, w), c) for w, c in zip(win, cap)]


@pytest.mark.parametrize("longest", [64, 65, 512, 513])
def test_layouts_in_place(longest):
    inst = wl.random_small(m=70, u=900, kmin=longest, kmax=longest, wmax=9, seed=longest)
    print(f"[gpu] layouts of requests of {longest} chunks", flush=True)
    for kind, rank in ((mpt.MPT_ORDER_ID, oracle.id_rank(inst)), (mpt.MPT_ORDER_POPULARITY, oracle.popularity_rank(inst))):
        want = oracle.global_order_layout(inst, rank)
        L = mpt.Layouts(inst)
        assert np.array_equal(L.global_order(kind).cpu().numpy(), want)
        mpt.mpt_global_order_layout(L.m, L.n_chunks, L.req_off, L.req_chunks, kind, L.req_chunks, L.workspace)
        assert np.array_equal(L.req_chunks.cpu().numpy(), want)


@pytest.mark.parametrize("m", [50, 5000])
@pytest.mark.parametrize("what,name", [("offsets", "MPT_E_INVALID"), ("end", "MPT_E_INVALID"), ("low", "MPT_E_RANGE"),
                                       ("high", "MPT_E_RANGE"), ("weight", "MPT_E_WEIGHT")])
def test_refusals(m, what, name):
    inst = wl.random_small(m=m, u=100, kmin=3, kmax=3, wmax=9, seed=m)
    L = mpt.Layouts(inst, n_configs=1)
    if what == "offsets":
        L.req_off[7] = 25               # above req_off[8] = 24
    elif what == "end":
        L.req_off[m] -= 1
    elif what in ("low", "high"):
        L.req_chunks[40] = -1 if what == "low" else 100
    else:
        L.chunk_w[int(inst.req_chunks[11])] = 0
    L.dfs.fill_(-3)
    print(f"[gpu] layouts refuse {what} m={m}", flush=True)
    calls = [lambda: L.cost(L.req_chunks), lambda: L.simulate(L.req_chunks, [0], [5])]
    if what != "weight":
        calls += [lambda: L.global_order(mpt.MPT_ORDER_ID), lambda: L.global_order(mpt.MPT_ORDER_POPULARITY)]
    for call in calls:
        with pytest.raises(mpt.MptError) as e:
            call()
        assert e.value.name == name
    assert (L.dfs == -3).all()
