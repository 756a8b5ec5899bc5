"""The greedy's request and demand lists at the edges of their routes: a wave
per request up to 64 chunks, a workgroup up to 512, a key sort above; chunks
held by every request and by none, empty requests, one request. Pair weights,
merges and layout against the oracle; a repeated chunk, a bad id, a bad weight
and bad offsets refused on every route."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_13692_amd import mpt
from paper_2609_13692_amd import workloads as wl

pytestmark = pytest.mark.gpu


def family(lens, u, seed, hot=0):
    """hot: chunks 0 .. hot - 1 are in every request that has room."""
    rng = np.random.default_rng(seed)
    sets = []
    for k in lens:
        h = list(range(min(hot, k)))
        sets.append(rng.permutation(h + (hot + rng.choice(u - hot, size=k - len(h), replace=False)).tolist()).tolist())
    return wl.from_sets(sets, rng.integers(1, 300, size=u).tolist(), u)


CASES = {
    "one": ([5], 9, 0), "none": ([0, 0, 0], 4, 0), "wave": ([64, 63, 1, 0, 64] * 9, 300, 0),
    "list": ([65, 64, 2, 0, 300] * 7, 700, 3), "list_max": ([512, 511, 257, 255, 1, 0], 900, 2),
    "sort": ([513, 512, 40, 0, 2000, 7], 2500, 1), "hot": ([9] * 1500, 4000, 4), "wide": ([30] * 40, 200000, 0),
}


@pytest.mark.parametrize("name", list(CASES))
def test_against_the_oracle(name):
    lens, u, hot = CASES[name]
    inst = family(lens, u, len(name), hot)
    print(f"[gpu] greedy lists {name} m={inst.m} nnz={inst.nnz}", flush=True)
    g = mpt.Greedy(inst)
    got = g.run()
    got.update(g.host())
    ref = oracle.greedy_solve(inst)
    for k in ("P", "merge_a", "merge_b", "gain", "parent", "orders"):
        assert np.array_equal(got[k], ref[k]), k
    assert got["mst"] == ref["mst"] and got["request_total"] == int(inst.weights[inst.req_chunks].sum())


@pytest.mark.parametrize("longest", [40, 300, 600])
@pytest.mark.parametrize("what,name", [("dup", "MPT_E_DUP"), ("low", "MPT_E_RANGE"), ("high", "MPT_E_RANGE"),
                                       ("weight", "MPT_E_WEIGHT"), ("offsets", "MPT_E_INVALID"),
                                       ("end", "MPT_E_INVALID")])
def test_refusals(longest, what, name):
    inst = family([20, longest, 10, 30], 1000, longest)
    g = mpt.Greedy(inst)
    if what == "dup":
        g.req_chunks[20 + longest - 1] = g.req_chunks[20]
    elif what in ("low", "high"):
        g.req_chunks[25] = -1 if what == "low" else 1000
    elif what == "weight":
        g.chunk_w[999] = 0
    elif what == "offsets":
        g.req_off[2] = 19
    else:
        g.req_off[4] -= 1
    print(f"[gpu] greedy refuses {what} longest={longest}", flush=True)
    for call in (g.pair_weights, g.hierarchy):
        with pytest.raises(mpt.MptError) as e:
            call()
        assert e.value.name == name
