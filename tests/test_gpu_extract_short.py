"""The order read-off at the edges of its one-launch route (at most 4096
request slots; 256 threads per request up to 1024, 1024 above): 1023 to 1025 and
4095 to 4097 slots; requests of 0, 1, 128 (ranks), 129 (tile sort), a wave's 256
keys and the merges' 512 and 1024, and of 4096 chunks; the stateless call and the
context. Orders
against the oracle's, and nothing written when the input is refused."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_13692_amd import mpt
from paper_2609_13692_amd import workloads as wl

pytestmark = pytest.mark.gpu


def family(lens, u, seed):
    rng = np.random.default_rng(seed)
    return wl.from_sets([rng.choice(u, size=k, replace=False).tolist() for k in lens],
                        rng.integers(1, 50, size=u).tolist(), u)


LENS = [[0], [1], [0, 0, 3], [512, 513, 1, 0], [511, 512, 513, 514, 700, 1, 2], [4095], [4096], [4097],
        [127, 128, 129, 130], [255, 256, 257], [511, 512], [511, 513], [1023, 0, 1], [1024], [1025], [1026, 128, 129], [3000],
        [2048, 2048], [2048, 2049], [1500, 0, 1500, 1000, 96], [63] * 12 + [900]]


@pytest.mark.parametrize("lens", LENS, ids=str)
def test_orders(lens):
    inst = family(lens, 5000, len(lens) + sum(lens))
    print(f"[gpu] extract {lens}", flush=True)
    ref = oracle.solve(inst)
    p = mpt.Problem(inst)
    p.run()
    assert np.array_equal(p.host_tables()["orders"], ref["orders"])
    ctx = mpt.Context("cuda")
    assert np.array_equal(ctx.run(inst)["orders"], ref["orders"])
    ctx.close()


@pytest.mark.parametrize("what", ["offsets", "split", "chunk"])
def test_refused_input_leaves_the_orders_alone(what):
    inst = family([30, 20, 40, 10, 5], 200, 3)
    p = mpt.Problem(inst)
    p.run()
    p.orders.fill_(-5)
    if what == "offsets":
        p.req_off[2] = 29               # below req_off[1] = 30
    elif what == "split":
        p.split[31] = 31
    else:
        p.req_chunks[-1] = 200
    print(f"[gpu] extract refuses {what}", flush=True)
    with pytest.raises(mpt.MptError) as e:
        p.extract()
    assert e.value.name == ("MPT_E_RANGE" if what == "chunk" else "MPT_E_INVALID")
    assert (p.orders == -5).all()
