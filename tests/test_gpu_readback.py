"""Results and small host instances that travel through the pinned blocks
(16 KiB each, a pool of 32): at the block's size, just past it, and from
several threads and streams at a time. Compared exactly with the oracle."""
import threading

import numpy as np
import pytest
import torch

import oracle
from paper_2609_13692_amd import mpt
from paper_2609_13692_amd import workloads as wl

pytestmark = pytest.mark.gpu


def instance(m, u, k, seed):
    rng = np.random.default_rng([seed, m, u])
    return wl.from_sets([rng.choice(u, size=k, replace=False).tolist() for _ in range(m)],
                        rng.integers(1, 300, size=u, dtype=np.int64), u)


def check(got, inst):
    ref = oracle.solve(inst)
    assert got["opt"] == ref["opt"]
    assert got["savings"] == int(inst.weights[inst.req_chunks].sum()) - ref["opt"]
    assert np.array_equal(np.asarray(got["orders"]), np.asarray(ref["orders"]))


# orders of 16380, 16384 and 16388 bytes; then host instances around 16 KiB
# (8 (m + 1) + 4 nnz + 8 u, each padded to 256 bytes)
@pytest.mark.parametrize("m,u,k", [(5, 1500, 819), (4, 1500, 1024), (1, 5000, 4097), (7, 1800, 20), (7, 1952, 20),
                                   (7, 2100, 20)])
def test_sizes_around_a_block(m, u, k):
    inst = instance(m, u, k, 1)
    print(f"[gpu] read-back m={m} u={u} nnz={inst.nnz}", flush=True)
    ctx = mpt.Context("cuda")
    check(ctx.run(inst), inst)
    check(ctx.run((inst.m, inst.n_chunks, torch.as_tensor(inst.weights).cuda(), torch.as_tensor(inst.req_off).cuda(),
                   torch.as_tensor(inst.req_chunks).cuda())), inst)
    ctx.close()


def test_threads_and_streams():
    insts = [[instance(4 + t % 5, 60 + 300 * i, 6 + t, 10 * t + i) for i in range(4)] for t in range(8)]
    failed = []

    def work(t):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                ctx = mpt.Context("cuda")
                for _ in range(5):
                    for inst in insts[t]:
                        check(ctx.run(inst), inst)
                        g = mpt.Greedy(inst)
                        out = g.run()
                        assert out["savings"] == int(g.gain[:inst.m - 1].sum())
                ctx.close()
        except BaseException as e:      # reported by the main thread
            failed.append((t, repr(e)))

    threads = [threading.Thread(target=work, args=(t,)) for t in range(len(insts))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed
