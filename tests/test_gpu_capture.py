"""Calls that return no host data, captured into a HIP graph: a context's solve
and read-off (one workgroup, short rows, long rows; one launch and key sort),
and the allocation-free solve of up to 12 requests. Every replay, with the
tables overwritten and other work in between, against the eager result."""
import numpy as np
import pytest
import torch

from paper_2609_13692_amd import mpt
from paper_2609_13692_amd import workloads as wl

pytestmark = pytest.mark.gpu
TABLES = (mpt.MPT_TABLE_C, mpt.MPT_TABLE_SPLIT, mpt.MPT_TABLE_ORDERS)


def instance(m, k):
    rng = np.random.default_rng([m, k])
    u = 3 * k + 40 * m
    return wl.from_sets([rng.choice(u, size=k, replace=False).tolist() for _ in range(m)],
                        rng.integers(1, 300, size=u).tolist(), u)


@pytest.mark.parametrize("m,k", [(9, 6), (12, 500), (16, 20), (21, 30), (24, 20)])
def test_context_solve_and_orders(m, k):
    inst = instance(m, k)
    s = torch.cuda.Stream()
    ctx = mpt.Context("cuda", s)
    with torch.cuda.stream(s):
        ctx.reserve(m, inst.n_chunks, inst.nnz)
        ctx.build_weights(m, inst.n_chunks, torch.as_tensor(inst.weights), torch.as_tensor(inst.req_off),
                          torch.as_tensor(inst.req_chunks))
        ctx.solve_exact(want_cost=False)
        ctx.extract_orders(to_host=False)
    want = [ctx.copy_table(t) for t in TABLES]
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=s):
        ctx.solve_exact(want_cost=False)
        ctx.extract_orders(to_host=False)
    base = ctx.workspace.data_ptr()
    for i in range(3):
        for t in TABLES:
            at, nbytes = ctx.table_device(t)
            ctx.workspace[at - base:at - base + nbytes].fill_(i + 1)
        eager = mpt.Problem(instance(8, 5)).run()
        torch.cuda.synchronize()
        print(f"[gpu] replay {i} m={m}", flush=True)
        graph.replay()
        torch.cuda.synchronize()
        assert eager == mpt.Problem(instance(8, 5)).run()
        for t, ref in zip(TABLES, want):
            got = ctx.copy_table(t)
            assert np.array_equal(got, ref), (t, i)
    assert ctx.optimum()[0] == int(want[0][-1])
    ctx.close()


@pytest.mark.parametrize("m", [3, 9, 12])
def test_allocation_free_solve(m):
    p = mpt.Problem(instance(m, 9))
    p.build()
    opt = p.solve()
    C, S = torch.empty_like(p.C), torch.empty_like(p.split)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        mpt.mpt_solve_exact_noalloc(m, p.W, C, S, s, want_cost=False)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        mpt.mpt_solve_exact_noalloc(m, p.W, C, S, s, want_cost=False)
    for i in range(3):
        C.fill_(i)
        S.fill_(i)
        assert p.solve() == opt
        torch.cuda.synchronize()
        print(f"[gpu] replay {i} m={m}", flush=True)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(C, p.C) and torch.equal(S, p.split)
