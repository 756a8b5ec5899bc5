"""The builds at the edges of their routes: one workgroup up to 16384 chunks
and 16384 slots with the W table (m up to 12), up to 16384 of both together
without it, several launches above; inputs in
device memory, in host memory (small and large) and inside the context's own
workspace. W and the demand sets against the oracle's; every refused input is
refused on either side of the limit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_13692_amd import mpt
from paper_2609_13692_amd import workloads as wl

pytestmark = pytest.mark.gpu
LIMIT = 16384


def family(m, u, nnz, seed, wmax=600):
    rng = np.random.default_rng(seed)
    lens = np.full(m, nnz // m)
    lens[: nnz % m] += 1
    return wl.from_sets([rng.choice(u, size=int(k), replace=False).tolist() for k in lens],
                        rng.integers(1, wmax + 1, size=u).tolist(), u)


def device(inst):
    return (torch.as_tensor(inst.weights, dtype=torch.int64).cuda(), torch.as_tensor(inst.req_off).cuda(),
            torch.as_tensor(inst.req_chunks, dtype=torch.int32).cuda())


def check(inst, W, sig):
    assert np.array_equal(W, oracle.intersection_weights(inst))
    assert np.array_equal(sig.view(np.uint32), oracle.demand_sets(inst))


SIZES = [(1, 1, 1), (2, 5, 0), (5, 0, 0), (12, LIMIT, LIMIT), (13, LIMIT, LIMIT), (12, LIMIT + 1, 100),
         (12, 9000, LIMIT + 1), (14, LIMIT + 1, LIMIT), (13, 9000, LIMIT + 1), (6, 70, 300), (16, 4095, 64), (17, 40000, 900),
         (13, LIMIT - 300, 300), (13, LIMIT - 299, 300), (19, 6000, LIMIT - 6000), (19, 6000, LIMIT - 5999)]


@pytest.mark.parametrize("m,u,nnz", SIZES)
def test_tables(m, u, nnz):
    inst = family(m, u, nnz, u + nnz)
    print(f"[gpu] build m={m} u={u} nnz={nnz}", flush=True)
    p = mpt.Problem(inst)
    p.build()
    check(inst, p.W.cpu().numpy(), p.sig.cpu().numpy()[:u])
    ctx = mpt.Context("cuda")
    ctx.reserve(m, u, nnz)
    for args in (device(inst), (torch.as_tensor(inst.weights), torch.as_tensor(inst.req_off),
                                torch.as_tensor(inst.req_chunks))):
        ctx.build_weights(m, u, *args)
        check(inst, ctx.copy_table(mpt.MPT_TABLE_W), ctx.copy_table(mpt.MPT_TABLE_SIG))
    # the instance the context keeps is the one it was given
    opt, _, _ = ctx.solve_exact()
    ref = oracle.solve(inst)
    assert opt == ref["opt"] and np.array_equal(ctx.extract_orders(), ref["orders"])
    ctx.close()


@pytest.mark.parametrize("m,u,nnz,one", [(12, LIMIT, LIMIT, True), (13, 8000, LIMIT - 8000, True),
                                         (13, 8000, LIMIT - 7999, False), (20, LIMIT, LIMIT, False)])
def test_one_workgroup_where_it_is_the_faster_side(m, u, nnz, one):
    """20 requests over 16384 chunks and slots: 65 us by one workgroup, 58 by
    the wide launches. The launches that ran, by their labels."""
    p = mpt.Problem(family(m, u, nnz, 1))
    p.build()
    mpt.profile_begin()
    p.build()
    labels = mpt.profile_end()
    assert ("build_init" not in labels) == one, labels


@pytest.mark.parametrize("m", [7, 13])
@pytest.mark.parametrize("nnz", [6, 4097, LIMIT, LIMIT + 1])
def test_slots_without_chunks(m, nnz):
    """An empty universe: request slots name no chunk. The build takes them on
    every route and W is 0; the stateless read-off refuses the ids, the
    context's, which looks at none, gives -1 for each."""
    off = np.minimum(np.arange(m + 1) * (nnz // 4), nnz)
    off[m] = nnz
    inst = wl.Instance(0, np.zeros(0, dtype=np.int64), off, np.arange(nnz, dtype=np.int32))
    print(f"[gpu] build without chunks m={m} nnz={nnz}", flush=True)
    p = mpt.Problem(inst)
    p.build()
    assert not p.W.any()
    assert p.solve() == 0
    with pytest.raises(mpt.MptError) as e:
        p.extract()
    assert e.value.name == "MPT_E_RANGE"
    for up in (lambda t: t, lambda t: t.cuda()):
        ctx = mpt.Context("cuda")
        ctx.reserve(m, 0, nnz)
        ctx.build_weights(m, 0, up(torch.as_tensor(inst.weights)), up(torch.as_tensor(inst.req_off)),
                          up(torch.as_tensor(inst.req_chunks)))
        assert not ctx.copy_table(mpt.MPT_TABLE_W).any()
        assert ctx.solve_exact()[:2] == (0, 0)
        assert (ctx.extract_orders() == -1).all()
        ctx.close()


def test_inputs_inside_the_workspace():
    """A rebuild on the context's own orders as request lists."""
    inst = family(9, 300, 200, 4)
    ctx = mpt.Context("cuda")
    ctx.run(inst)
    at, nbytes = ctx.table_device(mpt.MPT_TABLE_ORDERS)
    base = ctx.workspace.data_ptr()
    lists = ctx.workspace[at - base:at - base + nbytes].view(torch.int32)
    w, off, _ = device(inst)
    ctx.build_weights(inst.m, inst.n_chunks, w, off, lists)
    check(inst, ctx.copy_table(mpt.MPT_TABLE_W), ctx.copy_table(mpt.MPT_TABLE_SIG))
    ctx.close()


@pytest.mark.parametrize("u", [200, LIMIT + 200])
@pytest.mark.parametrize("m", [7, 13])
@pytest.mark.parametrize("what,name", [("offsets", "MPT_E_INVALID"), ("end", "MPT_E_INVALID"), ("low", "MPT_E_RANGE"),
                                       ("high", "MPT_E_RANGE"), ("dup", "MPT_E_DUP"), ("zero", "MPT_E_WEIGHT"),
                                       ("heavy", "MPT_E_WEIGHT"), ("unheld", "MPT_E_WEIGHT")])
def test_refusals(u, m, what, name):
    inst = family(m, u, 20 * m, 8)
    p = mpt.Problem(inst)
    if what == "offsets":
        p.req_off[2] = 19
    elif what == "end":
        p.req_off[m] = 20 * m - 1
    elif what in ("low", "high"):
        p.req_chunks[7] = -1 if what == "low" else u
    elif what == "dup":
        p.req_chunks[22] = p.req_chunks[21]
    elif what == "unheld":
        free = np.setdiff1d(np.arange(u), inst.req_chunks)
        p.chunk_w[int(free[-1])] = 0
    else:
        p.chunk_w[int(inst.req_chunks[3])] = 0 if what == "zero" else (1 << 32) + 1
    print(f"[gpu] build refuses {what} m={m} u={u}", flush=True)
    with pytest.raises(mpt.MptError) as e:
        p.build()
    assert e.value.name == name
    ctx = mpt.Context("cuda")
    ctx.reserve(m, u, inst.nnz)
    with pytest.raises(mpt.MptError) as e:
        ctx.build_weights(m, u, p.chunk_w, p.req_off, p.req_chunks)
    assert e.value.name == name
    ctx.close()
