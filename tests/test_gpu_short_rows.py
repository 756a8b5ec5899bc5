"""The exact DP on 2^9-entry rows (m = 13 .. 23, cross pairs chunked by the
library) at its limits: the smallest m, levels completed in one launch and in
two (m = 16 .. 18), the largest m, the three key widths and instances full of
ties. Integer results: compared exactly with the oracle, and for larger m
with the 2^12-entry rows, which a context with MPT_OPT_CHUNK_PAIRS takes."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_13692_amd import mpt
from paper_2609_13692_amd import workloads as wl

pytestmark = pytest.mark.gpu


def instance(m, width, seed, ties=False):
    """Weights scaled by a power of two until sum_i w(R_i) is in the range of
    the width; at the smallest m, where weights of at most 2^32 reach 64-bit
    keys only so, with longer requests."""
    rng = np.random.default_rng([seed, m])
    long = width == "u64" and m < 15
    u = (20 if long else 10) if ties else 12 * m
    longest = min(u, 70 if long else 14)
    sets = [rng.choice(u, size=int(rng.integers(0 if ties else 1, longest)), replace=False).tolist() for _ in range(m)]
    w = np.ones(u, dtype=np.int64) if ties else rng.integers(1, 400, size=u, dtype=np.int64)
    total = int(sum(w[s].sum() for s in sets))
    least, most = {"u32": (0, (1 << 20) - 1), "f64": ((1 << 20) - 1, 1 << (51 - m)), "u64": (1 << (51 - m), 1 << (61 - m))}[width]
    scale = 1
    while total * scale < least and int(w.max()) * scale <= 1 << 31:
        scale *= 2
    assert least <= total * scale < most, (m, width, ties)
    return wl.from_sets(sets, w * scale, u)


def tables(inst, chunk_pairs=0):
    ctx = mpt.Context("cuda")
    if chunk_pairs:
        ctx.set_option(mpt.MPT_OPT_CHUNK_PAIRS, chunk_pairs)
    ctx.reserve(inst.m, inst.n_chunks, inst.nnz)
    ctx.build_weights(inst.m, inst.n_chunks, torch.as_tensor(inst.weights), torch.as_tensor(inst.req_off),
                      torch.as_tensor(inst.req_chunks))
    opt, _, _ = ctx.solve_exact()
    out = opt, ctx.copy_table(mpt.MPT_TABLE_C)[1:], ctx.copy_table(mpt.MPT_TABLE_SPLIT)
    ctx.close()
    return out


WIDTHS = ["u32", "f64", "u64"]


@pytest.mark.parametrize("m", [13, 14, 16, 17])
@pytest.mark.parametrize("width", WIDTHS)
@pytest.mark.parametrize("ties", [False, True])
def test_against_the_oracle(m, width, ties):
    inst = instance(m, width, 3, ties)
    total = int(inst.weights[inst.req_chunks].sum())
    assert total < 1 << (61 - m)
    print(f"[gpu] short rows m={m} total={total}", flush=True)
    opt, C, split = tables(inst)
    ref = oracle.solve(inst)
    assert opt == ref["opt"]
    assert np.array_equal(C, ref["C"][1:])
    assert np.array_equal(split, ref["split"].astype(np.uint32))


@pytest.mark.parametrize("m", [18, 20, 21, 22, 23])
@pytest.mark.parametrize("width", WIDTHS)
@pytest.mark.parametrize("ties", [False, True])
def test_against_the_long_rows(m, width, ties):
    inst = instance(m, width, 4, ties)
    print(f"[gpu] short rows m={m} width={width}", flush=True)
    a, b = tables(inst), tables(inst, chunk_pairs=64)
    assert a[0] == b[0]
    assert np.array_equal(a[1], b[1])
    assert np.array_equal(a[2], b[2])


def test_where_the_long_rows_are_faster():
    """64-bit keys at m = 22 (2750 us on 2^12-entry rows, 2808 on short ones):
    the kernels that ran, by their labels."""
    for m, width, wide in ((21, "u64", False), (22, "u64", True), (22, "f64", False), (23, "u64", False),
                           (24, "u32", True)):
        inst = instance(m, width, 5)
        prob = mpt.Problem(inst)
        prob.build()
        print(f"[gpu] rows m={m} width={width}", flush=True)
        mpt.profile_begin()
        prob.solve()
        labels = mpt.profile_end()
        assert f"rb_cross_{width}" in labels
        assert ("rb_unpack" in labels) == wide, (m, width)


@pytest.mark.parametrize("m", [13, 15])
def test_element_aligned_tables(m):
    """C and split one element past a 16-byte boundary."""
    inst = instance(m, "u32", 6)
    prob = mpt.Problem(inst)
    prob.build()
    C = torch.full(((1 << m) + 1,), -7, dtype=torch.int64, device="cuda")[1:]
    S = torch.full(((1 << m) + 1,), -7, dtype=torch.int32, device="cuda")[1:]
    opt = mpt.mpt_solve_exact(m, prob.W, C, S, prob.workspace)
    ref = oracle.solve(inst)
    assert opt == ref["opt"] and int(C[0]) == mpt.MPT_COST_SENTINEL
    assert np.array_equal(C.cpu().numpy()[1:], ref["C"][1:])
    assert np.array_equal(S.cpu().numpy().view(np.uint32), ref["split"])
