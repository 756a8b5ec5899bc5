"""The one-workgroup DP: whole instances of m <= 12 requests (mpt_solve_exact
on a W table, every m) and row 0 of larger ones, at the limits of its key
widths: sum_i w(R_i) of 2^20 - 2 and 2^20 - 1 (32-bit / 64-bit keys) and
2^50 - 1 and 2^50 (64-bit keys / (cost, part) pairs). Integer results,
compared exactly with the oracle's DP on the same table."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_13692_amd import mpt

pytestmark = pytest.mark.gpu


def table(m, total, seed, sparse=False):
    """A W table with sum_i W({i}) = total: superset sums of a few weighted
    demand sets; unit sets of weight 0 or more make up the total."""
    rng = np.random.default_rng([seed, m])
    n = 1 << m
    f = np.zeros(n, dtype=np.int64)
    left = total
    for _ in range(0 if sparse else 3 * m):
        s = int(rng.integers(1, n))
        w = int(rng.integers(0, max(1, total // (4 * m * m))))
        f[s] += w
        left -= w * bin(s).count("1")
    f[1 << int(rng.integers(0, m))] += left          # (left > 0: at most 3/4 of the total is spent)
    assert left > 0
    for b in range(m):
        v = f.reshape(-1, 2, 1 << b)
        v[:, 0] += v[:, 1]
    assert sum(int(f[1 << i]) for i in range(m)) == total
    return f


TOTALS = [1, 700, (1 << 20) - 2, (1 << 20) - 1, (1 << 41) + 12345, (1 << 50) - 1, 1 << 50, (1 << 60) + 987654321]


@pytest.mark.parametrize("total", TOTALS, ids=lambda t: f"total={t}")
def test_every_small_m_at_every_width(total):
    for m in range(1, 13):
        W = table(m, total, 5, sparse=total < 100)
        print(f"[gpu] row dp m={m} total={total}", flush=True)
        dev = torch.as_tensor(W).cuda()
        # (C and split one element past a 16-byte boundary: element alignment is enough)
        C = torch.full((W.size + 1,), -7, dtype=torch.int64, device="cuda")[1:]
        S = torch.full((W.size + 1,), -7, dtype=torch.int32, device="cuda")[1:]
        opt = mpt.mpt_solve_exact(m, dev, C, S, mpt.alloc_workspace(m, 0))
        M, split = oracle.exact_dp(m, W)
        ref = oracle.cost_table(m, W, M)
        assert opt == ref[-1]
        assert int(C[0]) == mpt.MPT_COST_SENTINEL
        assert np.array_equal(C.cpu().numpy()[1:], ref[1:]), (m, total)
        assert np.array_equal(S.cpu().numpy().view(np.uint32), split), (m, total)


def test_ties_of_large_totals():
    """Costs that are small multiples of 2^48: (cost, part) pairs, many equal
    costs, the smallest part of each."""
    for m in range(2, 13):
        W = table(m, 40, 5, sparse=True) << 48
        W[: 1 << (m - 1)] += 1 << 48                  # (one chunk that all but the last request hold)
        print(f"[gpu] row dp ties m={m}", flush=True)
        dev = torch.as_tensor(W).cuda()
        C = torch.empty(W.size, dtype=torch.int64, device="cuda")
        S = torch.empty(W.size, dtype=torch.int32, device="cuda")
        mpt.mpt_solve_exact(m, dev, C, S, mpt.alloc_workspace(m, 0))
        M, split = oracle.exact_dp(m, W)
        assert np.array_equal(C.cpu().numpy()[1:], oracle.cost_table(m, W, M)[1:]), m
        assert np.array_equal(S.cpu().numpy().view(np.uint32), split), m


@pytest.mark.parametrize("m", [13, 14])
@pytest.mark.parametrize("total", [700, (1 << 20) - 1, (1 << 46) + 3])
def test_row0_of_larger_instances(m, total):
    W = table(m, total, 9)
    print(f"[gpu] row 0 m={m} total={total}", flush=True)
    dev = torch.as_tensor(W).cuda()
    C = torch.empty(W.size, dtype=torch.int64, device="cuda")
    S = torch.empty(W.size, dtype=torch.int32, device="cuda")
    mpt.mpt_solve_exact(m, dev, C, S, mpt.alloc_workspace(m, 0))
    M, split = oracle.exact_dp(m, W)
    ref = oracle.cost_table(m, W, M)
    assert np.array_equal(C.cpu().numpy()[1:], ref[1:])
    assert np.array_equal(S.cpu().numpy().view(np.uint32), split)
