// libmpt.so, Sections 7-8 of "Prefix Sharing Is a Sorting Problem":
// layouts, serving schedules and the radix cache.
//   mpt_global_order_layout  every request sorted by one chunk order: chunk
//                            id, or popularity (the global-order baselines)
//   mpt_layout_cost          trie cost (Eq. 1) of any layout, and the DFS
//                            serving order of its trie (Theorem 7)
//   mpt_cache_simulate       the prefill bill of serving a layout through a
//                            radix cache with least-recently-used leaf
//                            eviction, for many (reorder window, capacity)
//                            pairs at once (Section 8, 8.1)
//
// Trie cost. Sorted lexicographically, request s shares with all earlier
// requests exactly the longest common prefix (LCP) with its predecessor, so
// it adds the trie nodes past that LCP: the cost is a sum over requests of
// the weights past their LCP, and the sorted order is a DFS order of the
// trie. Nodes get ids in that order.
//
// Radix cache. Serving a request touches its whole path, so an ancestor is
// never older than a descendant, and the least-recently-used leaf is the
// deepest of the least-recently-used nodes: the policy is plain LRU over
// nodes, with each request's path touched from the leaf up. Such a cache
// always holds the longest prefix of its recency stack that fits, so an
// access hits iff the distinct weight accessed since its node's previous
// access, plus its own, fits the capacity. That stack distance does not
// depend on the capacity: configurations with the same window share one
// schedule, one access log and one pass that prices all their capacities,
// every log entry on its own thread.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <vector>

#include "common.h"
#include "keysort.h"
#include "mpt.h"
#include "seqsort.h"

namespace {

using mptlib::align256;
using mptlib::fail;
using mptlib::grid_for;
using mptlib::kListMax;
using mptlib::kListThreads;
using mptlib::kSegMax;
using mptlib::list_ranks;
using mptlib::LaunchScope;
using mptlib::seg_rank;
using mptlib::sort_keys;
using mptlib::seq_recs_bytes;
using mptlib::sort_requests;

constexpr int kWave = 64;

enum : uint32_t { LERR_INVALID = 1u, LERR_RANGE = 2u, LERR_WEIGHT = 8u, LERR_OVERFLOW = 16u };

struct LHeader {
    uint32_t err;
    uint32_t pad0;
    unsigned long long total;   // sum of the sequence weights
    unsigned long long cost;    // trie cost
    int64_t max_len;            // longest sequence
    int64_t pad[28];
};
static_assert(sizeof(LHeader) == 256, "header is one 256-byte block");

inline int64_t pow2_at_least(int64_t n) {
    int64_t p = 1;
    while (p < n) p <<= 1;
    return p;
}

struct LLayout {
    size_t ord, rank, recs, lcp, base, pn, nw, mtree, crank, cinv, keys, keys2, sched, log_off, logs, acc_start, prev, next, wsuf,
        snext, ssum, bnext, bsum, cfg_win, cfg_cap, cfg_off, cfg_list, costs, total;
    int64_t mpad;
};

// nnz bounds the trie's node count
LLayout l_layout(int m, int64_t n_chunks, int64_t nnz, int n_cfg) {
    LLayout L{};
    const size_t mm = (size_t)m, nz = (size_t)std::max<int64_t>(nnz, 1), nc = (size_t)std::max(n_cfg, 0);
    L.mpad = std::max<int64_t>(pow2_at_least(m), 1024);      // leaves of the segment tree
    // the most keys of one sort (two buffers)
    const size_t kn = (size_t)std::max(std::max<int64_t>(nnz, n_chunks), (int64_t)nc * std::max<int64_t>(m, nnz));
    const size_t nblk = (nz + 1023) / 1024;     // big sorted blocks of the access logs (kBigBlock entries)
    size_t o = align256(sizeof(LHeader));
    auto take = [&](size_t bytes) { size_t at = o; o = align256(o + std::max<size_t>(bytes, 1)); return at; };
    L.ord = take(4 * mm);
    L.rank = take(4 * mm);
    L.lcp = take(4 * mm);
    L.base = take(8 * (mm + 1));
    L.pn = take(4 * nz);
    L.nw = take(8 * nz);
    L.mtree = take(8 * (size_t)L.mpad);          // min segment tree over the LCPs
    L.crank = take(4 * (size_t)n_chunks);
    L.cinv = take(4 * (size_t)n_chunks);
    L.sched = take(4 * nc * mm);
    L.log_off = take(8 * nc * mm);
    L.logs = take(4 * nc * nz);
    L.acc_start = take(4 * nc * nz);
    L.prev = take(4 * nc * nz);
    L.next = take(4 * nc * nz);
    // the request sort is over before the first key sort, and those before the
    // sorted blocks of the logs are written
    const size_t shared = o;
    L.recs = take(2 * seq_recs_bytes(m));
    const size_t recs_end = o;
    o = shared;
    L.keys = take(8 * kn);
    L.keys2 = take(8 * kn);
    const size_t sorts_end = std::max(o, recs_end);
    o = shared;
    L.wsuf = take(8 * nc * nz);
    L.snext = take(4 * nc * nblk * 1024);
    L.ssum = take(8 * nc * nblk * 1024);
    L.bnext = take(4 * nc * nblk * 1024);
    L.bsum = take(8 * nc * nblk * 1024);
    o = std::max(o, sorts_end);
    L.cfg_win = take(8 * nc);
    L.cfg_cap = take(8 * nc);
    L.cfg_off = take(4 * (nc + 1));
    L.cfg_list = take(4 * nc);
    L.costs = take(8 * nc);
    L.total = o;
    return L;
}

// ---------------------------------------------------------------------------
// validation

// header and, where given, zero[0 .. n)
__global__ void k_l_begin(LHeader *h, int32_t *zero, int64_t n) {
    if (blockIdx.x == 0 && threadIdx.x == 0) { h->err = 0; h->total = 0; h->cost = 0; h->max_len = 0; }
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) zero[i] = 0;
}

constexpr int kCheckThreads = 256;
// the sum of v over the workgroup, on thread 0
__device__ inline uint64_t check_block_sum(uint64_t v, uint64_t (&red)[kCheckThreads / kWave]) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = v;
    __syncthreads();
    uint64_t sum = 0;
    for (int k = 0; k < kCheckThreads / kWave; ++k) sum += red[k];
    return sum;
}

// offsets, chunk ids and (w given) weights, the longest sequence and the total
// weight: one addition per workgroup (one per slot on the total's address was
// 25 us at 160088 slots, and the offsets on one workgroup 18 us)
__global__ __launch_bounds__(kCheckThreads) void k_l_check(int m, int64_t nnz, int64_t n_chunks,
                                                           const int64_t *__restrict__ off,
                                                           const int32_t *__restrict__ seqs,
                                                           const int64_t *__restrict__ w, LHeader *h) {
    __shared__ uint64_t red[kCheckThreads / kWave];
    const int64_t t0 = blockIdx.x * (int64_t)kCheckThreads + threadIdx.x, stride = (int64_t)gridDim.x * kCheckThreads;
    uint32_t err = 0;
    int64_t longest = 0;
    for (int64_t i = t0; i < m; i += stride) {
        const int64_t len = off[i + 1] - off[i];
        if (len < 0) err |= LERR_INVALID;
        longest = len > longest ? len : longest;
    }
    if (t0 == 0 && (off[0] != 0 || off[m] != nnz)) err |= LERR_INVALID;
    uint64_t total = 0;
    for (int64_t j = t0; j < nnz; j += stride) {
        const int32_t x = seqs[j];
        if (x < 0 || (int64_t)x >= n_chunks) { err |= LERR_RANGE; continue; }
        if (!w) continue;
        const int64_t wx = w[x];
        if (wx <= 0 || wx > MPT_MAX_CHUNK_WEIGHT) err |= LERR_WEIGHT;
        else total += (uint64_t)wx;
    }
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        const int64_t l = __shfl_xor(longest, o, kWave);
        longest = l > longest ? l : longest;
        err |= (uint32_t)__shfl_xor((int)err, o, kWave);
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        if (err) atomicOr(&h->err, err);
        if (longest > 0) atomicMax((long long *)&h->max_len, (long long)longest);
    }
    total = check_block_sum(total, red);
    if (threadIdx.x == 0 && total) atomicAdd(&h->total, (unsigned long long)total);
}

int l_read_errors(LHeader *h, hipStream_t s, int64_t *max_len = nullptr, int64_t *cost = nullptr) {
    LHeader hh;
    MPT_HIP_TRY(mptlib::read_back(&hh, h, sizeof hh, s));
    if (hh.err & LERR_INVALID) return fail(MPT_E_INVALID, "offsets are not a CSR offset array of length m+1 ending at nnz");
    if (hh.err & LERR_RANGE) return fail(MPT_E_RANGE, "a chunk id is outside [0, n_chunks)");
    if (hh.err & LERR_WEIGHT) return fail(MPT_E_WEIGHT, "a chunk weight is <= 0 or > 2^32");
    if (hh.total >= (1ull << 61)) return fail(MPT_E_OVERFLOW, "sum of sequence weights reaches 2^61");
    if (max_len) *max_len = hh.max_len;
    if (cost) *cost = (int64_t)hh.cost;
    return MPT_OK;
}

// ---------------------------------------------------------------------------
// global-order layouts

__global__ void k_l_fill_u64(uint64_t *p, int64_t n, uint64_t v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

// Demand of every chunk (into the rank array, zeroed). Popular chunks repeat
// in a quarter of the requests, and atomics on one address serialise
// device-wide (70 us at 160088 slots, one per slot), so each workgroup counts
// its slice in an LDS hash table first (linear probing; a slot that finds no
// entry is counted in memory directly).
constexpr int kCountThreads = 1024;
constexpr int kCountSlice = 4096;
constexpr int kCountBits = 13;
constexpr int kCountEntries = 1 << kCountBits;
constexpr int kCountProbes = 16;
__global__ __launch_bounds__(kCountThreads) void k_l_count(int64_t nnz, const int32_t *__restrict__ chunks,
                                                           int32_t *cnt, const LHeader *h) {
    __shared__ uint32_t key[kCountEntries], num[kCountEntries];     // chunk + 1 (0: empty), its slots
    if (h->err) return;
    for (int64_t s0 = (int64_t)blockIdx.x * kCountSlice; s0 < nnz; s0 += (int64_t)gridDim.x * kCountSlice) {
        for (int e = (int)threadIdx.x; e < kCountEntries; e += kCountThreads) { key[e] = 0u; num[e] = 0u; }
        __syncthreads();
        for (int64_t j = s0 + threadIdx.x; j < s0 + kCountSlice && j < nnz; j += kCountThreads) {
            const uint32_t x = (uint32_t)chunks[j];
            uint32_t slot = (x * 2654435761u) >> (32 - kCountBits);
            bool done = false;
            for (int p = 0; p < kCountProbes && !done; ++p) {
                uint32_t k = *(volatile uint32_t *)&key[slot];      // (most find their chunk there)
                if (k == 0u) k = atomicCAS(&key[slot], 0u, x + 1u);
                if (k == 0u || k == x + 1u) {
                    atomicAdd(&num[slot], 1u);
                    done = true;
                }
                slot = (slot + 1u) & (kCountEntries - 1u);
            }
            if (!done) atomicAdd(&cnt[x], 1);
        }
        __syncthreads();
        for (int e = (int)threadIdx.x; e < kCountEntries; e += kCountThreads)
            if (key[e]) atomicAdd(&cnt[key[e] - 1u], (int32_t)num[e]);
        __syncthreads();
    }
}

// popularity key of chunk x: demand descending, then id ascending
__global__ void k_l_pop_keys(int64_t n_chunks, const int32_t *cnt, uint64_t *keys) {
    for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < n_chunks; x += (int64_t)gridDim.x * blockDim.x)
        keys[x] = ((uint64_t)(0x7fffffffu - (uint32_t)cnt[x]) << 32) | (uint32_t)x;
}

// sorted popularity keys -> rank[x]
__global__ void k_l_pop_rank(int64_t n_chunks, const uint64_t *keys, int32_t *rank) {
    for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < n_chunks; r += (int64_t)gridDim.x * blockDim.x)
        rank[(uint32_t)(keys[r] & 0xffffffffu)] = (int32_t)r;
}

// key of slot j: its request in the high 32 bits, the chunk's position in
// the order in the low 32 bits (for the id order the position is the id)
__global__ void k_l_layout_keys(int m, int64_t nnz, const int64_t *req_off, const int32_t *chunks,
                                const int32_t *rank, int kind, uint64_t *keys) {
    for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < nnz; j += (int64_t)gridDim.x * blockDim.x) {
        int lo = 0, hi = m - 1;                 // request of slot j
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (req_off[mid] <= j) lo = mid; else hi = mid - 1;
        }
        const uint32_t x = (uint32_t)chunks[j];
        const uint32_t r = kind == MPT_ORDER_ID ? x : (uint32_t)rank[x];
        keys[j] = ((uint64_t)lo << 32) | r;
    }
}

// sorted keys -> sequences (position -> chunk through the inverse of rank)
__global__ void k_l_layout_out(int64_t nnz, const uint64_t *keys, const int32_t *inv, int kind, int32_t *seqs) {
    for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < nnz; j += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t r = (uint32_t)(keys[j] & 0xffffffffu);
        seqs[j] = kind == MPT_ORDER_ID ? (int32_t)r : inv[r];
    }
}

// the layout when every request has at most kListMax chunks: a wave per
// request (up to kSegMax chunks) or a workgroup per request orders its chunks
// by their position in the order (the id, or the popularity rank), ties by
// slot. With longer requests, or an error, nothing is done (the key sort's).
__global__ __launch_bounds__(kListThreads) void k_l_layout_short(int m, const int64_t *__restrict__ req_off,
                                                                 const int32_t *chunks,
                                                                 const int32_t *__restrict__ rank, int kind,
                                                                 int32_t *seqs, const LHeader *h) {
    __shared__ __align__(16) uint32_t stage[kListMax];
    if (h->err || h->max_len > kListMax) return;
    auto place = [&](int32_t x) { return kind == MPT_ORDER_ID ? (uint32_t)x : (uint32_t)rank[x]; };
    if (h->max_len <= kSegMax) {
        const int lane = (int)(threadIdx.x & (kWave - 1));
        const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) / kWave;
        for (int64_t i = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kWave; i < m; i += nwaves) {
            const int64_t o = req_off[i];
            const int n = (int)(req_off[i + 1] - o);
            const int32_t x = lane < n ? chunks[o + lane] : 0;
            bool dup;
            const int pos = seg_rank(lane < n ? place(x) : 0u, n, dup);
            if (lane < n) seqs[o + pos] = x;
        }
        return;
    }
    for (int64_t i = blockIdx.x; i < m; i += gridDim.x) {
        const int64_t o = req_off[i];
        // the chunks themselves, held until all of the request's are read
        int32_t x[kListMax / kListThreads];
        const int n = (int)(req_off[i + 1] - o);
        int q = 0;
        list_ranks(stage, n,
                   [&](int e) {
                       x[q] = chunks[o + e];
                       return place(x[q++]);
                   },
                   [&](int e, uint32_t, int pos, bool) { seqs[o + pos] = x[e / kListThreads]; });
        __syncthreads();
    }
}

__global__ void k_l_inverse(int64_t n, const int32_t *rank, int32_t *inv) {
    for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < n; x += (int64_t)gridDim.x * blockDim.x)
        inv[rank[x]] = (int32_t)x;
}

// ---------------------------------------------------------------------------
// trie cost, ranks, node ids

// position s of the sorted order: LCP with s-1, the weight it adds (one
// addition per workgroup), the count of its new nodes (into base[s + 1] for the
// scan), rank of its request
__global__ __launch_bounds__(kCheckThreads) void k_l_lcp(int m, const int32_t *__restrict__ ord,
                                                         const int64_t *__restrict__ off,
                                                         const int32_t *__restrict__ seqs,
                                                         const int64_t *__restrict__ w, int32_t *__restrict__ lcp,
                                                         int64_t *__restrict__ base, int32_t *__restrict__ rank,
                                                         LHeader *h) {
    __shared__ uint64_t red[kCheckThreads / kWave];
    if (h->err) return;
    uint64_t add = 0;
    for (int s = blockIdx.x * kCheckThreads + threadIdx.x; s < m; s += gridDim.x * kCheckThreads) {
        const int i = ord[s];
        const int64_t li = off[i + 1] - off[i];
        const int32_t *si = seqs + off[i];
        int64_t l = 0;
        if (s > 0) {
            const int p = ord[s - 1];
            const int64_t lp = off[p + 1] - off[p];
            const int32_t *sp = seqs + off[p];
            while (l < li && l < lp && si[l] == sp[l]) ++l;
        }
        for (int64_t j = l; j < li; ++j) add += (uint64_t)w[si[j]];
        lcp[s] = (int32_t)l;
        base[s + 1] = li - l;
        rank[i] = s;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) base[0] = 0;
    add = check_block_sum(add, red);
    if (threadIdx.x == 0 && add) atomicAdd(&h->cost, (unsigned long long)add);
}

// In-place scan of a[0 .. n) by one workgroup of 1024, inclusive or exclusive,
// kScanPer * 1024 entries at a time through LDS: coalesced reads and writes,
// kScanPer consecutive entries per thread in between. The sums stay below 2^31
// (at most nnz). (One entry per thread at a time was a round trip per 1024
// entries, 30 us at 20011.)
constexpr int kScanPer = 16;
template <bool INCL>
__device__ inline void scan_array(int64_t n, int64_t *a) {
    __shared__ int32_t buf[1024 * (kScanPer + 1)];       // one pad per thread's entries: no bank conflicts
    __shared__ int32_t sw[16];
    const int tid = (int)threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    int32_t carry = 0;
    for (int64_t b0 = 0; b0 < n; b0 += 1024 * kScanPer) {
        int64_t v[kScanPer];
#pragma unroll
        for (int q = 0; q < kScanPer; ++q) {
            const int e = q * 1024 + tid;
            v[q] = b0 + e < n ? a[b0 + e] : 0;
        }
#pragma unroll
        for (int q = 0; q < kScanPer; ++q) {
            const int e = q * 1024 + tid;
            buf[e + e / kScanPer] = (int32_t)v[q];
        }
        __syncthreads();
        int32_t x = 0, in[kScanPer];
#pragma unroll
        for (int q = 0; q < kScanPer; ++q) {
            const int32_t t = buf[tid * (kScanPer + 1) + q];
            in[q] = INCL ? x + t : x;
            x += t;
        }
        const int32_t own = x;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int32_t y = __shfl_up(x, o, kWave);
            if (lane >= o) x += y;
        }
        if (lane == kWave - 1) sw[wid] = x;
        __syncthreads();
        int32_t before = carry + x - own;
        for (int k = 0; k < 16; ++k) {
            before += k < wid ? sw[k] : 0;
            carry += sw[k];
        }
#pragma unroll
        for (int q = 0; q < kScanPer; ++q) buf[tid * (kScanPer + 1) + q] = before + in[q];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kScanPer; ++q) {
            const int e = q * 1024 + tid;
            if (b0 + e < n) a[b0 + e] = buf[e + e / kScanPer];
        }
        __syncthreads();
    }
}

// base[s] becomes the first node id of sorted position s, base[m] the node count
__global__ __launch_bounds__(1024) void k_l_scan(int m, int64_t *base) { scan_array<true>(m, base + 1); }

// weight of every trie node: sorted position s creates the nodes of depths
// LCP .. len-1 of its request, with ids base[s] + (j - LCP)
__global__ void k_l_node_weights(int m, const int32_t *ord, const int64_t *off, const int32_t *seqs, const int64_t *w,
                                 const int32_t *lcp, const int64_t *base, int64_t *nw) {
    for (int s = blockIdx.x * blockDim.x + threadIdx.x; s < m; s += gridDim.x * blockDim.x) {
        const int i = ord[s];
        const int64_t li = off[i + 1] - off[i], l = lcp[s], b = base[s];
        for (int64_t j = l; j < li; ++j) nw[b + (j - l)] = w[seqs[off[i] + j]];
    }
}

// node ids of every request's path. Request s (in sorted order) creates the
// nodes of depths LCP(s) .. len-1, with ids base[s] + (j - LCP(s)); a
// shallower depth j < LCP(s) holds the node of the previous request, and so
// on back to the last request t <= s with LCP(t) <= j, which created it. A
// min segment tree over the LCPs finds t in O(log m), so every slot of the
// layout is one independent thread.
constexpr int kTreeBlock = 2048;               // leaves of the subtree one workgroup builds in LDS

// leaves mtree[mpad + t] = LCP(t) (padding: INT32_MAX) and the levels of each
// workgroup's subtree of kTreeBlock leaves (heap order: node n has children
// 2n, 2n + 1; the root is 1)
__global__ __launch_bounds__(1024) void k_l_mtree_low(int m, int64_t mpad, const int32_t *lcp, int32_t *mtree) {
    __shared__ int32_t t[kTreeBlock];
    const int64_t S = min<int64_t>(kTreeBlock, mpad);
    const int64_t first = (int64_t)blockIdx.x * S;
    for (int64_t e = threadIdx.x; e < S; e += blockDim.x) {
        const int64_t leaf = first + e;
        const int32_t v = leaf < m ? lcp[leaf] : INT32_MAX;
        t[e] = v;
        mtree[mpad + leaf] = v;
    }
    __syncthreads();
    for (int64_t len = S >> 1, k = 1; len >= 1; len >>= 1, ++k) {
        int32_t v = 0;
        const int64_t e = threadIdx.x;
        if (e < len) v = min(t[2 * e], t[2 * e + 1]);
        __syncthreads();
        if (e < len) {
            t[e] = v;
            mtree[(mpad >> k) + (first >> k) + e] = v;
        }
        __syncthreads();
    }
}

// the levels above the subtrees, one workgroup
__global__ __launch_bounds__(1024) void k_l_mtree_top(int64_t top, int32_t *mtree) {
    for (int64_t len = top >> 1; len >= 1; len >>= 1) {
        for (int64_t n = len + threadIdx.x; n < 2 * len; n += blockDim.x) mtree[n] = min(mtree[2 * n], mtree[2 * n + 1]);
        __syncthreads();
    }
}

// last position t <= r whose LCP is at most j (exists: LCP(0) = 0)
__device__ inline int64_t last_at_most(const int32_t *mtree, int64_t mpad, int64_t r, int32_t j) {
    int64_t n = mpad + r;
    if (mtree[n] <= j) return r;
    while (n > 1) {
        if ((n & 1) && mtree[n - 1] <= j) { n -= 1; break; }   // the left neighbour's subtree holds one
        n >>= 1;
    }
    while (n < mpad) n = mtree[2 * n + 1] <= j ? 2 * n + 1 : 2 * n;
    return n - mpad;
}

__global__ void k_l_paths(int m, int64_t nnz, int64_t mpad, const int64_t *off, const int32_t *rank, const int32_t *lcp,
                          const int64_t *base, const int32_t *mtree, int32_t *pn) {
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < nnz; k += (int64_t)gridDim.x * blockDim.x) {
        // the request holding slot k: the last i with off[i] <= k
        int lo = 0, hi = m - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (off[mid] <= k) lo = mid; else hi = mid - 1;
        }
        const int64_t j = k - off[lo];
        const int64_t s = rank[lo];
        const int64_t t = j < lcp[s] ? last_at_most(mtree, mpad, s - 1, (int32_t)j) : s;
        pn[k] = (int32_t)(base[t] + (j - lcp[t]));
    }
}

// ---------------------------------------------------------------------------
// schedules and access logs

// key of request i under configuration c: window index, then the request's
// position in the DFS order (windowed DFS = sort inside every window)
__global__ void k_l_sched_keys(int m, int n_cfg, const int64_t *windows, const int32_t *rank, uint64_t *keys) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < (int64_t)n_cfg * m;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int c = (int)(e / m), i = (int)(e % m);
        const int64_t W = windows[c];
        const uint64_t win = (uint64_t)(i / W);
        keys[e] = ((uint64_t)c << 56) | (win << 28) | (uint64_t)rank[i];
    }
}

// sorted keys -> schedule of every configuration (request ids) and the
// access-log length of each served request
__global__ void k_l_sched_out(int m, int n_cfg, const uint64_t *keys, const int32_t *ord, const int64_t *off,
                              int32_t *sched, int64_t *log_off) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < (int64_t)n_cfg * m;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int r = (int)(keys[e] & ((1u << 28) - 1u));
        const int i = ord[r];
        sched[e] = i;
        log_off[e] = off[i + 1] - off[i];
    }
}

// exclusive scan of the log lengths of every configuration (one workgroup
// per configuration)
__global__ __launch_bounds__(1024) void k_l_log_scan(int m, int64_t *log_off) {
    scan_array<false>(m, log_off + (int64_t)blockIdx.x * m);
}

// the access log of every configuration: served requests in order, each
// path from its leaf up to the root
__global__ void k_l_logs(int m, int n_cfg, int64_t nnz, const int32_t *sched, const int64_t *log_off,
                         const int64_t *off, const int32_t *pn, int32_t *logs, int32_t *acc_start) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < (int64_t)n_cfg * m;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int c = (int)(e / m);
        const int i = sched[e];
        const int64_t li = off[i + 1] - off[i], at = log_off[e];
        int32_t *dst = logs + (int64_t)c * nnz + at;
        int32_t *st = acc_start + (int64_t)c * nnz + at;
        const int32_t *path = pn + off[i];
        for (int64_t j = 0; j < li; ++j) {
            dst[j] = path[li - 1 - j];
            st[j] = (int32_t)at;                 // where the request's accesses start
        }
    }
}

// ---------------------------------------------------------------------------
// the radix cache by stack distances
//
// Serving a request touches its whole path, each node of it more recently
// than its descendants, and every miss is inserted before the cache evicts
// (least-recently-used leaf first, which is the least-recently-used node,
// since an ancestor is never older than its descendants). By induction over
// the requests, the cache after each request holds exactly the longest
// prefix of the recency stack (nodes by latest access, most recent first)
// whose weight fits the capacity: the stack property of LRU (Mattson et al.,
// 1970), here with weights. So node v of the request whose accesses start at
// log position s is a hit iff it was accessed before and the nodes above it
// in the stack together with v fit: D + w(v) <= capacity, where D is the
// weight of the distinct nodes accessed between v's previous access p and s,
// i.e. the sum of w_j over log entries p < j < s whose node is not accessed
// again before s (next_j >= s). D does not depend on the capacity: one pass
// over a schedule's log bills all its capacities.

constexpr int kSmallBlock = 64, kBigBlock = 1024;   // log entries per sorted block

// sort keys of the access logs of schedules d0 .. d0 + nd - 1: (schedule,
// node, log position)
__global__ void k_l_acc_keys(int64_t nnz, int d0, int nd, int be, int bn, const int32_t *logs, uint64_t *keys) {
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < (int64_t)nd * nnz;
         k += (int64_t)gridDim.x * blockDim.x) {
        const int64_t dl = k / nnz, e = k % nnz;
        const uint64_t v = (uint64_t)logs[(d0 + dl) * nnz + e];
        keys[k] = ((uint64_t)dl << (bn + be)) | (v << be) | (uint64_t)e;
    }
}

// previous and next access of the same node (-1 / nnz when there is none);
// schedule d0 + dl holds sorted positions [dl nnz, (dl + 1) nnz)
__global__ void k_l_prev_next(int64_t nnz, int d0, int nd, int be, const uint64_t *keys, int32_t *prev,
                              int32_t *next) {
    const uint64_t emask = (1ull << be) - 1ull;
    const int64_t n = (int64_t)nd * nnz;
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t key = keys[k], grp = key >> be;
        const int64_t at = (d0 + k / nnz) * nnz + (int64_t)(key & emask);
        const bool has_prev = (k % nnz) > 0 && (keys[k - 1] >> be) == grp;
        const bool has_next = (k + 1) % nnz != 0 && (keys[k + 1] >> be) == grp;
        prev[at] = has_prev ? (int32_t)(keys[k - 1] & emask) : -1;
        next[at] = has_next ? (int32_t)(keys[k + 1] & emask) : (int32_t)nnz;
    }
}

// One workgroup per big block of one schedule's log. For every entry, the
// weight of the entries from it to the end of its small block (wsuf); and the
// small blocks, then the big one, sorted by next access descending with the
// running weight sum, so that the weight of a block's entries with next >= s is
// a prefix. Keys (next access inverted << 10 | entry), sorted in registers up
// to 256 and merged in LDS.
constexpr int kStackThreads = kBigBlock / 4;
__device__ inline int32_t stack_next(uint64_t key) { return (int32_t)(0x7fffffffll - (int64_t)(key >> 10)); }
__global__ __launch_bounds__(kStackThreads) void k_l_stack_blocks(int64_t nnz, int64_t nblk,
                                                                  const int32_t *__restrict__ logs,
                                                                  const int64_t *__restrict__ nw,
                                                                  const int32_t *__restrict__ next,
                                                                  int64_t *__restrict__ wsuf,
                                                                  int32_t *__restrict__ snext,
                                                                  int64_t *__restrict__ ssum,
                                                                  int32_t *__restrict__ bnext,
                                                                  int64_t *__restrict__ bsum) {
    using namespace mptlib::keysort_detail;
    __shared__ __align__(16) uint64_t t[2][kBigBlock];
    __shared__ int64_t ws[kBigBlock];
    __shared__ int64_t part[kStackThreads / kWave];
    const int tid = (int)threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    const int64_t d = blockIdx.x / nblk, b = blockIdx.x % nblk;
    const int64_t j0 = b * kBigBlock + tid * 4;
    uint64_t v[4];
    int64_t w[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t at = d * nnz + j0 + r;
        w[r] = 0;
        int32_t nx = -1;                                 // padding: never counted
        if (j0 + r < nnz) {
            w[r] = nw[logs[at]];
            nx = next[at];
        }
        ws[tid * 4 + r] = w[r];
        v[r] = ((uint64_t)(0x7fffffffll - nx) << 10) | (uint64_t)(tid * 4 + r);
    }
    {
        // 16 lanes hold a small block
        int64_t suf[4], x;
        suf[3] = w[3];
#pragma unroll
        for (int r = 2; r >= 0; --r) suf[r] = w[r] + suf[r + 1];
        x = suf[0];
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
            const int64_t y = __shfl_down(x, o, 16);
            if ((lane & 15) + o < 16) x += y;
        }
        x -= suf[0];                                     // the lanes after this one
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (j0 + r < nnz) wsuf[d * nnz + j0 + r] = suf[r] + x;
    }
    __syncthreads();
    const int64_t out = (d * nblk + b) * kBigBlock + tid * 4;
    // running sums of the sorted weights over WIDTH lanes, from start on
    auto emit = [&](int width, int64_t start, int32_t *on, int64_t *os) {
        int64_t pre[4], x = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) pre[r] = x += ws[v[r] & (kBigBlock - 1u)];
        const int64_t own = x;
        for (int o = 1; o < width; o <<= 1) {
            const int64_t y = __shfl_up(x, o, width);
            if ((lane & (width - 1)) >= o) x += y;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            on[out + r] = stack_next(v[r]);
            os[out + r] = start + x - own + pre[r];
        }
    };
    sort_wave64(v);
    emit(16, 0, snext, ssum);
    sort_wave256(v);
    int cur = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) t[0][tid * 4 + r] = v[r];
    __syncthreads();
    for (int run = 256; run < kBigBlock; run <<= 1, cur ^= 1) {
        merge_outputs(t[cur], run, tid * 4, v);
#pragma unroll
        for (int r = 0; r < 4; ++r) t[cur ^ 1][tid * 4 + r] = v[r];
        __syncthreads();
    }
    int64_t x = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) x += ws[v[r] & (kBigBlock - 1u)];
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) x += __shfl_xor(x, o, kWave);
    if (lane == 0) part[wid] = x;
    __syncthreads();
    int64_t start = 0;
    for (int k = 0; k < wid; ++k) start += part[k];
    emit(kWave, start, bnext, bsum);
}

// The weight of the entries with next access >= s in `count` <= 4 sorted blocks
// of SIZE entries that end at hi, hi - SIZE, ..., their searches in lockstep
template <int SIZE>
__device__ inline int64_t blocks_weight(const int32_t *bn, const int64_t *bs, int64_t hi, int count, int64_t s) {
    int lo[4], up[4];
    int64_t first[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        first[u] = hi - (int64_t)(u + 1) * SIZE;
        lo[u] = 0;
        up[u] = u < count ? SIZE : 0;
    }
    for (int left = SIZE; left > 0; left >>= 1) {
        int32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = lo[u] < up[u] ? bn[first[u] + ((lo[u] + up[u]) >> 1)] : 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (lo[u] >= up[u]) continue;
            const int mid = (lo[u] + up[u]) >> 1;
            if (v[u] >= s) lo[u] = mid + 1; else up[u] = mid;
        }
    }
    int64_t sum = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (lo[u] > 0) sum += bs[first[u] + lo[u] - 1];
    return sum;
}

// One thread per log entry of one schedule: its stack distance, then its bill
// under every capacity of the schedule, summed per workgroup in LDS and added
// to the configurations' costs. The stretch (p, s) is taken from its end: the
// part of a small block before s is the block's share less the weight of its
// entries from s on (those are accessed at s or later themselves), then small
// blocks down to a big block's end, big blocks, small blocks, and single
// entries up to the first small block. A distance that already misses the
// largest capacity misses them all, whatever is left of the stretch.
// Bound by the searches' reads: 250 us at 20011 requests and 114 at 4096; with
// one size of block (256), its edges entry by entry and no end to a search, 840
// and 162.
constexpr int kBillThreads = 256;
constexpr int kBillSingles = 96;      // stretches up to this are added entry by entry
__global__ __launch_bounds__(kBillThreads) void k_l_bill(int64_t nnz, int64_t nblk, const int32_t *__restrict__ prev,
                                                         const int32_t *__restrict__ next,
                                                         const int32_t *__restrict__ acc_start,
                                                         const int64_t *__restrict__ wsuf,
                                                         const int32_t *__restrict__ snext,
                                                         const int64_t *__restrict__ ssum,
                                                         const int32_t *__restrict__ bnext,
                                                         const int64_t *__restrict__ bsum,
                                                         const int32_t *__restrict__ cfg_off,
                                                         const int32_t *__restrict__ cfg_list,
                                                         const int64_t *__restrict__ caps,
                                                         unsigned long long *costs) {
    __shared__ unsigned long long acc[MPT_CACHE_MAX_CONFIGS];
    __shared__ int64_t cap[MPT_CACHE_MAX_CONFIGS];
    const int d = blockIdx.y;
    const int c0 = cfg_off[d], nc = cfg_off[d + 1] - c0;
    for (int k = threadIdx.x; k < nc; k += kBillThreads) {
        acc[k] = 0ull;
        cap[k] = caps[cfg_list[c0 + k]];
    }
    __syncthreads();
    int64_t largest = 0;
    for (int k = 0; k < nc; ++k) largest = cap[k] > largest ? cap[k] : largest;
    const int64_t e = blockIdx.x * (int64_t)kBillThreads + threadIdx.x;
    if (e < nnz) {
        const int64_t base = (int64_t)d * nnz;
        // the weight of entry q, given the suffix sums at it and after it
        auto weight = [&](int64_t q, int64_t at, int64_t after) {
            return at - ((q + 1) % kSmallBlock != 0 && q + 1 < nnz ? after : 0);
        };
        const int64_t w = weight(e, wsuf[base + e], e + 1 < nnz ? wsuf[base + e + 1] : 0);
        const int64_t p = prev[base + e];
        int64_t dist = -1;                               // -1: first access, a miss everywhere
        if (p >= 0) {
            const int64_t s = acc_start[base + e], j0 = p + 1;
            dist = 0;
            // a range of single entries, 8 in flight at a time
            auto singles = [&](int64_t from, int64_t to) {
                for (int64_t q = from; q < to; q += 8) {
                    int32_t nx[8];
                    int64_t wq[9];
#pragma unroll
                    for (int u = 0; u < 8; ++u) nx[u] = q + u < to ? next[base + q + u] : -1;
#pragma unroll
                    for (int u = 0; u < 9; ++u) wq[u] = q + u < nnz ? wsuf[base + q + u] : 0;
#pragma unroll
                    for (int u = 0; u < 8; ++u) dist += nx[u] >= s ? weight(q + u, wq[u], wq[u + 1]) : 0;
                }
            };
            if (s - j0 <= kBillSingles) {
                singles(j0, s);
            } else {
                const int64_t row = (int64_t)d * nblk * kBigBlock;
                const int32_t *sn = snext + row, *bn = bnext + row;
                const int64_t *ss = ssum + row, *bs = bsum + row;
                const int64_t lo64 = (j0 + kSmallBlock - 1) / kSmallBlock * kSmallBlock;
                const int64_t lo1k = (j0 + kBigBlock - 1) / kBigBlock * kBigBlock;
                int64_t hi = s / kSmallBlock * kSmallBlock;
                if (s > hi) dist += blocks_weight<kSmallBlock>(sn, ss, hi + kSmallBlock, 1, s) - wsuf[base + s];
                while (hi > lo64 && hi % kBigBlock != 0 && dist + w <= largest) {
                    const int64_t down = hi / kBigBlock * kBigBlock;
                    const int n = (int)min<int64_t>(4, (hi - (down > lo64 ? down : lo64)) / kSmallBlock);
                    dist += blocks_weight<kSmallBlock>(sn, ss, hi, n, s);
                    hi -= (int64_t)n * kSmallBlock;
                }
                while (hi > lo1k && hi % kBigBlock == 0 && dist + w <= largest) {
                    const int n = (int)min<int64_t>(4, (hi - lo1k) / kBigBlock);
                    dist += blocks_weight<kBigBlock>(bn, bs, hi, n, s);
                    hi -= (int64_t)n * kBigBlock;
                }
                while (hi > lo64 && dist + w <= largest) {
                    const int n = (int)min<int64_t>(4, (hi - lo64) / kSmallBlock);
                    dist += blocks_weight<kSmallBlock>(sn, ss, hi, n, s);
                    hi -= (int64_t)n * kSmallBlock;
                }
                if (dist + w <= largest) singles(j0, lo64);
            }
        }
        for (int k = 0; k < nc; ++k) {
            const bool miss = dist < 0 || dist + w > cap[k];
            if (miss) atomicAdd(&acc[k], (unsigned long long)w);
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < nc; k += kBillThreads)
        if (acc[k]) atomicAdd(&costs[cfg_list[c0 + k]], acc[k]);
}

// ---------------------------------------------------------------------------
// host side

int l_check(int m, int64_t n_chunks, int64_t nnz) {
    if (m < 1 || m > MPT_LAYOUT_MAX_M) return fail(MPT_E_INVALID, "m = %d outside [1, %d]", m, MPT_LAYOUT_MAX_M);
    if (n_chunks < 0 || n_chunks > MPT_MAX_CHUNKS) return fail(MPT_E_INVALID, "n_chunks = %lld out of range", (long long)n_chunks);
    if (nnz < 0 || nnz > (int64_t)INT32_MAX) return fail(MPT_E_INVALID, "nnz = %lld out of range", (long long)nnz);
    return MPT_OK;
}

int l_check_ws(const LLayout &L, void *ws, size_t bytes) {
    if (!ws) return fail(MPT_E_WORKSPACE, "workspace is NULL");
    if (((uintptr_t)ws & 255u) != 0) return fail(MPT_E_WORKSPACE, "workspace is not 256-byte aligned");
    if (bytes < L.total) return fail(MPT_E_WORKSPACE, "workspace has %zu bytes, needs %zu", bytes, L.total);
    return MPT_OK;
}

// validation + lexicographic order (to dfs too, where given) + LCPs + trie
// cost, with one synchronisation at the end; then, paths: the node ids
int l_prepare(int m, int64_t n_chunks, int64_t nnz, const int64_t *w, const int64_t *off, const int32_t *seqs,
              const LLayout &L, char *ws, hipStream_t s, bool paths, int32_t *dfs, int64_t *trie_cost) {
    LHeader *h = (LHeader *)ws;
    int32_t *ord = (int32_t *)(ws + L.ord), *rank = (int32_t *)(ws + L.rank), *lcp = (int32_t *)(ws + L.lcp);
    int64_t *base = (int64_t *)(ws + L.base);
    int rc;
    k_l_begin<<<grid_for(m, 256), 256, 0, s>>>(h, rank, m);
    k_l_check<<<grid_for(std::max<int64_t>(nnz, m), 2 * kCheckThreads, 1024), kCheckThreads, 0, s>>>(
        m, nnz, n_chunks, off, seqs, w, h);
    {
        LaunchScope ls("l_sort_requests", (double)m, s);
        if ((rc = sort_requests(ord, rank, dfs, m, off, seqs, ws + L.recs, &h->err, s))) return rc;
    }
    {
        LaunchScope ls("l_lcp", (double)nnz, s);
        k_l_lcp<<<grid_for(m, kCheckThreads, 4096), kCheckThreads, 0, s>>>(m, ord, off, seqs, w, lcp, base, rank, h);
    }
    MPT_HIP_TRY(hipGetLastError());
    if ((rc = l_read_errors(h, s, nullptr, trie_cost))) return rc;
    if (paths) {
        int32_t *pn = (int32_t *)(ws + L.pn), *mtree = (int32_t *)(ws + L.mtree);
        int64_t *nw = (int64_t *)(ws + L.nw);
        LaunchScope ls("l_paths", (double)nnz, s);
        k_l_scan<<<1, 1024, 0, s>>>(m, base);
        k_l_node_weights<<<grid_for(m, 256), 256, 0, s>>>(m, ord, off, seqs, w, lcp, base, nw);
        const int64_t sub = std::min<int64_t>(kTreeBlock, L.mpad);
        k_l_mtree_low<<<(unsigned)(L.mpad / sub), 1024, 0, s>>>(m, L.mpad, lcp, mtree);
        if (L.mpad > sub) k_l_mtree_top<<<1, 1024, 0, s>>>(L.mpad / sub, mtree);
        if (nnz > 0)
            k_l_paths<<<grid_for(nnz, 256), 256, 0, s>>>(m, nnz, L.mpad, off, rank, lcp, base, mtree, pn);
        MPT_HIP_TRY(hipGetLastError());
    }
    return MPT_OK;
}

}  // namespace

extern "C" size_t mpt_layout_workspace_bytes(int m, int64_t n_chunks, int64_t nnz, int n_configs) {
    if (m < 1 || m > MPT_LAYOUT_MAX_M || n_chunks < 0 || nnz < 0 || n_configs < 0 ||
        n_configs > MPT_CACHE_MAX_CONFIGS)
        return 0;
    return l_layout(m, n_chunks, nnz, n_configs).total;
}

extern "C" int mpt_global_order_layout(int m, int64_t n_chunks, int64_t nnz, const int64_t *req_off,
                                       const int32_t *req_chunks, int order_kind, int32_t *seqs, void *workspace,
                                       size_t workspace_bytes, void *stream) {
    mptlib::clear_error();
    return mptlib::guarded(__func__, [&]() -> int {
        int rc = l_check(m, n_chunks, nnz);
        if (rc) return rc;
        if (order_kind != MPT_ORDER_ID && order_kind != MPT_ORDER_POPULARITY)
            return fail(MPT_E_INVALID, "order_kind = %d is not MPT_ORDER_ID or MPT_ORDER_POPULARITY", order_kind);
        if (!req_off || (nnz > 0 && (!req_chunks || !seqs))) return fail(MPT_E_INVALID, "req_off, req_chunks and seqs must not be NULL");
        const LLayout L = l_layout(m, n_chunks, nnz, 0);
        if ((rc = l_check_ws(L, workspace, workspace_bytes))) return rc;
        hipStream_t s = (hipStream_t)stream;
        char *ws = (char *)workspace;
        LHeader *h = (LHeader *)ws;
        uint64_t *keys = (uint64_t *)(ws + L.keys), *keys2 = (uint64_t *)(ws + L.keys2), *sorted = nullptr;
        int32_t *rank = (int32_t *)(ws + L.crank), *inv = (int32_t *)(ws + L.cinv);
        const bool popular = order_kind == MPT_ORDER_POPULARITY;
        LaunchScope ls("l_global_order", (double)nnz, s);
        k_l_begin<<<grid_for(popular ? n_chunks : 1, 256), 256, 0, s>>>(h, rank, popular ? n_chunks : 0);
        k_l_check<<<grid_for(std::max<int64_t>(nnz, m), 2 * kCheckThreads, 1024), kCheckThreads, 0, s>>>(
            m, nnz, n_chunks, req_off, req_chunks, nullptr, h);
        if (nnz > 0) {
            if (popular) {
                // (count, id) keys of the chunks
                k_l_count<<<grid_for(nnz, kCountSlice, 1024), kCountThreads, 0, s>>>(nnz, req_chunks, rank, h);
                k_l_pop_keys<<<grid_for(n_chunks, 256), 256, 0, s>>>(n_chunks, rank, keys);
                if ((rc = sort_keys(keys, keys2, n_chunks, s, &sorted))) return rc;
                k_l_pop_rank<<<grid_for(n_chunks, 256), 256, 0, s>>>(n_chunks, sorted, rank);
            }
            // (workgroups for requests of more than kSegMax chunks, whose length the
            // host does not know; four requests each took 217 us for 100 of 512
            // chunks, where a wave per request does not notice the difference)
            k_l_layout_short<<<grid_for(m, 1, 4096), kListThreads, 0, s>>>(m, req_off, req_chunks, rank, order_kind, seqs, h);
        }
        MPT_HIP_TRY(hipGetLastError());
        int64_t max_len = 0;
        if ((rc = l_read_errors(h, s, &max_len))) return rc;
        if (max_len <= kListMax) return MPT_OK;
        if (popular) k_l_inverse<<<grid_for(n_chunks, 256), 256, 0, s>>>(n_chunks, rank, inv);
        k_l_layout_keys<<<grid_for(nnz, 256), 256, 0, s>>>(m, nnz, req_off, req_chunks, rank, order_kind, keys);
        if ((rc = sort_keys(keys, keys2, nnz, s, &sorted))) return rc;
        k_l_layout_out<<<grid_for(nnz, 256), 256, 0, s>>>(nnz, sorted, inv, order_kind, seqs);
        MPT_HIP_TRY(hipGetLastError());
        return MPT_OK;
    });
}

extern "C" int mpt_layout_cost(int m, int64_t n_chunks, int64_t nnz, const int64_t *chunk_w, const int64_t *seq_off,
                               const int32_t *seqs, int32_t *dfs_order, int64_t *trie_cost, void *workspace,
                               size_t workspace_bytes, void *stream) {
    mptlib::clear_error();
    return mptlib::guarded(__func__, [&]() -> int {
        int rc = l_check(m, n_chunks, nnz);
        if (rc) return rc;
        if (!seq_off || !trie_cost || (nnz > 0 && !seqs) || (n_chunks > 0 && !chunk_w))
            return fail(MPT_E_INVALID, "seq_off, seqs, chunk_w and trie_cost must not be NULL");
        const LLayout L = l_layout(m, n_chunks, nnz, 0);
        if ((rc = l_check_ws(L, workspace, workspace_bytes))) return rc;
        hipStream_t s = (hipStream_t)stream;
        char *ws = (char *)workspace;
        return l_prepare(m, n_chunks, nnz, chunk_w, seq_off, seqs, L, ws, s, false, dfs_order, trie_cost);
    });
}

extern "C" int mpt_cache_simulate(int m, int64_t n_chunks, int64_t nnz, const int64_t *chunk_w,
                                  const int64_t *seq_off, const int32_t *seqs, int n_configs,
                                  const int64_t *windows, const int64_t *capacities, int64_t *costs,
                                  int64_t *trie_cost, void *workspace, size_t workspace_bytes, void *stream) {
    mptlib::clear_error();
    return mptlib::guarded(__func__, [&]() -> int {
        int rc = l_check(m, n_chunks, nnz);
        if (rc) return rc;
        if (n_configs < 1 || n_configs > MPT_CACHE_MAX_CONFIGS)
            return fail(MPT_E_INVALID, "n_configs = %d outside [1, %d]", n_configs, MPT_CACHE_MAX_CONFIGS);
        if (!seq_off || !windows || !capacities || !costs || (nnz > 0 && !seqs) || (n_chunks > 0 && !chunk_w))
            return fail(MPT_E_INVALID, "seq_off, seqs, chunk_w, windows, capacities and costs must not be NULL");
        for (int c = 0; c < n_configs; ++c)
            if (capacities[c] < 0) return fail(MPT_E_INVALID, "capacity %d is negative", c);
        const LLayout L = l_layout(m, n_chunks, nnz, n_configs);
        if ((rc = l_check_ws(L, workspace, workspace_bytes))) return rc;
        hipStream_t s = (hipStream_t)stream;
        char *ws = (char *)workspace;
        int64_t tc = 0;
        if ((rc = l_prepare(m, n_chunks, nnz, chunk_w, seq_off, seqs, L, ws, s, true, nullptr, &tc))) return rc;
        if (trie_cost) *trie_cost = tc;
        // configurations: window <= 0 or > m means the whole stream. Equal
        // windows share one schedule (and log); cfg_off / cfg_list list the
        // configurations of every schedule.
        std::vector<int64_t> win;
        std::vector<int> sched_of(n_configs);
        for (int c = 0; c < n_configs; ++c) {
            const int64_t wc = (windows[c] <= 0 || windows[c] > m) ? m : windows[c];
            int d = 0;
            while (d < (int)win.size() && win[d] != wc) ++d;
            if (d == (int)win.size()) win.push_back(wc);
            sched_of[c] = d;
        }
        const int n_sched = (int)win.size();
        std::vector<int32_t> cfg_off(n_sched + 1, 0), cfg_list;
        for (int d = 0; d < n_sched; ++d) {
            for (int c = 0; c < n_configs; ++c)
                if (sched_of[c] == d) cfg_list.push_back(c);
            cfg_off[d + 1] = (int32_t)cfg_list.size();
        }
        // windows, capacities, offsets and lists go over in one copy: the four
        // arrays lie one after the other in the workspace
        int64_t *dev_win = (int64_t *)(ws + L.cfg_win), *dev_capacity = (int64_t *)(ws + L.cfg_cap);
        int32_t *dev_cfg_off = (int32_t *)(ws + L.cfg_off), *dev_cfg_list = (int32_t *)(ws + L.cfg_list);
        std::vector<char> image(L.cfg_list - L.cfg_win + sizeof(int32_t) * (size_t)n_configs);
        std::memcpy(image.data(), win.data(), sizeof(int64_t) * (size_t)n_sched);
        std::memcpy(image.data() + (L.cfg_cap - L.cfg_win), capacities, sizeof(int64_t) * (size_t)n_configs);
        std::memcpy(image.data() + (L.cfg_off - L.cfg_win), cfg_off.data(), sizeof(int32_t) * (size_t)(n_sched + 1));
        std::memcpy(image.data() + (L.cfg_list - L.cfg_win), cfg_list.data(), sizeof(int32_t) * (size_t)n_configs);
        MPT_HIP_TRY(hipMemcpyAsync(dev_win, image.data(), image.size(), hipMemcpyHostToDevice, s));
        uint64_t *keys = (uint64_t *)(ws + L.keys), *keys2 = (uint64_t *)(ws + L.keys2), *sorted = nullptr;
        int32_t *sched = (int32_t *)(ws + L.sched), *logs = (int32_t *)(ws + L.logs);
        int32_t *acc_start = (int32_t *)(ws + L.acc_start), *prev = (int32_t *)(ws + L.prev), *next = (int32_t *)(ws + L.next);
        int64_t *log_off = (int64_t *)(ws + L.log_off), *wsuf = (int64_t *)(ws + L.wsuf);
        const int32_t *ord = (const int32_t *)(ws + L.ord), *rank = (const int32_t *)(ws + L.rank);
        {
            LaunchScope ls("l_schedules", (double)n_sched * m, s);
            const int64_t sn = (int64_t)n_sched * m;
            k_l_sched_keys<<<grid_for(sn, 256), 256, 0, s>>>(m, n_sched, dev_win, rank, keys);
            if ((rc = sort_keys(keys, keys2, sn, s, &sorted))) return rc;
            k_l_sched_out<<<grid_for(sn, 256), 256, 0, s>>>(m, n_sched, sorted, ord, seq_off, sched,
                                                                              log_off);
            k_l_log_scan<<<n_sched, 1024, 0, s>>>(m, log_off);
            if (nnz > 0)
                k_l_logs<<<grid_for((int64_t)n_sched * m, 256), 256, 0, s>>>(m, n_sched, nnz, sched, log_off, seq_off,
                                                                             (const int32_t *)(ws + L.pn), logs, acc_start);
        }
        MPT_HIP_TRY(hipGetLastError());
        int64_t *dev_costs = (int64_t *)(ws + L.costs);
        k_l_fill_u64<<<1, 256, 0, s>>>((uint64_t *)dev_costs, n_configs, 0ull);
        if (nnz > 0) {
            {
                // previous and next access of every log entry: a sort of
                // (schedule, node, position) keys, as many schedules per sort as
                // the 63 key bits hold
                LaunchScope ls("l_reuse", (double)n_sched * nnz, s);
                auto bits = [](int64_t n) { int b = 1; while (b < 62 && ((int64_t)1 << b) < n) ++b; return b; };
                const int be = bits(nnz), bn = be;            // (nnz bounds the node count)
                const int gb = 63 - be - bn;                  // >= 1: nnz stays below 2^31
                const int group = gb >= 8 ? n_sched : std::min(n_sched, 1 << gb);
                for (int d0 = 0; d0 < n_sched; d0 += group) {
                    const int nd = std::min(group, n_sched - d0);
                    const int64_t an = (int64_t)nd * nnz;
                    k_l_acc_keys<<<grid_for(an, 256), 256, 0, s>>>(nnz, d0, nd, be, bn, logs, keys);
                    if ((rc = sort_keys(keys, keys2, an, s, &sorted))) return rc;
                    k_l_prev_next<<<grid_for(an, 256), 256, 0, s>>>(nnz, d0, nd, be, sorted, prev, next);
                }
            }
            LaunchScope ls("l_simulate", (double)n_configs * nnz, s);
            const int64_t nblk = (nnz + kBigBlock - 1) / kBigBlock;
            int32_t *snext = (int32_t *)(ws + L.snext), *bnext = (int32_t *)(ws + L.bnext);
            int64_t *ssum = (int64_t *)(ws + L.ssum), *bsum = (int64_t *)(ws + L.bsum);
            k_l_stack_blocks<<<(unsigned)(n_sched * nblk), kStackThreads, 0, s>>>(
                nnz, nblk, logs, (const int64_t *)(ws + L.nw), next, wsuf, snext, ssum, bnext, bsum);
            k_l_bill<<<dim3((unsigned)((nnz + kBillThreads - 1) / kBillThreads), (unsigned)n_sched), kBillThreads, 0, s>>>(
                nnz, nblk, prev, next, acc_start, wsuf, snext, ssum, bnext, bsum, dev_cfg_off, dev_cfg_list, dev_capacity,
                (unsigned long long *)dev_costs);
        }
        MPT_HIP_TRY(hipGetLastError());
        MPT_HIP_TRY(mptlib::read_back(costs, dev_costs, sizeof(int64_t) * n_configs, s));
        return MPT_OK;
    });
}
