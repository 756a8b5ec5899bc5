// libmpt.so, Sections 6.2-6.3 of "Prefix Sharing Is a Sorting Problem",
// for any number of requests up to MPT_GREEDY_MAX_M:
//   mpt_pair_weights         P[i][j] = w(R_i ∩ R_j)
//   mpt_greedy_hierarchy     the agglomerative common-prefix hierarchy H_g
//                            (Section 6.2, Theorem 6) and its layout
//   mpt_spanning_tree_bound  the maximum spanning tree of P, whence
//                            OPT_free >= sum_i w(R_i) - MST (Section 6.3)
//
// Every request's chunks are put in ascending order once; a counting sort of
// the slots by chunk gives the demand list S_x of every chunk.
// Pair weights are a scatter over the pairs of every demand list: request
// families of retrieval shape have small |S_x|, so this touches
// sum_x |S_x|^2 entries instead of a dense m x m x u contraction.
//
// The greedy's merges run in rounds over the whole chip: every round merges
// all pairs of clusters that are each other's best partner (merge values
// never grow, Theorem 6 part i, so each such pair is one of the greedy's
// merges), intersects their signatures, recomputes the new rows and only
// the best partners that can have changed. A sort of the merges by the
// lowest priority in their subtrees then gives the greedy's sequence.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>

#include "common.h"
#include "keysort.h"
#include "mpt.h"

namespace {

using mptlib::align256;
using mptlib::fail;
using mptlib::grid_for;
using mptlib::LaunchScope;
using mptlib::kListMax;
using mptlib::kListThreads;
using mptlib::kSegMax;
using mptlib::list_ranks;
using mptlib::seg_rank;
using mptlib::sort_keys;

constexpr int kWave = 64;

enum : uint32_t { GERR_INVALID = 1u, GERR_RANGE = 2u, GERR_DUP = 4u, GERR_WEIGHT = 8u, GERR_OVERFLOW = 16u };

// first 256 bytes of the workspace
struct GHeader {
    uint32_t err;
    uint32_t pad0;
    unsigned long long total;    // sum_i w(R_i), unsigned so it cannot wrap before the check
    int32_t n_rec;               // merge records so far
    int32_t lo;                  // first record of the current round
    int32_t n_resc[2];           // rows marked for a rescan, by round parity
    int32_t last_pairs;          // merges of the last finished round
    int32_t bv_done;             // spanning tree: 1 once one component is left
    unsigned long long dcursor;  // next free slot of the packed D lists
    int64_t max_len;             // longest request list
    unsigned long long dem_at;   // next free slot of the demand lists
    unsigned long long savings;  // sum of the merges' gains
    int64_t pad[23];
};
static_assert(sizeof(GHeader) == 256, "header is one 256-byte block");

struct GLayout {
    size_t keys1, keys2, rank, sig, sig_slot, sig_len, dem, dem_seg, V, best_v, best_p, active, last, touched, resc, live, dense, d_off,
        d_len, rec32, rec64, total;
};
// clusters that the greedy's last rounds, run by one workgroup, may start from
constexpr int kTailLive = 2048;
constexpr int kRec32 = 7;    // int32 arrays of the merge records
constexpr int kRec64 = 3;    // int64 arrays of the merge records

GLayout g_layout(int m, int64_t n_chunks, int64_t nnz) {
    GLayout L{};
    const size_t mm = (size_t)m;
    size_t o = align256(sizeof(GHeader));
    auto take = [&](size_t bytes) { size_t at = o; o = align256(o + std::max<size_t>(bytes, 1)); return at; };
    // the sort of long lists is over before the tail's dense matrix is written
    const size_t shared = o, dm = std::min<size_t>(mm, kTailLive);
    L.keys1 = take(8 * (size_t)std::max<int64_t>(nnz, 1));
    L.keys2 = take(8 * (size_t)std::max<int64_t>(nnz, 1));
    const size_t keys_end = o;
    o = shared;
    L.dense = take(8 * dm * dm);
    o = std::max(o, keys_end);
    L.rank = take(4 * (size_t)std::max<int64_t>(nnz, 1));
    L.sig = take(8 * (size_t)std::max<int64_t>(nnz, 1));   // the lists, then the D lists of long merges
    L.sig_slot = take(4 * (size_t)std::max<int64_t>(nnz, 1));
    L.sig_len = take(4 * mm);
    L.dem = take(4 * (size_t)std::max<int64_t>(nnz, 1));
    L.dem_seg = take(8 * (size_t)std::max<int64_t>(n_chunks, 1));
    L.V = take(8 * mm * mm);
    L.best_v = take(8 * mm);
    L.best_p = take(4 * mm);
    L.active = take(4 * mm);
    L.last = take(4 * mm);
    L.touched = take(4 * mm);
    L.resc = take(4 * mm);
    L.live = take(4 * mm);
    L.d_off = take(8 * (2 * mm));
    L.d_len = take(4 * (2 * mm));
    L.rec32 = take(4 * mm * kRec32);
    L.rec64 = take(8 * mm * kRec64);
    L.total = o;
    return L;
}

// ---------------------------------------------------------------------------
// block helpers

// (value, index) pair order of a maximum with ties to the smallest index
__device__ inline bool better(int64_t v, int32_t i, int64_t ov, int32_t oi) {
    return v > ov || (v == ov && (unsigned)i < (unsigned)oi);
}

__device__ inline void wave_best(int64_t &v, int32_t &i) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        const int64_t ov = __shfl_xor(v, off, kWave);
        const int32_t oi = __shfl_xor(i, off, kWave);
        if (better(ov, oi, v, i)) { v = ov; i = oi; }
    }
}

// exclusive prefix sum of one int per thread over the workgroup; returns
// the thread's offset, *total gets the sum
__device__ inline int block_scan(int x, int *total, int *sw) {
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    int incl = x;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int y = __shfl_up(incl, off, kWave);
        if (lane >= off) incl += y;
    }
    if (lane == kWave - 1) sw[wid] = incl;
    __syncthreads();
    int before = 0, all = 0;
    for (int k = 0; k < (int)(blockDim.x / kWave); ++k) {
        if (k < wid) before += sw[k];
        all += sw[k];
    }
    __syncthreads();
    *total = all;
    return before + incl - x;
}

// position of x in the ascending list a[0 .. n), or -1
__device__ inline int64_t find_sorted(const int32_t *a, int64_t n, int32_t x) {
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (a[mid] < x) lo = mid + 1; else hi = mid;
    }
    return (lo < n && a[lo] == x) ? lo : -1;
}

// ---------------------------------------------------------------------------
// validation and lists
//
// Demand lists by a counting sort of the slots, in three launches: the first
// counts every chunk's slots (and leaves each slot its place among its
// chunk's), the second gives every chunk a stretch of dem, the third writes.
// The stretches follow the order of their atomics and a list's requests come
// in no order: the lists are only summed over. A sort of (chunk, request) keys
// took two launches of 25 us and two more to read them (before that ten
// bitonic ones), and the total one atomic per slot on one address.

__global__ void k_g_begin(int64_t n_chunks, uint64_t *dem_seg, GHeader *h) {
    if (blockIdx.x == 0 && threadIdx.x == 0) { h->err = 0; h->total = 0; h->max_len = 0; h->dem_at = 0; }
    for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < n_chunks; x += (int64_t)gridDim.x * blockDim.x)
        dem_seg[x] = 0;
}

// Offsets, weights, chunk ids, sum_i w(R_i), the longest request, and the
// slots of every chunk counted into dem_seg[x]; rank[j]: slot j's place among
// its chunk's. Popular chunks are in a quarter of all requests, and atomics on
// one address serialise device-wide, so each workgroup counts its slice of the
// slots in an LDS hash table first (linear probing; a slot that finds no entry
// counts in memory directly) and adds each entry once.
constexpr int kCountThreads = 1024;
constexpr int kCountSlice = 4096;              // slots per workgroup pass
constexpr int kCountBits = 13;
constexpr int kCountEntries = 1 << kCountBits;
constexpr int kCountProbes = 16;
__global__ __launch_bounds__(kCountThreads) void k_g_check(int m, int64_t n_chunks, int64_t nnz,
                                                           const int64_t *__restrict__ req_off,
                                                           const int32_t *__restrict__ req_chunks,
                                                           const int64_t *__restrict__ w, uint64_t *dem_seg,
                                                           uint32_t *__restrict__ rank, GHeader *h) {
    constexpr int PER = kCountSlice / kCountThreads;
    __shared__ uint32_t key[kCountEntries];    // chunk + 1; 0: empty
    __shared__ uint32_t cnt[kCountEntries];    // its slots here, then its slots before this workgroup's
    __shared__ uint64_t red[kCountThreads / kWave];
    const int64_t t0 = blockIdx.x * (int64_t)kCountThreads + threadIdx.x, stride = (int64_t)gridDim.x * kCountThreads;
    const int lane = (int)(threadIdx.x & (kWave - 1));
    uint32_t err = 0;
    int64_t longest = 0;
    for (int64_t i = t0; i < m; i += stride) {
        const int64_t len = req_off[i + 1] - req_off[i];
        if (len < 0) err |= GERR_INVALID;
        longest = len > longest ? len : longest;
    }
    if (t0 == 0 && (req_off[0] != 0 || req_off[m] != nnz)) err |= GERR_INVALID;
    for (int64_t x = t0; x < n_chunks; x += stride)
        if (w[x] <= 0 || w[x] > MPT_MAX_CHUNK_WEIGHT) err |= GERR_WEIGHT;
    uint64_t total = 0;
    for (int64_t s0 = (int64_t)blockIdx.x * kCountSlice; s0 < nnz; s0 += (int64_t)gridDim.x * kCountSlice) {
        for (int e = (int)threadIdx.x; e < kCountEntries; e += kCountThreads) { key[e] = 0u; cnt[e] = 0u; }
        __syncthreads();
        int at[PER];                           // the slot's entry; -1: counted in memory or no slot
        uint32_t place[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int64_t j = s0 + q * kCountThreads + threadIdx.x;
            at[q] = -1;
            place[q] = 0;
            if (j >= nnz) continue;
            const int32_t x = req_chunks[j];
            if (x < 0 || (int64_t)x >= n_chunks) { err |= GERR_RANGE; continue; }
            const int64_t wx = w[x];
            if (wx > 0 && wx <= MPT_MAX_CHUNK_WEIGHT) total += (uint64_t)wx;
            uint32_t slot = ((uint32_t)x * 2654435761u) >> (32 - kCountBits);
            for (int p = 0; p < kCountProbes && at[q] < 0; ++p) {
                uint32_t k = *(volatile uint32_t *)&key[slot];      // (most find their chunk there)
                if (k == 0u) k = atomicCAS(&key[slot], 0u, (uint32_t)x + 1u);
                if (k == 0u || k == (uint32_t)x + 1u) {
                    at[q] = (int)slot;
                    place[q] = atomicAdd(&cnt[slot], 1u);
                }
                slot = (slot + 1u) & (kCountEntries - 1u);
            }
            if (at[q] < 0) rank[j] = (uint32_t)atomicAdd((unsigned long long *)&dem_seg[x], 1ull);
        }
        __syncthreads();
        for (int e = (int)threadIdx.x; e < kCountEntries; e += kCountThreads)
            if (key[e]) cnt[e] = (uint32_t)atomicAdd((unsigned long long *)&dem_seg[key[e] - 1u], (unsigned long long)cnt[e]);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if (at[q] >= 0) rank[s0 + q * kCountThreads + threadIdx.x] = cnt[at[q]] + place[q];
        __syncthreads();
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        total += __shfl_xor(total, off, kWave);
        const int64_t o = __shfl_xor(longest, off, kWave);
        longest = o > longest ? o : longest;
        err |= (uint32_t)__shfl_xor((int)err, off, kWave);
    }
    if (lane == 0) {
        red[threadIdx.x / kWave] = total;
        if (err) atomicOr(&h->err, err);
        if (longest > 0) atomicMax((long long *)&h->max_len, (long long)longest);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t sum = 0;
        for (int k = 0; k < kCountThreads / kWave; ++k) sum += red[k];
        if (sum) atomicAdd(&h->total, (unsigned long long)sum);
    }
}

// a stretch of dem for every chunk: dem_seg[x] = start << 32 | count
__global__ __launch_bounds__(kCountThreads) void k_g_stretches(int64_t n_chunks, uint64_t *dem_seg, GHeader *h) {
    __shared__ int sw[kCountThreads / kWave];
    __shared__ unsigned long long start;
    for (int64_t x0 = (int64_t)blockIdx.x * kCountThreads; x0 < n_chunks; x0 += (int64_t)gridDim.x * kCountThreads) {
        const int64_t x = x0 + threadIdx.x;
        const uint64_t c = x < n_chunks ? dem_seg[x] : 0;
        int total;
        const int before = block_scan((int)c, &total, sw);
        if (threadIdx.x == 0) start = total ? atomicAdd(&h->dem_at, (unsigned long long)total) : 0ull;
        __syncthreads();
        if (c) dem_seg[x] = ((start + (uint64_t)before) << 32) | c;
        __syncthreads();
    }
}

// Request lists (chunk ids ascending) into sig, with the check for repeated
// chunks, the demand lists, and sig_slot, where in dem a list entry's request
// stands. Lists of up to kSegMax chunks take a wave
// each, of up to kListMax a workgroup each; with a longer one, sig is left to
// a key sort. Nothing is done once an error is known.
__global__ __launch_bounds__(kListThreads) void k_g_lists(int m, const int64_t *__restrict__ req_off,
                                                          const int32_t *__restrict__ req_chunks,
                                                          const uint32_t *__restrict__ rank,
                                                          const uint64_t *__restrict__ dem_seg,
                                                          int32_t *__restrict__ sig, int32_t *__restrict__ sig_slot,
                                                          int32_t *__restrict__ sig_len, int32_t *__restrict__ dem,
                                                          GHeader *h) {
    __shared__ __align__(16) uint32_t stage[kListMax];
    if (h->err & ~GERR_DUP) return;            // (GERR_DUP is raised in this launch: no workgroup stops for it)
    const int64_t longest = h->max_len;
    const int lane = (int)(threadIdx.x & (kWave - 1));
    auto demand = [&](int64_t j, int32_t x, int i) {         // slot j's place in dem
        const int32_t at = (int32_t)(dem_seg[x] >> 32) + (int32_t)rank[j];
        dem[at] = (int32_t)i;
        return at;
    };
    if (longest <= kSegMax) {
        const int nwaves = (int)(gridDim.x * blockDim.x) / kWave;
        for (int i = (int)(blockIdx.x * blockDim.x + threadIdx.x) / kWave; i < m; i += nwaves) {
            const int64_t o = req_off[i];
            const int n = (int)(req_off[i + 1] - o);
            const int32_t c = lane < n ? req_chunks[o + lane] : 0;
            bool dup;
            const int pos = seg_rank((uint32_t)c, n, dup);
            if (lane < n) {
                sig_slot[o + pos] = demand(o + lane, c, i);
                sig[o + pos] = c;
                if (dup) atomicOr(&h->err, (uint32_t)GERR_DUP);
            }
            if (lane == 0) sig_len[i] = n;
        }
        return;
    }
    for (int i = (int)blockIdx.x; i < m; i += (int)gridDim.x) {
        const int64_t o = req_off[i];
        const int64_t n = req_off[i + 1] - o;
        if (threadIdx.x == 0) sig_len[i] = (int32_t)n;
        if (longest > kListMax) {
            for (int64_t e = threadIdx.x; e < n; e += kListThreads) demand(o + e, req_chunks[o + e], i);
        } else {
            list_ranks(stage, (int)n, [&](int e) { return (uint32_t)req_chunks[o + e]; },
                       [&](int e, uint32_t c, int pos, bool dup) {
                           sig[o + pos] = (int32_t)c;
                           sig_slot[o + pos] = demand(o + e, (int32_t)c, i);
                           if (dup) atomicOr(&h->err, (uint32_t)GERR_DUP);
                       });
            __syncthreads();
        }
    }
}

// (request, chunk) keys of every slot (valid input)
__global__ void k_g_keys(int m, int64_t nnz, const int64_t *req_off, const int32_t *req_chunks, uint64_t *keys) {
    for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < nnz; j += (int64_t)gridDim.x * blockDim.x) {
        int lo = 0, hi = m - 1;                     // request of slot j: last i with req_off[i] <= j
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (req_off[mid] <= j) lo = mid; else hi = mid - 1;
        }
        keys[j] = ((uint64_t)lo << 32) | (uint32_t)req_chunks[j];
    }
}

// sorted keys -> request lists; a repeated chunk inside a request is two
// equal adjacent keys. Slot j's entry stands in dem at its chunk's stretch +
// rank[j] (as k_g_lists wrote it), and in its list where the sorted keys of its
// request have it: a binary search in them, whatever the chunk's demand. (A
// look through the chunk's demand list took up to m reads: the pair weights of
// 1000 nested requests of 1001 to 2000 chunks took 4649 us with it, 2245 now.)
__global__ void k_g_sig_long(int m, int64_t nnz, const int64_t *req_off, const int32_t *req_chunks,
                             const uint64_t *keys, const uint64_t *dem_seg, const uint32_t *rank, int32_t *sig,
                             int32_t *sig_slot, GHeader *h) {
    for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < nnz; j += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t key = keys[j];
        sig[j] = (int32_t)(key & 0xffffffffu);
        if (j > 0 && key == keys[j - 1]) atomicOr(&h->err, (uint32_t)GERR_DUP);
        int a = 0, b = m - 1;                       // request of slot j: last i with req_off[i] <= j
        while (a < b) {
            const int mid = (a + b + 1) >> 1;
            if (req_off[mid] <= j) a = mid; else b = mid - 1;
        }
        const int32_t x = req_chunks[j];
        const uint64_t own = ((uint64_t)a << 32) | (uint32_t)x;
        int64_t lo = req_off[a], hi = req_off[a + 1];
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (keys[mid] < own) lo = mid + 1; else hi = mid;
        }
        sig_slot[lo] = (int32_t)(dem_seg[x] >> 32) + (int32_t)rank[j];
    }
}

// ---------------------------------------------------------------------------
// pair weights

// row a of P, a tile of kPairTile columns per workgroup: every chunk x of
// R_a adds w(x) to the columns of the requests in its demand list S_x (one
// wave per chunk, lanes along S_x), summed in LDS and written once. The
// row's tiles cover every column, so P needs no zeroing.
constexpr int kPairTile = 4096;
constexpr int kPairThreads = 256;
__global__ __launch_bounds__(kPairThreads) void k_g_pair_rows(int m, const int32_t *sig, const int64_t *req_off,
                                                              const int32_t *dem, const uint64_t *dem_seg,
                                                              const int64_t *w, int64_t *P, int sorted, const GHeader *h) {
    __shared__ unsigned long long row[kPairTile];
    const bool lists = sorted || h->max_len <= kListMax;
    if (h->err || !lists) return;              // (the lists are not there)
    const int tiles = (m + kPairTile - 1) / kPairTile;
    const int64_t a = blockIdx.x / tiles;
    const int c0 = (int)(blockIdx.x % tiles) * kPairTile;
    const int width = min(kPairTile, m - c0);
    for (int j = threadIdx.x; j < width; j += kPairThreads) row[j] = 0ull;
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    const int64_t s0 = req_off[a], s1 = req_off[a + 1];
    for (int64_t q = s0 + wid; q < s1; q += kPairThreads / kWave) {
        const int32_t x = sig[q];
        const unsigned long long wx = (unsigned long long)w[x];
        const uint64_t seg = dem_seg[x];
        const int32_t *holders = dem + (seg >> 32);
        const int n = (int)(seg & 0xffffffffu);
        for (int f = lane; f < n; f += kWave) {
            const int b = holders[f] - c0;
            if (b >= 0 && b < width) atomicAdd(&row[b], wx);
        }
    }
    __syncthreads();
    int64_t *out = P + a * (int64_t)m + c0;
    for (int j = threadIdx.x; j < width; j += kPairThreads) out[j] = (int64_t)row[j];
}

// ---------------------------------------------------------------------------
// agglomerative hierarchy

// best partner of every row: max over d != c of V[c][d], ties to the
// smallest d; one wave per row
__global__ void k_g_row_best(int m, const int64_t *V, int64_t *best_v, int32_t *best_p) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t row = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    if (row >= m) return;
    int64_t v = -1;
    int32_t p = -1;
    constexpr int U = 8;                         // columns per lane in flight (128 MiB: 24 us, 42 us one at a time)
    for (int d0 = lane; d0 < m; d0 += U * kWave) {
        int64_t x[U];
#pragma unroll
        for (int q = 0; q < U; ++q) x[q] = d0 + q * kWave < m ? V[row * m + d0 + q * kWave] : -2;
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int d = d0 + q * kWave;
            if (d < m && d != row && better(x[q], d, v, p)) { v = x[q]; p = d; }
        }
    }
    wave_best(v, p);
    if (lane == 0) { best_v[row] = v; best_p[row] = p; }
}

// The greedy's merges in rounds. Merge values never grow (Theorem 6 part
// i): a cluster formed from A and B shares with any C at most what A and B
// each share with C. Order pairs by (value desc, smaller name asc, larger
// name asc), where a cluster's name is its smallest request; the sequential
// greedy merges the first pair in this order every time. A pair (a, b) in
// which each is the other's best partner stays so under every other merge,
// so the sequential greedy merges it at some point: every round merges all
// such mutual-best pairs of positive value at once (the first pair overall
// is always one), until no positive value is left. The rounds produce the
// greedy's merges, not its sequence; the sequence is the pair order itself.
// A merge X that forms a cluster taking part in a later merge Y of names
// p < q comes first: X's value is at least Y's, and if equal, the parts
// named p and q already shared that value when X was chosen (their
// signatures contain those of Y's clusters), so X's pair preceded (p, q).
struct Rac {
    int m;
    const int64_t *w;
    const int64_t *req_off;     // start of each cluster's signature in sig
    int32_t *sig;               // signatures, ascending, shrinking in place
    int32_t *sig_slot;          // where in dem the entry's cluster stands
    int32_t *sig_len;
    int32_t *dem;               // the clusters holding each chunk (-1: no longer); stretch of chunk x: dem_seg[x]
    const uint64_t *dem_seg;
    int64_t *V;                 // V[a][c] = w(I(a) ∩ I(c)) for live a, c
    int64_t *best_v;
    int32_t *best_p;
    int32_t *act;               // 1 while the name is a live cluster
    int32_t *last;              // last merge record into each name (-1: a leaf)
    int32_t *touched;           // round in which the name last merged
    int32_t *resc;              // rows whose best partner is recomputed this round
    // merge records, in the order the rounds produce them
    int32_t *ra, *rb, *rca, *rcb, *rpos, *rdal, *rdbl;
    int64_t *rgain, *rdao, *rdbo;
    int64_t nnz;                // D(v) = I(v) \ I(parent(v)) lies in sig, or from sig[nnz] on (at most nnz entries)
    int32_t *live;              // the tail's clusters, ascending
    int64_t *dense;             // their V
    int64_t *d_off;
    int32_t *d_len;
    int32_t *merge_a, *merge_b;
    int64_t *gain;
    int32_t *node_parent;
    GHeader *h;
};

__device__ inline uint64_t lanes_below(int lane) { return (1ull << lane) - 1ull; }

__global__ void k_rac_init(Rac R) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    for (int64_t r = t0; r < R.m; r += stride) { R.act[r] = 1; R.last[r] = -1; R.touched[r] = -1; R.rpos[r] = 0; }
    for (int64_t v = t0; v < 2 * (int64_t)R.m - 1; v += stride) { R.node_parent[v] = -1; R.d_off[v] = 0; R.d_len[v] = 0; }
    if (t0 == 0) {
        R.h->n_rec = 0;
        R.h->lo = 0;
        R.h->n_resc[0] = 0;
        R.h->n_resc[1] = 0;
        R.h->last_pairs = -1;
        R.h->dcursor = 0;
    }
}

// whether z is among the ascending values y of the wave's lanes (INT32_MAX:
// none), by shuffles: six halvings of 64
__device__ inline bool lane_find(int32_t y, int32_t z) {
    int at = 0;
#pragma unroll
    for (int h = 32; h > 0; h >>= 1) at += __shfl(y, at + h - 1, kWave) < z ? h : 0;
    return __shfl(y, at, kWave) == z;
}

// One wave merges clusters a and b as record i: I(C) = I(A) ∩ I(B) in place of
// I(A), D(B) = I(B) \ I(A) and D(A) = I(A) \ I(B), and the merges that formed A
// and B; b and what a loses leave the demand lists. Lists of up to 64 chunks
// are read once and matched in registers, and the D lists stay where their
// chunks were: D(A) behind what is left of A's list, D(B) in front of B's,
// which no cluster reads any more. Longer ones search each other in memory and
// move their D lists to sig + nnz, at reserve(entries) on lane 0. rec(): the
// record's number, asked for once the lists' reads are under way. Returns
// |I(C)|, or -1 (cannot happen) when there is no room.
template <class Rec, class Reserve>
__device__ inline int merge_pair(const Rac &R, int32_t a, int32_t b, int64_t oa, int64_t na, int64_t ob, int64_t nb,
                                 int64_t gain, int round, Rec &&rec, Reserve &&reserve) {
    const int lane = threadIdx.x & (kWave - 1);
    const int32_t la = R.last[a], lb = R.last[b];
    int32_t *sa = R.sig + oa, *sb = R.sig + ob, *ta = R.sig_slot + oa;
    const int32_t *tb = R.sig_slot + ob;
    int64_t kept = 0, d_a, d_b;                  // where the D lists lie in sig
    int64_t i;
    if (na <= kWave && nb <= kWave) {
        int32_t x = INT32_MAX, z = INT32_MAX, xt = 0, zt = 0;
        if (lane < na) { x = sa[lane]; xt = ta[lane]; }
        if (lane < nb) { z = sb[lane]; zt = tb[lane]; }
        i = rec();
        if (i < 0) return -1;
        const bool in_b = lane_find(z, x) && lane < na;
        const bool in_a = lane_find(x, z) && lane < nb;
        const uint64_t mb = __ballot(lane < nb && !in_a), mi = __ballot(in_b), mo = __ballot(lane < na && !in_b);
        kept = __popcll(mi);
        if (lane < nb) R.dem[zt] = -1;
        if (lane < nb && !in_a) sb[__popcll(mb & lanes_below(lane))] = z;
        if (in_b) {
            const int at = __popcll(mi & lanes_below(lane));
            sa[at] = x;
            ta[at] = xt;
        } else if (lane < na) {
            sa[kept + __popcll(mo & lanes_below(lane))] = x;
            R.dem[xt] = -1;
        }
        d_a = oa + kept;
        d_b = ob;
    } else {
        i = rec();
        if (i < 0) return -1;
        for (int64_t base = 0; base < na; base += kWave) {
            const int64_t e = base + lane;
            kept += __popcll(__ballot(e < na && find_sorted(sb, nb, sa[e]) >= 0));
        }
        const int64_t dlen = na + nb - 2 * kept;
        unsigned long long dstart = 0;
        if (lane == 0) dstart = reserve((unsigned long long)dlen);
        dstart = __shfl(dstart, 0, kWave);
        if ((int64_t)dstart + dlen > R.nnz) return -1;
        int32_t *dbuf = R.sig + R.nnz;
        int64_t dcur = (int64_t)dstart;
        d_b = R.nnz + dcur;
        d_a = d_b + (nb - kept);
        for (int64_t base = 0; base < nb; base += kWave) {
            const int64_t e = base + lane;
            bool keep = false;
            int32_t z = 0;
            if (e < nb) { z = sb[e]; keep = find_sorted(sa, na, z) < 0; R.dem[tb[e]] = -1; }
            const uint64_t mk = __ballot(keep);
            if (keep) dbuf[dcur + __popcll(mk & lanes_below(lane))] = z;
            dcur += __popcll(mk);
        }
        // in place: a lane writes at or below the entry it read, and the
        // entries above the current 64 are not written yet
        int64_t k = 0;
        for (int64_t base = 0; base < na; base += kWave) {
            const int64_t e = base + lane;
            int32_t x = 0, xt = 0;
            bool in_b = false;
            if (e < na) { x = sa[e]; xt = ta[e]; in_b = find_sorted(sb, nb, x) >= 0; }
            const uint64_t mi = __ballot(in_b);
            const uint64_t mo = __ballot(e < na && !in_b);
            if (in_b) {
                const int64_t at = k + __popcll(mi & lanes_below(lane));
                sa[at] = x;
                ta[at] = xt;
            } else if (e < na) {
                dbuf[dcur + __popcll(mo & lanes_below(lane))] = x;
                R.dem[xt] = -1;
            }
            k += __popcll(mi);
            dcur += __popcll(mo);
        }
    }
    if (lane == 0) {
        R.ra[i] = a;
        R.rb[i] = b;
        R.rgain[i] = gain;
        R.sig_len[a] = (int32_t)kept;
        R.act[b] = 0;
        R.touched[a] = round;
        R.touched[b] = round;
        R.rca[i] = la;
        R.rcb[i] = lb;
        R.last[a] = (int32_t)i;
        R.rdbo[i] = d_b;
        R.rdbl[i] = (int32_t)(nb - kept);
        R.rdao[i] = d_a;
        R.rdal[i] = (int32_t)(na - kept);
    }
    return (int)kept;
}

// One wave per row a: if a and its best partner b > a are mutual best with
// positive value, a new merge record i (a, b, value) is taken and the wave
// merges the pair. The pair test reads only values that no merge of the round
// writes (best values and partners; a partner b that a merge deactivates fails
// the test b > best partner as well), so merging while other waves still test
// finds the same pairs. Record numbers within a round follow the atomic
// order; the sequence is recovered by sorting on the pair order.
__global__ void k_rac_pairs_merge(Rac R, int round) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) / kWave;
    for (int64_t a = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kWave; a < R.m; a += nwaves) {
        // (read together: a wave's time is its chain of dependent reads)
        const int32_t live = R.act[a], b = R.best_p[a];
        const int64_t v = R.best_v[a];
        if (!live || v <= 0 || b <= (int32_t)a || R.best_p[b] != (int32_t)a) continue;
        const int kept = merge_pair(
            R, (int32_t)a, b, R.req_off[a], R.sig_len[a], R.req_off[b], R.sig_len[b], v, round,
            [&]() {
                int i = 0;
                if (lane == 0) i = atomicAdd(&R.h->n_rec, 1);
                i = __shfl(i, 0, kWave);
                return i < R.m - 1 ? (int64_t)i : -1;
            },
            [&](unsigned long long n) { return atomicAdd(&R.h->dcursor, n); });
        if (kept < 0 && lane == 0) atomicOr(&R.h->err, (uint32_t)GERR_INVALID);   // cannot happen
    }
}

// The clusters that hold the chunks of a list, walked by whole waves: add(c, w)
// for every chunk y of list[0 .. kept) and live cluster c holding it (the
// merged cluster itself among them), w = w(y). 64 chunks at a time, a lane
// each; the entries of their demand lists are laid end to end and taken first,
// first + stride, ... (first + a multiple of stride below the sum), each lane
// finding its chunk by shuffles, four entries in flight. Entries of clusters
// that merged away or lost the chunk read -1.
template <class Add>
__device__ inline void walk_holders(const Rac &R, const int32_t *list, int kept, int first, int stride, Add &&add) {
    const int lane = (int)(threadIdx.x & (kWave - 1));
    for (int base = 0; base < kept; base += kWave) {
        const bool has = base + lane < kept;
        const int32_t y = has ? list[base + lane] : 0;
        const uint64_t seg = has ? R.dem_seg[y] : 0;
        const int64_t wy = has ? R.w[y] : 0;
        const int n = (int)(seg & 0xffffffffu);
        int upto = n;                                     // entries of this lane's chunk and those before it
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int q = __shfl_up(upto, o, kWave);
            if (lane >= o) upto += q;
        }
        const int total = __shfl(upto, kWave - 1, kWave);
        const int shift = (int)(seg >> 32) - (upto - n);  // entry t lies at t + shift
        constexpr int U = 4;
        for (int t0 = 0; t0 < total; t0 += U * stride) {  // (the same turns for every lane)
            int32_t c[U];
            int64_t wt[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int t = t0 + u * stride + first;
                int at = 0;                               // chunks that end at or before entry t
#pragma unroll
                for (int hlf = 32; hlf > 0; hlf >>= 1) at += __shfl(upto, at + hlf - 1, kWave) <= t ? hlf : 0;
                const int sh = __shfl(shift, at, kWave);
                wt[u] = __shfl(wy, at, kWave);
                c[u] = t < total ? R.dem[t + sh] : -1;
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (c[u] >= 0) add(c[u], wt[u]);
        }
    }
}

// The new clusters' rows: a workgroup per merge and tile of kPairTile columns
// sums w(y) over the chunks y of the merged list into the columns of the
// clusters that hold y, in LDS, and writes what changed: the row of a by its
// own merge (columns of clusters merged in the same round included: both sides
// compute the same value), the column entry of every other row here. The work
// is the holders of the merged list, and the time a chain of seven reads, 10 to
// 12 us whatever the lists are; intersecting the list with every column's list
// took 33 us in the first 16 rounds of 701 requests of up to 100 chunks.
// The same launch marks the rows whose best partner may have changed: the new
// clusters, the rows whose best partner was merged away, and those whose value
// with a best partner that lives on as a new cluster fell (no other row's best
// can change: values only fall, and the partner is the smallest name at its
// value). Of the rows whose best partner merged, that leaves a third to a half
// at m = 4096.
constexpr int kRowThreads = 512;
__global__ __launch_bounds__(kRowThreads) void k_rac_rows(Rac R, int round) {
    __shared__ unsigned long long row[kPairTile];
    constexpr int PER = kPairTile / kRowThreads;             // columns per thread
    const int lo = R.h->lo, hi = min(R.h->n_rec, R.m - 1);
    if (hi <= lo) return;                        // nothing merged, nothing to rescan
    const int64_t m = R.m;
    const int tid = (int)threadIdx.x;
    const int tiles = (R.m + kPairTile - 1) / kPairTile;
    for (int64_t f = blockIdx.x; f < (int64_t)(hi - lo) * tiles; f += gridDim.x) {
        const int32_t a = R.ra[lo + f / tiles];
        const int c0 = (int)(f % tiles) * kPairTile;
        const int width = min(kPairTile, R.m - c0);
        // the old row, on its way while the holders are walked
        int64_t va[PER];
        int32_t live[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int j = tid + u * kRowThreads;
            va[u] = j < width ? R.V[a * m + c0 + j] : 0;
            live[u] = j < width ? R.act[c0 + j] : 0;
            row[j] = 0ull;
        }
        __syncthreads();
        walk_holders(R, R.sig + R.req_off[a], R.sig_len[a], tid, kRowThreads, [&](int32_t c, int64_t w) {
            if (c >= c0 && c < c0 + width) atomicAdd(&row[c - c0], (unsigned long long)w);
        });
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int j = tid + u * kRowThreads;
            if (!live[u] || c0 + j == a) continue;
            const int64_t x = c0 + j, v = (int64_t)row[j];
            if (v == va[u]) continue;
            R.V[a * m + x] = v;
            if (R.touched[x] == round) continue;
            R.V[x * m + a] = v;
            if (R.best_p[x] == a) R.resc[atomicAdd(&R.h->n_resc[round & 1], 1)] = (int32_t)x;
        }
        __syncthreads();
    }
    for (int64_t x = blockIdx.x * (int64_t)kRowThreads + tid; x < m; x += (int64_t)gridDim.x * kRowThreads) {
        if (!R.act[x]) continue;
        const int32_t p = R.best_p[x];
        if (R.touched[x] == round || (p >= 0 && !R.act[p]))
            R.resc[atomicAdd(&R.h->n_resc[round & 1], 1)] = (int32_t)x;
    }
}

// one workgroup per marked row: best partner, ties to the smallest index;
// each thread loads 8 columns before comparing them. Block 0 also closes
// the round: the next round's records start at the current count, and its
// rescan counter starts at 0.
constexpr int kRescThreads = 512;
__global__ __launch_bounds__(kRescThreads) void k_rac_rescan(Rac R, int round) {
    __shared__ int64_t sv[kRescThreads / kWave];
    __shared__ int32_t si[kRescThreads / kWave];
    const int n = R.h->n_resc[round & 1];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        R.h->last_pairs = R.h->n_rec - R.h->lo;
        R.h->lo = R.h->n_rec;
        R.h->n_resc[(round + 1) & 1] = 0;
    }
    const int64_t m = R.m;
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    constexpr int U = 8;
    for (int j = blockIdx.x; j < n; j += gridDim.x) {
        const int32_t x = R.resc[j];
        const int64_t *row = R.V + x * m;
        int64_t v = -1;
        int32_t p = -1;
        for (int64_t d0 = threadIdx.x; d0 < m; d0 += (int64_t)kRescThreads * U) {
            int64_t val[U];
            int32_t live[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t d = d0 + (int64_t)u * kRescThreads;
                val[u] = d < m ? row[d] : -1;
                live[u] = d < m ? R.act[d] : 0;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int32_t d = (int32_t)(d0 + (int64_t)u * kRescThreads);
                if (live[u] && d != x && better(val[u], d, v, p)) { v = val[u]; p = d; }
            }
        }
        wave_best(v, p);
        if (lane == 0) { sv[wid] = v; si[wid] = p; }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int k = 1; k < kRescThreads / kWave; ++k)
                if (better(sv[k], si[k], v, p)) { v = sv[k]; p = si[k]; }
            R.best_v[x] = v;
            R.best_p[x] = p;
        }
        __syncthreads();
    }
}

constexpr int kChainThreads = 1024;

// The tail's clusters: the live ones in ascending order (one workgroup), and
// their part of V as a dense matrix (a workgroup per row): the tail reads whole
// rows of it from one CU, whose reads cost a line each in V's scattered columns
// (22 us a round there, m = 4096, 500 clusters left).
__global__ __launch_bounds__(kChainThreads) void k_rac_live(Rac R) {
    __shared__ int scan_w[kChainThreads / kWave];
    int done = 0;
    for (int base = 0; base < R.m; base += kChainThreads) {
        const int r = base + (int)threadIdx.x;
        const int live = r < R.m && R.act[r];
        int tot;
        const int at = done + block_scan(live, &tot, scan_w);
        if (live) R.live[at] = r;
        done += tot;
    }
}

// The demand lists without the entries that left them, a wave per chunk; the
// clusters' lists learn their entries' new places.
__global__ void k_rac_tidy(Rac R, int64_t n_chunks, uint64_t *dem_seg) {
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) / kWave;
    for (int64_t x = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kWave; x < n_chunks; x += nwaves) {
        const uint64_t seg = dem_seg[x];
        const int start = (int)(seg >> 32), n = (int)(seg & 0xffffffffu);
        int k = 0;
        for (int base = 0; base < n; base += kWave) {
            const int32_t c = base + lane < n ? R.dem[start + base + lane] : -1;
            const uint64_t left = __ballot(c >= 0);
            if (c >= 0) {
                const int at = start + k + __popcll(left & lanes_below(lane));
                const int64_t o = R.req_off[c], e = find_sorted(R.sig + o, R.sig_len[c], (int32_t)x);
                R.dem[at] = c;           // (at or below the entry read)
                if (e >= 0) R.sig_slot[o + e] = at;
            }
            k += __popcll(left);
        }
        if (lane == 0 && k != n) dem_seg[x] = ((uint64_t)start << 32) | (uint64_t)k;
    }
}

__global__ __launch_bounds__(256) void k_rac_dense(Rac R, int L) {
    const int64_t i = blockIdx.x, x = R.live[i];
    for (int j = threadIdx.x; j < L; j += 256) R.dense[i * L + j] = R.V[x * R.m + R.live[j]];
}

// All remaining rounds by one workgroup, once few clusters are left and few
// pairs merge per round: the same rounds as the three kernels above, with the
// live clusters' names, best partners and lists' places in LDS and barriers in
// the place of launches. A round of one to a dozen merges spends its time in
// dependent reads (of the lists, their holders, the rows to rescan), not in work
// for 256 CUs: 15 us here at m = 4096 (40 rounds from 650 clusters on), 24 us
// for three launches and as much as 10 more for their gaps, and no round is
// launched in vain (the batches ran up to 31 empty ones).
// Every round merges at least one pair of the live clusters, so the loop ends
// after fewer than kTailLive rounds.
constexpr int kTailThreads = 1024;
// (pairs of the last round) x (live clusters) up to which the tail takes over
// (20000: 8 rounds earlier, 270 us more in the tail and 240 us less before it at
// m = 4096, and 415 against 200 us at 701 long requests), and (pairs of the last
// round)^2 x (mean request length), for long lists: a round's merges share the
// waves, so a merge takes the longer the more there are, where the chip's rounds
// take as long as one merge. Whole hierarchies of m requests of k chunks over u
// by the tail alone and by the chip's rounds alone, in us: m = 40, k = 500, u =
// 2000 (24500) 629 and 690; 100, 100, 400 (28900) 351 and 391; 100, 150, 500
// (43350) 461 and 614, with the tail after eight rounds of the chip 430; 200,
// 100, 400 (115600) 626 and 548, so 478; 200, 500, 1000 3081 and 1495, so 1428;
// 200, 5000, 10000 29700 and 12500, so 12500.
constexpr int64_t kTailWork = 8192;
constexpr int64_t kTailEntries = 40000;
constexpr int kTailAcc = 3 * kTailLive;
struct TailLds {
    int64_t bv[kTailLive];               // best value
    int64_t off[kTailLive];              // the list: sig[off .. off + len)
    int32_t len[kTailLive];
    int32_t stamp[kTailLive];            // round in which the cluster last merged
    uint16_t id[kTailLive];              // names, ascending
    uint16_t bp[kTailLive];              // place of the best partner; kNoPlace: none
    uint16_t queue[kTailLive];           // places of the rows to rescan
    uint16_t pa[kTailLive / 2], pb[kTailLive / 2];
    uint8_t dead[kTailLive];
    uint16_t place[MPT_GREEDY_MAX_M];    // name -> place
    unsigned long long acc[kTailAcc];    // new rows in the making
    int n_pairs, n_queue;
    unsigned long long dcursor;
};
constexpr uint16_t kNoPlace = 0xffffu;
__global__ __launch_bounds__(kTailThreads) void k_rac_tail(Rac R, int L, int round) {
    __shared__ TailLds T;
    const int tid = (int)threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    constexpr int kWaves = kTailThreads / kWave;
    for (int i = tid; i < L; i += kTailThreads) {
        T.id[i] = (uint16_t)R.live[i];
        T.place[R.live[i]] = (uint16_t)i;
    }
    __syncthreads();
    for (int i = tid; i < L; i += kTailThreads) {
        const int32_t x = T.id[i], p = R.best_p[x];
        T.bp[i] = p >= 0 ? T.place[p] : kNoPlace;        // (the best partner of a live cluster is live)
        T.bv[i] = R.best_v[x];
        T.off[i] = R.req_off[x];
        T.len[i] = R.sig_len[x];
        T.stamp[i] = -1;
        T.dead[i] = 0;
    }
    int n_rec = min(R.h->n_rec, R.m - 1);
    if (tid == 0) T.dcursor = R.h->dcursor;
    for (;; ++round) {
        if (tid == 0) { T.n_pairs = 0; T.n_queue = 0; }
        __syncthreads();
        for (int i = tid; i < L; i += kTailThreads) {
            const uint16_t p = T.bp[i];
            if (T.dead[i] || T.bv[i] <= 0 || p == kNoPlace || (int)p <= i || (int)T.bp[p] != i) continue;
            const int f = atomicAdd(&T.n_pairs, 1);
            T.pa[f] = (uint16_t)i;
            T.pb[f] = p;
        }
        __syncthreads();
        const int np = T.n_pairs;
        if (np == 0 || n_rec + np > R.m - 1) break;      // (the second cannot happen)
        for (int f = wv; f < np; f += kWaves) {
            const int ia = T.pa[f], ib = T.pb[f];
            const int32_t a = T.id[ia], b = T.id[ib];
            const int kept = merge_pair(R, a, b, T.off[ia], T.len[ia], T.off[ib], T.len[ib], T.bv[ia], round,
                                        [&]() { return (int64_t)(n_rec + f); },
                                        [&](unsigned long long n) { return atomicAdd(&T.dcursor, n); });
            if (lane == 0) {
                if (kept < 0) atomicOr(&R.h->err, (uint32_t)GERR_INVALID);       // cannot happen
                T.len[ia] = max(kept, 0);
                T.dead[ib] = 1;
                T.stamp[ia] = round;
                T.stamp[ib] = round;
            }
        }
        n_rec += np;
        __syncthreads();
        // the new rows: as many merges at a time as the LDS holds rows for, the
        // waves shared out among them
        const int par = min(min(np, kWaves), kTailAcc / L), per = kWaves / par;
        for (int f0 = 0; f0 < np; f0 += par) {
            const int slot = wv / per, f = f0 + slot;
            const bool mine = slot < par && f < np;
            const int first = (wv % per) * kWave + lane, stride = per * kWave;
            unsigned long long *acc = T.acc + (size_t)slot * L;
            if (mine)
                for (int c = first; c < L; c += stride) acc[c] = 0ull;
            __syncthreads();
            if (mine) {
                const int ia = T.pa[f];
                walk_holders(R, R.sig + T.off[ia], T.len[ia], first, stride, [&](int32_t c, int64_t w) {
                    atomicAdd(&acc[T.place[c]], (unsigned long long)w);
                });
            }
            __syncthreads();
            if (mine) {
                const int64_t ia = T.pa[f];
                constexpr int U = 4;
                for (int d0 = first; d0 < L; d0 += U * stride) {
                    int64_t va[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int d = d0 + u * stride;
                        va[u] = d < L && d != ia && !T.dead[d] ? R.dense[ia * L + d] : -1;
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        if (va[u] < 0) continue;
                        const int64_t d = d0 + u * stride, v = (int64_t)acc[d];
                        if (v == va[u]) continue;
                        R.dense[ia * L + d] = v;
                        if (T.stamp[d] == round) continue;
                        R.dense[d * L + ia] = v;
                        if ((int64_t)T.bp[d] == ia) T.queue[atomicAdd(&T.n_queue, 1)] = (uint16_t)d;
                    }
                }
            }
            __syncthreads();                             // the rows' LDS is the next merges'
        }
        for (int i = tid; i < L; i += kTailThreads) {
            if (T.dead[i]) continue;
            const uint16_t p = T.bp[i];
            if (T.stamp[i] == round || (p != kNoPlace && T.dead[p]))
                T.queue[atomicAdd(&T.n_queue, 1)] = (uint16_t)i;
        }
        __syncthreads();
        // best partners of the queued rows, a wave each, two rows in flight
        for (int q = wv; q < T.n_queue; q += 2 * kWaves) {
            const int qq[2] = {q, q + kWaves < T.n_queue ? q + kWaves : q};
            int64_t v[2] = {-1, -1};
            int32_t p[2] = {-1, -1};
            for (int d0 = lane; d0 < L; d0 += 8 * kWave) {
                int64_t x[2][8];
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int d = d0 + u * kWave, i = T.queue[qq[k]];
                        x[k][u] = d < L && d != i && !T.dead[d] ? R.dense[(int64_t)i * L + d] : -2;
                    }
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (x[k][u] >= 0 && better(x[k][u], d0 + u * kWave, v[k], p[k])) {
                            v[k] = x[k][u];
                            p[k] = d0 + u * kWave;
                        }
            }
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                wave_best(v[k], p[k]);
                if (lane == 0) {
                    T.bv[T.queue[qq[k]]] = v[k];
                    T.bp[T.queue[qq[k]]] = p[k] < 0 ? kNoPlace : (uint16_t)p[k];
                }
            }
        }
        __syncthreads();
    }
    if (tid == 0) {
        R.h->n_rec = n_rec;
        R.h->lo = n_rec;
        R.h->last_pairs = 0;
        R.h->dcursor = T.dcursor;
    }
}

// position of every record in the greedy's sequence: the records before it
// in the pair order (gain descending, names ascending). Blocks take a tile of
// records (x) against a tile of kRankTileY others, held in LDS, and add their
// counts (positions start at 0). 64 others a block and four comparisons in
// flight: with 256, one after the other, the 3700 records of m = 4096 took 28
// us.
constexpr int kRankThreads = 256;
constexpr int kRankTileY = 64;
__global__ __launch_bounds__(kRankThreads) void k_rac_rank(Rac R, int n) {
    __shared__ int64_t tg[kRankTileY];
    __shared__ uint32_t tn[kRankTileY];
    const int i = blockIdx.x * kRankThreads + threadIdx.x;
    const int j0 = blockIdx.y * kRankTileY;
    const int j = j0 + (int)threadIdx.x;
    if ((int)threadIdx.x < kRankTileY) {         // a record past the end comes after every other
        tg[threadIdx.x] = j < n ? R.rgain[j] : -1;
        tn[threadIdx.x] = j < n ? (uint32_t)R.ra[j] << 14 | (uint32_t)R.rb[j] : ~0u;
    }
    __syncthreads();
    if (i >= n) return;
    const int64_t g = R.rgain[i];
    const uint32_t names = (uint32_t)R.ra[i] << 14 | (uint32_t)R.rb[i];
    int pos = 0;
#pragma unroll 4
    for (int k = 0; k < kRankTileY; ++k) pos += tg[k] > g || (tg[k] == g && tn[k] < names) ? 1 : 0;
    if (pos) atomicAdd(&R.rpos[i], pos);
}
static_assert(MPT_GREEDY_MAX_M <= 1 << 14, "two names in 28 bits");

// tree node of merge record i is m + its position; leaves are 0 .. m - 1
__device__ inline int32_t rec_node(const Rac &R, int32_t rec, int32_t leaf) {
    return rec >= 0 ? R.m + R.rpos[rec] : leaf;
}

__global__ void k_rac_emit(Rac R, int n) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const int t = R.rpos[i];
        const int32_t a = R.ra[i], b = R.rb[i];
        R.merge_a[t] = a;
        R.merge_b[t] = b;
        R.gain[t] = R.rgain[i];
        const int32_t node = R.m + t;
        const int32_t na = rec_node(R, R.rca[i], a), nb = rec_node(R, R.rcb[i], b);
        R.node_parent[na] = node;
        R.node_parent[nb] = node;
        R.d_off[na] = R.rdao[i];
        R.d_len[na] = R.rdal[i];
        R.d_off[nb] = R.rdbo[i];
        R.d_len[nb] = R.rdbl[i];
    }
}

// Every remaining pair shares nothing: the merges take the two smallest
// live names in turn (n0, n1), (n0, n2), ... with gain 0, and every
// merged signature is empty, so D(child) is the child's whole signature
// (the root's whole signature if only one cluster is left) and the
// chain's own nodes emit nothing. Live names in ascending order, one
// round of the workgroup at a time.
__global__ __launch_bounds__(kChainThreads) void k_rac_chain(Rac R, int t0) {
    __shared__ int scan_w[kChainThreads / kWave];
    __shared__ int32_t first_name;
    __shared__ unsigned long long savings;
    const int m = R.m, tid = threadIdx.x;
    if (tid == 0) { first_name = -1; savings = 0ull; }
    __syncthreads();
    // SAV(H): the gains of the merges found (k_rac_emit; the chain's are 0)
    unsigned long long sum = 0;
    for (int t = tid; t < t0; t += kChainThreads) sum += (unsigned long long)R.gain[t];
    if (sum) atomicAdd(&savings, sum);
    int done = 0;                                // live names ranked so far
    for (int base = 0; base < m; base += kChainThreads) {
        const int r = base + tid;
        const int live = r < m && R.act[r];
        int tot;
        const int rank = done + block_scan(live, &tot, scan_w);
        if (live) {
            const int32_t node = rec_node(R, R.last[r], r);
            R.d_off[node] = R.req_off[r];
            R.d_len[node] = R.sig_len[r];
            if (rank == 0) {
                first_name = r;
            } else {
                const int tt = t0 + rank - 1;    // the merge that takes r
                if (tt < m - 1) {
                    R.merge_b[tt] = r;
                    R.gain[tt] = 0;
                    R.node_parent[node] = m + tt;
                }
            }
        }
        done += tot;
        __syncthreads();
    }
    const int n_live = done;
    // the chain: node m+t0 holds the first two names, node m+t0+k holds
    // node m+t0+k-1 and the name of rank k+1
    for (int k = tid; k + 1 < n_live && t0 + k < m - 1; k += kChainThreads) {
        R.merge_a[t0 + k] = first_name;
        R.d_off[m + t0 + k] = 0;
        R.d_len[m + t0 + k] = 0;
        if (k > 0) R.node_parent[m + t0 + k - 1] = m + t0 + k;
    }
    if (tid == 0 && n_live >= 2) R.node_parent[rec_node(R, R.last[first_name], first_name)] = m + t0;
    if (tid == 0 && t0 + n_live - 1 != m - 1) atomicOr(&R.h->err, GERR_INVALID);
    if (tid == 0) R.h->savings = savings;      // (added before the first barrier of the loop above: m >= 1)
}

// pi_i: walk from leaf i to the root, placing D(v) of every node on the
// path right to left (the root's list comes first); one wave per request.
// The zero-gain merges (nodes m + chain_from and up) emit nothing and
// every node above one of them is one of them, so a walk ends there.
__global__ void k_g_orders(int m, int64_t nnz, const int64_t *req_off, const int32_t *node_parent,
                           const int32_t *sig, const int64_t *d_off, const int32_t *d_len, int32_t *order_chunks,
                           int chain_from, GHeader *h) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    if (i >= m) return;
    int64_t end = req_off[i + 1];
    const int64_t begin = req_off[i];
    int steps = 0;
    for (int v = (int)i; v >= 0 && steps < 2 * m; v = node_parent[v], ++steps) {
        if (v >= 2 * m - 1) { if (lane == 0) atomicOr(&h->err, GERR_INVALID); return; }
        if (v >= m + chain_from) break;
        const int64_t len = d_len[v];
        if (len < 0 || end - len < begin || d_off[v] < 0 || d_off[v] + len > 2 * nnz) {
            if (lane == 0) atomicOr(&h->err, GERR_INVALID);
            return;
        }
        const int32_t *src = sig + d_off[v];
        for (int64_t e = lane; e < len; e += kWave) order_chunks[end - len + e] = src[e];
        end -= len;
    }
    if (end != begin && lane == 0) atomicOr(&h->err, GERR_INVALID);
}

// ---------------------------------------------------------------------------
// maximum spanning tree (Boruvka). Edges are ordered by (weight desc, then
// the pair (lo, hi) of their endpoints ascending), a strict total order, so
// every round's chosen edges form a forest plus mutual pairs and no cycle
// can close. Every round at least halves the number of components; the
// complete graph keeps an edge between any two, so ceil(log2 m) rounds
// leave one. The tree's weight does not depend on which order breaks ties.

__device__ inline uint32_t edge_id(int u, int v) {
    const uint32_t lo = (uint32_t)min(u, v), hi = (uint32_t)max(u, v);
    return (lo << 14) | hi;                      // m <= 2^14
}

// Borůvka's rounds after the last component has formed change nothing:
// k_bv_merge raises h->bv_done when a root finds no edge out of its
// component (P is complete, so that root's component holds every vertex),
// and the later rounds' kernels return at once.
__global__ void k_bv_init(int m, int32_t *comp, int64_t *vw, int64_t *cw, GHeader *h) {
    for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < m; v += gridDim.x * blockDim.x) {
        comp[v] = v;
        vw[v] = -1;
        cw[v] = -1;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        h->total = 0;
        h->bv_done = 0;
    }
}

// *p = max(*p, v) for a value that only rises: an atomic only where it would
// still raise it (all vertices of a large component share p, and atomics on one
// address serialise: a round of two components took 52 us, others 28)
__device__ inline void raise_best(int64_t *p, int64_t v) {
    if (__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < v) atomicMax((long long *)p, (long long)v);
}

// best edge of every vertex to another component (one wave per vertex),
// folded into its component's best weight
__global__ void k_bv_vertex(int m, const int64_t *P, const int32_t *comp, int64_t *vw, uint32_t *ve, int64_t *cw,
                            const GHeader *h) {
    if (h->bv_done) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t u = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    if (u >= m) return;
    const int32_t cu = comp[u];
    int64_t bw = vw[u];
    uint32_t be = bw >= 0 ? ve[u] : ~0u;
    // the vertex's best edge of an earlier round stays its best while it
    // leaves the component (the edges to choose from only get fewer)
    if (bw >= 0 && comp[(int64_t)(be >> 14) == u ? be & 0x3fffu : be >> 14] != cu) {
        if (lane == 0) raise_best(&cw[cu], bw);
        return;
    }
    bw = -1;
    be = ~0u;
    // eight columns per lane in flight (twelve rounds at m = 4096, five of
    // them real: 219 us, one column at a time 254 us)
    constexpr int U = 8;
    for (int v0 = lane; v0 < m; v0 += U * kWave) {
        int64_t x[U];
        int32_t c[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int v = v0 + q * kWave;
            x[q] = v < m ? P[u * m + v] : -1;
            c[q] = v < m ? comp[v] : cu;
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const uint32_t e = edge_id((int)u, v0 + q * kWave);
            if (c[q] != cu && (x[q] > bw || (x[q] == bw && e < be))) { bw = x[q]; be = e; }
        }
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        const int64_t ow = __shfl_xor(bw, off, kWave);
        const uint32_t oe = (uint32_t)__shfl_xor((int)be, off, kWave);
        if (ow > bw || (ow == bw && oe < be)) { bw = ow; be = oe; }
    }
    if (lane == 0) {
        vw[u] = bw; ve[u] = be;
        if (bw >= 0) raise_best(&cw[cu], bw);
    }
}

// The rest of a round, by one workgroup with barriers between its phases and
// the components, hooks and best edges in LDS: the smallest edge among the
// vertices that reach their component's best weight; every component hooks onto
// the component across its best edge, except the smaller one of a mutual pair,
// and the hooking side adds the edge weight; every vertex follows the hooks to
// its new root; the components' best weights are cleared for the next round.
// Four launches over m entries took 14 us and three more gaps, this kernel with
// its arrays in memory 20 us (the walks to the roots are chains of reads).
constexpr int kBvThreads = 1024;
__global__ __launch_bounds__(kBvThreads) void k_bv_merge(int m, int32_t *comp, const int64_t *vw, const uint32_t *ve,
                                                         int64_t *cw, GHeader *h) {
    __shared__ uint32_t ce[MPT_GREEDY_MAX_M];
    __shared__ uint16_t cp[MPT_GREEDY_MAX_M], par[MPT_GREEDY_MAX_M];
    __shared__ uint32_t done;
    const int tid = (int)threadIdx.x;
    if (h->bv_done) return;
    if (tid == 0) done = 0;
    for (int v = tid; v < m; v += kBvThreads) {
        cp[v] = (uint16_t)comp[v];
        ce[v] = ~0u;
    }
    __syncthreads();
    constexpr int U = 4;                               // vertices per thread in flight
    for (int u0 = tid; u0 < m; u0 += U * kBvThreads) {
        int64_t w[U], best[U];
        uint32_t e[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int u = u0 + q * kBvThreads;
            w[q] = u < m ? vw[u] : -1;
            e[q] = u < m ? ve[u] : ~0u;
            best[q] = u < m ? cw[cp[u]] : 0;
        }
#pragma unroll
        for (int q = 0; q < U; ++q)
            if (w[q] >= 0 && w[q] == best[q]) atomicMin(&ce[cp[u0 + q * kBvThreads]], e[q]);
    }
    __syncthreads();
    uint64_t sum = 0;
    for (int c = tid; c < m; c += kBvThreads) {
        int to = c;
        if (cp[c] == c) {
            const uint32_t e = ce[c];
            if (e == ~0u) {
                done = 1;                              // no edge out: one component is left
            } else {
                const int lo = (int)(e >> 14), hi = (int)(e & 0x3fffu);
                const int d = cp[lo] == c ? cp[hi] : cp[lo];
                if (!(ce[d] == e && c < d)) {          // else d hooks onto c
                    to = d;
                    sum += (uint64_t)cw[c];
                }
            }
        }
        par[c] = (uint16_t)to;
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) sum += __shfl_xor(sum, off, kWave);
    if ((tid & (kWave - 1)) == 0 && sum) atomicAdd(&h->total, (unsigned long long)sum);
    __syncthreads();                                   // (cw is read before it is cleared)
    if (done) {
        if (tid == 0) h->bv_done = 1;
        return;
    }
    for (int v = tid; v < m; v += kBvThreads) {
        int r = cp[v];
        for (int guard = 0; guard < m && par[r] != r; ++guard) r = par[r];
        comp[v] = r;
        cw[v] = -1;
    }
}
static_assert(MPT_GREEDY_MAX_M <= 1 << 14, "vertices in 16 bits, edges in 28");

// ---------------------------------------------------------------------------
// host side

int g_check_common(int m, int64_t n_chunks, int64_t nnz) {
    if (m < 1 || m > MPT_GREEDY_MAX_M) return fail(MPT_E_INVALID, "m = %d outside [1, %d]", m, MPT_GREEDY_MAX_M);
    if (n_chunks < 0 || n_chunks > MPT_MAX_CHUNKS) return fail(MPT_E_INVALID, "n_chunks = %lld out of range", (long long)n_chunks);
    if (nnz < 0 || nnz > (int64_t)INT32_MAX) return fail(MPT_E_INVALID, "nnz = %lld out of range", (long long)nnz);
    return MPT_OK;
}

int g_check_ws(const GLayout &L, void *ws, size_t bytes) {
    if (!ws) return fail(MPT_E_WORKSPACE, "workspace is NULL");
    if (((uintptr_t)ws & 255u) != 0) return fail(MPT_E_WORKSPACE, "workspace is not 256-byte aligned");
    if (bytes < L.total) return fail(MPT_E_WORKSPACE, "workspace has %zu bytes, needs %zu", bytes, L.total);
    return MPT_OK;
}

int g_read_errors(GHeader *h, hipStream_t s, int64_t *request_total = nullptr, int64_t *max_len = nullptr,
                  int64_t *savings = nullptr) {
    GHeader hh;
    MPT_HIP_TRY(mptlib::read_back(&hh, h, sizeof hh, s));
    if (hh.err & GERR_INVALID) return fail(MPT_E_INVALID, "req_off is not a CSR offset array of length m+1 ending at nnz");
    if (hh.err & GERR_RANGE) return fail(MPT_E_RANGE, "a chunk id is outside [0, n_chunks)");
    if (hh.err & GERR_WEIGHT) return fail(MPT_E_WEIGHT, "a chunk weight is <= 0 or > 2^32");
    if (hh.err & GERR_DUP) return fail(MPT_E_DUP, "a chunk is repeated inside one request");
    if (hh.total >= (1ull << 61)) return fail(MPT_E_OVERFLOW, "sum of request weights reaches 2^61");
    if (request_total) *request_total = (int64_t)hh.total;
    if (max_len) *max_len = hh.max_len;
    if (savings) *savings = (int64_t)hh.savings;
    return MPT_OK;
}

// Validate the instance and build the request lists, the demand lists and the
// pair weights, with one synchronisation at the end to report errors (two with
// requests of more than kListMax chunks, whose lists a key sort puts in order).
int g_prepare(int m, int64_t n_chunks, int64_t nnz, const int64_t *chunk_w, const int64_t *req_off,
              const int32_t *req_chunks, int64_t *P, const GLayout &L, char *ws, hipStream_t s,
              int64_t *request_total = nullptr) {
    GHeader *h = (GHeader *)ws;
    int32_t *sig = (int32_t *)(ws + L.sig), *sig_len = (int32_t *)(ws + L.sig_len), *dem = (int32_t *)(ws + L.dem);
    int32_t *sig_slot = (int32_t *)(ws + L.sig_slot);
    uint64_t *dem_seg = (uint64_t *)(ws + L.dem_seg);
    uint32_t *rank = (uint32_t *)(ws + L.rank);
    const int64_t blocks = (int64_t)m * ((m + kPairTile - 1) / kPairTile);
    auto pairs = [&](int sorted) {
        LaunchScope ls("g_pairs", 8.0 * (double)m * m, s);
        k_g_pair_rows<<<(unsigned)blocks, kPairThreads, 0, s>>>(m, sig, req_off, dem, dem_seg, chunk_w, P, sorted, h);
    };
    {
        LaunchScope ls("g_lists", (double)nnz, s);
        k_g_begin<<<grid_for(n_chunks, 256), 256, 0, s>>>(n_chunks, dem_seg, h);
        k_g_check<<<grid_for(std::max<int64_t>(nnz, std::max<int64_t>(m, n_chunks / 4)), kCountSlice, 1024),
                    kCountThreads, 0, s>>>(m, n_chunks, nnz, req_off, req_chunks, chunk_w, dem_seg, rank, h);
        if (n_chunks > 0)
            k_g_stretches<<<grid_for(n_chunks, kCountThreads), kCountThreads, 0, s>>>(n_chunks, dem_seg, h);
        k_g_lists<<<grid_for(m, 1, 4096), kListThreads, 0, s>>>(m, req_off, req_chunks, rank, dem_seg, sig, sig_slot,
                                                               sig_len, dem, h);
    }
    pairs(0);
    MPT_HIP_TRY(hipGetLastError());
    int64_t max_len = 0;
    int rc = g_read_errors(h, s, request_total, &max_len);
    if (rc || max_len <= kListMax) return rc;
    uint64_t *sorted = nullptr;
    {
        LaunchScope ls("g_sort", (double)nnz, s);
        k_g_keys<<<grid_for(nnz, 256), 256, 0, s>>>(m, nnz, req_off, req_chunks, (uint64_t *)(ws + L.keys1));
        if ((rc = sort_keys((uint64_t *)(ws + L.keys1), (uint64_t *)(ws + L.keys2), nnz, s, &sorted))) return rc;
        k_g_sig_long<<<grid_for(nnz, 256), 256, 0, s>>>(m, nnz, req_off, req_chunks, sorted, dem_seg, rank, sig,
                                                           sig_slot, h);
    }
    pairs(1);
    MPT_HIP_TRY(hipGetLastError());
    return g_read_errors(h, s, request_total);
}

}  // namespace

extern "C" size_t mpt_greedy_workspace_bytes(int m, int64_t n_chunks, int64_t nnz) {
    if (m < 1 || m > MPT_GREEDY_MAX_M || n_chunks < 0 || nnz < 0) return 0;
    return g_layout(m, n_chunks, nnz).total;
}

extern "C" int mpt_pair_weights(int m, int64_t n_chunks, int64_t nnz, const int64_t *chunk_w, const int64_t *req_off,
                                const int32_t *req_chunks, int64_t *P, int64_t *request_total, void *workspace,
                                size_t workspace_bytes, void *stream) {
    mptlib::clear_error();
    return mptlib::guarded(__func__, [&]() -> int {
        int rc = g_check_common(m, n_chunks, nnz);
        if (rc) return rc;
        if (!req_off || !P) return fail(MPT_E_INVALID, "req_off and P must not be NULL");
        if (n_chunks > 0 && !chunk_w) return fail(MPT_E_INVALID, "chunk_w must not be NULL");
        if (nnz > 0 && !req_chunks) return fail(MPT_E_INVALID, "req_chunks must not be NULL");
        const GLayout L = g_layout(m, n_chunks, nnz);
        if ((rc = g_check_ws(L, workspace, workspace_bytes))) return rc;
        return g_prepare(m, n_chunks, nnz, chunk_w, req_off, req_chunks, P, L, (char *)workspace, (hipStream_t)stream,
                         request_total);
    });
}

extern "C" int mpt_greedy_hierarchy(int m, int64_t n_chunks, int64_t nnz, const int64_t *chunk_w,
                                    const int64_t *req_off, const int32_t *req_chunks, int32_t *merge_a,
                                    int32_t *merge_b, int64_t *gain, int32_t *node_parent, int32_t *order_chunks,
                                    int64_t *savings, void *workspace, size_t workspace_bytes, void *stream) {
    mptlib::clear_error();
    return mptlib::guarded(__func__, [&]() -> int {
        int rc = g_check_common(m, n_chunks, nnz);
        if (rc) return rc;
        if (!req_off || !node_parent) return fail(MPT_E_INVALID, "req_off and node_parent must not be NULL");
        if (m > 1 && (!merge_a || !merge_b || !gain)) return fail(MPT_E_INVALID, "merge_a, merge_b and gain must not be NULL");
        if (n_chunks > 0 && !chunk_w) return fail(MPT_E_INVALID, "chunk_w must not be NULL");
        if (nnz > 0 && !req_chunks) return fail(MPT_E_INVALID, "req_chunks must not be NULL");
        const GLayout L = g_layout(m, n_chunks, nnz);
        if ((rc = g_check_ws(L, workspace, workspace_bytes))) return rc;
        hipStream_t s = (hipStream_t)stream;
        char *ws = (char *)workspace;
        int64_t *V = (int64_t *)(ws + L.V);
        if ((rc = g_prepare(m, n_chunks, nnz, chunk_w, req_off, req_chunks, V, L, ws, s))) return rc;
        Rac R{};
        R.m = m;
        R.w = chunk_w;
        R.req_off = req_off;
        R.sig = (int32_t *)(ws + L.sig);
        R.sig_slot = (int32_t *)(ws + L.sig_slot);
        R.sig_len = (int32_t *)(ws + L.sig_len);
        R.dem = (int32_t *)(ws + L.dem);
        R.dem_seg = (const uint64_t *)(ws + L.dem_seg);
        R.V = V;
        R.best_v = (int64_t *)(ws + L.best_v);
        R.best_p = (int32_t *)(ws + L.best_p);
        R.act = (int32_t *)(ws + L.active);
        R.last = (int32_t *)(ws + L.last);
        R.touched = (int32_t *)(ws + L.touched);
        R.resc = (int32_t *)(ws + L.resc);
        int32_t *r32 = (int32_t *)(ws + L.rec32);
        int32_t **f32[kRec32] = {&R.ra, &R.rb, &R.rca, &R.rcb, &R.rpos, &R.rdal, &R.rdbl};
        for (int k = 0; k < kRec32; ++k) *f32[k] = r32 + (size_t)k * m;
        int64_t *r64 = (int64_t *)(ws + L.rec64);
        int64_t **f64[kRec64] = {&R.rgain, &R.rdao, &R.rdbo};
        for (int k = 0; k < kRec64; ++k) *f64[k] = r64 + (size_t)k * m;
        R.nnz = std::max<int64_t>(nnz, 1);
        R.live = (int32_t *)(ws + L.live);
        R.dense = (int64_t *)(ws + L.dense);
        R.d_off = (int64_t *)(ws + L.d_off);
        R.d_len = (int32_t *)(ws + L.d_len);
        R.merge_a = merge_a;
        R.merge_b = merge_b;
        R.gain = gain;
        R.node_parent = node_parent;
        R.h = (GHeader *)ws;
        {
            LaunchScope ls("g_row_best", 8.0 * (double)m * m, s);
            k_g_row_best<<<(m + 3) / 4, 4 * kWave, 0, s>>>(m, V, R.best_v, R.best_p);
            k_rac_init<<<grid_for(2 * (int64_t)m, 256), 256, 0, s>>>(R);
        }
        // Rounds in batches without host synchronisation, until the rest is the
        // tail's (k_rac_tail, which needs no further look); a round that finds no
        // pair changes nothing, so the batch's last round tells whether the rounds
        // are over. The first round merges about a sixth of the clusters, so an
        // instance whose first round would be the tail's goes there at once.
        int n_rec = 0;
        {
            LaunchScope ls("g_rounds", (double)(m - 1), s);
            const int g_rec = std::max(1, std::min(4096, (m + 3) / 4));        // waves: one per row
            const int g_cols = std::max(1, std::min(2048, m / 2 * ((m + kPairTile - 1) / kPairTile)));   // workgroups: one per merge and tile
            const int g_resc = std::max(1, std::min(m, 2048));                  // workgroups: one per marked row
            int64_t pairs = (m + 5) / 6;
            for (int round = 0;;) {
                const int64_t live = m - n_rec;
                const bool tail = live <= kTailLive && pairs * live <= kTailWork &&
                                  pairs * pairs * nnz <= kTailEntries * m;
                if (tail) {
                    k_rac_live<<<1, kChainThreads, 0, s>>>(R);
                    k_rac_dense<<<(unsigned)live, 256, 0, s>>>(R, (int)live);
                    // (one look at every chunk: not worth it for a universe far
                    // larger than the requests)
                    if (round > 0 && n_chunks <= ((int64_t)1 << 20))
                        k_rac_tidy<<<grid_for(n_chunks, 4, 8192), 4 * kWave, 0, s>>>(R, n_chunks,
                                                                                    (uint64_t *)(ws + L.dem_seg));
                    k_rac_tail<<<1, kTailThreads, 0, s>>>(R, (int)live, round);
                } else {
                    for (int k = 0; k < 8; ++k, ++round) {
                        k_rac_pairs_merge<<<g_rec, 4 * kWave, 0, s>>>(R, round);
                        k_rac_rows<<<g_cols, kRowThreads, 0, s>>>(R, round);
                        k_rac_rescan<<<g_resc, kRescThreads, 0, s>>>(R, round);
                    }
                }
                MPT_HIP_TRY(hipGetLastError());
                GHeader hh;
                MPT_HIP_TRY(mptlib::read_back(&hh, R.h, sizeof hh, s));
                if (hh.err) return fail(MPT_E_INTERNAL, "greedy rounds left an inconsistent state");   // cannot happen
                n_rec = std::min(hh.n_rec, m - 1);
                pairs = hh.last_pairs;
                if (pairs == 0) break;
                if (tail || round > m + 32) return fail(MPT_E_INTERNAL, "greedy rounds do not end");   // cannot happen
            }
        }
        {
            LaunchScope ls("g_sequence", (double)m, s);
            if (n_rec > 0) {
                const unsigned tx = (unsigned)((n_rec + kRankThreads - 1) / kRankThreads);
                const unsigned ty = (unsigned)((n_rec + kRankTileY - 1) / kRankTileY);
                k_rac_rank<<<dim3(tx, ty), kRankThreads, 0, s>>>(R, n_rec);
                k_rac_emit<<<grid_for(n_rec, 256), 256, 0, s>>>(R, n_rec);
            }
            k_rac_chain<<<1, kChainThreads, 0, s>>>(R, n_rec);
        }
        MPT_HIP_TRY(hipGetLastError());
        if (order_chunks) {
            LaunchScope ls("g_orders", 4.0 * (double)nnz, s);
            k_g_orders<<<(m + 3) / 4, 4 * kWave, 0, s>>>(m, nnz, req_off, node_parent, R.sig, R.d_off, R.d_len,
                                                         order_chunks, n_rec, R.h);
            MPT_HIP_TRY(hipGetLastError());
        }
        return g_read_errors(R.h, s, nullptr, nullptr, savings);
    });
}

extern "C" int mpt_spanning_tree_bound(int m, const int64_t *P, int64_t *mst_weight, void *workspace,
                                       size_t workspace_bytes, void *stream) {
    mptlib::clear_error();
    return mptlib::guarded(__func__, [&]() -> int {
        if (m < 1 || m > MPT_GREEDY_MAX_M) return fail(MPT_E_INVALID, "m = %d outside [1, %d]", m, MPT_GREEDY_MAX_M);
        if (!P || !mst_weight) return fail(MPT_E_INVALID, "P and mst_weight must not be NULL");
        if (!workspace) return fail(MPT_E_WORKSPACE, "workspace is NULL");
        if (((uintptr_t)workspace & 255u) != 0) return fail(MPT_E_WORKSPACE, "workspace is not 256-byte aligned");
        // header, then the vertices' components, best weights and edges and the
        // components' best weights (24 m bytes of the documented 32 m)
        const size_t mm = (size_t)m, a4 = align256(4 * mm), a8 = align256(8 * mm);
        const size_t off_comp = align256(sizeof(GHeader)), off_vw = off_comp + a4, off_ve = off_vw + a8,
                     off_cw = off_ve + a4, need = off_comp + 4 * a4 + 2 * a8;
        if (workspace_bytes < need) return fail(MPT_E_WORKSPACE, "workspace has %zu bytes, needs %zu", workspace_bytes, need);
        hipStream_t s = (hipStream_t)stream;
        GHeader *h = (GHeader *)workspace;
        char *ws = (char *)workspace;
        int32_t *comp = (int32_t *)(ws + off_comp);
        int64_t *vw = (int64_t *)(ws + off_vw), *cw = (int64_t *)(ws + off_cw);
        uint32_t *ve = (uint32_t *)(ws + off_ve);
        int rounds = 0;
        while ((1 << rounds) < m) ++rounds;
        const int gv = grid_for(m, 256);
        k_bv_init<<<gv, 256, 0, s>>>(m, comp, vw, cw, h);
        for (int r = 0; r < rounds; ++r) {
            LaunchScope ls("g_boruvka", 8.0 * (double)m * m, s);
            k_bv_vertex<<<(m + 3) / 4, 4 * kWave, 0, s>>>(m, P, comp, vw, ve, cw, h);
            k_bv_merge<<<1, kBvThreads, 0, s>>>(m, comp, vw, ve, cw, h);
        }
        MPT_HIP_TRY(hipGetLastError());
        unsigned long long total = 0;
        MPT_HIP_TRY(mptlib::read_back(&total, &h->total, sizeof total, s));
        *mst_weight = (int64_t)total;
        return MPT_OK;
    });
}
