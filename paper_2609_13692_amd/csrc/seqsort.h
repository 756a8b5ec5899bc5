// Lexicographic sort of requests by their chunk sequences (a CSR of
// sequences: off[m+1], seqs[off[m]]); a proper prefix sorts first, equal
// sequences by request index. Up to kSeqRankMax requests by ranks counted over
// all pairs; above, tiles of requests ranked the same way and merged eight runs
// at a time. Every request's first kSeqLdsDepth chunks are packed into words
// whose order is the sequence order on them, so that a comparison reads the
// sequences only when two agree on all of those. Shared by the library's source
// files.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "common.h"

namespace mptlib {

constexpr int kSeqLdsDepth = 8;               // leading chunks of each request in its words

// a < b in sequence order, from chunk kSeqLdsDepth on (the first kSeqLdsDepth
// chunks are equal and both sequences are longer)
__device__ inline bool seq_less_tail(int a, int b, const int64_t *off, const int32_t *seqs) {
    const int64_t la = off[a + 1] - off[a], lb = off[b + 1] - off[b];
    const int32_t *sa = seqs + off[a], *sb = seqs + off[b];
    const int64_t n = la < lb ? la : lb;
    for (int64_t j = kSeqLdsDepth; j < n; ++j)
        if (sa[j] != sb[j]) return sa[j] < sb[j];
    if (la != lb) return la < lb;
    return a < b;
}

// Up to kSeqRankMax requests the order comes from ranks: the position of
// request i is the number of requests before it (a strict total order, so the
// ranks are a permutation), counted over all pairs. Workgroup (x, y) takes 256
// requests i, one per thread, against 64 requests j staged in LDS. The words:
// four 64-bit words of two biased chunks (chunk + 1, 0 past the end; chunk ids
// are validated to lie in [0, n_chunks)), so that the word order is the
// sequence order on those chunks with a proper prefix first; sequences equal
// there are ordered by length, or by index, or, when both go on past them, by
// seq_less_tail. m^2 comparisons with no dependent stages, 16 us at m = 4096. A
// layout cost takes, by ranks and by merges: 51 and 62 us at m = 4096, 57 and 65
// at 5000, 64 and 65 at 6000, 76 and 66 at 8192; where all requests share their
// first 16 chunks, so that most comparisons read the sequences, 217 and 306 at
// 4096, 637 and 329 at 5000. The line keeps clear of the latter.
constexpr int kSeqRankMax = 4096;
constexpr int kSeqRankTile = 256;         // requests i per workgroup, one per thread
constexpr int kSeqRankTileY = 64;         // requests j per workgroup, staged in LDS
static_assert(kSeqLdsDepth == 8 && kSeqRankTile % 8 == 0 && kSeqRankTileY % 8 == 0,
              "four words of two chunks; eight requests compared at a time");

__device__ inline void seq_words(int i, const int64_t *off, const int32_t *seqs, ulonglong2 &a, ulonglong2 &b) {
    const int64_t len = off[i + 1] - off[i];
    const int32_t *si = seqs + off[i];
    uint32_t c[kSeqLdsDepth];
#pragma unroll
    for (int j = 0; j < kSeqLdsDepth; ++j) c[j] = j < len ? (uint32_t)si[j] + 1u : 0u;
    auto word = [&](int q) { return ((uint64_t)c[2 * q] << 32) | c[2 * q + 1]; };
    a = make_ulonglong2(word(0), word(1));
    b = make_ulonglong2(word(2), word(3));
}

// requests of equal words: x before y
__device__ inline bool seq_less_equal_words(int x, int y, const int64_t *off, const int32_t *seqs) {
    const int64_t lx = off[x + 1] - off[x], ly = off[y + 1] - off[y];
    if (lx > kSeqLdsDepth && ly > kSeqLdsDepth) return seq_less_tail(x, y, off, seqs);
    return lx < ly || (lx == ly && x < y);
}

// How many of the requests j0 .. j0 + n - 1, words ya / yb in LDS, come before
// request i with words xa, xb. Eight at a time: their first two words (every
// thread reads the same ones) are compared without a branch, and only requests
// that agree on those four chunks are looked at again; with all four words and
// the tie in one branching step, a comparison took 350 cycles.
__device__ inline int count_before(const ulonglong2 *ya, const ulonglong2 *yb, int n, int j0, int i, ulonglong2 xa,
                                   ulonglong2 xb, const int64_t *off, const int32_t *seqs) {
    int count = 0;
    for (int j = 0; j < n; j += 8) {
        ulonglong2 y[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) y[u] = ya[j + u];       // (the arrays hold a multiple of 8)
        uint32_t ties = 0;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const bool in = j + u < n;
            const bool same = y[u].x == xa.x;
            count += in && (y[u].x < xa.x || (same && y[u].y < xa.y)) ? 1 : 0;
            ties |= in && same && y[u].y == xa.y ? 1u << u : 0u;
        }
        while (ties) {
            const int k = j + __ffs(ties) - 1;
            ties &= ties - 1u;
            const ulonglong2 b = yb[k];
            const bool lt = b.x != xb.x ? b.x < xb.x : b.y != xb.y ? b.y < xb.y
                            : j0 + k != i && seq_less_equal_words(j0 + k, i, off, seqs);
            count += lt ? 1 : 0;
        }
    }
    return count;
}

static __global__ __launch_bounds__(kSeqRankTile) void k_l_seq_rank(int m, const int64_t *off, const int32_t *seqs,
                                                                    int32_t *rank, const uint32_t *err) {
    __shared__ ulonglong2 ya[kSeqRankTileY], yb[kSeqRankTileY];
    if (err && *err) return;
    const int j0 = blockIdx.y * kSeqRankTileY;
    const int ny = min(kSeqRankTileY, m - j0);
    if ((int)threadIdx.x < ny) seq_words(j0 + (int)threadIdx.x, off, seqs, ya[threadIdx.x], yb[threadIdx.x]);
    const int i = blockIdx.x * kSeqRankTile + (int)threadIdx.x;
    ulonglong2 xa = make_ulonglong2(0, 0), xb = xa;
    if (i < m) seq_words(i, off, seqs, xa, xb);
    __syncthreads();
    if (i >= m) return;
    const int count = count_before(ya, yb, ny, j0, i, xa, xb, off, seqs);
    if (count) atomicAdd(&rank[i], count);
}

// ord[rank[i]] = i, to copy too, where given
static __global__ void k_l_rank_scatter(int m, const int32_t *rank, int32_t *ord, int32_t *copy, const uint32_t *err) {
    if (err && *err) return;
    for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < m; p += gridDim.x * blockDim.x) {
        const int32_t r = rank[p];
        ord[r] = (int32_t)p;
        if (copy) copy[r] = (int32_t)p;
    }
}

// The merge sort's records: a request's four words, side by side so that one
// line holds them, and its index.
struct SeqRecs {
    ulonglong2 *w;
    int32_t *id;
};
inline size_t seq_recs_bytes(int m) {                     // one buffer of them
    return m <= kSeqRankMax ? 0 : align256(32 * (size_t)m) + align256(4 * (size_t)m);
}
inline SeqRecs seq_recs(char *at, int m) {
    return {(ulonglong2 *)at, (int32_t *)(at + align256(32 * (size_t)m))};
}

// record i, words a and b, before the record with words ka, kb and index kid
__device__ inline bool rec_before(const SeqRecs &R, int64_t i, ulonglong2 a, ulonglong2 b, ulonglong2 ka, ulonglong2 kb,
                                  int kid, const int64_t *off, const int32_t *seqs) {
    const bool tie = a.x == ka.x && a.y == ka.y && b.x == kb.x && b.y == kb.y;
    if (tie) return seq_less_equal_words(R.id[i], kid, off, seqs);
    return a.x != ka.x ? a.x < ka.x : a.y != ka.y ? a.y < ka.y : b.x != kb.x ? b.x < kb.x : b.y < kb.y;
}

// Tiles of kSeqRun requests, in order: ranks over all pairs of the tile, each
// request's by kTileParts threads (one thread per request was 22 us, the chain
// of its comparisons)
constexpr int kSeqRun = 256;
constexpr int kTileParts = 4;
static __global__ __launch_bounds__(kSeqRun * kTileParts) void k_l_seq_tiles(int m, const int64_t *off,
                                                                             const int32_t *seqs, SeqRecs out,
                                                                             const uint32_t *err) {
    constexpr int PER = kSeqRun / kTileParts;
    __shared__ ulonglong2 ya[kSeqRun], yb[kSeqRun];
    __shared__ int32_t rank[kSeqRun];
    if (err && *err) return;
    const int base = blockIdx.x * kSeqRun, e = (int)threadIdx.x % kSeqRun, part = (int)threadIdx.x / kSeqRun;
    const int i = base + e, n = min(kSeqRun, m - base);
    if (part == 0) {
        ya[e] = yb[e] = make_ulonglong2(0, 0);
        if (i < m) seq_words(i, off, seqs, ya[e], yb[e]);
        rank[e] = 0;
    }
    __syncthreads();
    const ulonglong2 xa = ya[e], xb = yb[e];
    const int j = part * PER;
    if (i < m && j < n) {
        const int count = count_before(ya + j, yb + j, min(PER, n - j), base + j, i, xa, xb, off, seqs);
        if (count) atomicAdd(&rank[e], count);
    }
    __syncthreads();
    if (part == 0 && i < m) {
        const int64_t at = base + rank[e];
        out.w[2 * at] = xa;
        out.w[2 * at + 1] = xb;
        out.id[at] = i;
    }
}

// Eight sorted runs of `run` records (a multiple of kSeqRun; the last ones
// shorter or empty) into one, as the key sort's merges: a workgroup takes
// kSeqRun consecutive records of a run, its waves find where the first and the
// last of them fall in every sibling (64 probes at a time, a wave per search),
// and each record searches those stretches, kMergeParts threads sharing its
// siblings. LAST: only ord (and copy) are written.
// Bound by a chain of about ten reads of records other XCDs wrote: 10 to 11 us
// (20 with one thread per record). A sort of 20011 requests takes 45 us in four
// launches, the bitonic one between tiles of 1024 took 250 us in 26.
constexpr int kSeqFan = 8;
constexpr int kMergeParts = 4;
template <bool LAST>
__global__ __launch_bounds__(kSeqRun * kMergeParts) void k_l_seq_merge(int m, int64_t run, SeqRecs in, SeqRecs out,
                                                                       const int64_t *off, const int32_t *seqs,
                                                                       int32_t *ord, int32_t *copy,
                                                                       const uint32_t *err) {
    constexpr int S = kSeqFan - 1, Q = (S + kMergeParts - 1) / kMergeParts;     // siblings; of one thread
    static_assert(2 * S <= kSeqRun * kMergeParts / 64, "a wave per search");
    __shared__ int64_t bound[2][S];
    __shared__ int32_t before[kSeqRun];
    if (err && *err) return;
    const int tid = (int)threadIdx.x, wv = tid >> 6;
    const int64_t lane = tid & 63;
    const int64_t n = m, i0 = (int64_t)blockIdx.x * kSeqRun;
    const int64_t own = i0 / run, g0 = own / kSeqFan * kSeqFan;
    const int r = (int)(own - g0);
    const int64_t last = (i0 + kSeqRun < n ? i0 + kSeqRun : n) - 1;
    auto first_of = [&](int q) {                             // where sibling q starts
        const int64_t s0 = (g0 + (q < r ? q : q + 1)) * run;
        return s0 < n ? s0 : n;
    };
    const int e = tid % kSeqRun, part = tid / kSeqRun;
    const int64_t i = i0 + e <= last ? i0 + e : last;
    const ulonglong2 ka = in.w[2 * i], kb = in.w[2 * i + 1];
    const int kid = in.id[i];
    if (part == 0) before[e] = 0;
    if (wv < 2 * S) {
        const int q = wv >> 1;                               // sibling q: first record, then last
        const int64_t k = (wv & 1) ? last : i0;
        const ulonglong2 wa = in.w[2 * k], wb = in.w[2 * k + 1];
        const int wid = in.id[k];
        int64_t lo = first_of(q), end = lo + run < n ? lo + run : n;
        while (lo < end) {
            const int64_t step = (end - lo + 63) >> 6, at = lo + (lane + 1) * step - 1;
            const int64_t get = at < end ? at : i0;
            const ulonglong2 a = in.w[2 * get], b = in.w[2 * get + 1];
            const bool lt = at < end && rec_before(in, at, a, b, wa, wb, wid, off, seqs);
            lo += (int64_t)__popcll(__ballot(lt)) * step;
            end = lo + step - 1 < end ? lo + step - 1 : end;
        }
        if (lane == 0) bound[wv & 1][q] = lo;
    }
    __syncthreads();
    if (i0 + e <= last) {
        int64_t lo[Q], hi[Q], from[Q], most = 0;
#pragma unroll
        for (int u = 0; u < Q; ++u) {
            const int q = part * Q + u;
            from[u] = lo[u] = q < S ? bound[0][q] : 0;
            hi[u] = q < S ? bound[1][q] : 0;
            most = hi[u] - lo[u] > most ? hi[u] - lo[u] : most;
        }
        for (; most > 0; most >>= 1) {
            ulonglong2 a[Q], b[Q];
#pragma unroll
            for (int u = 0; u < Q; ++u) {
                const int64_t get = lo[u] < hi[u] ? (lo[u] + hi[u]) >> 1 : i;
                a[u] = in.w[2 * get];
                b[u] = in.w[2 * get + 1];
            }
#pragma unroll
            for (int u = 0; u < Q; ++u) {
                if (lo[u] >= hi[u]) continue;
                const int64_t mid = (lo[u] + hi[u]) >> 1;
                if (rec_before(in, mid, a[u], b[u], ka, kb, kid, off, seqs)) lo[u] = mid + 1; else hi[u] = mid;
            }
        }
        int32_t mine = 0;
#pragma unroll
        for (int u = 0; u < Q; ++u) mine += (int32_t)(lo[u] - from[u]);
        if (mine) atomicAdd(&before[e], mine);
    }
    __syncthreads();
    if (part != 0 || i0 + e > last) return;
    int64_t pos = i0 + e + (g0 - own) * run + before[e];
#pragma unroll
    for (int q = 0; q < S; ++q) pos += bound[0][q] - first_of(q);
    if (LAST) {
        ord[pos] = kid;
        if (copy) copy[pos] = kid;
    } else {
        out.w[2 * pos] = ka;
        out.w[2 * pos + 1] = kb;
        out.id[pos] = kid;
    }
}

// ord[0 .. m) gets the request ids 0 .. m-1 in order; copy (nullable) too.
// rank: m entries of scratch, zeroed; recs: 2 * seq_recs_bytes(m) bytes of
// scratch. err (nullable): device error bits of the input; nothing is read or
// written once they are set.
inline int sort_requests(int32_t *ord, int32_t *rank, int32_t *copy, int m, const int64_t *off, const int32_t *seqs,
                         char *recs, const uint32_t *err, hipStream_t s) {
    if (m <= kSeqRankMax) {
        const unsigned tx = (unsigned)((m + kSeqRankTile - 1) / kSeqRankTile);
        const unsigned ty = (unsigned)((m + kSeqRankTileY - 1) / kSeqRankTileY);
        k_l_seq_rank<<<dim3(tx, ty), kSeqRankTile, 0, s>>>(m, off, seqs, rank, err);
        k_l_rank_scatter<<<grid_for(m, 256), 256, 0, s>>>(m, rank, ord, copy, err);
        MPT_HIP_TRY(hipGetLastError());
        return MPT_OK;
    }
    const unsigned blocks = (unsigned)((m + kSeqRun - 1) / kSeqRun);
    SeqRecs a = seq_recs(recs, m), b = seq_recs(recs + seq_recs_bytes(m), m);
    k_l_seq_tiles<<<blocks, kSeqRun * kTileParts, 0, s>>>(m, off, seqs, a, err);
    for (int64_t run = kSeqRun; run < m; run *= kSeqFan) {      // (m > kSeqRun: at least one merge)
        if (run * kSeqFan >= m) k_l_seq_merge<true><<<blocks, kSeqRun * kMergeParts, 0, s>>>(m, run, a, b, off, seqs, ord, copy, err);
        else k_l_seq_merge<false><<<blocks, kSeqRun * kMergeParts, 0, s>>>(m, run, a, b, off, seqs, ord, copy, err);
        const SeqRecs t = a;
        a = b;
        b = t;
    }
    MPT_HIP_TRY(hipGetLastError());
    return MPT_OK;
}
static_assert(kSeqRankMax >= kSeqRun, "the merges write the order");

}  // namespace mptlib
