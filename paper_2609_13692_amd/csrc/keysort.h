// Sort of n uint64 keys, ascending, on the caller's stream, between two
// buffers of n keys; and the order of one short list. Shared by the library's
// source files.
//
// Tiles of kSortTile keys are sorted by one workgroup each, then up to 8 runs
// are merged at a time: every key finds its position in each sibling run and
// is written there. Few dependent launches: 32768 keys take two (a bitonic
// sort between tiles took ten), a million four (45).
// What bounds it: latency. The tile sort: LDS traffic and its round trips (15
// us; bitonic in LDS, 78 stages, 37). A merge: three or four dependent reads of
// keys that another XCD wrote (10 to 12 us for eight runs at 32768 keys; with
// each key's binary search in global memory 21). The two launches of 32768
// keys took 25 us, the bitonic sort's ten 87; the seven sorts of a cache step
// at 20011 requests (100K and 800K keys among them) 210 us, before 550.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "common.h"

namespace mptlib {

constexpr int kSortThreads = 1024;
constexpr int kSortPer = 4;                              // keys per thread
constexpr int kSortTile = kSortThreads * kSortPer;       // keys sorted in LDS per workgroup

namespace keysort_detail {

// the key of lane ^ X (X one of the patterns below), by DPP where one or two
// of its patterns give it
template <int X> __device__ inline uint32_t lane_xor32(uint32_t v) {
    auto dpp = [](uint32_t u, auto c) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)u, decltype(c)::value, 0xF, 0xF, false); };
    if constexpr (X == 1) return dpp(v, std::integral_constant<int, 0xB1>{});           // quad_perm [1,0,3,2]
    else if constexpr (X == 2) return dpp(v, std::integral_constant<int, 0x4E>{});      // quad_perm [2,3,0,1]
    else if constexpr (X == 3) return dpp(v, std::integral_constant<int, 0x1B>{});      // quad_perm [3,2,1,0]
    else if constexpr (X == 7) return dpp(v, std::integral_constant<int, 0x141>{});     // row_half_mirror
    else if constexpr (X == 15) return dpp(v, std::integral_constant<int, 0x140>{});    // row_mirror
    else if constexpr (X == 4) return lane_xor32<3>(lane_xor32<7>(v));
    else if constexpr (X == 8) return lane_xor32<7>(lane_xor32<15>(v));
    else return (uint32_t)__shfl_xor((int)v, X, 64);
}
template <int X> __device__ inline uint64_t lane_xor(uint64_t v) {
    return ((uint64_t)lane_xor32<X>((uint32_t)(v >> 32)) << 32) | lane_xor32<X>((uint32_t)v);
}
__device__ inline void order2(uint64_t &a, uint64_t &b) {        // a <= b afterwards
    const bool sw = b < a;
    const uint64_t x = sw ? b : a, y = sw ? a : b;
    a = x;
    b = y;
}
// exchange with lane ^ X: the lane whose top bit of X is clear keeps the
// smaller key; FLIP: with the partner's mirrored register (3 - r)
template <int X, bool FLIP> __device__ inline void cross(uint64_t (&v)[kSortPer]) {
    constexpr int top = X >= 32 ? 32 : X >= 16 ? 16 : X >= 8 ? 8 : X >= 4 ? 4 : X >= 2 ? 2 : 1;
    const bool low = ((threadIdx.x & 63u) & (uint32_t)top) == 0;
    uint64_t o[kSortPer];
#pragma unroll
    for (int r = 0; r < kSortPer; ++r) o[r] = lane_xor<X>(v[FLIP ? kSortPer - 1 - r : r]);
#pragma unroll
    for (int r = 0; r < kSortPer; ++r) v[r] = ((o[r] < v[r]) == low) ? o[r] : v[r];
}
// (a key equal to its partner's stays on both sides: the two are the same)

// The 256 keys of a wave, key lane * 4 + r in v[r]: a bitonic sort whose
// merges of k keys start by pairing i with i ^ (k - 1), so that every exchange
// leaves the smaller key at the lower index. sort_wave64 stops at runs of 64
// (16 lanes), sort_wave256 goes on from there.
__device__ inline void half2(uint64_t (&v)[kSortPer]) {      // strides 2, 1
    order2(v[0], v[2]); order2(v[1], v[3]);
    order2(v[0], v[1]); order2(v[2], v[3]);
}
__device__ inline void sort_wave64(uint64_t (&v)[kSortPer]) {
    order2(v[0], v[1]); order2(v[2], v[3]);               // k = 2
    order2(v[0], v[3]); order2(v[1], v[2]);               // k = 4
    order2(v[0], v[1]); order2(v[2], v[3]);
    cross<1, true>(v); half2(v);                          // k = 8
    cross<3, true>(v); cross<1, false>(v); half2(v);      // 16
    cross<7, true>(v); cross<2, false>(v); cross<1, false>(v); half2(v);
    cross<15, true>(v); cross<4, false>(v); cross<2, false>(v); cross<1, false>(v); half2(v);
}
__device__ inline void sort_wave256(uint64_t (&v)[kSortPer]) {
    cross<31, true>(v); cross<8, false>(v); cross<4, false>(v); cross<2, false>(v); cross<1, false>(v); half2(v);
    cross<63, true>(v); cross<16, false>(v); cross<8, false>(v); cross<4, false>(v); cross<2, false>(v);
    cross<1, false>(v); half2(v);                         // 256
}
// kSortPer consecutive outputs, from o on, of the merge of each pair of sorted
// runs of `run` keys in t: the split of the two runs at the first output by a
// binary search, then one comparison per output
__device__ inline void merge_outputs(const uint64_t *t, int run, int o, uint64_t (&v)[kSortPer]) {
    const int diag = o & (2 * run - 1);
    const uint64_t *A = t + (o - diag), *B = A + run;
    int lo = diag > run ? diag - run : 0, hi = diag < run ? diag : run;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (A[mid] <= B[diag - 1 - mid]) lo = mid + 1; else hi = mid;
    }
    int a = lo, b = diag - lo;
    uint64_t ka = a < run ? A[a] : 0, kb = b < run ? B[b] : 0;
#pragma unroll
    for (int r = 0; r < kSortPer; ++r) {
        const bool take_a = b >= run || (a < run && ka <= kb);
        v[r] = take_a ? ka : kb;
        a += take_a ? 1 : 0;
        b += take_a ? 0 : 1;
        if (take_a) ka = a < run ? A[a] : 0;
        else kb = b < run ? B[b] : 0;
    }
}

// tiles of kSortTile keys: 256 keys per wave in registers, then the runs
// merged in LDS, every thread its four outputs
// (in place: a workgroup has read all of its tile before it writes)
static __global__ __launch_bounds__(kSortThreads) void k_sort_tile(uint64_t *keys, int64_t n) {
    __shared__ __align__(16) uint64_t t[2][kSortTile];
    const int64_t base = (int64_t)blockIdx.x * kSortTile;
    const int tid = (int)threadIdx.x, lane = tid & 63, wv = tid >> 6;
    uint64_t v[kSortPer];
#pragma unroll
    for (int r = 0; r < kSortPer; ++r) {
        const int64_t i = base + wv * 256 + r * 64 + lane;
        v[r] = i < n ? keys[i] : ~0ull;                     // padding sorts last
    }
    sort_wave64(v);
    sort_wave256(v);
    const int o = tid * kSortPer;                         // this thread's first output
#pragma unroll
    for (int r = 0; r < kSortPer; ++r) t[0][o + r] = v[r];
    __syncthreads();
    int cur = 0;
    for (int run = 256; run < kSortTile; run <<= 1, cur ^= 1) {
        merge_outputs(t[cur], run, o, v);
#pragma unroll
        for (int r = 0; r < kSortPer; ++r) t[cur ^ 1][o + r] = v[r];
        __syncthreads();
    }
    // coalesced: consecutive threads, consecutive keys
    for (int e = tid; e < kSortTile; e += kSortThreads)
        if (base + e < n) keys[base + e] = t[cur][e];
}

// The number of keys in the sorted stretch [lo, end) that come before `key`
// (equal ones included where eq), for U independent searches by one wave: 64
// probes at once cut a stretch to a 64th, so a run of 4096 takes two dependent
// reads, not twelve.
template <int U>
__device__ inline void wave_counts(const uint64_t *__restrict__ in, const uint64_t (&key)[U], const bool (&eq)[U],
                                   int64_t (&lo)[U], int64_t (&end)[U]) {
    const int64_t lane = (int64_t)(threadIdx.x & 63u);
    for (;;) {
        uint64_t k[U];
        int64_t step[U];
        bool any = false;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            step[u] = (end[u] - lo[u] + 63) >> 6;
            any = any || step[u] > 0;
            const int64_t at = lo[u] + (lane + 1) * step[u] - 1;
            k[u] = step[u] > 0 && at < end[u] ? in[at] : ~0ull;
        }
        if (!any) return;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (step[u] == 0) continue;
            const int64_t at = lo[u] + (lane + 1) * step[u] - 1;
            const bool before = at < end[u] && (eq[u] ? k[u] <= key[u] : k[u] < key[u]);
            lo[u] += (int64_t)__popcll(__ballot(before)) * step[u];
            // the stretch's next probe is not before the key, or past its end
            end[u] = lo[u] + step[u] - 1 < end[u] ? lo[u] + step[u] - 1 : end[u];
        }
    }
}

// R sorted runs of `run` keys (a multiple of kMergeKeys; the last ones shorter
// or empty) into one: key i of run r goes to its place in its run plus the
// number of keys before it in each sibling run (equal keys of earlier runs
// come first). A workgroup takes kMergeKeys consecutive keys of a run: its
// waves find where the first and the last of them fall in every sibling, those
// stretches go to LDS, and each key searches there (in global memory where
// together they do not fit).
constexpr int kMergeKeys = 256;
constexpr int kMergeLds = 4096;
template <int R>
__global__ __launch_bounds__(kMergeKeys) void k_sort_merge(const uint64_t *__restrict__ in,
                                                           uint64_t *__restrict__ out, int64_t n, int64_t run) {
    constexpr int S = R - 1;                               // siblings
    constexpr int U = (2 * S + 3) / 4;                     // searches per wave: first and last key in each sibling
    __shared__ uint64_t st[kMergeLds];
    __shared__ int64_t bound[2][S];                        // where the stretch of each sibling starts and ends
    const int tid = (int)threadIdx.x, wv = tid >> 6;
    for (int64_t i0 = (int64_t)blockIdx.x * kMergeKeys; i0 < n; i0 += (int64_t)gridDim.x * kMergeKeys) {
        const int64_t own = i0 / run, g0 = own / R * R;    // own run, first run of its group
        const int r = (int)(own - g0);
        const int64_t last = (i0 + kMergeKeys < n ? i0 + kMergeKeys : n) - 1;
        const uint64_t key = in[i0 + tid <= last ? i0 + tid : last];
        {
            const uint64_t ends[2] = {in[i0], in[last]};
            uint64_t k[U];
            bool eq[U];
            int64_t lo[U], end[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int task = wv * U + u, q = task >> 1;      // sibling q: first key, then last
                const int sib = q < r ? q : q + 1;
                const int64_t s0 = (g0 + sib) * run, s1 = s0 + run;
                k[u] = (task & 1) ? ends[1] : ends[0];
                eq[u] = sib < r;
                lo[u] = s0 < n ? s0 : n;
                end[u] = q < S ? (s1 < n ? s1 : n) : lo[u];
            }
            wave_counts<U>(in, k, eq, lo, end);
            if ((tid & 63) == 0) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int task = wv * U + u;
                    if (task < 2 * S) bound[task & 1][task >> 1] = lo[u];
                }
            }
        }
        __syncthreads();
        int64_t b0[S], cnt[S];
        int off[S];
        int64_t total = 0;
        int64_t most = 0;
        int64_t pos = i0 + tid;                            // own place: g0 * run + (i - own * run), i = i0 + tid
        pos += (g0 - own) * run;
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const int sib = q < r ? q : q + 1;
            const int64_t s0 = (g0 + sib) * run;
            b0[q] = bound[0][q];
            cnt[q] = bound[1][q] - b0[q];
            off[q] = (int)(total < kMergeLds ? total : kMergeLds);
            total += cnt[q];
            most = cnt[q] > most ? cnt[q] : most;
            pos += b0[q] - (s0 < n ? s0 : n);              // all keys before the stretch
        }
        const bool staged = total <= kMergeLds;
        if (staged) {
            uint64_t v[S];
#pragma unroll
            for (int q = 0; q < S; ++q) v[q] = tid < cnt[q] ? in[b0[q] + tid] : 0ull;
#pragma unroll
            for (int q = 0; q < S; ++q) {
                if (tid < cnt[q]) st[off[q] + tid] = v[q];
                for (int64_t x = tid + kMergeKeys; x < cnt[q]; x += kMergeKeys) st[off[q] + x] = in[b0[q] + x];
            }
        }
        __syncthreads();
        if (i0 + tid <= last) {
            int64_t lo[S], hi[S];
#pragma unroll
            for (int q = 0; q < S; ++q) {
                lo[q] = 0;
                hi[q] = cnt[q];
            }
            for (int64_t left = most; left > 0; left >>= 1) {
#pragma unroll
                for (int q = 0; q < S; ++q) {
                    if (lo[q] >= hi[q]) continue;
                    const int64_t mid = (lo[q] + hi[q]) >> 1;
                    const uint64_t k = staged ? st[off[q] + mid] : in[b0[q] + mid];
                    const bool before = q < r ? k <= key : k < key;      // (sibling q < r is run q)
                    if (before) lo[q] = mid + 1; else hi[q] = mid;
                }
            }
#pragma unroll
            for (int q = 0; q < S; ++q) pos += lo[q];
            out[pos] = key;
        }
        __syncthreads();
    }
}

}  // namespace keysort_detail

// Short segments: the position of lane e's entry (key r, e < n <= 64) in
// its wave's segment, ascending by key, ties by lane: the number of lanes f
// < n with a smaller key, or an equal one and f < e. dup: some other lane
// holds an equal key. One shuffle per lane of the segment.
constexpr int kSegMax = 64;
__device__ inline int seg_rank(uint32_t r, int n, bool &dup) {
    const int e = (int)(threadIdx.x & 63u);
    int pos = 0;
    dup = false;
    for (int f = 0; f < n; ++f) {
        const uint32_t o = (uint32_t)__shfl((int)r, f, 64);
        pos += (o < r || (o == r && f < e)) ? 1 : 0;
        dup = dup || (o == r && f != e);
    }
    return pos;
}

// The same for segments of up to kListMax entries, by a workgroup of
// kListThreads: the entries key(e) < 2^32 - 1, e < n, are staged in LDS (16-byte
// aligned) and put(e, key, position, dup) is called for each. n^2 comparisons;
// the staged keys are read 16 at a time, and ties looked at again. The greedy's
// lists of 100 requests of 512 chunks take 17 us (72 with one key at a time,
// each a round trip to LDS; the key sort of 513 chunks each two launches of 25
// us). The caller ends its use of `stage` with a barrier before the next call.
constexpr int kListMax = 512;
constexpr int kListThreads = 256;
template <class KeyOf, class Put>
__device__ inline void list_ranks(uint32_t (&stage)[kListMax], int n, KeyOf &&key, Put &&put) {
    constexpr int U = 16;
    static_assert(kListMax % U == 0, "whole batches");
    const int padded = (n + U - 1) / U * U;                // entries past n: above every key
    for (int e = (int)threadIdx.x; e < padded; e += kListThreads) stage[e] = e < n ? key(e) : ~0u;
    __syncthreads();
    for (int e = (int)threadIdx.x; e < n; e += kListThreads) {
        const uint32_t r = stage[e];
        int pos = 0, same = 0;                             // smaller keys, equal ones
        for (int f = 0; f < n; f += U) {
            uint32_t o[U];
#pragma unroll
            for (int u = 0; u < U; u += 4) {
                const uint4 v = *reinterpret_cast<const uint4 *>(&stage[f + u]);
                o[u] = v.x; o[u + 1] = v.y; o[u + 2] = v.z; o[u + 3] = v.w;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                pos += o[u] < r ? 1 : 0;
                same += o[u] == r ? 1 : 0;
            }
        }
        if (same > 1)
            for (int f = 0; f < e; ++f) pos += stage[f] == r ? 1 : 0;
        put(e, r, pos, same > 1);
    }
}

// Sorts keys[0 .. n) with tmp[0 .. n) as the other buffer (the buffers do not
// overlap); *sorted is the one that holds the result.
inline int sort_keys(uint64_t *keys, uint64_t *tmp, int64_t n, hipStream_t s, uint64_t **sorted) {
    using namespace keysort_detail;
    *sorted = keys;
    if (n <= 0) return MPT_OK;
    uint64_t *a = keys, *b = tmp;
    k_sort_tile<<<(unsigned)((n + kSortTile - 1) / kSortTile), kSortThreads, 0, s>>>(a, n);
    const int grid = grid_for(n, kMergeKeys, 16384);
    for (int64_t run = kSortTile; run < n;) {
        const int64_t runs = (n + run - 1) / run;
        const int fan = runs > 4 ? 8 : runs > 2 ? 4 : 2;
        if (fan == 2) k_sort_merge<2><<<grid, kMergeKeys, 0, s>>>(a, b, n, run);
        else if (fan == 4) k_sort_merge<4><<<grid, kMergeKeys, 0, s>>>(a, b, n, run);
        else k_sort_merge<8><<<grid, kMergeKeys, 0, s>>>(a, b, n, run);
        run *= fan;
        uint64_t *t = a;
        a = b;
        b = t;
    }
    MPT_HIP_TRY(hipGetLastError());
    *sorted = a;
    return MPT_OK;
}

}  // namespace mptlib
