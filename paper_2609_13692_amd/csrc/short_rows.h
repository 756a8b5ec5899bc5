// Phase 2 for mid-sized instances: the row-blocked DP of mpt.hip on rows of
// 2^9 entries (included by mpt.hip, which describes the scheme and the keys).
//
// With 2^12-entry rows an instance of m = 13 .. 21 requests has few rows per
// level (at most 126 for 256 CUs) and a level's time is the finishing of one row
// (10 in-row levels and 3^9 block convolutions on one CU, 30 us on 32-bit keys,
// 41 us on 64-bit ones), whatever the number of CUs. With 2^9 entries a row has 7 in-row
// levels and 3^6 convolutions, there are eight times as many rows, and one
// wave takes a row pair by itself in four steps (lifted on the top middle
// bit: 3^5 = 243 base steps in 64 lanes of at most 4), so that the pairs need
// no barrier. Against that, a row pair carries 3^9 candidates for two rows of
// traffic instead of 3^12, which is what counts for large m (short_rows_pay).
//
// Tables: one row-major table T of tagged entries (C(X) << m | X in the
// representation of Key<E>; E = uint32_t, the narrow keys: C(X) << 9 | X_L).
// A B row's tags are cleared on the way into LDS. W is read and C and split
// are written in mask order, scattered by rows: at these sizes the tables
// stay in cache, and three transposing launches (16 us) fall away.
namespace sr {

using rb::CB;
using rb::Key;
using rb::NB;
using rb::cdeposit;
using rb::conv_full;
using rb::cpop;
using rb::deposit;

constexpr int L = 9;                       // row bits
constexpr int R2 = L - CB;                 // middle bits
constexpr int ROW = 1 << L;
constexpr int NS2 = 1 << R2;               // blocks per row
// Four waves: three (192) took 570 us where four take 544 (m = 21, 32-bit keys;
// on doubles 786 and 757), six and eight 664 and 541 (doubles 1041 and 960: 148
// registers leave three waves a SIMD, which they do not fill).
constexpr int THREADS = 256;
constexpr int kMaxChunks = 32;             // chunks of one row's pairs

constexpr int TOP = NS2 / 2;               // the top middle bit, E
constexpr int WAVES = THREADS / kWave;

// block of middle mask x2 at slot x2, its low four bits flipped where bit 4 is
// set: an involution, linear over GF(2), that keeps E and spreads the lanes
// of a wave over the 16 groups of LDS banks (the 64 lanes' block reads take
// 36 passes of 16 lanes where 32 is the least; unflipped 58)
__host__ __device__ constexpr uint32_t slot_of(uint32_t x2) { return x2 ^ ((x2 & 16u) ? 15u : 0u); }
// a row: planes of 16-byte pieces, block at slot s in piece s of each plane
template <class E> __host__ __device__ constexpr uint32_t pos(uint32_t slot, int x) {
    constexpr int P = 16 / (int)sizeof(E);
    return (uint32_t)(x / P) * (uint32_t)(NS2 * P) + slot * (uint32_t)P + (uint32_t)(x % P);
}
template <class E> __device__ inline void load_blk(const E *row, uint32_t slot, E (&v)[NB]) {
    constexpr int P = 16 / (int)sizeof(E);
    const __uint128_t *p = reinterpret_cast<const __uint128_t *>(row) + slot;
#pragma unroll
    for (int q = 0; q < NB / P; ++q) {
        const __uint128_t t = p[q * NS2];
#pragma unroll
        for (int i = 0; i < P; ++i) {
            if constexpr (P == 4) v[P * q + i] = (uint32_t)(t >> (32 * i));
            else v[P * q + i] = Key<E>::from_bits((uint64_t)(t >> (64 * i)));
        }
    }
}

// Work items: lanes that hold a run of cnt consecutive submasks A2 of S2,
// S2 | first A2 << 8 | cnt << 16 | log2(lanes of this S2) << 24 | 1 << 31
// (0: none). The lanes of one S2 are an aligned group.
//   cross   a row pair, on the middle bits below E: A2 runs over all
//           submasks, at most 4 per lane
//   self[k] the self pair's level k = |S2|: all but A2 = S2
struct Items { uint32_t cross[kWave]; uint32_t self[R2 + 1][THREADS]; bool ok; };
constexpr Items make_items() {
    Items t{};
    t.ok = true;
    auto group = [&](uint32_t *v, int lanes, int &at, int s2, int run, int n) {
        const int k = cpop(s2);
        int lg = 0;
        while ((run << lg) < (1 << k)) ++lg;
        if (at % (1 << lg) != 0 || at + (1 << lg) > lanes) { t.ok = false; return; }
        for (int j = 0; j < (1 << lg); ++j) {
            const int first = j * run, left = n - first, cnt = left < 0 ? 0 : left < run ? left : run;
            v[at++] = (uint32_t)s2 | (cdeposit((uint32_t)first, (uint32_t)s2) << 8) | ((uint32_t)cnt << 16) |
                      ((uint32_t)lg << 24) | (1u << 31);
        }
    };
    int at = 0;
    for (int k = R2 - 1; k >= 0; --k)
        for (int s = 0; s < TOP; ++s)
            if (cpop(s) == k && t.ok) group(t.cross, kWave, at, s, 4, 1 << k);
    t.self[0][0] = 1u << 31;
    for (int k = 1; k <= R2; ++k) {
        at = 0;
        for (int s = 0; s < NS2; ++s)
            if (cpop(s) == k && t.ok) group(t.self[k], THREADS, at, s, k == 4 ? 2 : 1, (1 << k) - 1);
    }
    return t;
}
constexpr Items kItems = make_items();
static_assert(kItems.ok, "the items of a row pair fit a wave's lanes, those of every level the workgroup's");
__constant__ Items c_items = kItems;

template <class E> using Weight = typename std::conditional<sizeof(E) == 4, uint32_t, uint64_t>::type;

// a wave's row pair; the finishing reuses the first two waves' rows
template <class E> struct alignas(16) Lds {
    E row[WAVES][2][ROW];  // [wave][A side, B side]
    uint64_t acc[ROW];     // best key of every entry (as order(): unsigned order is key order)
    __device__ E *own() { return row[0][0]; }             // row S_H
    __device__ E *zero() { return row[0][1]; }            // row 0
    __device__ Weight<E> *w() { return reinterpret_cast<Weight<E> *>(row[1][0]); }
    __device__ uint32_t *split() { return reinterpret_cast<uint32_t *>(row[1][1]); }
};

// LDS exchange between the lanes of one wave: LDS operations of a wave run in
// order, so only the compiler has to keep them so
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// a candidate's key in its lane -> 64 bits whose unsigned order is the
// order of (cost, A); narrow keys carry A_H beside them
template <class E> __device__ inline uint64_t order(E k, uint32_t a_h) {
    if constexpr (sizeof(E) == 4) return k == Key<E>::none() ? ~0ull : ((uint64_t)k << 32) | a_h;
    else return Key<E>::bits(k);
}
template <class E> __device__ inline uint64_t order_none() { return order<E>(Key<E>::none(), 0u); }

// minimum of a key over an aligned group of 2^lg lanes, as unsigned 64-bit
// (the high words, then the low words of the lanes that hold the least one)
__device__ inline uint64_t group_min(uint64_t key, uint32_t lg) {
    const uint32_t seg = lg < 4u ? 1u << lg : 16u, h = (uint32_t)(key >> 32);
    const uint32_t hi = rb::group_min32(h, seg);
    const uint32_t lo = rb::group_min32(h == hi ? (uint32_t)key : ~0u, seg);
    return ((uint64_t)hi << 32) | lo;
}
// the lanes' best keys of block S2 into acc, one LDS atomic per group and entry
template <class E>
__device__ inline void flush(const uint64_t (&key)[NB], uint32_t s2, uint32_t lg, uint64_t *acc) {
#pragma unroll
    for (int x = 0; x < NB; ++x) {
        const uint64_t g = group_min(key[x], lg);
        if ((threadIdx.x & ((1u << lg) - 1u)) == 0 && g != order_none<E>())
            atomicMin((unsigned long long *)&acc[(s2 << CB) | (uint32_t)x], (unsigned long long)g);
    }
}

// low bits of an entry's words that hold its tag
template <class E> __device__ inline uint32_t tag_bits(int m) {
    if constexpr (sizeof(E) == 4) return ROW - 1u;
    else if constexpr (std::is_same<E, double>::value) return ((1u << m) - 1u) << 1;
    else return (1u << m) - 1u;
}
// (a native vector: arrays of the HIP vector types held across a loop went
// to private memory, and the loads with them)
typedef uint32_t Piece __attribute__((ext_vector_type(4)));
template <class E> __device__ inline Piece clear_tags(Piece v, uint32_t keep) {
    v.x &= keep;
    v.z &= keep;
    if constexpr (sizeof(E) == 4) {
        v.y &= keep;
        v.w &= keep;
    }
    return v;
}

// W of row S_H, two entries per thread (in entry order), before the work
// whose waits then cover these loads
constexpr int W_PER = (ROW + THREADS - 1) / THREADS;
template <class E> __device__ inline void load_w(int m, uint32_t sh, const int64_t *__restrict__ W, Weight<E> (&w)[W_PER]) {
#pragma unroll
    for (int r = 0; r < W_PER; ++r) {
        const uint32_t e = threadIdx.x + (uint32_t)(r * THREADS);
        w[r] = e < (uint32_t)ROW ? (Weight<E>)W[sh | (e << (m - L))] : 0;
    }
}

// Completes row S_H (non-empty): s.acc holds its cross-pair keys. post, given
// for the row of the full set alone, receives C of the full set (host memory).
// A level's lanes convolve one or two block pairs, take the minima over the
// lanes of their S2 in registers and go on, all of them, with the block's own
// chain; the group's first lane writes the block. One barrier per level.
// What bounds it: seven levels of one dependent chain each (a level 1 row
// alone takes 8.4 us on 32-bit keys and 11.5 us on doubles, launch included;
// 16.6 and 19.7 us with the minima combined by LDS atomics, two barriers per
// level and 64-bit integers in place of doubles in the chain).
template <class E>
__device__ inline void finish_row(int m, uint32_t sh, const Weight<E> (&w_in)[W_PER], Lds<E> &s, E *__restrict__ T,
                                  int64_t *__restrict__ C, uint32_t *__restrict__ split, int64_t *post) {
    constexpr bool NARROW = sizeof(E) == 4;
    const int tid = (int)threadIdx.x, H = m - L;
    E *rS = s.own(), *r0 = s.zero();
    Weight<E> *ws = s.w();
    uint32_t *spl = s.split();
    constexpr int PIECES = ROW * (int)sizeof(E) / 16;
    const uint32_t keep = ~tag_bits<E>(m);
    for (int p = tid; p < PIECES; p += THREADS)
        reinterpret_cast<Piece *>(r0)[p] = clear_tags<E>(reinterpret_cast<const Piece *>(T)[p], keep);
#pragma unroll
    for (int r = 0; r < W_PER; ++r)
        if (tid + r * THREADS < ROW) ws[tid + r * THREADS] = w_in[r];
    uint32_t items[R2 + 1];
#pragma unroll
    for (int k = 0; k <= R2; ++k) items[k] = c_items.self[k][tid];
    lds_barrier();
    const bool single = (sh & (sh - 1u)) == 0;
    const uint64_t mask = ((uint64_t)1 << m) - 1u;
    E b0[NB];
    load_blk<E>(r0, 0u, b0);
#pragma unroll
    for (int k = 0; k <= R2; ++k) {
        const uint32_t it = items[k];
        if (it >> 31) {
            const uint32_t s2 = it & 0xffu, lg = (it >> 24) & 15u, slot = slot_of(s2), tag = s2 << CB;
            uint64_t kacc[NB];
            Weight<E> w[NB];
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                kacc[x] = s.acc[tag | (uint32_t)x];
                w[x] = ws[tag | (uint32_t)x];
            }
            // A2 a proper submask of S2
            E best[NB];
#pragma unroll
            for (int x = 0; x < NB; ++x) best[x] = Key<E>::none();
            if (k > 0) {
                uint32_t a2 = (it >> 8) & 0xffu;
#pragma unroll
                for (int i = 0; i < (k == 4 ? 2 : 1); ++i) {
                    if ((uint32_t)i < ((it >> 16) & 15u)) {
                        const uint32_t sa = slot_of(a2);
                        E a[NB], b[NB];
                        load_blk<E>(rS, sa, a);
                        load_blk<E>(r0, slot ^ sa, b);
                        conv_full<E>(a, b, best);
                    }
                    a2 = ((a2 | ~s2) + 1u) & s2;
                }
                // (a level's groups are of one size: 2^lg lanes, lg of k alone)
                constexpr int kLog[R2 + 1] = {0, 0, 2, 3, 3, 5, 6};
                const uint32_t seg = kLog[k] < 4 ? 1u << kLog[k] : 16u;
#pragma unroll
                for (int x = 0; x < NB; ++x) {
                    if constexpr (NARROW) {
                        best[x] = rb::group_min32(best[x], seg);
                    } else {
                        best[x] = Key<E>::from_bits(group_min(Key<E>::bits(best[x]), (uint32_t)kLog[k]));
                    }
#pragma unroll
                    for (int off = 16; off < (1 << kLog[k]); off <<= 1)
                        best[x] = Key<E>::min(best[x], __shfl_xor(best[x], off, kWave));
                }
            }
            // A2 = S2: A = (S_H, S2, A1) holds lowbit(S), B = (0, 0, S1 ^ A1)
            // is in block 0 of row 0; S1 in order of popcount
            const bool leaf0 = k == 0 && single;
            uint32_t sp[NB];
            E entry[NB];
            if constexpr (NARROW) {
                uint32_t out[NB];
#pragma unroll
                for (int pc = 0; pc <= CB; ++pc) {
#pragma unroll
                    for (int s1 = 0; s1 < NB; ++s1) {
                        if (cpop(s1) != pc) continue;
                        const uint32_t nacc = (uint32_t)(kacc[s1] >> 32), aacc = (uint32_t)kacc[s1];
                        uint32_t nk = best[s1];
#pragma unroll
                        for (int a1 = 0; a1 < NB; ++a1) {
                            if ((a1 & ~s1) || a1 == s1) continue;
                            const uint32_t c = out[a1] + b0[s1 ^ a1];
                            nk = c < nk ? c : nk;
                        }
                        const bool leaf = s1 == 0 && leaf0;
                        const uint32_t key = nk < nacc ? nk : nacc;
                        out[s1] = ((leaf ? w[s1] : (key >> L) - w[s1]) << L) | tag | (uint32_t)s1;
                        // off the chain: equal narrow keys go to the smaller A_H
                        const uint32_t a_h = nk < nacc || (nk == nacc && sh < aacc) ? sh : aacc;
                        sp[s1] = leaf ? 0u : ((key & (ROW - 1u)) << H) | a_h;
                        entry[s1] = out[s1];
                    }
                }
            } else {
                const uint32_t base = sh | (tag << H);
#pragma unroll
                for (int pc = 0; pc <= CB; ++pc) {
#pragma unroll
                    for (int s1 = 0; s1 < NB; ++s1) {
                        if (cpop(s1) != pc) continue;
                        E kb = Key<E>::min(Key<E>::from_bits(kacc[s1]), best[s1]);
#pragma unroll
                        for (int a1 = 0; a1 < NB; ++a1) {
                            if ((a1 & ~s1) || a1 == s1) continue;
                            kb = Key<E>::min(kb, Key<E>::add(entry[a1], b0[s1 ^ a1]));
                        }
                        const uint64_t key = Key<E>::key_value(Key<E>::bits(kb)), wm = w[s1] << m;
                        const bool leaf = s1 == 0 && leaf0;
                        const uint64_t c = leaf ? wm : (key & ~mask) - wm;
                        sp[s1] = leaf ? 0u : (uint32_t)(key & mask);
                        entry[s1] = Key<E>::entry(c | base | ((uint32_t)s1 << H));
                    }
                }
            }
            if ((tid & ((1 << lg) - 1)) == 0) {
#pragma unroll
                for (int x = 0; x < NB; ++x) {
                    rS[pos<E>(slot, x)] = entry[x];
                    spl[tag | (uint32_t)x] = sp[x];
                }
            }
        }
        lds_barrier();
    }
    for (int p = tid; p < PIECES; p += THREADS)
        reinterpret_cast<Piece *>(T + ((size_t)sh << L))[p] = reinterpret_cast<const Piece *>(rS)[p];
    for (uint32_t e = (uint32_t)tid; e < (uint32_t)ROW; e += THREADS) {
        const E v = rS[pos<E>(slot_of(e >> CB), (int)(e & (NB - 1u)))];
        const uint32_t at = sh | (e << H);
        int64_t c;
        if constexpr (NARROW) c = (int64_t)(v >> L);
        else c = (int64_t)(Key<E>::entry_value(v) >> m);
        C[at] = c;
        split[at] = spl[e];
        if (post && e == (uint32_t)ROW - 1u) *post = c;
    }
}

// One level's cross pairs: a workgroup takes chunk id % chunks (of per_chunk
// pairs) of one row, its waves the chunk's pairs in turn. Lanes hold the best
// keys of their two blocks (S2 and S2 | E) across the pairs. chunks == 1: the
// workgroup completes the row as well; otherwise it leaves its keys in
// partial, a row of 2^9 words per workgroup. A pair's rows reach the wave's
// LDS through registers, loaded while the pair before runs.
// What bounds it: VALU issue and the waits of few waves. A wave's pair is 520
// VALU instructions on 32-bit keys (486 of them candidates: v_add_u32,
// v_min3_u32), 660 on doubles; at m = 20, h = 7 (20790 pairs) a launch takes
// 33 us, 0.62 of the issue rate. Three waves per pair with a barrier each and
// a block load per convolution operand took 42 us.
template <class E>
__global__ __launch_bounds__(THREADS) void k_sr_cross(int m, int h, uint32_t n_pairs, uint32_t chunks,
                                                      uint32_t per_chunk, const int64_t *__restrict__ W,
                                                      E *__restrict__ T, int64_t *__restrict__ C,
                                                      uint32_t *__restrict__ split, int64_t *post, uint64_t *__restrict__ partial) {
    __shared__ Lds<E> s;
    constexpr int PIECES = ROW * (int)sizeof(E) / 16;
    constexpr int PER = PIECES / kWave;          // 16-byte pieces of a row per lane
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1u);
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid / kWave));
    const uint32_t id = xcd_block(blockIdx.x, gridDim.x);
    const uint32_t sh = unrank_colex(id / chunks, h, m - L);
    const uint32_t first = (id % chunks) * per_chunk + wave;
    const uint32_t end = (id % chunks + 1u) * per_chunk;
    const uint32_t last = end < n_pairs ? end : n_pairs;
    Weight<E> w[W_PER];
    if (chunks == 1) load_w<E>(m, sh, W, w);
    for (uint32_t e = tid; e < (uint32_t)ROW; e += THREADS) s.acc[e] = order_none<E>();
    lds_barrier();
    if (first < last) {
        const uint32_t low = sh & (0u - sh), rest = sh ^ low;
        const uint32_t keep = ~tag_bits<E>(m);
        const uint32_t it = c_items.cross[lane];
        const uint32_t s2 = it & 0xffu, cnt = (it >> 16) & 15u;
        uint32_t sa[4];
        {
            uint32_t a2 = (it >> 8) & 0xffu;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                sa[i] = slot_of(a2);
                a2 = ((a2 | ~s2) + 1u) & s2;
            }
        }
        const uint32_t slot = slot_of(s2);
        E *rA = s.row[wave][0], *rB = s.row[wave][1];
        Piece st_a[PER], st_b[PER];
        auto fetch = [&](uint32_t a_h) {
            const Piece *pa = reinterpret_cast<const Piece *>(T + ((size_t)a_h << L)) + lane;
            const Piece *pb = reinterpret_cast<const Piece *>(T + ((size_t)(sh ^ a_h) << L)) + lane;
#pragma unroll
            for (int r = 0; r < PER; ++r) st_a[r] = pa[r * kWave];
#pragma unroll
            for (int r = 0; r < PER; ++r) st_b[r] = pb[r * kWave];
        };
        E best0[NB], best1[NB];
        uint32_t ah0[NB], ah1[NB];
#pragma unroll
        for (int x = 0; x < NB; ++x) {
            best0[x] = best1[x] = Key<E>::none();
            ah0[x] = ah1[x] = 0;
        }
        const uint32_t step = deposit((uint32_t)WAVES, rest);
        uint32_t ap = deposit(first, rest);
        fetch(low | ap);
        for (uint32_t q = first; q < last; q += WAVES) {
            const uint32_t a_h = low | ap;
            wave_sync();                             // the pair before has been read
#pragma unroll
            for (int r = 0; r < PER; ++r) {
                reinterpret_cast<Piece *>(rA)[r * kWave + lane] = st_a[r];
                reinterpret_cast<Piece *>(rB)[r * kWave + lane] = clear_tags<E>(st_b[r], keep);
            }
            wave_sync();
            ap = ((ap | ~rest) + step) & rest;
            if (q + WAVES < last) fetch(low | ap);
            E old0[NB], old1[NB];
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                old0[x] = best0[x];
                old1[x] = best1[x];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if ((uint32_t)i < cnt) {
                    E a[NB], b[NB], t[NB];
                    load_blk<E>(rA, sa[i], a);
                    load_blk<E>(rB, slot ^ sa[i], b);
                    conv_full<E>(a, b, best0);
                    load_blk<E>(rB, (slot ^ sa[i]) + TOP, t);
                    conv_full<E>(a, t, best1);
                    load_blk<E>(rA, sa[i] + TOP, t);
                    conv_full<E>(t, b, best1);
                }
            }
            if constexpr (sizeof(E) == 4) {
                // (a wave's pairs come in increasing A_H: an equal key keeps the earlier one)
#pragma unroll
                for (int x = 0; x < NB; ++x) {
                    ah0[x] = best0[x] < old0[x] ? a_h : ah0[x];
                    ah1[x] = best1[x] < old1[x] ? a_h : ah1[x];
                }
            }
        }
        uint64_t key[NB];
#pragma unroll
        for (int x = 0; x < NB; ++x) key[x] = order<E>(best0[x], ah0[x]);
        flush<E>(key, s2, (it >> 24) & 15u, s.acc);
#pragma unroll
        for (int x = 0; x < NB; ++x) key[x] = order<E>(best1[x], ah1[x]);
        flush<E>(key, s2 | (uint32_t)TOP, (it >> 24) & 15u, s.acc);
    }
    lds_barrier();
    if (chunks == 1) {
        finish_row<E>(m, sh, w, s, T, C, split, post);
    } else {
        for (uint32_t e = tid; e < (uint32_t)ROW; e += THREADS) partial[(size_t)id * ROW + e] = s.acc[e];
    }
}

// completes the rows of one level from their chunks' keys
template <class E>
__global__ __launch_bounds__(THREADS) void k_sr_final(int m, int h, uint32_t chunks, const int64_t *__restrict__ W,
                                                      E *__restrict__ T, int64_t *__restrict__ C,
                                                      uint32_t *__restrict__ split, int64_t *post,
                                                      const uint64_t *__restrict__ partial) {
    __shared__ Lds<E> s;
    const uint32_t sh = unrank_colex(blockIdx.x, h, m - L);
    Weight<E> w[W_PER];
    load_w<E>(m, sh, W, w);
    // 16 bytes of a chunk per lane, sixteen chunks in flight
    const ulonglong2 *src = reinterpret_cast<const ulonglong2 *>(partial + (size_t)blockIdx.x * chunks * ROW);
    for (uint32_t p = threadIdx.x; p < (uint32_t)ROW / 2; p += THREADS) {
        ulonglong2 v = src[p];
        for (uint32_t c = 1; c < chunks; c += 16) {
            ulonglong2 o[16];
#pragma unroll
            for (uint32_t j = 0; j < 16; ++j) o[j] = src[(size_t)(c + j < chunks ? c + j : 0u) * (ROW / 2) + p];
#pragma unroll
            for (uint32_t j = 0; j < 16; ++j) {
                v.x = o[j].x < v.x ? o[j].x : v.x;
                v.y = o[j].y < v.y ? o[j].y : v.y;
            }
        }
        reinterpret_cast<ulonglong2 *>(s.acc)[p] = v;
    }
    finish_row<E>(m, sh, w, s, T, C, split, post);
}

// row 0, the DP over the 9 in-row requests alone, by one workgroup
template <class E>
__global__ __launch_bounds__(rb::THREADS) void k_sr_row0(int m, const int64_t *__restrict__ W, E *__restrict__ T,
                                                         int64_t *__restrict__ C, uint32_t *__restrict__ split) {
    typedef Weight<E> D;
    __shared__ __align__(16) D t[rb::ROW];
    __shared__ __align__(16) D acc[rb::ROW];
    const int H = m - L;
    int own_k;
    uint32_t own_s2;
    D w[NB];
    rb::row_block(R2, own_k, own_s2);
#pragma unroll
    for (int x = 0; x < NB; ++x) w[x] = own_k >= 0 ? (D)W[((own_s2 << CB) | (uint32_t)x) << H] : 0;
    rb::row_dp<D>(R2, own_k, own_s2, w, t, acc);
    for (uint32_t e = threadIdx.x; e < (uint32_t)ROW; e += rb::THREADS) {
        const D c = t[rb::row_pos<D>(rb::slot_of(e >> CB), (int)(e & (NB - 1u)))] >> rb::L;
        const uint32_t at = pos<E>(slot_of(e >> CB), (int)(e & (NB - 1u)));
        if constexpr (sizeof(E) == 4) T[at] = (c << L) | e;
        else T[at] = Key<E>::entry(((uint64_t)c << m) | ((uint64_t)e << H));
        C[e << H] = e ? (int64_t)c : kInf;
        split[e << H] = (uint32_t)acc[e] << H;
    }
}

}  // namespace sr
