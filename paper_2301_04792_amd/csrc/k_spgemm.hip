// C = A B, Gustavson's row-by-row sparse product (Sec. 5.3 names it as the
// extension of SpMM: one kernel sizes each output row, the output is
// allocated, a second kernel multiplies).  Row i of C is the union of the
// rows of B selected by row i of A, each scaled by the A entry.
//
// Work per row is its product count p_i = sum over A entries of the length
// of the selected B row, which ranges from a few to millions on power-law
// inputs.  Rows are sorted into four tiers by p_i, each with its own
// accumulator:
//   tier 0 (p_i <= 32):    an 8-lane group per row, eight rows per wavefront,
//                           sorted in registers;
//   tier 1 (p_i <= 256):   one wavefront per row; the products, keyed by
//                           (column, product index), are bitonic-sorted in
//                           registers; equal columns are then adjacent, in
//                           product order;
//   tier 2 (p_i <= 4096):  one block per row, the same;
//   tier 3 (larger):       blocks of a work queue (32 to 512), a row at a time:
//                           a column bitmap gives the columns in order, and the
//                           products are added by column.  Up to 2^18 columns
//                           the bitmap and the sums are in LDS; beyond, each
//                           block owns a slot of global memory (1 GiB in all)
//                           with a dense float accumulator and a two-level
//                           bitmap, and the products are enumerated by the
//                           group_mapped_scan schedule over the row's A
//                           entries (tiles) and their B rows (atoms).
// The count pass runs the same tiers without values and writes each row's
// column count; an int64 scan turns them into C's row offsets.  Tiers 1 and
// 2 sum each column's products in product order (deterministic); tier 3
// adds them with float atomics (order varies run to run).
#include "lb_device.h"
#include "lb_internal.h"
#include "lb_schedule.hpp"

namespace lbk {
using namespace lb;

namespace {

constexpr int kTier0 = 32;  // an 8-lane group per row, 8 rows per wavefront
constexpr int kTier0Bits = 27;  // C's columns fit this many bits (wider ones: tier 1)
constexpr int kTier1 = 256;
constexpr int kTier2 = 4096;
constexpr int kBlock = 256;
constexpr int kBitBlock = 1024;
constexpr int kBitChunk = 16 * kBitBlock;  // columns emitted together, 16 a thread
constexpr int64_t kBitCols = 1 << 18;
constexpr int kBitSums = 1 << 14;  // entries of C summed together
constexpr int kBitPasses = 4;

struct gemm_args {
    int32_t m, n;
    const int32_t *a_ro, *a_ci;
    const float *a_val;
    const int32_t *b_ro, *b_ci;
    const float *b_val;
    const int64_t *prod;   // products per row
    int32_t *lists;        // tier lists: [0, m) tier 1, [m, 2m) tier 2, [2m, 3m) tier 3, [3m, 4m) tier 0
    int32_t *list_len;     // counters of tiers 1, 2, 3, the tier-3 work-queue ticket, the tier-0 counter
    int32_t *c_ro;         // count pass: per-row column counts; compute pass: C's row offsets
    int32_t *c_ci;
    float *c_val;
    float *slot_acc;       // tier 3: slots x n floats
    uint32_t *slot_bits;   // tier 3: slots x (n/32 words + n/1024 summary words)
    int64_t slot_words;    // words per slot bitmap (level 0 then level 1)
};

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------- products per row and tiers

// Both forms also zero the counters that the kernels after them append by, in
// place of a fill launch of 3 us and its gap.
__device__ __forceinline__ void clear_counters(const gemm_args &g) {
    if (blockIdx.x == 0 && threadIdx.x < 5) g.list_len[threadIdx.x] = 0;
}

// A wavefront per row of A (rows of eight or more entries on average).
__global__ __launch_bounds__(256) void gemm_products_rows(gemm_args g, int64_t *__restrict__ prod) {
    clear_counters(g);
    const group_mapped<kWave, csr_tile_set> sch{{g.a_ro, g.m, 0}};
    for (int64_t i : sch.tiles()) {
        int64_t p = 0;
        for (int64_t e : sch.atoms(sch.ts.tile(i))) {
            const int32_t j = g.a_ci[e];
            p += g.b_ro[j + 1] - g.b_ro[j];
        }
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) p += __shfl_xor(p, off, kWave);
        if (sch.lane() == 0) prod[i] = p;
    }
}

// For short rows: a block takes kProdRows rows and strides their entries, which
// are one range of A's; an entry's row is found among the row ends in LDS and its
// B row's length added to the row's LDS counter (exact, int64).    (Rows dealt
// to wavefronts 64 at a time, a segmented scan per step, took 30 us for 1M rows
// of five.)
constexpr int kProdRows = 512;
__global__ __launch_bounds__(256) void gemm_products(gemm_args g, int64_t *__restrict__ prod) {
    __shared__ int32_t s_end[kProdRows];
    __shared__ unsigned long long s_cnt[kProdRows];
    clear_counters(g);
    const int tid = threadIdx.x;
    const int64_t r0 = static_cast<int64_t>(blockIdx.x) * kProdRows;
    const int32_t rows = static_cast<int32_t>(g.m - r0 < kProdRows ? g.m - r0 : kProdRows);
    for (int q = tid; q < kProdRows; q += 256) {
        s_end[q] = g.a_ro[r0 + 1 + (q < rows ? q : rows - 1)];
        s_cnt[q] = 0;
    }
    const int32_t e0 = g.a_ro[r0];
    __syncthreads();
    const int32_t e1 = s_end[rows - 1];
    constexpr int U = 4;  // entries in flight per thread
    for (int64_t b = e0; b < e1; b += U * 256) {  // uniform across the block
        int32_t len[U], row[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t e = b + tid + u * 256;
            len[u] = -1;
            if (e < e1) {
                const int32_t j = g.a_ci[e];
                len[u] = g.b_ro[j + 1] - g.b_ro[j];
            }
            row[u] = 0;  // the first row whose end is past e
        }
#pragma unroll
        for (int step = kProdRows / 2; step > 0; step >>= 1) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (s_end[row[u] + step - 1] <= b + tid + u * 256) row[u] += step;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (len[u] > 0) atomicAdd(s_cnt + row[u], static_cast<unsigned long long>(len[u]));
    }
    __syncthreads();
    for (int q = tid; q < rows; q += 256) prod[r0 + q] = static_cast<int64_t>(s_cnt[q]);
}

// Rows into their tier's list.  A block takes kClassRows consecutive rows
// in two passes: it counts its rows per tier (per wavefront, then in LDS),
// reserves its stretch of each list with one atomicAdd per tier, and writes
// each wavefront's rows from its own offset in that stretch.  (One atomic per
// wavefront and tier put ~16k atomics on the one counter of a 1M-row
// matrix whose rows share a tier, ~200 µs of serialized atomics; blocks of 1024
// rows still 17 µs.)
constexpr int kClassRows = 4096;
constexpr int kClassBlock = 1024;
constexpr int kClassWaves = kClassBlock / kWave;

__device__ __forceinline__ int gemm_tier_of(int64_t p, int32_t n) {
    if (p <= kTier0) return p < 0 ? -1 : (n < (1 << kTier0Bits) ? 3 : 0);
    return p <= kTier1 ? 0 : (p <= kTier2 ? 1 : 2);
}

__global__ __launch_bounds__(kClassBlock) void gemm_classify(gemm_args g) {
    __shared__ int32_t s_cnt[kClassWaves][4];  // [wavefront][list]
    __shared__ int32_t s_base[4];
    const int w = wave_id(), lane = lane_id();
    const int64_t r0 = static_cast<int64_t>(blockIdx.x) * kClassRows;
    const int64_t r1 = r0 + kClassRows < g.m ? r0 + kClassRows : g.m;
    // pass 1: this wavefront's rows per list (list t holds tier t + 1 for t < 3, tier 0 for t = 3)
    int32_t cnt[4] = {0, 0, 0, 0};
    for (int64_t i0 = r0 + w * kWave; i0 < r1; i0 += kClassBlock) {  // uniform per wavefront
        const int64_t i = i0 + lane;
        const int t = gemm_tier_of(i < r1 ? g.prod[i] : -1, g.n);
#pragma unroll
        for (int q = 0; q < 4; ++q) cnt[q] += __popcll(__ballot(t == q));
    }
    if (lane == 0)
        for (int q = 0; q < 4; ++q) s_cnt[w][q] = cnt[q];
    __syncthreads();
    if (threadIdx.x < 4) {
        const int q = threadIdx.x;
        int32_t total = 0;
        for (int v = 0; v < kClassWaves; ++v) total += s_cnt[v][q];
        s_base[q] = total > 0 ? atomicAdd(g.list_len + (q == 3 ? 4 : q), total) : 0;
    }
    __syncthreads();
    // pass 2: the same rows in the same order, each list from this wavefront's offset
    int32_t off[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        off[q] = s_base[q];
        for (int v = 0; v < w; ++v) off[q] += s_cnt[v][q];
    }
    for (int64_t i0 = r0 + w * kWave; i0 < r1; i0 += kClassBlock) {
        const int64_t i = i0 + lane;
        const int t = gemm_tier_of(i < r1 ? g.prod[i] : -1, g.n);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint64_t mask = __ballot(t == q);
            if (t == q)
                g.lists[static_cast<int64_t>(q) * g.m + off[q] + __popcll(mask & ((1ull << lane) - 1))] =
                    static_cast<int32_t>(i);
            off[q] += __popcll(mask);
        }
    }
}

// ---------------------------------------------------------------- tiers 0, 1 and 2: sort in registers

// Exchange with lane gl ^ D of an aligned group of eight lanes (DPP: no LDS).
template <int D>
__device__ __forceinline__ uint32_t swap8(uint32_t v) {
    static_assert(D == 1 || D == 2 || D == 4, "lane distances in eight lanes");
    auto dpp = [](uint32_t x, auto ctrl) {
        return static_cast<uint32_t>(
            __builtin_amdgcn_update_dpp(0, static_cast<int>(x), decltype(ctrl)::value, 0xF, 0xF, false));
    };
    if constexpr (D == 1) return dpp(v, std::integral_constant<int, 0xB1>{});  // quad_perm [1,0,3,2]
    if constexpr (D == 2) return dpp(v, std::integral_constant<int, 0x4E>{});  // quad_perm [2,3,0,1]
    // half-row mirror (gl ^ 7), then quad_perm [3,2,1,0] (gl ^ 3)
    return dpp(dpp(v, std::integral_constant<int, 0x141>{}), std::integral_constant<int, 0x1B>{});
}

// Ascending bitonic sort of 32 keys held by eight lanes, lane gl elements
// 4 gl .. 4 gl + 3: distances 1 and 2 are inside a lane, 4, 8 and 16 are lane
// exchanges.
__device__ __forceinline__ void sort32(uint32_t (&k)[4], int gl) {
    auto pair = [](uint32_t &x, uint32_t &y, bool up) {
        const uint32_t lo = x < y ? x : y, hi = x < y ? y : x;
        x = up ? lo : hi;
        y = up ? hi : lo;
    };
    auto inside = [&](bool up) {  // distances 2, then 1
        pair(k[0], k[2], up), pair(k[1], k[3], up);
        pair(k[0], k[1], up), pair(k[2], k[3], up);
    };
    auto across = [&](auto dist, bool up) {
        constexpr int D = decltype(dist)::value;
        const bool keep_min = ((gl & D) == 0) == up;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t o = swap8<D>(k[r]);
            const uint32_t lo = k[r] < o ? k[r] : o, hi = k[r] < o ? o : k[r];
            k[r] = keep_min ? lo : hi;
        }
    };
    using d1 = std::integral_constant<int, 1>;
    using d2 = std::integral_constant<int, 2>;
    using d4 = std::integral_constant<int, 4>;
    pair(k[0], k[1], true), pair(k[2], k[3], false);
    inside((gl & 1) == 0);
    const bool up8 = (gl & 2) == 0, up16 = (gl & 4) == 0;
    across(d1{}, up8), inside(up8);
    across(d2{}, up16), across(d1{}, up16), inside(up16);
    across(d4{}, true), across(d2{}, true), across(d1{}, true), inside(true);
}

// Tier 0: an 8-lane group per row (p <= 32), eight rows per wavefront.  The
// products are expanded into LDS and sorted in registers, four per lane, by one
// 32-bit key (column, product index), so n < 2^kTier0Bits; a value is fetched
// by its product index once its place is known.  (A 32-element network of
// 64-bit keys and values in LDS took 234 us for the count and 443 for the
// compute pass of the 1024 x 1024 stencil squared, 26.2M products.)
template <bool COMPUTE>
__global__ __launch_bounds__(kBlock) void gemm_tier0(gemm_args g) {
    constexpr int GL = 8;
    constexpr int GPB = kBlock / GL;
    constexpr int STRIDE = kTier0 + 4;  // 16-byte rows whose starts spread over the banks
    __shared__ __align__(16) uint32_t s_key[GPB][STRIDE];
    __shared__ float s_val[GPB][COMPUTE ? STRIDE : 1];
    const int gl = threadIdx.x & (GL - 1), gi = threadIdx.x / GL;
    uint32_t *key = s_key[gi];
    float *val = s_val[gi];
    const int32_t rows = g.list_len[4];
    const int64_t groups = static_cast<int64_t>(gridDim.x) * GPB;
    for (int64_t r = static_cast<int64_t>(blockIdx.x) * GPB + gi; r < rows; r += groups) {
        const int32_t i = g.lists[3 * static_cast<int64_t>(g.m) + r];
        const int32_t a0 = g.a_ro[i], a1 = g.a_ro[i + 1];
        const int32_t out0 = COMPUTE ? g.c_ro[i] : 0;
        int32_t p = 0;
        for (int32_t c0 = a0; c0 < a1; c0 += GL) {  // uniform over the group
            const int32_t e = c0 + gl;
            int32_t f0 = 0, len = 0;
            float a = 0.f;
            if (e < a1) {
                const int32_t j = g.a_ci[e];
                if constexpr (COMPUTE) a = g.a_val[e];
                f0 = g.b_ro[j];
                len = g.b_ro[j + 1] - f0;
            }
            const int32_t incl = group_scan_incl<GL>(len);
            const int32_t start = p + incl - len;
            constexpr int U = 6;  // loads in flight per lane
            for (int32_t t0 = 0; t0 < len; t0 += U) {
                int32_t c[U];
                float b[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int32_t f = f0 + (t0 + u < len ? t0 + u : len - 1);
                    c[u] = g.b_ci[f];
                    if constexpr (COMPUTE) b[u] = g.b_val[f];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int32_t q = start + t0 + u;
                    if (t0 + u < len) {
                        key[q] = (static_cast<uint32_t>(c[u]) << 5) | static_cast<uint32_t>(q);
                        if constexpr (COMPUTE) val[q] = a * b[u];
                    }
                }
            }
            p += __shfl(incl, GL - 1, GL);
        }
        for (int32_t q = p + gl; q < kTier0; q += GL) key[q] = 0xffffffffu;  // sorts after every real key
        wave_sync();
        uint32_t k[4];
        {
            const uint4 k4 = *reinterpret_cast<const uint4 *>(key + 4 * gl);
            k[0] = k4.x, k[1] = k4.y, k[2] = k4.z, k[3] = k4.w;
        }
        sort32(k, gl);
        // heads of the runs of equal columns among the first p elements
        const uint32_t before = static_cast<uint32_t>(__shfl_up(static_cast<int>(k[3]), 1, GL));
        bool head[4];
        int32_t cnt = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t last = q ? k[q - 1] : before;
            head[q] = 4 * gl + q < p && ((q == 0 && gl == 0) || (k[q] >> 5) != (last >> 5));
            cnt += head[q] ? 1 : 0;
        }
        const int32_t upto = group_scan_incl<GL>(cnt);
        if constexpr (COMPUTE) {
            float v[4];
            seg_t mine{0.f, 0};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v[q] = 4 * gl + q < p ? val[k[q] & (kTier0 - 1)] : 0.f;
                mine = head[q] ? seg_t{v[q], 1} : seg_t{mine.v + v[q], mine.f};
            }
            const seg_t incl = group_seg_scan_incl<GL>(mine);
            const float open = __shfl_up(incl.v, 1, GL);
            const int after = __shfl_down(static_cast<int>(head[0]), 1, GL);  // the next lane starts a run
            float sum = gl ? open : 0.f;
            int32_t at = out0 + upto - cnt - 1;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                sum = head[q] ? v[q] : sum + v[q];
                at += head[q] ? 1 : 0;
                const bool next = q < 3 ? head[q < 3 ? q + 1 : 3] : (after != 0 && gl < GL - 1);
                if (4 * gl + q < p && (next || 4 * gl + q == p - 1)) {
                    g.c_ci[at] = static_cast<int32_t>(k[q] >> 5);
                    g.c_val[at] = sum;
                }
            }
        } else {
            if (gl == GL - 1) g.c_ro[i] = upto;
        }
        wave_sync();
    }
}

// Exchange with lane ^ D of the wavefront.
__device__ __forceinline__ uint32_t lane_swap(uint32_t v, int d) {  // d is a constant where it is called
    switch (d) {
        case 1: return swap8<1>(v);
        case 2: return swap8<2>(v);
        case 4: return swap8<4>(v);
        case 8:  // row_ror:8
            return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x128, 0xF, 0xF, false));
        default: return __shfl_xor(v, d, kWave);
    }
}
__device__ __forceinline__ uint64_t lane_swap(uint64_t v, int d) {
    return static_cast<uint64_t>(lane_swap(static_cast<uint32_t>(v >> 32), d)) << 32 |
           lane_swap(static_cast<uint32_t>(v), d);
}

// The threads of one row: a wavefront or a block.
template <int T>
struct row_team {
    static __device__ __forceinline__ int rank() { return threadIdx.x & (T - 1); }
    static __device__ __forceinline__ void sync() {
        if constexpr (T == kWave)
            wave_sync();
        else
            __syncthreads();
    }
    static __device__ __forceinline__ int32_t scan_incl(int32_t v, int32_t *s_wave) {
        if constexpr (T == kWave)
            return group_scan_incl<kWave>(v);
        else
            return block_scan_incl<T>(v, s_wave);
    }
    static __device__ __forceinline__ float open_sum(seg_t x, seg_t *s_wave) {  // exclusive segmented scan
        if constexpr (T == kWave) {
            const seg_t incl = group_seg_scan_incl<kWave>(x);
            const float v = __shfl_up(incl.v, 1, kWave);
            return rank() ? v : 0.f;
        } else {
            seg_t tot;
            return block_seg_scan_excl<T>(x, s_wave, tot).v;
        }
    }
};

// The products of a row dealt to T threads: EN entries of A at a time.
template <int T, int EN, bool COMPUTE>
struct row_deal {
    int32_t start[EN], from[EN];  // first product of an A entry; its B row begins at from + start
    float a[COMPUTE ? EN : 1];
    int32_t total;
    int32_t wave[T / kWave];
};

// Calls body(q, column of B, product) for every product q of the entries [a0, a1)
// of A.  The products of EN entries are dealt to the threads in order, each
// finding its entry among the starts in LDS, so B rows are read coalesced whatever
// their lengths.  Every thread of the team calls it; the LDS is free afterwards.
// q is exact up to 2^32 products; without VALUES the product is 0.
template <bool VALUES, int T, int EN, bool COMPUTE, typename F>
__device__ __forceinline__ void each_product(const gemm_args &g, row_deal<T, EN, COMPUTE> &l, int32_t a0, int32_t a1,
                                             F body) {
    using team = row_team<T>;
    const int t = team::rank();
    uint32_t base = 0;
    for (int32_t c0 = a0; c0 < a1; c0 += EN) {
        const int32_t e = c0 + t;
        int32_t f0 = 0, n = 0;
        float a = 0.f;
        if (t < EN && e < a1) {
            const int32_t j = g.a_ci[e];
            if constexpr (VALUES) a = g.a_val[e];
            f0 = g.b_ro[j];
            n = g.b_ro[j + 1] - f0;
        }
        const int32_t incl = team::scan_incl(n, l.wave);
        if (t < EN) {
            l.start[t] = incl - n;
            l.from[t] = f0 - (incl - n);
            if constexpr (VALUES) l.a[t] = a;
        }
        if (t == T - 1) l.total = incl;
        team::sync();
        const uint32_t end = l.total;
        constexpr int U = 4;  // products in flight per thread
        for (uint32_t q0 = t; q0 < end; q0 += U * T) {
            int32_t q[U], w[U], c[U];
            float b[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                q[u] = static_cast<int32_t>(q0 + u * T < end ? q0 + u * T : end - 1);
                w[u] = 0;
            }
#pragma unroll
            for (int s = EN / 2; s > 0; s >>= 1) {  // the last entry that starts at or before q
#pragma unroll
                for (int u = 0; u < U; ++u) w[u] += l.start[w[u] + s] <= q[u] ? s : 0;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int32_t f = l.from[w[u]] + q[u];
                c[u] = g.b_ci[f];
                if constexpr (VALUES) b[u] = g.b_val[f];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (q0 + u * T < end) {
                    if constexpr (VALUES)
                        body(base + q[u], c[u], l.a[w[u]] * b[u]);
                    else
                        body(base + q[u], c[u], 0.f);
                }
            }
        }
        base += end;
        team::sync();
    }
}

// LDS of one row of at most P products on T threads.
template <int T, int P, typename K, bool COMPUTE>
struct row_lds {
    K key[P];                    // keys in product order; then of the exchange; then the columns of C
    float val[COMPUTE ? P : 1];  // products; then the values of C
    row_deal<T, T, COMPUTE> deal;
    seg_t seg[T / kWave];
};

// Ascending bitonic sort of T * E keys, thread t elements E t .. E t + E - 1:
// distances below E are inside a thread, below 64 E lane exchanges, the rest go
// through LDS (x, T * E keys).
template <int T, int E, typename K>
__device__ __forceinline__ void sort_keys(K (&k)[E], int t, K *x) {
#pragma unroll
    for (int size = 2; size <= T * E; size <<= 1) {
#pragma unroll
        for (int j = size >> 1; j > 0; j >>= 1) {
            if (j >= E) {
                const int d = j / E;
                const bool keep_min = ((t & d) == 0) == ((t & (size / E)) == 0);
                if (d >= kWave) {
#pragma unroll
                    for (int e = 0; e < E; ++e) x[e * T + t] = k[e];
                    row_team<T>::sync();
                }
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const K o = d < kWave ? lane_swap(k[e], d) : x[e * T + (t ^ d)];
                    k[e] = (k[e] < o) == keep_min ? k[e] : o;
                }
                if (d >= kWave) row_team<T>::sync();
            } else {
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    if ((e & j) == 0) {
                        const bool up = size < E ? (e & size) == 0 : (t & (size / E)) == 0;
                        const K p = k[e], q = k[e | j];
                        const bool keep = (p < q) == up;
                        k[e] = keep ? p : q;
                        k[e | j] = keep ? q : p;
                    }
                }
            }
        }
    }
}

// The p products of a row, already in l.key (column << BITS | product) and l.val:
// sorted, equal columns summed in product order, written from out0 (compute), or
// the columns counted (returned by the last thread).
template <int T, int P, int E, int BITS, typename K, bool COMPUTE>
__device__ __forceinline__ int32_t reduce_row(const gemm_args &g, row_lds<T, P, K, COMPUTE> &l, int32_t p,
                                              int32_t out0) {
    using team = row_team<T>;
    const int t = team::rank();
    K k[E];
#pragma unroll
    for (int e = 0; e < E; ++e) k[e] = e * T + t < p ? l.key[e * T + t] : ~static_cast<K>(0);  // sorts last
    team::sync();
    sort_keys<T, E, K>(k, t, l.key);
    // the neighbours' keys
    l.key[t] = k[E - 1];
    K before, after;
    if constexpr (T == kWave) {
        team::sync();
        before = l.key[t ? t - 1 : 0];
        team::sync();
        l.key[t] = k[0];
        team::sync();
        after = l.key[t < T - 1 ? t + 1 : t];
    } else {
        l.key[T + t] = k[0];
        team::sync();
        before = l.key[t ? t - 1 : 0];
        after = l.key[T + (t < T - 1 ? t + 1 : t)];
    }
    bool head[E + 1];  // of a run of equal columns
    int32_t cnt = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const K last = e ? k[e ? e - 1 : 0] : before;
        head[e] = E * t + e < p && (E * t + e == 0 || (k[e] >> BITS) != (last >> BITS));
        cnt += head[e] ? 1 : 0;
    }
    head[E] = E * t + E >= p || (after >> BITS) != (k[E - 1] >> BITS);
    const int32_t upto = team::scan_incl(cnt, l.deal.wave);
    if constexpr (COMPUTE) {
        float v[E];
        seg_t mine{0.f, 0};
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const bool in = E * t + e < p;
            v[e] = in ? l.val[static_cast<uint32_t>(k[e]) & ((1u << BITS) - 1)] : 0.f;
            mine = head[e] ? seg_t{v[e], 1} : seg_t{mine.v + v[e], mine.f};
        }
        float sum = team::open_sum(mine, l.seg);
        if (t == T - 1) l.deal.total = upto;
        team::sync();  // keys and products have been read: C's entries take their place
        int32_t at = upto - cnt - 1;
        uint32_t *col = reinterpret_cast<uint32_t *>(l.key);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            sum = head[e] ? v[e] : sum + v[e];
            at += head[e] ? 1 : 0;
            if (E * t + e < p && (E * t + e == p - 1 || head[e + 1])) {
                col[at] = static_cast<uint32_t>(k[e] >> BITS);
                l.val[at] = sum;
            }
        }
        team::sync();
        const int32_t total = l.deal.total;
        for (int32_t q = t; q < total; q += T) {
            g.c_ci[out0 + q] = static_cast<int32_t>(col[q]);
            g.c_val[out0 + q] = l.val[q];
        }
    }
    return upto;
}

// Tiers 1 (a wavefront per row, up to 256 products) and 2 (a block per row, up to
// 4096).  The products are sorted in registers by (column, product index), which
// fits 32 bits where C has at most 2^(32 - BITS) columns (K), and a value is
// fetched by its product index once its place is known.  50,378 power-law rows
// squared: block rows 67 us to compute and 50 to count, wavefront rows 12 and 10;
// 50,000 rows of 1 to 32 entries: 257, 154, 37 and 29.  (An LDS network of
// 64-bit keys and values, expanded by a thread per B row, took 600, 494, 55 and
// 40; 911, 534, 126 and 89.)
template <int T, int P, int BITS, typename K, bool COMPUTE>
__global__ __launch_bounds__(kBlock) void gemm_sort_rows(gemm_args g, const int32_t *__restrict__ list,
                                                         const int32_t *__restrict__ len) {
    using team = row_team<T>;
    constexpr int PER = kBlock / T;  // rows of a block
    __shared__ row_lds<T, P, K, COMPUTE> s_row[PER];
    const int t = team::rank();
    row_lds<T, P, K, COMPUTE> &l = s_row[threadIdx.x / T];
    const int32_t rows = *len;
    const int64_t step = static_cast<int64_t>(gridDim.x) * PER;
    for (int64_t r = static_cast<int64_t>(blockIdx.x) * PER + threadIdx.x / T; r < rows; r += step) {  // uniform in the team
        const int32_t i = list[r];
        const int32_t p = static_cast<int32_t>(g.prod[i]);
        const int32_t a0 = g.a_ro[i], a1 = g.a_ro[i + 1];
        each_product<COMPUTE>(g, l.deal, a0, a1, [&](uint32_t q, int32_t c, float v) {
            l.key[q] = static_cast<K>(c) << BITS | q;
            if constexpr (COMPUTE) l.val[q] = v;
        });
        const int32_t out0 = COMPUTE ? g.c_ro[i] : 0;
        int32_t upto;  // the smallest network that holds the products
        if constexpr (T == kWave) {
            if (p <= T)
                upto = reduce_row<T, P, 1, BITS, K, COMPUTE>(g, l, p, out0);
            else if (p <= 2 * T)
                upto = reduce_row<T, P, 2, BITS, K, COMPUTE>(g, l, p, out0);
            else
                upto = reduce_row<T, P, 4, BITS, K, COMPUTE>(g, l, p, out0);
        } else {
            if (p <= 2 * T)
                upto = reduce_row<T, P, 2, BITS, K, COMPUTE>(g, l, p, out0);
            else if (p <= 4 * T)
                upto = reduce_row<T, P, 4, BITS, K, COMPUTE>(g, l, p, out0);
            else if (p <= 8 * T)
                upto = reduce_row<T, P, 8, BITS, K, COMPUTE>(g, l, p, out0);
            else
                upto = reduce_row<T, P, 16, BITS, K, COMPUTE>(g, l, p, out0);
        }
        if constexpr (!COMPUTE) {
            if (t == T - 1) g.c_ro[i] = upto;
        }
        team::sync();
    }
}

template <int T, int P, int BITS>
void sort_rows(const gemm_args &g, const int32_t *list, const int32_t *len, uint32_t grid, bool compute,
               hipStream_t s) {
    const bool narrow = g.n <= (1ll << (32 - BITS));
    if (compute) {
        if (narrow)
            hipLaunchKernelGGL((gemm_sort_rows<T, P, BITS, uint32_t, true>), dim3(grid), dim3(kBlock), 0, s, g, list, len);
        else
            hipLaunchKernelGGL((gemm_sort_rows<T, P, BITS, uint64_t, true>), dim3(grid), dim3(kBlock), 0, s, g, list, len);
    } else {
        if (narrow)
            hipLaunchKernelGGL((gemm_sort_rows<T, P, BITS, uint32_t, false>), dim3(grid), dim3(kBlock), 0, s, g, list, len);
        else
            hipLaunchKernelGGL((gemm_sort_rows<T, P, BITS, uint64_t, false>), dim3(grid), dim3(kBlock), 0, s, g, list, len);
    }
}

// ---------------------------------------------------------------- tier 3: dense slot per block

// The slots that gemm_tier3 will use start clear (it clears what it used): as
// many as there are rows, up to `slots`.  Clearing all of them took 190 us (1 GiB
// of sums at n = 1M) where no row was this large.
template <bool COMPUTE>
__global__ __launch_bounds__(256) void gemm_clear_slots(gemm_args g, int64_t slots) {
    const int64_t used = g.list_len[2] < slots ? g.list_len[2] : slots;
    for (int64_t q : grid_stride_range(0, used * g.slot_words)) g.slot_bits[q] = 0u;
    if constexpr (COMPUTE)
        for (int64_t q : grid_stride_range(0, used * g.n)) g.slot_acc[q] = 0.f;
}

// More than kBitCols columns.  A block per slot; a block past the rows leaves, so
// the slots that the queue's rows use are the first ones.
template <bool COMPUTE>
__global__ __launch_bounds__(kBlock) void gemm_tier3(gemm_args g) {
    using sched = group_mapped_scan<kBlock, indexed_tile_set>;
    __shared__ typename sched::storage s_st[1];
    __shared__ int32_t s_wi[kBlock / kWave];
    __shared__ int32_t s_slot;
    __shared__ int32_t s_int;
    const int tid = threadIdx.x;
    if (static_cast<int32_t>(blockIdx.x) >= g.list_len[2]) return;  // uniform
    const int64_t nw0 = (static_cast<int64_t>(g.n) + 31) / 32;  // level-0 words: a bit per column
    float *acc = g.slot_acc + static_cast<int64_t>(blockIdx.x) * g.n;
    uint32_t *bits = g.slot_bits + static_cast<int64_t>(blockIdx.x) * g.slot_words;
    uint32_t *summary = bits + nw0;  // level 1: a bit per level-0 word
    const queue_rounds rows{g.list_len + 3, &s_slot, 1, g.list_len[2]};
    for (int64_t r : rows) {  // uniform across the block
        const int32_t i = g.lists[2 * static_cast<int64_t>(g.m) + r];
        const int32_t a0 = g.a_ro[i], a1 = g.a_ro[i + 1];
        // the row's A entries are the tiles; entry e selects B row a_ci[e]
        sched sch(indexed_tile_set{g.a_ci + a0, g.b_ro, a1 - a0}, s_st);
        int32_t mine = 0;  // columns this thread set first (count pass)
        const int64_t chunks = (static_cast<int64_t>(a1 - a0) + kBlock - 1) / kBlock;
        for (int64_t c = 0; c < chunks; ++c) {
            const int32_t total = sch.load(c);
            for (int64_t at : sch.atoms(total)) {
                const int32_t q = sch.get_tile(static_cast<int32_t>(at));
                const int32_t f = sch.atom(static_cast<int32_t>(at), q);
                const int32_t col = g.b_ci[f];
                const uint32_t bit = 1u << (col & 31);
                const uint32_t old = atomicOr(bits + (col >> 5), bit);
                if (old == 0) atomicOr(summary + (col >> 10), 1u << ((col >> 5) & 31));
                if constexpr (COMPUTE) {
                    const int32_t e = a0 + static_cast<int32_t>(c) * kBlock + q;
                    atomicAdd(acc + col, g.a_val[e] * g.b_val[f]);
                } else {
                    if (!(old & bit)) ++mine;
                }
            }
            sch.done();
        }
        __threadfence();
        __syncthreads();
        // walk the bitmap in column order: per summary word (32 level-0 words,
        // 1024 columns) a thread counts, the block scans, then it emits
        const int64_t nw1 = (nw0 + 31) / 32;
        int32_t written = 0;
        const int32_t out0 = COMPUTE ? g.c_ro[i] : 0;
        for (int64_t s0 = 0; s0 < nw1; s0 += kBlock) {  // uniform across the block
            const int64_t s = s0 + tid;
            const uint32_t sw = s < nw1 ? summary[s] : 0u;
            int32_t cnt = 0;
            if constexpr (COMPUTE) {
                for (uint32_t m = sw; m; m &= m - 1) cnt += __popc(bits[s * 32 + __ffs(m) - 1]);
            }
            const int32_t incl = block_scan_incl<kBlock>(cnt, s_wi);
            int32_t pos = written + incl - cnt;
            for (uint32_t m = sw; m; m &= m - 1) {
                const int64_t wi = s * 32 + __ffs(m) - 1;
                uint32_t word = bits[wi];
                if constexpr (COMPUTE) {
                    for (; word; word &= word - 1) {
                        const int32_t col = static_cast<int32_t>(wi * 32 + __ffs(word) - 1);
                        g.c_ci[out0 + pos] = col;
                        g.c_val[out0 + pos] = acc[col];
                        acc[col] = 0.f;
                        ++pos;
                    }
                }
                bits[wi] = 0u;
            }
            if (s < nw1) summary[s] = 0u;
            if (tid == kBlock - 1) s_int = incl;
            __syncthreads();
            written += s_int;
            __syncthreads();
        }
        if constexpr (!COMPUTE) {
            const int32_t incl = block_scan_incl<kBlock>(mine, s_wi);
            if (tid == kBlock - 1) g.c_ro[i] = incl;
        }
        __threadfence();
        __syncthreads();
    }
}

// Up to kBitCols columns: the row's bitmap is in LDS (dynamic, a multiple of
// kBitChunk columns), and counting never leaves it.  The compute pass enumerates
// the products once for the bitmap, turns it into the place of every 16 columns'
// first entry, writes the columns, and sums by place: kBitSums entries of C at a
// time in LDS, the products enumerated again for each (a pass costs 3.6 ps a
// product over the device, a global float atomic 48).  A row of more than
// kBitPasses times that adds into the block's slot instead: one long row alone is
// bound by its own block's passes.  kBitCols: the bitmap and the places take 64
// KB, beside 64 KB of sums.  50,378 power-law rows squared: 143 us to compute and 31 to
// count, against 627 and 281 with bitmap and sums in the slot.
template <bool COMPUTE>
__global__ __launch_bounds__(kBitBlock) void gemm_tier3_bits(gemm_args g) {
    constexpr int T = kBitBlock;
    extern __shared__ uint32_t s_bits[];  // the bitmap; compute: the place of each 16 columns in their chunk (16 bits)
    __shared__ row_deal<T, kBlock, COMPUTE> s_deal;
    __shared__ float s_sum[COMPUTE ? kBitSums : 1];
    __shared__ int32_t s_place[COMPUTE ? kBitCols / kBitChunk : 1];  // first entry of a chunk
    __shared__ int32_t s_slot;
    static_assert(kBitSums * 4 >= kBitChunk * 2, "a chunk's columns are listed in the sums");
    const int t = threadIdx.x;
    if (static_cast<int32_t>(blockIdx.x) >= g.list_len[2]) return;  // uniform
    const int32_t chunks = (g.n + kBitChunk - 1) / kBitChunk;
    const int32_t words = chunks * (kBitChunk / 32);
    for (int32_t w = t; w < words; w += T) s_bits[w] = 0u;
    __syncthreads();
    const queue_rounds rows{g.list_len + 3, &s_slot, 1, g.list_len[2]};
    for (int64_t r : rows) {  // uniform across the block
        const int32_t i = g.lists[2 * static_cast<int64_t>(g.m) + r];
        const int32_t a0 = g.a_ro[i], a1 = g.a_ro[i + 1];
        each_product<false>(g, s_deal, a0, a1,
                            [&](uint32_t, int32_t c, float) { atomicOr(s_bits + (c >> 5), 1u << (c & 31)); });
        if constexpr (COMPUTE) {
            const uint16_t *half = reinterpret_cast<uint16_t *>(s_bits);  // 16 columns per thread and chunk
            uint16_t *place = reinterpret_cast<uint16_t *>(s_bits + words);
            uint16_t *list = reinterpret_cast<uint16_t *>(s_sum);
            const int32_t out0 = g.c_ro[i];
            int32_t out = 0;
            for (int32_t k = 0; k < chunks; ++k) {  // uniform across the block
                uint32_t m = half[k * T + t];
                const int32_t cnt = __popc(m);
                const int32_t incl = block_scan_incl<T>(cnt, s_deal.wave);
                place[k * T + t] = static_cast<uint16_t>(incl - cnt);  // below kBitChunk where m != 0
                if (t == T - 1) s_deal.total = incl, s_place[k] = out;
                for (int32_t at = incl - cnt; m; m &= m - 1)
                    list[at++] = static_cast<uint16_t>(t * 16 + __ffs(static_cast<int>(m)) - 1);
                __syncthreads();
                const int32_t total = s_deal.total;
                for (int32_t q = t; q < total; q += T) g.c_ci[out0 + out + q] = k * kBitChunk + list[q];
                out += total;
                __syncthreads();
            }
            if (out <= kBitPasses * kBitSums) {
                for (int32_t p0 = 0; p0 < out; p0 += kBitSums) {
                    const int32_t here = out - p0 < kBitSums ? out - p0 : kBitSums;
                    for (int32_t q = t; q < here; q += T) s_sum[q] = 0.f;
                    __syncthreads();
                    each_product<true>(g, s_deal, a0, a1, [&](uint32_t, int32_t c, float v) {
                        const int32_t at = s_place[c / kBitChunk] + place[c >> 4] +
                                           __popc(half[c >> 4] & ((1u << (c & 15)) - 1)) - p0;
                        if (at >= 0 && at < here) unsafeAtomicAdd(s_sum + at, v);
                    });
                    for (int32_t q = t; q < here; q += T) g.c_val[out0 + p0 + q] = s_sum[q];
                    __syncthreads();
                }
            } else {
                float *acc = g.slot_acc + static_cast<int64_t>(blockIdx.x) * g.n;
                each_product<true>(g, s_deal, a0, a1, [&](uint32_t, int32_t c, float v) { unsafeAtomicAdd(acc + c, v); });
                __threadfence();
                __syncthreads();
                for (int32_t q = t; q < out; q += T) {
                    const int32_t c = g.c_ci[out0 + q];
                    g.c_val[out0 + q] = acc[c];
                    acc[c] = 0.f;
                }
                __threadfence();  // the slot is clear before the next row adds to it
            }
            for (int32_t w = t; w < words; w += T) s_bits[w] = 0u;
        } else {
            int32_t cnt = 0;
            for (int32_t w = t; w < words; w += T) {
                cnt += __popc(s_bits[w]);
                s_bits[w] = 0u;
            }
            const int32_t incl = block_scan_incl<T>(cnt, s_deal.wave);
            if (t == T - 1) g.c_ro[i] = incl;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------- int64 scan of the row counts

constexpr int kScanTile = 2048;

// Per tile of 2048 counts (int32, in c_ro): in-tile exclusive prefix (int64) and the tile total.
__global__ __launch_bounds__(256) void gemm_scan_tiles(const int32_t *__restrict__ cnt, int64_t m,
                                                       int64_t *__restrict__ pre, int64_t *__restrict__ tile_sum) {
    __shared__ int64_t s_w[256 / kWave];
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanTile + threadIdx.x * 8;
    int64_t v[8];
    int64_t sum = 0;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        v[u] = base + u < m ? cnt[base + u] : 0;
        sum += v[u];
    }
    int64_t incl = sum;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int64_t o = __shfl_up(incl, off, kWave);
        if (lane_id() >= off) incl += o;
    }
    if (lane_id() == kWave - 1) s_w[wave_id()] = incl;
    __syncthreads();
    for (int k = 0; k < wave_id(); ++k) incl += s_w[k];
    int64_t run = incl - sum;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        if (base + u < m) pre[base + u] = run;
        run += v[u];
    }
    if (threadIdx.x == 255) tile_sum[blockIdx.x] = incl;
}

// One block: exclusive prefix of the tile totals (m / 2048 of them) and the
// grand total (one thread took 60 us for 513 tiles).
constexpr int kTotalsBlock = 1024;
__global__ __launch_bounds__(kTotalsBlock) void gemm_scan_totals(int64_t *__restrict__ tile_sum, int64_t nb,
                                                                 int64_t *__restrict__ total) {
    __shared__ int64_t s_w[kTotalsBlock / kWave];
    int64_t carry = 0;
    for (int64_t b0 = 0; b0 < nb; b0 += kTotalsBlock) {  // uniform across the block
        const int64_t b = b0 + threadIdx.x;
        const int64_t v = b < nb ? tile_sum[b] : 0;
        int64_t incl = v;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int64_t o = __shfl_up(incl, off, kWave);
            if (lane_id() >= off) incl += o;
        }
        if (lane_id() == kWave - 1) s_w[wave_id()] = incl;
        __syncthreads();
        int64_t sum = 0;
#pragma unroll
        for (int k = 0; k < kTotalsBlock / kWave; ++k) {
            if (k < wave_id()) incl += s_w[k];
            sum += s_w[k];
        }
        if (b < nb) tile_sum[b] = carry + incl - v;
        carry += sum;
        __syncthreads();
    }
    if (threadIdx.x == 0) *total = carry;
}

// C's row offsets (int32) where the total fits; the host checks the total first.
__global__ __launch_bounds__(256) void gemm_scan_write(const int64_t *__restrict__ pre,
                                                       const int64_t *__restrict__ tile_pre,
                                                       const int64_t *__restrict__ total, int64_t m,
                                                       int32_t *__restrict__ c_ro) {
    for (int64_t i : grid_stride_range(0, m)) c_ro[i] = static_cast<int32_t>(pre[i] + tile_pre[i / kScanTile]);
    if (blockIdx.x == 0 && threadIdx.x == 0) c_ro[m] = static_cast<int32_t>(*total);
}

int64_t capped(int64_t work, int64_t per) {
    const int64_t b = (work + per - 1) / per;
    return b < 1 ? 1 : (b > 4096 ? 4096 : b);
}

}  // namespace

// ---------------------------------------------------------------- workspace

struct gemm_ws {
    int64_t *prod, *pre, *tile_sum, *total;
    int32_t *lists, *list_len;
    float *slot_acc;
    uint32_t *slot_bits;
    int64_t slot_words;
};

static gemm_ws gemm_carve(void *base, int64_t m, int64_t n) {
    char *p = static_cast<char *>(base);
    gemm_ws w;
    w.prod = reinterpret_cast<int64_t *>(p);
    p += align256(static_cast<size_t>(m) * 8);
    w.pre = reinterpret_cast<int64_t *>(p);
    p += align256(static_cast<size_t>(m) * 8);
    w.tile_sum = reinterpret_cast<int64_t *>(p);
    p += align256(static_cast<size_t>(m / kScanTile + 2) * 8);
    w.total = reinterpret_cast<int64_t *>(p);
    p += 256;
    w.lists = reinterpret_cast<int32_t *>(p);
    p += align256(static_cast<size_t>(4 * m) * 4);
    w.list_len = reinterpret_cast<int32_t *>(p);
    p += 256;
    w.slot_words = (n + 31) / 32 + ((n + 31) / 32 + 31) / 32;
    w.slot_acc = reinterpret_cast<float *>(p);
    p += align256(static_cast<size_t>(spgemm_slots(n)) * n * 4);
    w.slot_bits = reinterpret_cast<uint32_t *>(p);
    return w;
}

size_t spgemm_ws_bytes(int64_t m, int64_t n) {
    const int64_t words = (n + 31) / 32 + ((n + 31) / 32 + 31) / 32;
    return 2 * align256(static_cast<size_t>(m) * 8) + align256(static_cast<size_t>(m / kScanTile + 2) * 8) + 256 +
           align256(static_cast<size_t>(4 * m) * 4) + 256 + align256(static_cast<size_t>(spgemm_slots(n)) * n * 4) +
           align256(static_cast<size_t>(spgemm_slots(n)) * words * 4);
}

static hipError_t gemm_pass(const spgemm_dev &P, int32_t *c_ro, int32_t *c_ci, float *c_val, void *ws, bool compute,
                            hipStream_t s) {
    const gemm_ws w = gemm_carve(ws, P.m, P.n);
    gemm_args g{P.m, P.n, P.a_ro, P.a_ci, P.a_val, P.b_ro, P.b_ci, P.b_val, w.prod, w.lists, w.list_len,
                c_ro, c_ci, c_val, w.slot_acc, w.slot_bits, w.slot_words};
    hipError_t e;
    {
        prof_scope p(s, "spgemm_products");
        // short rows (fewer than 8 entries on average) share wavefronts; longer ones get one each
        if (P.m > 0 && static_cast<int64_t>(P.a_nnz) < 8 * static_cast<int64_t>(P.m)) {
            const int64_t blocks = (static_cast<int64_t>(P.m) + kProdRows - 1) / kProdRows;
            hipLaunchKernelGGL(gemm_products, dim3(static_cast<uint32_t>(blocks)), dim3(256), 0, s, g, w.prod);
        } else {
            constexpr int GPB = group_block<kWave>::GPB;  // grid-stride: at most 2^16 blocks
            const int64_t want = (static_cast<int64_t>(P.m) + GPB - 1) / GPB;
            const int64_t grid = want < 1 ? 1 : (want < 65536 ? want : 65536);
            hipLaunchKernelGGL(gemm_products_rows, dim3(static_cast<uint32_t>(grid)), dim3(256), 0, s, g, w.prod);
        }
        const int64_t cb = (static_cast<int64_t>(P.m) + kClassRows - 1) / kClassRows;
        hipLaunchKernelGGL(gemm_classify, dim3(static_cast<uint32_t>(cb < 1 ? 1 : cb)), dim3(kClassBlock), 0, s, g);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const int64_t slots = spgemm_slots(P.n);
    const bool bits_in_lds = P.n <= kBitCols;
    // slots hold the rows of too many entries for LDS, and the bitmaps past kBitCols
    if (compute && P.n > kBitPasses * kBitSums)
        hipLaunchKernelGGL(gemm_clear_slots<true>, dim3(1024), dim3(256), 0, s, g, slots);
    else if (!bits_in_lds)
        hipLaunchKernelGGL(gemm_clear_slots<false>, dim3(256), dim3(256), 0, s, g, slots);
    // one launch per tier (each reads its list's length on the device)
    const uint32_t grid12 = static_cast<uint32_t>(capped(P.m, 1) < 2048 ? capped(P.m, 1) : 2048);
    const char *names[2][4] = {{"spgemm_count_t0", "spgemm_count_t1", "spgemm_count_t2", "spgemm_count_t3"},
                               {"spgemm_compute_t0", "spgemm_compute_t1", "spgemm_compute_t2", "spgemm_compute_t3"}};
    const int c = compute ? 1 : 0;
    {
        prof_scope p(s, names[c][0]);
        if (compute)
            hipLaunchKernelGGL(gemm_tier0<true>, dim3(grid12), dim3(kBlock), 0, s, g);
        else
            hipLaunchKernelGGL(gemm_tier0<false>, dim3(grid12), dim3(kBlock), 0, s, g);
    }
    {
        prof_scope p(s, names[c][1]);
        sort_rows<kWave, kTier1, 8>(g, w.lists, w.list_len, grid12, compute, s);
    }
    {
        prof_scope p(s, names[c][2]);
        sort_rows<kBlock, kTier2, 12>(g, w.lists + P.m, w.list_len + 1, grid12, compute, s);
    }
    {
        prof_scope p(s, names[c][3]);
        const size_t bitmap = static_cast<size_t>((P.n + kBitChunk - 1) / kBitChunk) * (kBitChunk / 8);
        if (bits_in_lds && compute)
            hipLaunchKernelGGL(gemm_tier3_bits<true>, dim3(static_cast<uint32_t>(slots)), dim3(kBitBlock), 2 * bitmap, s, g);
        else if (bits_in_lds)
            hipLaunchKernelGGL(gemm_tier3_bits<false>, dim3(static_cast<uint32_t>(slots)), dim3(kBitBlock), bitmap, s, g);
        else if (compute)
            hipLaunchKernelGGL(gemm_tier3<true>, dim3(static_cast<uint32_t>(slots)), dim3(kBlock), 0, s, g);
        else
            hipLaunchKernelGGL(gemm_tier3<false>, dim3(static_cast<uint32_t>(slots)), dim3(kBlock), 0, s, g);
    }
    e = hipGetLastError();
    return e;
}

hipError_t spgemm_count(const spgemm_dev &P, int32_t *c_ro, int64_t *total_host, void *ws, hipStream_t s) {
    hipError_t e = gemm_pass(P, c_ro, nullptr, nullptr, ws, false, s);
    if (e != hipSuccess) return e;
    const gemm_ws w = gemm_carve(ws, P.m, P.n);
    const int64_t nb = (static_cast<int64_t>(P.m) + kScanTile - 1) / kScanTile;
    if (nb > 0)
        hipLaunchKernelGGL(gemm_scan_tiles, dim3(static_cast<uint32_t>(nb)), dim3(256), 0, s, c_ro,
                           static_cast<int64_t>(P.m), w.pre, w.tile_sum);
    hipLaunchKernelGGL(gemm_scan_totals, dim3(1), dim3(kTotalsBlock), 0, s, w.tile_sum, nb, w.total);
    hipLaunchKernelGGL(gemm_scan_write, dim3(static_cast<uint32_t>(capped(P.m, 256))), dim3(256), 0, s, w.pre,
                       w.tile_sum, w.total, static_cast<int64_t>(P.m), c_ro);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = hipMemcpyAsync(total_host, w.total, sizeof(int64_t), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    return e;
}

hipError_t spgemm_compute(const spgemm_dev &P, const int32_t *c_ro, int32_t *c_ci, float *c_val, void *ws,
                          hipStream_t s) {
    return gemm_pass(P, const_cast<int32_t *>(c_ro), c_ci, c_val, ws, true, s);
}

}  // namespace lbk
