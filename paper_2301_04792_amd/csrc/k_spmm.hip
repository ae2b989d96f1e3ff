// Merge-path SpMM (Sec. 5.3) and the batched persistent form, for gfx950.
//
// Y[r, :] = sum_j values[j] * X[col_idx[j], :].  The SpMM listing of
// Sec. 5.3 wraps the SpMV loop in a loop over B's columns; here the column
// loop sits inside the atom loop instead, so the matrix is read once for all
// columns (k <= 64).
//
// Per unit (the merge-path split and carry handling of k_merge.hip), two
// consumers:
//  * one column (merge_spmm_consume): the products values[j] * X[col_idx[j]]
//    of every nonzero are staged in LDS with all loads of a lane issued
//    before the first wait, then the threads walk their merge items over LDS
//    (the SpMV consumer's scheme);
//  * more columns (merge_spmm_rows): LDS holds the row ends and each
//    nonzero's X row and value; groups of lanes share the unit's merge items
//    and each lane keeps a few columns' sums.
//  Both finish with one segmented scan over all columns.
//
// Batched: matrices stored back to back form one block-diagonal matrix
// whose merged sequence of sum(m_b) row ends and sum(nnz_b) nonzeros is cut
// into units of W items by the split launch.  One persistent launch (grid =
// CUs x resident blocks) then loops over the units (Sec. 5.1 persistent
// ranges; every block leaves once its unit index passes the last unit).
// A nonzero's X row is col_base[b] + col_idx[j] for the matrix b that owns
// it: two wavefronts find the matrices of the unit's first and last rows;
// only a unit that straddles matrices searches the owner per nonzero.
#include "lb_device.h"
#include "lb_internal.h"

namespace lbk {
using namespace lb;

constexpr int kMaxCols = 64;  // columns of a call (checked by the caller)

// V consecutive values of an X row.  The row may start at any multiple of the
// element size (an odd stride or first column): the type says so, and one
// load of V elements serves on gfx950 whatever the alignment.
template <int V>
__device__ __forceinline__ void load_cols(const float *p, float (&o)[V]) {
    struct __attribute__((packed, aligned(4))) cols {
        float v[V];
    };
    const cols t = *reinterpret_cast<const cols *>(p);
#pragma unroll
    for (int e = 0; e < V; ++e) o[e] = t.v[e];
}
template <int V>
__device__ __forceinline__ void load_cols(const bf16_bits *p, float (&o)[V]) {
    static_assert(V % 2 == 0, "pairs of BF16");
    struct __attribute__((packed, aligned(2))) cols {
        uint32_t w[V / 2];
    };
    const cols t = *reinterpret_cast<const cols *>(p);
#pragma unroll
    for (int e = 0; e < V / 2; ++e) {
        o[2 * e] = __uint_as_float(t.w[e] << 16);
        o[2 * e + 1] = __uint_as_float(t.w[e] & 0xffff0000u);
    }
}
template <int V>
__device__ __forceinline__ void store_cols(float *p, const float (&o)[V]) {
    struct __attribute__((packed, aligned(4))) cols {
        float v[V];
    };
    cols t;
#pragma unroll
    for (int e = 0; e < V; ++e) t.v[e] = o[e];
    *reinterpret_cast<cols *>(p) = t;
}

// One column.
template <int BLOCK, int ITEMS, bool BATCHED, typename VT>
__global__ __launch_bounds__(BLOCK) void merge_spmm_consume(
    int32_t rows, int32_t nnz, int32_t T, const int32_t *__restrict__ ro, const int32_t *__restrict__ ci,
    const VT *__restrict__ val, const VT *__restrict__ X, int64_t ldx, float *__restrict__ Y, int64_t ldy,
    const int32_t *__restrict__ part_i, const int32_t *__restrict__ part_j, int32_t *__restrict__ carry_row,
    float *__restrict__ carry_val, const int32_t *__restrict__ part_mat, const int64_t *__restrict__ nnz_base,
    const int64_t *__restrict__ col_base) {
    constexpr int W = BLOCK * ITEMS;
    __shared__ float s_buf[W];  // row ends (int) [0, nrows), then products
    __shared__ seg_t s_wave[BLOCK / kWave];

    const int tid = threadIdx.x;
    // XCD-aware order for the persistent launch: blocks are dealt round-robin
    // to the 8 XCDs (block b runs on XCD b % 8), so XCD x takes the contiguous
    // eighth [x * per, (x + 1) * per) of the units and its L2 holds only the
    // X rows of its own matrices.  Without BATCHED: one unit per block.
    int32_t u, u_end, u_step;
    if constexpr (BATCHED) {
        const int32_t per = (T + kXcds - 1) / kXcds;
        const int32_t xcd = blockIdx.x % kXcds;
        u = xcd * per + blockIdx.x / kXcds;
        u_end = (xcd + 1) * per < T ? (xcd + 1) * per : T;
        u_step = gridDim.x / kXcds;  // the grid is a multiple of kXcds
    } else {
        u = blockIdx.x, u_end = T, u_step = gridDim.x;
    }
    for (; u < u_end; u += u_step) {
        const int32_t i0 = part_i[u], j0 = part_j[u], i1 = part_i[u + 1], j1 = part_j[u + 1];
        const int32_t nrows = i1 - i0, nnzs = j1 - j0;
        int32_t *s_re = reinterpret_cast<int32_t *>(s_buf);
        float *s_pv = s_buf + nrows;

        int32_t mat_lo = 0, mat_hi = 0;
        if constexpr (BATCHED) mat_lo = part_mat[u], mat_hi = part_mat[u + 1];

        // unconditional loads with indices clamped into the unit
        const int32_t re_last = i1 > i0 ? i1 : i0 + 1 <= rows ? i0 + 1 : rows;
        const int32_t nz_last = nnzs > 0 ? j1 - 1 : (j0 < nnz ? j0 : nnz - 1);
        int32_t re[ITEMS], xrow[ITEMS];  // xrow: X row of the nonzero (the batch's total columns fit int32)
        VT vv[ITEMS];
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            const int32_t rk = i0 + 1 + tid + q * BLOCK;
            const int32_t jk = j0 + tid + q * BLOCK;
            re[q] = ro[rk < re_last ? rk : re_last];
            xrow[q] = ld_stream(ci + (jk < nz_last ? jk : nz_last));
            vv[q] = ld_stream(val + (jk < nz_last ? jk : nz_last));
        }
        if constexpr (BATCHED) {
            if (mat_lo == mat_hi) {
                const int32_t cb = static_cast<int32_t>(col_base[mat_lo]);
#pragma unroll
                for (int q = 0; q < ITEMS; ++q) xrow[q] += cb;
            } else {
#pragma unroll
                for (int q = 0; q < ITEMS; ++q) {
                    const int32_t jk = j0 + tid + q * BLOCK;
                    const int64_t j = jk < nz_last ? jk : nz_last;
                    int32_t lo = mat_lo, hi = mat_hi;  // nnz_base[mat_lo] <= j
                    while (lo < hi) {
                        const int32_t mid = (lo + hi + 1) >> 1;
                        if (nnz_base[mid] <= j)
                            lo = mid;
                        else
                            hi = mid - 1;
                    }
                    xrow[q] += static_cast<int32_t>(col_base[lo]);
                }
            }
        }
        float g[ITEMS];
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) g[q] = to_f32(X[static_cast<int64_t>(xrow[q]) * ldx]);
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            const int k = tid + q * BLOCK;
            if (k < nrows) s_re[k] = re[q] - j0;
            if (k < nnzs) s_pv[k] = to_f32(vv[q]) * g[q];
        }
        __syncthreads();

        const int32_t total = nrows + nnzs;
        const int32_t d = tid * ITEMS < total ? tid * ITEMS : total;
        const int32_t dend = d + ITEMS < total ? d + ITEMS : total;
        int32_t lo = d - nnzs > 0 ? d - nnzs : 0;
        int32_t hi = d < nrows ? d : nrows;
        while (lo < hi) {
            const int32_t mid = (lo + hi) >> 1;
            if (s_re[mid] + mid < d)
                lo = mid + 1;
            else
                hi = mid;
        }
        int32_t it = lo, jt = d - lo;

        float acc = 0.f, first_sum = 0.f;
        int32_t first = -1;
        for (int32_t q = d; q < dend; ++q) {
            if (it < nrows && s_re[it] <= jt) {
                if (first < 0) {
                    first = it;
                    first_sum = acc;
                } else {
                    Y[static_cast<int64_t>(i0 + it) * ldy] = acc;
                }
                acc = 0.f;
                ++it;
            } else {
                acc += s_pv[jt];
                ++jt;
            }
        }

        seg_t tot;
        const seg_t in = block_seg_scan_excl<BLOCK>(seg_t{acc, first >= 0}, s_wave, tot);
        if (first >= 0) Y[static_cast<int64_t>(i0 + first) * ldy] = first_sum + in.v;
        if (tid == 0) {
            carry_row[u] = i1;
            carry_val[u] = tot.v;
        }
        // the scan ended with a barrier: LDS is free for the next unit
    }
}

// More than one column.  A group of 2^lg lanes owns (ITEMS << lg) consecutive
// merge items of the unit, each lane V neighbouring columns of them (16 bytes
// of X: 4 float or 8 BF16; 4 or 2 columns where k is smaller), so one load
// instruction of a wavefront fetches 64 >> lg whole X rows.  Lane l's columns
// start at min(l * V, kc - V): where kc is no multiple of V the last lanes
// overlap, load nothing past the row and store equal values twice.
// kAhead rows of X are in flight per lane, whatever row boundaries lie between
// them (the group's nonzeros are one range of the unit's).
// Bound: the X rows.  k = 32, 500,003 power-law rows, 11.7M nonzeros: 240 us,
// 6.2 TB/s of 128-byte X rows (885 us as four passes of eight columns, a lane
// per nonzero run, one dependent gather at a time).  k = 8, 512 matrices, 436M
// nonzeros: 3.37 ms, 0.86 L2 requests a nonzero (4.57 ms in that form); a CU's
// L1 has 256 lines, each held until its request is back, which bounds requests
// in flight (139 G nonzeros/s with X in L2, 106 with 200,000-row members).
// kAhead 2, 4 and 16: 3.86, 3.89 and 4.00 ms; k = 32: 253, 254 and 242 us.
// ONE: a lane holds the whole row (k = 2 and 4) and owns ITEMS merge items, four to
// eight, of which eight rows ahead would load most twice: four are in flight.
// 500,000 rows of 9, k = 2 42.8 us, 55.9 with eight (units of 256 x 4 there); BF16,
// k = 4 42.6 and 56.8.  BF16, k = 8: two lanes of four columns 62.2 us, one of eight
// 76.8.
constexpr int kAhead = 8;
constexpr int kAheadOne = 4;

template <int BLOCK, int ITEMS, int V, bool ONE, bool BATCHED, typename VT>
__global__ __launch_bounds__(BLOCK) void merge_spmm_rows(
    int32_t rows, int32_t nnz, int32_t T, int32_t kc, int lg, const int32_t *__restrict__ ro,
    const int32_t *__restrict__ ci, const VT *__restrict__ val, const VT *__restrict__ X, int64_t ldx,
    float *__restrict__ Y, int64_t ldy, const int32_t *__restrict__ part_i, const int32_t *__restrict__ part_j,
    int32_t *__restrict__ carry_row, float *__restrict__ carry_val, const int32_t *__restrict__ part_mat,
    const int64_t *__restrict__ nnz_base, const int64_t *__restrict__ col_base) {
    constexpr int W = BLOCK * ITEMS;
    constexpr int NW = BLOCK / kWave;
    constexpr int AHEAD = ONE ? kAheadOne : kAhead;
    __shared__ int32_t s_buf[W];  // row ends [0, nrows), then X rows of the nonzeros [nrows, nrows + nnzs)
    __shared__ float s_val[W];
    __shared__ float s_wv[NW * kMaxCols];
    __shared__ int s_wf[NW];

    const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
    const int lpn = 1 << lg;
    const int sub = tid & (lpn - 1);  // the lane's place in its group
    const int32_t c0 = sub * V < kc - V ? sub * V : kc - V;
    int32_t u, u_end, u_step;
    if constexpr (BATCHED) {
        const int32_t per = (T + kXcds - 1) / kXcds;
        const int32_t xcd = blockIdx.x % kXcds;
        u = xcd * per + blockIdx.x / kXcds;
        u_end = (xcd + 1) * per < T ? (xcd + 1) * per : T;
        u_step = gridDim.x / kXcds;
    } else {
        u = blockIdx.x, u_end = T, u_step = gridDim.x;
    }
    for (; u < u_end; u += u_step) {
        const int32_t i0 = part_i[u], j0 = part_j[u], i1 = part_i[u + 1], j1 = part_j[u + 1];
        const int32_t nrows = i1 - i0, nnzs = j1 - j0;
        int32_t *s_re = s_buf;
        int32_t *s_xr = s_buf + nrows;
        int32_t mat_lo = 0, mat_hi = 0;
        if constexpr (BATCHED) mat_lo = part_mat[u], mat_hi = part_mat[u + 1];

        const int32_t re_last = i1 > i0 ? i1 : i0 + 1 <= rows ? i0 + 1 : rows;
        const int32_t nz_last = nnzs > 0 ? j1 - 1 : (j0 < nnz ? j0 : nnz - 1);
        int32_t re[ITEMS], cc[ITEMS];
        VT vv[ITEMS];
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            const int32_t k = tid + q * BLOCK;
            const int32_t rk = i0 + 1 + k;
            const int32_t jk = j0 + k;
            re[q] = ro[rk < re_last ? rk : re_last];
            cc[q] = ld_stream(ci + (jk < nz_last ? jk : nz_last));
            vv[q] = ld_stream(val + (jk < nz_last ? jk : nz_last));
        }
        if constexpr (BATCHED) {
            if (mat_lo == mat_hi) {
                const int32_t cb = static_cast<int32_t>(col_base[mat_lo]);
#pragma unroll
                for (int q = 0; q < ITEMS; ++q) cc[q] += cb;
            } else {
#pragma unroll
                for (int q = 0; q < ITEMS; ++q) {
                    const int32_t jk = j0 + tid + q * BLOCK;
                    const int64_t j = jk < nz_last ? jk : nz_last;
                    int32_t lo = mat_lo, hi = mat_hi;  // nnz_base[mat_lo] <= j
                    while (lo < hi) {
                        const int32_t mid = (lo + hi + 1) >> 1;
                        if (nnz_base[mid] <= j)
                            lo = mid;
                        else
                            hi = mid - 1;
                    }
                    cc[q] += static_cast<int32_t>(col_base[lo]);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            const int k = tid + q * BLOCK;
            if (k < nrows) s_re[k] = re[q] - j0;
            if (k < nnzs) {
                s_xr[k] = cc[q];
                s_val[k] = to_f32(vv[q]);
            }
        }
        __syncthreads();

        // the split at both ends of the group's items
        const int32_t total = nrows + nnzs;
        const int32_t per = ITEMS << lg;
        const int32_t d = (tid >> lg) * per < total ? (tid >> lg) * per : total;
        const int32_t dend = d + per < total ? d + per : total;
        int32_t lo = d - nnzs > 0 ? d - nnzs : 0, hi = d < nrows ? d : nrows;
        int32_t lo1 = dend - nnzs > 0 ? dend - nnzs : 0, hi1 = dend < nrows ? dend : nrows;
        while (lo < hi || lo1 < hi1) {
            const int32_t mid = (lo + hi) >> 1, mid1 = (lo1 + hi1) >> 1;
            if (lo < hi) {
                if (s_re[mid] + mid < d)
                    lo = mid + 1;
                else
                    hi = mid;
            }
            if (lo1 < hi1) {
                if (s_re[mid1] + mid1 < dend)
                    lo1 = mid1 + 1;
                else
                    hi1 = mid1;
            }
        }
        const int32_t it0 = lo, it1 = lo1, jt1 = dend - lo1;

        // a row's products are summed in fours (part, half), the pairs of fours in
        // acc: a group's chain is otherwise ITEMS << lg additions long and rounds worse
        float acc[V], part[V], half[V], first_sum[V];
#pragma unroll
        for (int c = 0; c < V; ++c) acc[c] = part[c] = half[c] = first_sum[c] = 0.f;
        int32_t it = it0;
        auto fold = [&]() {
#pragma unroll
            for (int c = 0; c < V; ++c) {
                acc[c] += half[c] + part[c];
                half[c] = part[c] = 0.f;
            }
        };
        auto close_row = [&]() {
            if (it == it0) {  // waits for the earlier groups' part
#pragma unroll
                for (int c = 0; c < V; ++c) first_sum[c] = acc[c];
            } else {
                store_cols<V>(Y + static_cast<int64_t>(i0 + it) * ldy + c0, acc);
            }
#pragma unroll
            for (int c = 0; c < V; ++c) acc[c] = 0.f;
            ++it;
        };
        int32_t end = it < it1 ? s_re[it] : INT32_MAX;  // the nonzero before which row it closes
        const VT *xc = X + c0;
        for (int32_t j = d - lo; j < jt1; j += AHEAD) {
            float g[AHEAD][V], v[AHEAD];
#pragma unroll
            for (int a = 0; a < AHEAD; ++a) {
                const int32_t ja = j + a < jt1 ? j + a : jt1 - 1;
                v[a] = s_val[ja];
                load_cols<V>(xc + static_cast<int64_t>(s_xr[ja]) * ldx, g[a]);
            }
#pragma unroll
            for (int a = 0; a < AHEAD; ++a) {
                if (a == AHEAD / 2) {
#pragma unroll
                    for (int c = 0; c < V; ++c) {
                        half[c] = part[c];
                        part[c] = 0.f;
                    }
                }
                if (j + a < jt1) {
                    while (end <= j + a) {
                        fold();
                        close_row();
                        end = it < it1 ? s_re[it] : INT32_MAX;
                    }
#pragma unroll
                    for (int c = 0; c < V; ++c) part[c] += v[a] * g[a][c];
                }
            }
            fold();
        }
        while (it < it1) close_row();

        // segmented scan of the groups' trailing sums: over the wavefront's
        // groups, then over the wavefronts through LDS (seg_t's operator)
        float inc[V];
        int f = it1 > it0;
#pragma unroll
        for (int c = 0; c < V; ++c) inc[c] = acc[c];
        for (int off = lpn; off < kWave; off <<= 1) {
            const int pf = __shfl_up(f, off, kWave);
#pragma unroll
            for (int c = 0; c < V; ++c) {
                const float pv = __shfl_up(inc[c], off, kWave);
                if (lane >= off) inc[c] = f ? inc[c] : pv + inc[c];
            }
            if (lane >= off) f |= pf;
        }
        if (lane >= kWave - lpn) {
            s_wf[w] = f;
#pragma unroll
            for (int c = 0; c < V; ++c) s_wv[w * kMaxCols + sub * V + c] = inc[c];
        }
        __syncthreads();
        float pre[V], all[V];
#pragma unroll
        for (int c = 0; c < V; ++c) pre[c] = all[c] = 0.f;
#pragma unroll
        for (int q = 0; q < NW; ++q) {
            const int fq = s_wf[q];
#pragma unroll
            for (int c = 0; c < V; ++c) {
                const float vq = s_wv[q * kMaxCols + sub * V + c];
                if (q < w) pre[c] = fq ? vq : pre[c] + vq;
                all[c] = fq ? vq : all[c] + vq;
            }
        }
        const int ef = __shfl_up(f, lpn, kWave);
        float in[V];
#pragma unroll
        for (int c = 0; c < V; ++c) {
            const float ev = __shfl_up(inc[c], lpn, kWave);
            in[c] = first_sum[c] + (lane >= lpn ? (ef ? ev : pre[c] + ev) : pre[c]);
        }
        if (it1 > it0) store_cols<V>(Y + static_cast<int64_t>(i0 + it0) * ldy + c0, in);
        if (tid < lpn) {
            if (tid == 0) carry_row[u] = i1;
            store_cols<V>(carry_val + static_cast<int64_t>(u) * kc + c0, all);
        }
        __syncthreads();  // LDS is free for the next unit
    }
}

// Resident blocks (CUs x occupancy) for the persistent launch.
template <typename K>
static int resident_grid(K kernel, int block) {
    int dev = 0, cus = 256, per_cu = 1;
    if (hipGetDevice(&dev) == hipSuccess) {
        (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block, 0);
    }
    return cus * (per_cu > 0 ? per_cu : 1);
}

struct spmm_problem {
    int32_t rows, nnz;
    const int32_t *ro, *ci;
    const void *val;
    int32_t count;
    const int64_t *row_base, *nnz_base, *col_base;
};

// Persistent grid for the batched form (a multiple of kXcds, at most the
// resident blocks), else a block per unit.
template <bool BATCHED, typename K>
static uint32_t spmm_grid(K kern, int block, int64_t T) {
    if (!BATCHED) return static_cast<uint32_t>(T);
    const int resident = resident_grid(kern, block);
    const int64_t per = (T + kXcds - 1) / kXcds;
    const int64_t slots = per < resident / kXcds ? per : resident / kXcds;
    return static_cast<uint32_t>(kXcds * (slots > 0 ? slots : 1));
}

template <int BLOCK, int ITEMS, int V, bool BATCHED, typename VT>
static hipError_t spmm_rows_launch(const spmm_problem &P, const merge_ws &w, const int32_t *part_mat, int64_t T,
                                   const VT *X, int32_t kc, int64_t ldx, float *Y, int64_t ldy, hipStream_t s) {
    int lg = 0;
    while ((V << lg) < kc) ++lg;
    auto kern = merge_spmm_rows<BLOCK, ITEMS, V, false, BATCHED, VT>;
    if constexpr (V <= 4) {
        if (lg == 0) kern = merge_spmm_rows<BLOCK, ITEMS, V, true, BATCHED, VT>;
    }
    prof_scope p(s, BATCHED ? "batched_consume" : "merge_consume");
    hipLaunchKernelGGL(kern, dim3(spmm_grid<BATCHED>(kern, BLOCK, T)), dim3(BLOCK), 0, s, P.rows, P.nnz,
                       static_cast<int32_t>(T), kc, lg, P.ro, P.ci, static_cast<const VT *>(P.val), X, ldx, Y, ldy,
                       w.part_i, w.part_j, w.carry_row, w.carry_val, part_mat, P.nnz_base, P.col_base);
    return hipGetLastError();
}

// One pass over kc columns: the consume, then the carry fix-up.
template <int BLOCK, int ITEMS, bool BATCHED, typename VT>
static hipError_t spmm_pass(const spmm_problem &P, const merge_ws &w, const int32_t *part_mat, int64_t T, const VT *X,
                            int32_t kc, int64_t ldx, float *Y, int64_t ldy, hipStream_t s) {
    hipError_t e;
    if (kc == 1) {
        auto kern = merge_spmm_consume<BLOCK, ITEMS, BATCHED, VT>;
        prof_scope p(s, BATCHED ? "batched_consume" : "merge_consume");
        hipLaunchKernelGGL(kern, dim3(spmm_grid<BATCHED>(kern, BLOCK, T)), dim3(BLOCK), 0, s, P.rows, P.nnz,
                           static_cast<int32_t>(T), P.ro, P.ci, static_cast<const VT *>(P.val), X, ldx, Y, ldy,
                           w.part_i, w.part_j, w.carry_row, w.carry_val, part_mat, P.nnz_base, P.col_base);
        e = hipGetLastError();
    } else {
        switch (spmm_lane_cols(kc, sizeof(VT) == 2)) {
            case 2: e = spmm_rows_launch<BLOCK, ITEMS, 2, BATCHED, VT>(P, w, part_mat, T, X, kc, ldx, Y, ldy, s); break;
            case 4: e = spmm_rows_launch<BLOCK, ITEMS, 4, BATCHED, VT>(P, w, part_mat, T, X, kc, ldx, Y, ldy, s); break;
            default:
                e = spmm_rows_launch<BLOCK, ITEMS, (sizeof(VT) == 2 ? 8 : 4), BATCHED, VT>(P, w, part_mat, T, X, kc, ldx,
                                                                                          Y, ldy, s);
        }
    }
    if (e != hipSuccess) return e;
    return launch_fixup(T, P.rows, kc, w.carry_row, w.carry_val, Y, ldy, s, BATCHED ? "batched_fixup" : "merge_fixup");
}

// One split launch, then passes of at most kc_max columns (the carries that
// the workspace holds).
template <int BLOCK, int ITEMS, bool BATCHED, typename VT>
static hipError_t run_spmm(const spmm_problem &P, const VT *X, int32_t k, int64_t ldx, float *Y, int64_t ldy, void *ws,
                           int32_t kc_max, hipStream_t s) {
    constexpr int W = BLOCK * ITEMS;
    const int64_t T = merge_units(P.rows, P.nnz, W);
    const merge_ws w = merge_ws_carve(ws, T);
    // batched: the matrix of every unit boundary, after the carries
    int32_t *part_mat =
        BATCHED ? reinterpret_cast<int32_t *>(static_cast<char *>(ws) + merge_ws_bytes(T, kc_max)) : nullptr;
    hipError_t e = merge_partition(P.ro, P.rows, P.nnz, W, static_cast<int32_t>(T), w.part_i, w.part_j, s,
                                   BATCHED ? P.row_base : nullptr, P.count, part_mat);
    for (int32_t c0 = 0; c0 < k && e == hipSuccess; c0 += kc_max) {
        const int32_t kc = k - c0 < kc_max ? k - c0 : kc_max;
        e = spmm_pass<BLOCK, ITEMS, BATCHED, VT>(P, w, part_mat, T, X + c0, kc, ldx, Y + c0, ldy, s);
    }
    return e;
}

template <bool BATCHED>
static hipError_t dispatch(const spmm_problem &P, lb_dtype_t dt, const void *X, int32_t k, int64_t ldx, float *Y,
                           int64_t ldy, int block, int items, void *ws, int32_t kc_max, hipStream_t s) {
#define X_(B, I)                                                                                                  \
    if (block == B && items == I) {                                                                               \
        if (dt == LB_BF16)                                                                                        \
            return run_spmm<B, I, BATCHED, bf16_bits>(P, static_cast<const bf16_bits *>(X), k, ldx, Y, ldy, ws, kc_max, s); \
        return run_spmm<B, I, BATCHED, float>(P, static_cast<const float *>(X), k, ldx, Y, ldy, ws, kc_max, s);   \
    }
    LB_MERGE_CONFIGS(X_)
#undef X_
    return hipErrorInvalidValue;
}

hipError_t merge_spmm(const csr_dev &A, const void *X, int32_t k, int64_t ldx, float *Y, int64_t ldy, int block,
                      int items, void *ws, int32_t kc_max, hipStream_t s) {
    const spmm_problem P{A.rows, A.nnz, A.ro, A.ci, A.val, 0, nullptr, nullptr, nullptr};
    return dispatch<false>(P, A.dt, X, k, ldx, Y, ldy, block, items, ws, kc_max, s);
}

size_t batched_ws_bytes(const batch_dev &B, int block, int items, int kc) {
    const int64_t T = merge_units(B.total_rows, B.total_nnz, static_cast<int64_t>(block) * items);
    return merge_ws_bytes(T, kc) + align256(static_cast<size_t>(T + 1) * 4);
}

hipError_t batched_spmm(const batch_dev &B, const void *X, int32_t k, float *Y, int block, int items, void *ws,
                        int32_t kc_max, hipStream_t s) {
    const spmm_problem P{B.total_rows, B.total_nnz, B.ro, B.ci, B.val, B.count, B.row_base, B.nnz_base, B.col_base};
    return dispatch<true>(P, B.dt, X, k, static_cast<int64_t>(k), Y, static_cast<int64_t>(k), block, items, ws, kc_max,
                          s);
}

}  // namespace lbk
