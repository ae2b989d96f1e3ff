// The scatter out[c] += sum of products with column c, for gfx950, without a
// global atomic per nonzero.
//
// The backward's dx = A^T dy and the CSC product both add one product per
// nonzero into a scattered target.  As global float atomics they run at the
// L2's rate for scattered atomics, about 21 G/s.  Here the products of a unit
// are sorted by target range and each range is summed in LDS:
//   1. bin_products: a block per merge-path unit of kBinW items labels its
//                    nonzeros with their rows (the backward's walk), forms the
//                    products (and dvalues), sorts them by bin (kBinCols
//                    targets) in LDS and writes them to the unit's own stretch
//                    of the product array: the product and its target within
//                    the bin (16 bits), 6 bytes a nonzero, and the start of
//                    every bin's run.  A unit whose columns lie within kBinW of
//                    each other (a stencil's) is summed in LDS at once, and its
//                    window of targets added to out;
//   2. bin_sum:      a block per bin and range of units adds the units' runs of
//                    its bin into float64 sums of the bin's targets in LDS and
//                    adds those to out (one coalesced
//                    float atomic per target and range of units).
// The sums are float64 so that a target with thousands of terms (a capped row
// of a power-law matrix in the CSC product) loses little to their order: terms
// that lanes of a wavefront share are added in float32 first (at most six
// additions deep, 6 * 2^-24 of their absolute sum), and so are the results of
// the blocks that hold parts of a target.
// Bytes a nonzero: 8 read, 6 written and 6 read, all streams, in place of one
// scattered atomic.  (With the bins whole in memory, each unit's run of a bin
// placed after the last unit's, a counting pass over the columns came first:
// 30 us for 30.8M nonzeros, and the runs' partial lines cost another 10.)
#include "lb_device.h"
#include "lb_internal.h"

namespace lbk {
using namespace lb;

namespace {

constexpr int kBinBlock = 512;
constexpr int kBinItems = 8;
constexpr int kBinW = kBinBlock * kBinItems;
constexpr int kSumBlock = 1024;
constexpr int kSumWaves = kSumBlock / kWave;
constexpr int kBinShift = 13;
constexpr int kBinCols = 1 << kBinShift;  // targets per bin: 64 KB of float64 sums, two blocks a CU
constexpr int kBinMax = 512;              // bins (kBinBlock counters)
constexpr int kBinRuns = 16;    // runs of equal bins in a wavefront up to which they are counted whole
constexpr int kBinShared = 8;   // lanes with one target from which they are summed before LDS
constexpr int kRangeMax = 512;  // units of a bin_sum block at most: what a bin that takes all nonzeros leaves to one
static_assert(kBinMax <= kBinBlock && kRangeMax <= kSumBlock, "one thread per bin, one lane per unit of a range");

struct bin_ws {
    int32_t *part_i, *part_j;  // the split at every unit boundary, T + 1 each
    int32_t *start;            // [unit][bin]: first entry of the bin's run in the unit; nb + 1 each
    float *prod;               // products, each unit's in bin order
    uint16_t *key;             // their targets within the bin
};

size_t bin_carve(void *base, int64_t n, int64_t T, int64_t nnz, bin_ws *w) {
    const int64_t nb = (n + kBinCols - 1) >> kBinShift;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        char *p = static_cast<char *>(base) + o;
        o += align256(bytes);
        return p;
    };
    bin_ws v{};
    v.part_i = reinterpret_cast<int32_t *>(take(static_cast<size_t>(T + 1) * 4));
    v.part_j = reinterpret_cast<int32_t *>(take(static_cast<size_t>(T + 1) * 4));
    v.start = reinterpret_cast<int32_t *>(take(static_cast<size_t>((nb + 1) * T) * 4));
    v.prod = reinterpret_cast<float *>(take(static_cast<size_t>(nnz) * 4));
    v.key = reinterpret_cast<uint16_t *>(take(static_cast<size_t>(nnz) * 2));
    if (w) *w = v;
    return o;
}

// Units of a bin_sum block, a multiple of its wavefronts: about 1024 blocks where
// there are units enough.
int32_t bin_range(int64_t T, int64_t nb) {
    const int64_t r = T * nb / 1024 / kSumWaves * kSumWaves;
    return static_cast<int32_t>(r < kSumWaves ? kSumWaves : (r < kRangeMax ? r : kRangeMax));
}

// Counts one entry per lane in cnt[bin] (LDS; bin < 0: none) and returns its
// place among the counted ones.  Sorted columns of a long row put runs of
// neighbouring lanes in one bin, which then queue on its counter: with few runs
// the first lane of each counts for all of it (counting a power-law matrix's
// columns took 101 us lane by lane, 30 so).
__device__ __forceinline__ int32_t bin_add(int32_t *cnt, int32_t bin) {
    const int lane = lane_id();
    // the lane before (wave_shr:1), -2 for lane 0
    const int32_t prev = __builtin_amdgcn_update_dpp(-2, bin, 0x138, 0xF, 0xF, false);
    const uint64_t heads = __ballot(prev != bin);
    if (__popcll(heads) > kBinRuns) return bin >= 0 ? atomicAdd(cnt + bin, 1) : 0;  // uniform
    const uint64_t upto = heads & ((2ull << lane) - 1), later = heads & ~((2ull << lane) - 1);
    const int first = kWave - 1 - __clzll(static_cast<long long>(upto));
    const int end = later ? __ffsll(static_cast<unsigned long long>(later)) - 1 : kWave;
    int32_t at = 0;
    if (lane == first && bin >= 0) at = atomicAdd(cnt + bin, end - first);
    return __shfl(at, first) + lane - first;
}

template <typename VT, bool WANT_DV>
__global__ __launch_bounds__(kBinBlock) void bin_products(
    int32_t rows, int32_t nnz, int32_t nb, const int32_t *__restrict__ ro, const int32_t *__restrict__ ci, const VT *__restrict__ val, const VT *__restrict__ x,
    const float *__restrict__ dy, float *__restrict__ dvalues, const int32_t *__restrict__ part_i,
    const int32_t *__restrict__ part_j, int32_t *__restrict__ start, float *__restrict__ prod,
    uint16_t *__restrict__ key, float *__restrict__ out, bool windows) {
    // row ends and row labels, then the products in bin order; columns in bin
    // order.  In their place: the float64 sums of a window
    __shared__ double s_win[kBinW];
    int32_t *s_buf = reinterpret_cast<int32_t *>(s_win);
    int32_t *s_col = s_buf + kBinW;
    __shared__ int32_t s_cnt[kBinMax], s_start[kBinMax];
    __shared__ int32_t s_wave[kBinBlock / kWave];
    __shared__ int32_t s_lo[kBinBlock / kWave], s_hi[kBinBlock / kWave];

    const int tid = threadIdx.x;
    const int32_t b = blockIdx.x;
    if (tid < nb) s_cnt[tid] = 0;
    const int32_t i0 = part_i[b], j0 = part_j[b];
    const int32_t i1 = part_i[b + 1], j1 = part_j[b + 1];
    const int32_t nrows = i1 - i0, nnzs = j1 - j0;
    int32_t *s_re = s_buf;
    int32_t *s_row = s_buf + nrows;
    // unconditional loads with indices clamped into the unit (see k_merge.hip)
    const int32_t *ro_u = ro + (i0 + 1 < rows ? i0 + 1 : rows);
    const int32_t jb = j0 < nnz ? j0 : nnz - 1;
    const int32_t *ci_u = ci + jb;
    const VT *val_u = val + jb;
    const uint32_t re_last = nrows > 0 ? nrows - 1 : 0, nz_last = nnzs > 0 ? nnzs - 1 : 0;
    int32_t cc[kBinItems];
    VT vv[kBinItems];
    {
        int32_t re[kBinItems];
#pragma unroll
        for (int u = 0; u < kBinItems; ++u) {
            const uint32_t k = tid + u * kBinBlock;
            re[u] = *at_off(ro_u, k < re_last ? k : re_last);
            cc[u] = ld_stream(at_off(ci_u, k < nz_last ? k : nz_last));
            vv[u] = ld_stream(at_off(val_u, k < nz_last ? k : nz_last));
        }
#pragma unroll
        for (int u = 0; u < kBinItems; ++u) {
            const int k = tid + u * kBinBlock;
            if (k < nrows) s_re[k] = re[u] - j0;
        }
    }
    // the range of the unit's columns
    int32_t cmin = INT32_MAX, cmax = -1;
    if (windows) {  // uniform
#pragma unroll
        for (int u = 0; u < kBinItems; ++u) {
            if (tid + u * kBinBlock < nnzs) {
                cmin = cc[u] < cmin ? cc[u] : cmin;
                cmax = cc[u] > cmax ? cc[u] : cmax;
            }
        }
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) {
            const int32_t l = __shfl_xor(cmin, off), h = __shfl_xor(cmax, off);
            cmin = l < cmin ? l : cmin;
            cmax = h > cmax ? h : cmax;
        }
        if (lane_id() == 0) s_lo[wave_id()] = cmin, s_hi[wave_id()] = cmax;
    }
    __syncthreads();
    if (windows) {
#pragma unroll
        for (int w = 0; w < kBinBlock / kWave; ++w) {
            cmin = s_lo[w] < cmin ? s_lo[w] : cmin;
            cmax = s_hi[w] > cmax ? s_hi[w] : cmax;
        }
    }
    const bool window = windows && cmax >= cmin && cmax - cmin < kBinW;  // uniform

    // the entry's place among the unit's entries of its bin (any order)
    int32_t rank[kBinItems];
#pragma unroll
    for (int u = 0; u < kBinItems; ++u) {
        const int k = tid + u * kBinBlock;
        rank[u] = window ? 0 : bin_add(s_cnt, k < nnzs ? cc[u] >> kBinShift : -1);
    }
    // label every nonzero with its row
    const int32_t all = nrows + nnzs;
    const int32_t d = tid * kBinItems < all ? tid * kBinItems : all;
    const int32_t dend = d + kBinItems < all ? d + kBinItems : all;
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
    for (int32_t q = d; q < dend; ++q) {
        if (it < nrows && s_re[it] <= jt)
            ++it;
        else
            s_row[jt++] = it;
    }
    __syncthreads();

    const float *dy_u = dy + i0;
    const uint32_t row_last = rows - 1 - i0 < nrows ? rows - 1 - i0 : nrows;  // i0 < rows where nnzs > 0
    float pr[kBinItems];
    {
        float g[kBinItems], xv[kBinItems];
#pragma unroll
        for (int u = 0; u < kBinItems; ++u) {
            const int k = tid + u * kBinBlock;
            // labels exist for k < nnzs; other lanes read a valid row and discard it
            const uint32_t lab = nnzs > 0 ? s_row[k < nnzs ? k : nnzs - 1] : 0;
            g[u] = nnzs > 0 ? *at_off(dy_u, lab < row_last ? lab : row_last) : 0.f;
            if constexpr (WANT_DV) xv[u] = to_f32(x[cc[u]]);
        }
#pragma unroll
        for (int u = 0; u < kBinItems; ++u) {
            const uint32_t k = tid + u * kBinBlock;
            pr[u] = to_f32(vv[u]) * g[u];
            if constexpr (WANT_DV) {
                if (static_cast<int32_t>(k) < nnzs) *at_off(dvalues + j0, k) = g[u] * xv[u];
            }
        }
    }
    if (window) {  // sum them here
        __syncthreads();  // the labels have been read
        const int32_t width = cmax - cmin + 1;
        for (int32_t c = tid; c < width; c += kBinBlock) s_win[c] = 0.0;
        if (tid < nb) start[static_cast<int64_t>(b) * (nb + 1) + tid] = 0;
        if (tid == 0) start[static_cast<int64_t>(b) * (nb + 1) + nb] = 0;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kBinItems; ++u)
            if (tid + u * kBinBlock < nnzs) unsafeAtomicAdd(s_win + (cc[u] - cmin), static_cast<double>(pr[u]));
        __syncthreads();
        for (int32_t c = tid; c < width; c += kBinBlock) {
            const float v = static_cast<float>(s_win[c]);
            if (v != 0.f) unsafeAtomicAdd(out + cmin + c, v);
        }
        return;
    }
    // first place of each bin in the unit
    const int32_t cnt = tid < nb ? s_cnt[tid] : 0;
    const int32_t incl = block_scan_incl<kBinBlock>(cnt, s_wave);  // (its barriers: the labels have been read)
    if (tid < nb) {
        s_start[tid] = incl - cnt;
        start[static_cast<int64_t>(b) * (nb + 1) + tid] = incl - cnt;
        if (tid == nb - 1) start[static_cast<int64_t>(b) * (nb + 1) + nb] = nnzs;
    }
    __syncthreads();
    float *s_prod = reinterpret_cast<float *>(s_buf);
#pragma unroll
    for (int u = 0; u < kBinItems; ++u) {
        const int k = tid + u * kBinBlock;
        if (k < nnzs) {
            const int32_t p = s_start[cc[u] >> kBinShift] + rank[u];
            s_prod[p] = pr[u];
            s_col[p] = cc[u];
        }
    }
    __syncthreads();
    float *prod_u = prod + j0;
    uint16_t *key_u = key + j0;
    for (int32_t p = tid; p < nnzs; p += kBinBlock) {
        *at_off(prod_u, static_cast<uint32_t>(p)) = s_prod[p];
        *at_off(key_u, static_cast<uint32_t>(p)) = static_cast<uint16_t>(s_col[p] & (kBinCols - 1));
    }
}

// Adds v to the bin's sum k, for the lanes with `in`.  A target that many lanes
// share (a capped row in the CSC product) is summed over them first: 84 us
// against 115 for 30.8M entries of which half fall on a few targets.  In float32:
// in float64, two lane moves a step, the CSC product of a 1M-row power-law matrix
// took 233 us against 225, its error 7.8e-8 against 8.2e-8.
__device__ __forceinline__ void bin_sum_add(double *sum, float v, uint16_t k, bool in) {
    const int32_t k0 = __builtin_amdgcn_readfirstlane(k);
    const bool same = in && k == k0;
    if (__popcll(__ballot(same)) >= kBinShared) {  // uniform
        const float t = group_sum_dpp<kWave>(same ? v : 0.f);
        if (lane_id() == kWave - 1) unsafeAtomicAdd(sum + k0, static_cast<double>(t));
        in = in && !same;
    }
    if (in) unsafeAtomicAdd(sum + k, static_cast<double>(v));
}

// Block -> (bin, range of units): the blocks of one XCD take the bins of one
// range after the other, so the lines that the runs of neighbouring bins share
// are in its L2.  The grid has nb * 8 * ceil(ranges / 8) blocks.
__global__ __launch_bounds__(kSumBlock) void bin_sum(int32_t nb, int32_t n, int32_t T, int32_t range,
                                                     const int32_t *__restrict__ part_j,
                                                     const int32_t *__restrict__ start,
                                                     const float *__restrict__ prod,
                                                     const uint16_t *__restrict__ key, float *__restrict__ out) {
    __shared__ double s_sum[kBinCols];
    __shared__ int32_t s_at[kRangeMax], s_len[kRangeMax];
    const int tid = threadIdx.x, lane = lane_id();
    const int32_t i = static_cast<int32_t>(blockIdx.x / kXcds);
    const int32_t bin = i % nb;
    const int64_t u0 = (static_cast<int64_t>(i / nb) * kXcds + blockIdx.x % kXcds) * range;
    if (u0 >= T) return;  // uniform
    const int32_t units = T - u0 < range ? static_cast<int32_t>(T - u0) : range;
    int32_t len = 0;
    if (tid < units) {
        const int32_t *st = start + (u0 + tid) * (nb + 1) + bin;
        len = st[1] - st[0];
        s_at[tid] = part_j[u0 + tid] + st[0];
        s_len[tid] = len;
    }
    if (!__syncthreads_or(len)) return;  // no unit of the range has the bin (out is cleared)
    for (int c = tid; c < kBinCols; c += kSumBlock) s_sum[c] = 0.0;
    __syncthreads();
    constexpr int R = 8;  // runs, or 64-entry pieces of one, in flight per wavefront
    for (int32_t t = wave_id(); t < units; t += R * kSumWaves) {
        float v[R];
        uint16_t k[R];
        int32_t at[R], ln[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {  // uniform over the wavefront
            const int32_t q = t + r * kSumWaves;
            ln[r] = q < units ? s_len[q] : 0;
            at[r] = ln[r] > 0 ? s_at[q] : 0;  // an empty run reads entry 0 and adds nothing
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int32_t e = at[r] + (lane < ln[r] ? lane : 0);
            v[r] = prod[e];
            k[r] = key[e];
        }
#pragma unroll
        for (int r = 0; r < R; ++r) bin_sum_add(s_sum, v[r], k[r], lane < ln[r]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            for (int32_t o = kWave; o < ln[r]; o += R * kWave) {  // the rest of a long run
                float lv[R];
                uint16_t lk[R];
#pragma unroll
                for (int p = 0; p < R; ++p) {
                    const int32_t e = o + p * kWave + lane;
                    lv[p] = prod[at[r] + (e < ln[r] ? e : 0)];
                    lk[p] = key[at[r] + (e < ln[r] ? e : 0)];
                }
#pragma unroll
                for (int p = 0; p < R; ++p) bin_sum_add(s_sum, lv[p], lk[p], o + p * kWave + lane < ln[r]);
            }
        }
    }
    __syncthreads();
    const int32_t c0 = bin << kBinShift;
    for (int c = tid; c < kBinCols && c0 + c < n; c += kSumBlock) {
        const float v = static_cast<float>(s_sum[c]);
        if (v != 0.f) unsafeAtomicAdd(out + c0 + c, v);
    }
}

}  // namespace

bool bins_pay(int64_t rows, int64_t n, int64_t nnz, bool by_rows) {
    if (n > static_cast<int64_t>(kBinMax) * kBinCols || nnz < kBinMinNnz) return false;
    if (by_rows) {
        const bool dense = n <= 2 ? rows <= 4 * nnz : 4 * rows <= 3 * nnz;
        if (n <= 8 && (n == 1 ? 3 : n) * nnz <= 8000000 && dense) return false;
        if (8 * rows <= nnz) return true;
    }
    const int64_t nb = (n + kBinCols - 1) >> kBinShift, starts = (nb + 1) * merge_units(rows, nnz, kBinW);
    return (nb <= 4 ? 44 : 22) * nnz > 9 * n + 2 * rows + 30 * starts + 5800000;
}

size_t bins_ws_bytes(int64_t rows, int64_t n, int64_t nnz) {
    return bin_carve(nullptr, n, merge_units(rows, nnz, kBinW), nnz, nullptr);
}

template <typename VT>
static hipError_t run_bins(const csr_dev &A, const void *x, const float *dy, float *dx, float *dvalues, void *ws,
                           hipStream_t s) {
    const int64_t T = merge_units(A.rows, A.nnz, kBinW);
    bin_ws w;
    bin_carve(ws, A.cols, T, A.nnz, &w);
    const int32_t nb = (A.cols + kBinCols - 1) >> kBinShift;
    const int32_t t = static_cast<int32_t>(T);
    // (the split launch also clears dx)
    const hipError_t e = merge_partition(A.ro, A.rows, A.nnz, kBinW, t, w.part_i, w.part_j, s, nullptr, 0, nullptr,
                                         dx, A.cols);
    if (e != hipSuccess) return e;
    prof_scope p(s, "backward");
    // Windows where targets have few terms on average (a stencil's five): the
    // windows of a matrix with few columns would all meet on them.
    const bool windows = A.nnz <= int64_t(64) * A.cols;
    const dim3 grid(static_cast<uint32_t>(T)), block(kBinBlock);
    const VT *val = static_cast<const VT *>(A.val);
    const VT *xv = static_cast<const VT *>(x);
    if (dvalues)
        hipLaunchKernelGGL((bin_products<VT, true>), grid, block, 0, s, A.rows, A.nnz, nb, A.ro, A.ci, val, xv, dy,
                           dvalues, w.part_i, w.part_j, w.start, w.prod, w.key, dx, windows);
    else
        hipLaunchKernelGGL((bin_products<VT, false>), grid, block, 0, s, A.rows, A.nnz, nb, A.ro, A.ci, val, xv, dy,
                           dvalues, w.part_i, w.part_j, w.start, w.prod, w.key, dx, windows);
    const int32_t range = bin_range(T, nb);
    const int64_t ranges = (T + range - 1) / range;
    hipLaunchKernelGGL(bin_sum, dim3(static_cast<uint32_t>((ranges + kXcds - 1) / kXcds * kXcds * nb)), dim3(kSumBlock),
                       0, s, nb, A.cols, t, range, w.part_j, w.start, w.prod, w.key, dx);
    return hipGetLastError();
}

hipError_t binned_backward(const csr_dev &A, const void *x, const float *dy, float *dx, float *dvalues, void *ws,
                           hipStream_t s) {
    if (A.dt == LB_BF16) return run_bins<bf16_bits>(A, x, dy, dx, dvalues, ws, s);
    return run_bins<float>(A, x, dy, dx, dvalues, ws, s);
}

}  // namespace lbk
