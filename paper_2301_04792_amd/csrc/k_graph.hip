// Graph traversal written on the public schedules of lb_schedule.hpp: the
// SSSP example of Sec. 5.3 and BFS (named in Sec. 6).  A graph is a CSR
// tile set read as adjacency: vertex u's out-edges are the atoms of tile u,
// edge e goes to col_idx[e] and weighs w[e].
//
// Iteration i takes frontier F_i, a compacted list of vertex ids (the tiles
// of an indexed_tile_set), and relaxes every out-edge of its vertices under
// the chosen schedule; the vertices that improve form F_{i+1}, each listed
// once.  The host launches again while the frontier holds vertices (Sec. 5.3).
//  * SSSP: dist is float32.  The offer dist[u] + w is one float32 addition
//    and an atomic minimum on the bit pattern keeps the smaller value
//    (non-negative floats order like their int32 bit patterns).  A vertex
//    joins F_{i+1} at most once: it carries the iteration that last queued
//    it, so nothing is cleared between iterations.
//  * BFS: depth is int32, -1 = unvisited; the compare-and-swap from -1 to
//    i + 1 that succeeds claims the vertex.
// Appends are aggregated per block: the merge-path advance places a unit's
// new vertices with a block prefix sum and one 64-bit atomicAdd; the other
// schedules stage them in an LDS buffer and reserve its stretch with one
// atomicAdd per block (per round for the prefix-sum form).  Pushes past the
// buffer fall back to one atomicAdd per wavefront.
//
// An iteration is one launch, persistent (the resident grid), that reads the
// frontier size from device memory, so the host enqueues a batch of
// iterations without waiting and reads the size once per batch to stop.  (The
// merge-path advance may take several small frontiers in one launch.)
// Three rotating counters: launch i reads counter i % 3, appends to
// (i + 1) % 3 and zeroes (i + 2) % 3, the one launch i + 1 appends to (and
// launch i - 1 last read), so no memset and no host round trip is needed.
#include <math.h>

#include "lb_device.h"
#include "lb_internal.h"
#include "lb_schedule.hpp"

namespace lbk {
using namespace lb;

namespace {

constexpr int32_t kUnvisited = -1;

struct trav_args {
    const int32_t *ro;
    const int32_t *ci;
    const float *w;
    float *dist;        // SSSP
    int32_t *depth;     // BFS
    int32_t *stamp;     // SSSP: iteration that last queued each vertex
    const int32_t *q_in;
    int32_t *q_out;
    const int32_t *cnt_in;
    int32_t *cnt_out;
    int32_t *cnt_clear;
    int32_t *rounds;    // non-empty frontiers processed
    int32_t *ticket;        // work queue of this launch (LB_WORK_QUEUE)
    int32_t *ticket_clear;  // the next launch's work queue, zeroed here
    int32_t iter;
};

// Appends v for every active lane with `want`; every active lane of the
// wavefront calls it (inactive lanes take no part in the ballot).
__device__ __forceinline__ void frontier_push(bool want, int32_t v, int32_t *q_out, int32_t *cnt_out) {
    const uint64_t m = __ballot(want);
    if (m == 0) return;
    const int leader = __ffsll(static_cast<unsigned long long>(m)) - 1;
    int32_t base = 0;
    if (lane_id() == leader) base = atomicAdd(cnt_out, __popcll(m));
    base = __shfl(base, leader);
    if (want) q_out[base + __popcll(m & ((1ull << lane_id()) - 1))] = v;
}

// Block-staged appends for the thread- and group-mapped advances: a push
// takes its slot in an LDS buffer from an LDS counter (one LDS atomic per
// wavefront), and flush() reserves the buffer's stretch of the next
// frontier with one global atomic per block, then copies it out.  Pushes
// past the buffer's capacity go straight to the frontier.  One global atomic
// per wavefront and step put every wavefront of the grid on the one frontier
// counter; staging takes that counter off the critical path.
template <int CAP>
struct staged_frontier {
    int32_t *buf;  // LDS, CAP entries
    int32_t *n;    // LDS: entries pushed (may exceed CAP: the rest went straight out)
    int32_t *base; // LDS: the block's first slot in the frontier
    // every thread of the block calls it, before the first push
    __device__ void start() {
        if (threadIdx.x == 0) *n = 0;
        __syncthreads();
    }
    // every active lane of the wavefront calls it
    __device__ void push(bool want, int32_t v, int32_t *q_out, int32_t *cnt_out) {
        const uint64_t m = __ballot(want);
        if (m == 0) return;
        const int leader = __ffsll(static_cast<unsigned long long>(m)) - 1;
        int32_t pos0 = 0;
        if (lane_id() == leader) pos0 = atomicAdd(n, __popcll(m));
        pos0 = __shfl(pos0, leader);
        const int32_t pos = pos0 + __popcll(m & ((1ull << lane_id()) - 1));
        const bool spill = want && pos >= CAP;
        if (want && !spill) buf[pos] = v;
        frontier_push(spill, v, q_out, cnt_out);
    }
    // every thread of the block calls it; the buffer is empty afterwards
    __device__ void flush(int32_t *q_out, int32_t *cnt_out) {
        __syncthreads();
        const int32_t k = *n < CAP ? *n : CAP;
        if (threadIdx.x == 0) *base = k > 0 ? atomicAdd(cnt_out, k) : 0;
        __syncthreads();
        for (int32_t i = threadIdx.x; i < k; i += blockDim.x) q_out[*base + i] = buf[i];
        __syncthreads();
        if (threadIdx.x == 0) *n = 0;
        __syncthreads();
    }
};
constexpr int kStageCap = 2048;

// Relaxes edge e of a vertex whose distance is du; returns true when the
// target v must join the next frontier.
template <bool BFS>
__device__ __forceinline__ bool relax(const trav_args &t, float du, int32_t e, int32_t &v) {
    v = t.ci[e];
    if constexpr (BFS) {
        // a stale read can only show -1 for a claimed vertex: the CAS decides
        if (t.depth[v] != kUnvisited) return false;
        return atomicCAS(t.depth + v, kUnvisited, t.iter + 1) == kUnvisited;
    } else {
        const float offer = du + t.w[e];
        // distances only decrease, so a stale read is >= the current value:
        // an offer that does not beat it cannot beat the current one
        if (!(offer < t.dist[v])) return false;
        const int32_t old = atomicMin(reinterpret_cast<int32_t *>(t.dist) + v, __float_as_int(offer));
        if (!(offer < __int_as_float(old))) return false;
        return atomicExch(t.stamp + v, t.iter) != t.iter;
    }
}

__device__ __forceinline__ int32_t frontier_size(const trav_args &t) {
    const int32_t nf = *t.cnt_in;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *t.cnt_clear = 0;
        *t.ticket_clear = 0;
        if (nf > 0) *t.rounds += 1;
    }
    return nf;
}

template <bool BFS>
__device__ __forceinline__ float tile_dist(const trav_args &t, int32_t u) {
    if constexpr (BFS)
        return 0.f;
    else
        return t.dist[u];
}

template <bool BFS>
__global__ __launch_bounds__(1024) void advance_thread_kernel(trav_args t) {
    __shared__ int32_t s_buf[kStageCap];
    __shared__ int32_t s_n, s_base;
    staged_frontier<kStageCap> out{s_buf, &s_n, &s_base};
    out.start();
    const int32_t nf = frontier_size(t);
    const thread_mapped<indexed_tile_set> sch{{t.q_in, t.ro, nf}};
    for (int64_t p : sch.tiles()) {
        const tile_ref tile = sch.ts.tile(p);
        const float du = tile_dist<BFS>(t, tile.id);
        for (int64_t e : sch.atoms(tile)) {
            int32_t v;
            const bool want = relax<BFS>(t, du, static_cast<int32_t>(e), v);
            out.push(want, v, t.q_out, t.cnt_out);
        }
    }
    out.flush(t.q_out, t.cnt_out);
}

template <int G, bool BFS>
__global__ __launch_bounds__(group_block<G>::BLOCK) void advance_group_kernel(trav_args t) {
    __shared__ int32_t s_buf[kStageCap];
    __shared__ int32_t s_n, s_base;
    staged_frontier<kStageCap> out{s_buf, &s_n, &s_base};
    out.start();
    const int32_t nf = frontier_size(t);
    const group_mapped<G, indexed_tile_set> sch{{t.q_in, t.ro, nf}};
    for (int64_t p : sch.tiles()) {
        const tile_ref tile = sch.ts.tile(p);
        const float du = tile_dist<BFS>(t, tile.id);
        for (int64_t e : sch.atoms(tile)) {
            int32_t v;
            const bool want = relax<BFS>(t, du, static_cast<int32_t>(e), v);
            out.push(want, v, t.q_out, t.cnt_out);
        }
    }
    out.flush(t.q_out, t.cnt_out);
}

template <int G, bool BFS, bool QUEUE>
__global__ __launch_bounds__(group_block<G>::BLOCK) void advance_scan_kernel(trav_args t) {
    using sched = group_mapped_scan<G, indexed_tile_set>;
    __shared__ typename sched::storage st[sched::GPB];
    __shared__ int32_t s_slot;
    __shared__ int32_t s_buf[kStageCap];
    __shared__ int32_t s_n, s_base;
    staged_frontier<kStageCap> out{s_buf, &s_n, &s_base};
    out.start();
    const int32_t nf = frontier_size(t);
    sched sch(indexed_tile_set{t.q_in, t.ro, nf}, st);
    auto round_body = [&](int64_t round) {  // called by every thread of the block
        const int32_t total = sch.load(round);
        for (int64_t a : sch.atoms(total)) {
            const int32_t q = sch.get_tile(static_cast<int32_t>(a));
            const int32_t u = sch.tile(q);
            const int32_t e = sch.atom(static_cast<int32_t>(a), q);
            int32_t v;
            const bool want = relax<BFS>(t, tile_dist<BFS>(t, u), e, v);
            out.push(want, v, t.q_out, t.cnt_out);
        }
        out.flush(t.q_out, t.cnt_out);  // per round: the buffer never holds more than one round
        sch.done();
    };
    if constexpr (QUEUE) {
        const int64_t rounds = ((static_cast<int64_t>(nf) + G - 1) / G + sched::GPB - 1) / sched::GPB;
        for (int64_t round : sch.queued_rounds(t.ticket, &s_slot, claim_batch(rounds))) round_body(round);
    } else {
        for (int64_t round : sch.rounds()) round_body(round);  // uniform across the block
    }
}

// ---------------------------------------------------------------- merge-path over the frontier
//
// One launch per iteration, or several small ones.  The frontier carries its own "row offsets": the
// vertices that have out-edges are stored in slots with the exclusive prefix sum
// of their degrees, because a block reserves its new vertices' slots and edges
// with one 64-bit atomicAdd (slots in the low word, edges in the high one), so
// slot order and edge order agree.  Offsets are kept for even slots only (the
// odd one's is the even one's plus its degree), which fits both frontiers' into
// n + 1 words.  A vertex without out-edges takes no slot; it only marks the
// next frontier as non-empty.  A unit is kEdgeUnit consecutive edges of the
// frontier, whoever owns them: blocks take equal contiguous ranges of units, find
// the first slot by a search over the offsets, stage the slots of a unit in
// LDS, and each thread takes kEdgeItems edges strided by the block.  Every load
// of a kind (targets and weights, then target states, then atomics) is in flight
// for all of a thread's edges together: a walk of one edge after the other
// waited for three dependent loads each.  The earlier form's four launches per
// iteration for the offsets (degree scan in three, split) are gone.  1M-vertex
// power-law graph, 30.8M edges: BFS 576 -> 365 us, SSSP 2.48 -> 1.55 ms; a
// 200 x 200 grid, BFS in 335 iterations, 7.2 -> 3.4 ms (with kSmallIters 1.66).  512 x 4 edges: 256 x 8
// has fewer wavefronts for the LDS a unit takes (396 us, 1.64 ms), 1024 x 2 fewer
// blocks (504 us, 1.86 ms).  Bound: the random target states (24M in 180 us) and
// returning atomics, both device-wide.

constexpr int kEdgeBlock = 512;
constexpr int kEdgeItems = 4;
constexpr int kEdgeUnit = kEdgeBlock * kEdgeItems;
// slots staged: a unit overlaps at most kEdgeUnit + 1, after one of its first
// pair, and pairs are loaded kEdgeBlock at a time
constexpr int kEdgeSlots = (kEdgeUnit / 2 + 2 + kEdgeBlock - 1) / kEdgeBlock * kEdgeBlock * 2;

// New vertices a block holds before it reserves their slots: with one atomic per
// unit the blocks of a large iteration queued on the one counter (12k atomics).
constexpr int kEdgeNew = 2 * kEdgeUnit;

struct edge_args {
    const int32_t *off_in;  // offset of slot 2t at t
    int32_t *off_out;
    const unsigned long long *pk_in;  // slots | edges << 32 of the frontier
    unsigned long long *pk_out, *pk_clear;
    const int32_t *done_in;  // iterations before this launch
    int32_t *done_out;
    int32_t max_iter;
};

// A frontier of one unit of edges or less is the work of one block, which goes on
// with the next one itself, up to this many iterations a launch: it knows the next
// frontier's size, and a launch, its gap and its start cost more than the unit: a
// grid of 200 x 200, 399 iterations, BFS 3.76 ms launched one by one (9.4 us an
// iteration), 1.87 so (4.7); SSSP 4.11 and 2.22.
constexpr int32_t kSmallIters = 256;

// Inclusive prefix sum over the block of a 64-bit value; s_wave holds BLOCK/64.
template <int BLOCK>
__device__ __forceinline__ unsigned long long block_scan_incl64(unsigned long long v, unsigned long long *s_wave) {
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const unsigned long long o = __shfl_up(v, off, kWave);
        if (lane_id() >= off) v += o;
    }
    if (lane_id() == kWave - 1) s_wave[wave_id()] = v;
    __syncthreads();
    unsigned long long pre = 0;
#pragma unroll
    for (int k = 0; k < BLOCK / kWave; ++k)
        if (k < wave_id()) pre += s_wave[k];
    __syncthreads();
    return v + pre;
}

template <bool BFS>
__global__ __launch_bounds__(kEdgeBlock) void advance_merge_kernel(trav_args t, edge_args x) {
    __shared__ int32_t s_off[kEdgeSlots];   // first edge of the slot
    __shared__ int32_t s_base[kEdgeSlots];  // edge e of the frontier, in this slot, is edge s_base + e of the graph
    __shared__ float s_du[BFS ? 1 : kEdgeSlots];
    __shared__ int32_t s_new[kEdgeNew];  // vertices for the next frontier
    __shared__ unsigned long long s_wave[kEdgeBlock / kWave];
    __shared__ unsigned long long s_got, s_next;
    __shared__ int32_t s_iwave[kEdgeBlock / kWave];
    __shared__ int32_t s_pair, s_held;
    const int tid = threadIdx.x;
    const bool live = *t.cnt_in != 0;
    const unsigned long long pk = *x.pk_in;
    int32_t iter = *x.done_in;
    const bool stop = iter >= x.max_iter;  // the frontier is left as it is
    int32_t nf = static_cast<int32_t>(pk & 0xffffffffu), E = static_cast<int32_t>(pk >> 32);
    const int32_t units = stop ? 0 : E / kEdgeUnit + (E % kEdgeUnit != 0);
    const bool single = units == 1;  // the last block's, which publishes the next frontier
    if (blockIdx.x == 0 && tid == 0) {
        *t.cnt_clear = 0;
        *x.pk_clear = 0;
        if (!single) *x.done_out = iter + (live && !stop);
        if (stop) *t.cnt_out = live;
    }
    // contiguous ranges of units: block b takes [b * units / grid, (b + 1) * units / grid)
    const int32_t u0 = static_cast<int32_t>(static_cast<int64_t>(blockIdx.x) * units / gridDim.x);
    const int32_t u1 = static_cast<int32_t>(static_cast<int64_t>(blockIdx.x + 1) * units / gridDim.x);
    if (u0 >= u1) return;  // uniform
    if (single) {
        if (tid == 0) s_pair = 0;
    } else if (wave_id() == 0) {  // the last pair that starts at or before the range's first edge
        const int32_t *off = x.off_in;
        const int32_t c = group_count_below<kWave>(0, (nf + 1) / 2, u0 * kEdgeUnit + 1, [off](int32_t q) { return off[q]; });
        if (lane_id() == 0) s_pair = c - 1;
    }
    __syncthreads();
    int32_t small = 0;  // iterations of this launch, by one block
    auto goes_on = [&](unsigned long long next) {
        const uint32_t edges = static_cast<uint32_t>(next >> 32);
        return edges > 0 && edges <= kEdgeUnit && small + 1 < kSmallIters && iter + 1 < x.max_iter;
    };
    // Slots and edges for the n vertices held, a contiguous share per thread.
    auto flush_new = [&](int32_t n) {  // every thread of the block
        if (n == 0) return;
        constexpr int S = kEdgeNew / kEdgeBlock;
        const int32_t per = (n + kEdgeBlock - 1) / kEdgeBlock;
        int32_t v[S], deg[S];
#pragma unroll
        for (int i = 0; i < S; ++i) {
            const int32_t k = tid * per + i;
            const bool in = i < per && k < n;
            v[i] = in ? s_new[k] : 0;
            deg[i] = in ? t.ro[v[i] + 1] - t.ro[v[i]] : 0;
        }
        unsigned long long mine = 0;
#pragma unroll
        for (int i = 0; i < S; ++i)
            if (deg[i] > 0) mine += (static_cast<unsigned long long>(deg[i]) << 32) | 1u;
        const unsigned long long incl = block_scan_incl64<kEdgeBlock>(mine, s_wave);
        if (tid == kEdgeBlock - 1) {
            s_next = incl;
            s_got = 0;
            if (!single) {
                if (incl) s_got = atomicAdd(x.pk_out, incl);
                *t.cnt_out = 1;
            }
        }
        __syncthreads();
        unsigned long long at = s_got + (incl - mine);
        if (single && goes_on(s_next)) {  // uniform: staged for this block's next iteration
#pragma unroll
            for (int i = 0; i < S; ++i) {
                if (deg[i] > 0) {
                    const uint32_t pos = static_cast<uint32_t>(at);
                    const int32_t off = static_cast<int32_t>(at >> 32);
                    s_off[pos] = off;
                    s_base[pos] = t.ro[v[i]] - off;
                    // the atomics' value: a line of this CU's L1 may be older
                    if constexpr (!BFS)
                        s_du[pos] = __hip_atomic_load(t.dist + v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    at += (static_cast<unsigned long long>(deg[i]) << 32) | 1u;
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < S; ++i) {
                if (deg[i] > 0) {
                    const uint32_t pos = static_cast<uint32_t>(at);
                    t.q_out[pos] = v[i];
                    if ((pos & 1) == 0) x.off_out[pos >> 1] = static_cast<int32_t>(at >> 32);
                    at += (static_cast<unsigned long long>(deg[i]) << 32) | 1u;
                }
            }
        }
        __syncthreads();
    };
    for (;; ++small) {  // uniform across the block
        int32_t held = 0, fresh = 0;
        for (int32_t u = u0; u < u1; ++u) {  // uniform across the block
            const int32_t e0 = u * kEdgeUnit;
            const int32_t n = E - e0 < kEdgeUnit ? E - e0 : kEdgeUnit;  // its edges
            const int32_t e1 = e0 + n, npairs = (nf + 1) / 2;
            const int32_t p0 = s_pair;
            int32_t slots = small ? nf : 0;  // staged: by the iteration before, or of pairs that begin in the unit or before it
            for (int32_t b = 0; small == 0; b += kEdgeBlock) {  // uniform
                const int32_t q = p0 + b + tid, at = 2 * (b + tid);
                int32_t o0 = INT32_MAX, o1 = INT32_MAX;
                if (q < npairs) {
                    o0 = x.off_in[q];
                    if (o0 < e1) {
                        const bool two = 2 * q + 1 < nf;
                        const int32_t v0 = t.q_in[2 * q], v1 = t.q_in[two ? 2 * q + 1 : 2 * q];
                        const int32_t f0 = t.ro[v0], l0 = t.ro[v0 + 1], f1 = t.ro[v1];
                        if (two) o1 = o0 + (l0 - f0);
                        s_base[at] = f0 - o0;
                        s_base[at + 1] = f1 - o1;
                        if constexpr (!BFS) {
                            s_du[at] = t.dist[v0];
                            s_du[at + 1] = t.dist[v1];
                        }
                    }
                }
                s_off[at] = o0;
                s_off[at + 1] = o1;
                const int32_t pairs = __syncthreads_count(o0 < e1);
                slots += 2 * pairs;
                if (pairs < kEdgeBlock) break;
            }
            // each edge's slot: the last with s_off <= e
            int32_t slot[kEdgeItems];
#pragma unroll
            for (int i = 0; i < kEdgeItems; ++i) slot[i] = 0;
            int32_t step = 1;
            while (step < slots) step <<= 1;
            for (step >>= 1; step > 0; step >>= 1) {  // uniform
#pragma unroll
                for (int i = 0; i < kEdgeItems; ++i) {
                    const int32_t at = slot[i] + step;
                    if (at < slots && s_off[at < slots ? at : 0] - e0 <= tid + i * kEdgeBlock) slot[i] = at;
                }
            }
            int32_t v[kEdgeItems];
            float offer[kEdgeItems];
            bool want[kEdgeItems];
#pragma unroll
            for (int i = 0; i < kEdgeItems; ++i) {
                const int32_t e = tid + i * kEdgeBlock;
                want[i] = e < n;
                v[i] = 0;
                offer[i] = 0.f;
                if (want[i]) {
                    const int32_t g = s_base[slot[i]] + e0 + e;
                    v[i] = ld_stream(t.ci + g);
                    if constexpr (!BFS) offer[i] = ld_stream(t.w + g);
                }
                if (e == n - 1) s_pair = p0 + slot[i] / 2;  // the next unit begins in this pair or after it
            }
            // the target's state, which only falls (SSSP) or is claimed once (BFS): a
            // stale read lets an offer through to the atomic, which decides
            if constexpr (BFS) {
                int32_t seen[kEdgeItems];
#pragma unroll
                for (int i = 0; i < kEdgeItems; ++i) seen[i] = want[i] ? t.depth[v[i]] : 0;
#pragma unroll
                for (int i = 0; i < kEdgeItems; ++i)
                    if (want[i] && seen[i] == kUnvisited) seen[i] = atomicCAS(t.depth + v[i], kUnvisited, iter + 1);
#pragma unroll
                for (int i = 0; i < kEdgeItems; ++i) want[i] = want[i] && seen[i] == kUnvisited;
            } else {
                float seen[kEdgeItems];
#pragma unroll
                for (int i = 0; i < kEdgeItems; ++i) {
                    offer[i] = s_du[slot[i]] + offer[i];
                    seen[i] = want[i] ? t.dist[v[i]] : 0.f;
                }
#pragma unroll
                for (int i = 0; i < kEdgeItems; ++i) {
                    want[i] = want[i] && offer[i] < seen[i];
                    if (want[i])
                        seen[i] = __int_as_float(
                            atomicMin(reinterpret_cast<int32_t *>(t.dist) + v[i], __float_as_int(offer[i])));
                }
                int32_t last[kEdgeItems];
#pragma unroll
                for (int i = 0; i < kEdgeItems; ++i) {
                    want[i] = want[i] && offer[i] < seen[i];
                    last[i] = want[i] ? atomicExch(t.stamp + v[i], iter) : 0;
                }
#pragma unroll
                for (int i = 0; i < kEdgeItems; ++i) want[i] = want[i] && last[i] != iter;
            }
            // the unit's new vertices join the block's
            int32_t mine = 0;
#pragma unroll
            for (int i = 0; i < kEdgeItems; ++i) mine += want[i] ? 1 : 0;
            const int32_t incl = block_scan_incl<kEdgeBlock>(mine, s_iwave);
            int32_t at = held + incl - mine;
#pragma unroll
            for (int i = 0; i < kEdgeItems; ++i)
                if (want[i]) s_new[at++] = v[i];
            if (tid == kEdgeBlock - 1) s_held = held + incl;
            __syncthreads();
            held = s_held;  // (the next unit's scan orders this read before the next write)
            fresh = held;
            if (held > kEdgeNew - kEdgeUnit || u + 1 == u1) {  // uniform
                flush_new(held);
                held = 0;
            }
        }
        if (!single) return;
        const unsigned long long next = fresh ? s_next : 0;
        nf = static_cast<int32_t>(next & 0xffffffffu);
        E = static_cast<int32_t>(next >> 32);
        const bool on = goes_on(next);
        ++iter;
        if (!on) {
            if (tid == 0) {
                *x.pk_out = next;
                *t.cnt_out = fresh != 0;
                *x.done_out = iter;
            }
            return;
        }
    }
}

template <bool BFS>
__global__ __launch_bounds__(256) void traversal_init_kernel(int32_t n, int32_t source, float *dist,
                                                             int32_t *depth, int32_t *stamp, int32_t *q0,
                                                             int32_t *counters, const int32_t *ro, int32_t *off0,
                                                             unsigned long long *pk, int32_t *done) {
    for (int64_t v : grid_stride_range(0, n)) {
        if constexpr (BFS) {
            depth[v] = v == source ? 0 : kUnvisited;
        } else {
            dist[v] = v == source ? 0.f : INFINITY;
            stamp[v] = -1;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        q0[0] = source;
        counters[0] = 1;  // F_0 = {source}
        counters[1] = 0;
        counters[2] = 0;
        counters[3] = 0;  // rounds
        counters[4] = 0;  // work-queue tickets of the first two launches
        counters[5] = 0;
        // merge-path: the source's slot and edges
        const int32_t d = ro[source + 1] - ro[source];
        off0[0] = 0;
        pk[0] = d > 0 ? (static_cast<unsigned long long>(d) << 32) | 1u : 0u;
        pk[1] = pk[2] = 0;
        done[0] = 0;
    }
}

template <typename K>
int resident_blocks(K kernel, int block) {
    int dev = 0, cus = 256, per_cu = 1;
    if (hipGetDevice(&dev) == hipSuccess) {
        (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block, 0);
    }
    return cus * (per_cu > 0 ? per_cu : 1);
}

template <typename K>
hipError_t launch_advance(K kernel, int block, int grid, const trav_args &t, hipStream_t s) {
    const int g = grid > 0 ? grid : resident_blocks(kernel, block);
    hipLaunchKernelGGL(kernel, dim3(static_cast<uint32_t>(g)), dim3(block), 0, s, t);
    return hipGetLastError();
}

template <bool BFS>
hipError_t advance_merge(const trav_cfg &c, const trav_ws &w, const trav_args &t, int32_t max_iter, hipStream_t s) {
    const int32_t i = t.iter;
    const edge_args x{w.off[i & 1], w.off[(i + 1) & 1], w.pk + i % 3, w.pk + (i + 1) % 3, w.pk + (i + 2) % 3,
                      w.done + i % 3, w.done + (i + 1) % 3, max_iter};
    hipLaunchKernelGGL(advance_merge_kernel<BFS>, dim3(static_cast<uint32_t>(c.grid)), dim3(kEdgeBlock), 0, s, t, x);
    return hipGetLastError();
}

template <bool BFS>
hipError_t advance(const trav_cfg &c, const trav_ws &w, const trav_args &t, int32_t max_iter, hipStream_t s) {
    prof_scope p(s, BFS ? "bfs_advance" : "sssp_advance");
    if (c.kind == LB_MERGE_PATH) return advance_merge<BFS>(c, w, t, max_iter, s);
    if (c.kind == LB_THREAD_MAPPED) return launch_advance(advance_thread_kernel<BFS>, c.block, c.grid, t, s);
#define LB_G(G)                                                                                               \
    if (c.group == G) {                                                                                       \
        if (c.kind == LB_WORK_QUEUE)                                                                          \
            return launch_advance(advance_scan_kernel<G, BFS, true>, group_block<G>::BLOCK, c.grid, t, s);     \
        if (c.tiles_per_group == 1)                                                                           \
            return launch_advance(advance_group_kernel<G, BFS>, group_block<G>::BLOCK, c.grid, t, s);          \
        return launch_advance(advance_scan_kernel<G, BFS, false>, group_block<G>::BLOCK, c.grid, t, s);        \
    }
    LB_TRAVERSAL_GROUPS(LB_G)
#undef LB_G
    return hipErrorInvalidValue;
}

template <bool BFS>
hipError_t run_traversal(const csr_dev &G, int32_t source, float *dist, int32_t *depth, trav_cfg c,
                         int32_t max_iter, int32_t *iterations, bool *converged, void *ws, hipStream_t s) {
    const trav_ws w = trav_ws_carve(ws, G.rows);
    {
        prof_scope p(s, "traversal_init");
        const int64_t blocks = (static_cast<int64_t>(G.rows) + 255) / 256;
        hipLaunchKernelGGL(traversal_init_kernel<BFS>, dim3(static_cast<uint32_t>(blocks < 8192 ? blocks : 8192)),
                           dim3(256), 0, s, G.rows, source, dist, depth, w.stamp, w.queue[0], w.counters, G.ro, w.off[0], w.pk,
                           w.done);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    trav_args t{G.ro, G.ci, static_cast<const float *>(G.val), dist, depth, w.stamp,
                nullptr, nullptr, nullptr, nullptr, nullptr, w.counters + 3, nullptr, nullptr, 0};
    // The size is read after 4, 8, 12, 16, 28, 32, 60, 92, ... launches: a power-law
    // graph ends within 16, and what is launched past the end is wasted (28 for 13);
    // a long chain or grid pays for each wait.  Read at 32 after 16, a graph of 20
    // iterations paid for more launches than at 28 (work queue, 100,000 vertices of
    // three edges, BFS 1.03 ms against 0.93).
    int32_t launched = 0;
    if (c.kind == LB_MERGE_PATH && c.grid <= 0) c.grid = resident_blocks(advance_merge_kernel<BFS>, kEdgeBlock);
    int32_t host[kTravDone + 3] = {}, rounds = 0;
    *converged = false;
    for (;;) {
        const int32_t batch = launched < 16 ? 4 : (launched < 28 ? 12 : (launched < 32 ? 4 : (launched < 60 ? 28 : 32)));
        for (int k = 0; k < batch && launched < max_iter; ++k, ++launched) {
            t.iter = launched;
            t.q_in = w.queue[launched & 1];
            t.q_out = w.queue[(launched + 1) & 1];
            t.cnt_in = w.counters + launched % 3;
            t.cnt_out = w.counters + (launched + 1) % 3;
            t.cnt_clear = w.counters + (launched + 2) % 3;
            t.ticket = w.counters + 4 + (launched & 1);
            t.ticket_clear = w.counters + 4 + ((launched + 1) & 1);
            const hipError_t e = advance<BFS>(c, w, t, max_iter, s);
            if (e != hipSuccess) return e;
        }
        hipError_t e = hipMemcpyAsync(host, w.counters, sizeof host, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return e;
        rounds = c.kind == LB_MERGE_PATH ? host[kTravDone + launched % 3] : host[3];
        if (host[launched % 3] == 0) {
            *converged = true;
            break;
        }
        if (rounds >= max_iter || launched >= max_iter) break;  // a launch is at least one iteration
    }
    if (iterations) *iterations = rounds;
    return hipSuccess;
}

}  // namespace

bool traversal_group_supported(int g) {
#define LB_G(G) if (g == G) return true;
    LB_TRAVERSAL_GROUPS(LB_G)
#undef LB_G
    return false;
}

hipError_t sssp(const csr_dev &G, int32_t source, float *dist, const trav_cfg &c, int32_t max_iter,
                int32_t *iterations, bool *converged, void *ws, hipStream_t s) {
    return run_traversal<false>(G, source, dist, nullptr, c, max_iter, iterations, converged, ws, s);
}

hipError_t bfs(const csr_dev &G, int32_t source, int32_t *depth, const trav_cfg &c, int32_t max_iter,
               int32_t *iterations, bool *converged, void *ws, hipStream_t s) {
    return run_traversal<true>(G, source, nullptr, depth, c, max_iter, iterations, converged, ws, s);
}

}  // namespace lbk
