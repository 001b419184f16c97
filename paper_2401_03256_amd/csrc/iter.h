// Device code of one PageRank iteration, shared by the single-graph
// engines (rank.hip) and the multi-graph serving loop (serve.hip).  The
// layout and the marking rules are described at the top of rank.hip.
#pragma once

#include <type_traits>

#include "common.h"

namespace dfpr {

// Index loads in flight per lane and round of a gather (each lane still
// adds its entries in index order, so the value does not change the sums).
// Measured on R-MAT scale 22: 8 beats 4, 6, 10, 12 and 16.
#ifndef DFPR_UNROLL
#define DFPR_UNROLL 8
#endif
// Minimum waves per SIMD the iteration kernels are compiled for (the second
// launch bound).  The kernels now fit 6-7 waves without spills; asking for
// eight is slower on R-MAT scale 22.
#ifndef DFPR_ITER_WAVES_PER_SIMD
#define DFPR_ITER_WAVES_PER_SIMD 5
#endif
// Index loads are streamed once per iteration; marking them non-temporal
// leaves more of L2 to the gathered contributions (4% on R-MAT scale 22;
// the same marking on the gathers themselves halves the speed).
#ifndef DFPR_NT_IDX
#define DFPR_NT_IDX 1
#endif
constexpr int kUnroll = DFPR_UNROLL;   // loads in flight per lane and round

// Data that other workgroups change during the launch that reads it.  A
// launch per iteration reads and writes it with ordinary accesses, the
// kernel boundary making one iteration's writes visible to the next (COH
// false).  The resident loop (k_resident in rank.hip) runs many iterations
// in one launch and uses relaxed agent-scope accesses (COH true): they pass
// over the vector L1, and a barrier between iterations needs no cache
// write-back or invalidate.  Random 8-byte gathers of this kind run at the
// speed of ordinary ones (205 against 212 G/s from 512 KB, equal from 8 MB).
template <bool COH, class T>
__device__ __forceinline__ T ld(const T *p)
{
    if constexpr (COH) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else return *p;
}
template <bool COH, class T>
__device__ __forceinline__ void st(T *p, T v)
{
    if constexpr (COH) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = v;
}

// x, as a value that nothing computed from it before can be reused for.  The
// compiler otherwise computes the addresses of the resident loop once before
// the iterations, keeps them in scratch memory (104 bytes a lane) and loads
// them back in each: R-MAT scale 13 1093 against 1058 us a call, 300 x 300 grid
// 834 against 806 us.
__device__ __forceinline__ uint32_t fresh(uint32_t x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// Largest of a non-negative value over the first `LANES` lanes of a wave (16 or
// 64), in all of them: moves between lanes in the vector unit, where shuffles
// go through LDS at some 100 cycles a step.
template <int CTRL>
__device__ __forceinline__ double max_step(double x)
{
    const int lo = __double2loint(x), hi = __double2hiint(x);
    return fmax(x, __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xF, 0xF, false),
                                    __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xF, 0xF, false)));
}
template <int LANES>
__device__ __forceinline__ double wave_max(double x)
{
    static_assert(LANES == 16 || LANES == kWave, "one row of lanes, or all four");
    x = max_step<0x111>(x);         // row_shr 1, 2, 4, 8: the last lane of each row
    x = max_step<0x112>(x);
    x = max_step<0x114>(x);
    x = max_step<0x118>(x);
    if constexpr (LANES == kWave) {
        x = max_step<0x142>(x);     // row_bcast 15, 31: the last lane of the wave
        x = max_step<0x143>(x);
    }
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), LANES - 1),
                            __builtin_amdgcn_readlane(__double2loint(x), LANES - 1));
}

// This wave's stores and atomics so far have reached the point where
// agent-scope loads find them.
__device__ __forceinline__ void drain_stores()
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// What the lanes of a wave left in LDS before is there for all of them after: the
// hardware runs a wave's accesses in order, the fence keeps the compiler from
// moving them.
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Whether this is the last workgroup of the grid to get here; the others'
// atomics and agent-scope stores before the call are then visible to its
// agent-scope loads.  Every thread calls it.  A workgroup arrives at one of
// kTickets counters and the last of each at one more, since arrivals at one
// address take 13 ns each; the last of all clears them.
__device__ __forceinline__ bool last_block(uint32_t *tick, int *s_last)
{
    drain_stores();
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t n = gridDim.x, b = blockIdx.x, t = b % kTickets;
        const uint32_t mine = (n - t + kTickets - 1) / kTickets, used = min(n, (uint32_t)kTickets);
        int last = 0;
        if (atomicAdd(&tick[t], 1u) == mine - 1 && atomicAdd(&tick[kTickets], 1u) == used - 1) {
            last = 1;
            for (int k = 0; k <= kTickets; k++) st<true>(&tick[k], 0u);
        }
        *s_last = last;
    }
    __syncthreads();
    return *s_last != 0;
}

// Index loads.  In a launch per iteration they are streamed: marked
// non-temporal so that they do not displace gathered contributions from L2.
// The resident loop reads the same indices every iteration and keeps them.
template <bool COH = false>
__device__ __forceinline__ int32_t load_idx(const int32_t *p)
{
#if DFPR_NT_IDX
    if constexpr (!COH) return __builtin_nontemporal_load(p);
#endif
    return *p;
}

// Contributions of the first kHubRows vertices (the highest in-degrees, and
// with them the most out-edges) are copied into LDS by each workgroup of a
// sweep that walks the full schedule, and gathers from those sources read
// LDS instead of going through the vector L1 and L2.  On R-MAT scale 22 the
// first 2048 sources take 17% of the gathers; 16 KB per workgroup keeps
// seven workgroups per CU, and a static sweep runs 4.5% faster (4096
// entries halve the workgroups per CU and are slower).  0 switches it off.
#ifndef DFPR_HUB
#define DFPR_HUB 2048
#endif
constexpr uint32_t kHubRows = DFPR_HUB;

// The LDS copy a workgroup gathers from: n entries (0: none).
struct Hub {
    const double *d;    // FP64 contributions
    const float *f;     // FP32 contributions (precision form)
    uint32_t n;
};

struct IterArgs {
    int32_t n;
    const uint32_t *in_beg, *in_cnt;
    const int32_t *in_idx;
    const uint32_t *out_beg, *out_cnt;
    const int32_t *out_idx;
    const double *Rc, *Cc;      // read
    double *Rn, *Cn;            // written
    const float *C32c;          // FP32 contributions read (precision form)
    float *C32n;                // FP32 contributions written
    uint32_t *stamp, *xstamp;
    int32_t *bins;              // class lists (sparse mode), n entries each
    Ctl *ctl;
    Ctl *mirror;                // host-visible copy of the control block, or NULL
    double *dr_part;            // kFoldSlots slots of the L-inf of Delta r
    double *rmax_part;          //   ... of the largest new rank
    unsigned long long *cnt_part;   // kCounters per slot
    double base_rank;           // (1 - alpha) / n
    double alpha, tol, ftol;
    uint32_t sbase;             // stamp base of the call
    uint32_t sparse_limit;
    uint32_t heavy;             // class lists: rows of more out-edges mark with plain stores
    int32_t it, max_iters;
    int32_t n_stride;
    uint32_t long_row;          // launches: FP64 rows of more in-edges take kLongParts parts
    uint32_t hub;               // contributions to copy into LDS (0: none)
    struct Stage *stage;        // resident loop: the workgroup's new list entries
};

__device__ __forceinline__ int lane_id() { return __lane_id(); }

// In-degree class of internal id v (its id range, Ctl::cls; the self-loop
// rows are in class 0).
__device__ __forceinline__ int class_of_id(const IterArgs &a, int32_t v)
{
    int c = kBins - 1;
#pragma unroll
    for (int k = 1; k < kBins; k++) c -= (uint32_t)v >= a.ctl->cls[k] ? 1 : 0;
    return c;
}

struct Acc {
    double dr_max = 0.0;
    double r_max = 0.0;
    // rows, edges, xrows, xedges of this lane: each below the graph's edge
    // slots (under 2^32), so 32 bits per lane; widened for the fold
    uint32_t c[kCounters] = {0, 0, 0, 0};
    double ftol = 0.0;          // frontier tolerance in effect
    bool plain = false;         // expansions mark with plain stores (Ctl::plain_marks)
};

// The contributions of the sources in i (-1: none), those below n_hub from the
// LDS copy and the others from memory.  The resident loop reads LDS for all of
// them first and then memory over it: with both kinds of load in one branch
// the compiler waits for one before it issues the next into the same register
// (a sweep of R-MAT scale 18 from host ranks: 3153 against 2974 us).  The
// launch kernels, whose LDS copy takes a sixth of the gathers, have no
// register left for that (R-MAT scale 22 29.8 against 31.6 ms).
template <bool COH, class T>
__device__ __forceinline__ void load_contribs(const T *hub, uint32_t n_hub, const T *C,
                                              const int32_t (&i)[kUnroll], T (&c)[kUnroll])
{
    if constexpr (COH) {
        if (n_hub) {
#pragma unroll
            for (int j = 0; j < kUnroll; j++) c[j] = hub[min((uint32_t)i[j], n_hub - 1)];
        } else {
#pragma unroll
            for (int j = 0; j < kUnroll; j++) c[j] = (T)0;
        }
#pragma unroll
        for (int j = 0; j < kUnroll; j++)
            if (i[j] >= (int32_t)n_hub) c[j] = ld<COH>(C + i[j]);
    } else {
#pragma unroll
        for (int j = 0; j < kUnroll; j++)
            c[j] = i[j] < 0 ? (T)0 : (uint32_t)i[j] < n_hub ? hub[i[j]] : ld<COH>(C + i[j]);
    }
}

// Sum of the contributions of in-edges idx[k] for k = first, first + step,
// ... < cnt, added in that order.  FP64, or (F32) FP32 contributions added
// with Kahan's compensated summation and returned as sum - compensation in
// FP64.
template <bool F32, bool COH>
__device__ __forceinline__ double gather_sum(const IterArgs &a, const Hub &hub, const int32_t *idx,
                                    uint32_t first, uint32_t step, uint32_t cnt)
{
    if (!F32) {
        double s = 0.0;
        for (uint32_t k0 = first; k0 < cnt; k0 += step * kUnroll) {
            int32_t i[kUnroll];
#pragma unroll
            for (int j = 0; j < kUnroll; j++) {
                const uint32_t k = k0 + j * step;
                i[j] = k < cnt ? load_idx<COH>(idx + k) : -1;
            }
            double c[kUnroll];
            load_contribs<COH>(hub.d, hub.n, a.Cc, i, c);
#pragma unroll
            for (int j = 0; j < kUnroll; j++)
                if (i[j] >= 0) s += c[j];
        }
        return s;
    } else {
        float ks = 0.0f, kc = 0.0f;
        for (uint32_t k0 = first; k0 < cnt; k0 += step * kUnroll) {
            int32_t i[kUnroll];
#pragma unroll
            for (int j = 0; j < kUnroll; j++) {
                const uint32_t k = k0 + j * step;
                i[j] = k < cnt ? load_idx<COH>(idx + k) : -1;
            }
            float c[kUnroll];
            load_contribs<COH>(hub.f, hub.n, a.C32c, i, c);
#pragma unroll
            for (int j = 0; j < kUnroll; j++) {
                if (i[j] >= 0) {
                    const float y = c[j] - kc;
                    const float t = ks + y;
                    kc = (t - ks) - y;
                    ks = t;
                }
            }
        }
        return (double)ks - (double)kc;
    }
}

// New entries of the class lists of one workgroup of the resident loop, kept
// in LDS until the workgroup has processed its rows: one atomic per class and
// workgroup on the list lengths instead of one per wave, round and class
// (atomics on one address take 13 ns each).
struct Stage {
    uint32_t cnt[kBins];        // entries per class
    uint32_t n;                 // all entries
    uint32_t cap;               // room in item
    uint32_t base[kBins];
    uint2 *item;                // vertex, class << 28 | position among the class's entries
};

// Wave-aggregated append of the lanes with `take` set to the class lists.
// Every lane of the wave calls it.
template <bool COH = false>
__device__ __forceinline__ void append_to_bins(bool take, int32_t x, int cls, Ctl *ctl, int32_t *bins,
                                      uint32_t stride, Stage *stage = nullptr)
{
    if constexpr (COH) {
        if (take) {
            const uint32_t at = atomicAdd(&stage->n, 1u);
            if (at < stage->cap) {
                const uint32_t k = atomicAdd(&stage->cnt[cls], 1u);
                stage->item[at] = make_uint2((uint32_t)x, (uint32_t)cls << 28 | k);
            } else {
                st<true>(&bins[(size_t)cls * stride + atomicAdd(&ctl->live[cls], 1u)], x);
            }
        }
        return;
    }
    unsigned long long pend = __ballot(take);
    const int lane = lane_id();
    const unsigned long long below = (1ull << lane) - 1ull;
    while (pend) {
        const int leader = __ffsll((long long)pend) - 1;
        const int c = __shfl(cls, leader);
        const unsigned long long mine = __ballot(take && cls == c);
        uint32_t base = 0;
        if (lane == leader) base = atomicAdd(&ctl->live[c], (uint32_t)__popcll(mine));
        base = __shfl(base, leader);
        if (take && cls == c) st<COH>(&bins[(size_t)c * stride + base + __popcll(mine & below)], x);
        pend &= ~mine;
    }
}

// Mark the out-neighbours of w with stamp `sv`.  The calling lanes take
// positions lane0, lane0 + step, ... (lane0 < step); every lane of every
// calling wave runs the same number of rounds.
template <bool SPARSE, bool COH>
__device__ __forceinline__ void mark_out_row(const IterArgs &a, int32_t w, uint32_t lane0, uint32_t step,
                                    uint32_t sv)
{
    const uint32_t ob = a.out_beg[w], oc = a.out_cnt[w];
    for (uint32_t k0 = 0; k0 < oc; k0 += step * kUnroll) {
        int32_t x[kUnroll];
#pragma unroll
        for (int j = 0; j < kUnroll; j++) {
            const uint32_t k = k0 + lane0 + j * step;
            x[j] = k < oc ? load_idx<COH>(a.out_idx + ob + k) : -1;
        }
        uint32_t sx[kUnroll];
#pragma unroll
        for (int j = 0; j < kUnroll; j++)
            sx[j] = x[j] < 0 ? 0xFFFFFFFFu
                    : SPARSE && COH ? atomicMax(&a.stamp[x[j]], sv) : ld<COH>(a.stamp + x[j]);
#pragma unroll
        for (int j = 0; j < kUnroll; j++) {
            bool nw = false;
            if (sx[j] < a.sbase) {
                if (SPARSE) nw = COH || atomicMax(&a.stamp[x[j]], sv) < a.sbase;
                else st<COH>(a.stamp + x[j], sv);
            }
            if (SPARSE) {
                const int cls = nw ? class_of_id(a, x[j]) : 0;
                append_to_bins<COH>(nw, x[j], cls, a.ctl, a.bins, a.n_stride, a.stage);
            }
        }
    }
}

// On the class lists, a row with more out-edges than this marks them with
// plain stores, like the full schedule does, and moves the call to the full
// schedule from the next iteration on: its out-row alone would fill a good
// part of the lists of launches (an eighth), and one workgroup appending them
// entry by entry (an atomic per out-edge) stalls the whole iteration.  The
// resident loop's longer lists do not move the line: R-MAT scale 20, a batch of
// two, 0.85 ms of iterations, and 1.24 with an eighth of its lists.
__device__ __forceinline__ bool heavy_in_sparse(const IterArgs &a, uint32_t oc)
{
    return oc > a.heavy;
}

// Expansion of the rows of a wave whose lanes have `deg` > 0 out-edges
// starting at `ob` (`incl` = inclusive prefix sum of `deg` over the wave,
// `total` its last value): every lane takes one out-edge per round, so
// rows with few out-edges share rounds and list appends.  Every lane of
// the wave calls it with the same `total`.
template <bool SPARSE, bool COH>
__device__ __forceinline__ void expand_rows(const IterArgs &a, uint32_t incl, uint32_t deg, uint32_t ob,
                                   uint32_t total, uint32_t sv)
{
    const int lane = lane_id();
    for (uint32_t t0 = 0; t0 < total; t0 += kWave) {
        const uint32_t t = t0 + lane;
        const uint32_t tt = min(t, total - 1);
        // owner: the first lane whose inclusive sum exceeds tt
        int j = 0;
#pragma unroll
        for (int step = kWave / 2; step > 0; step >>= 1)
            if (__shfl(incl, j + step - 1) <= tt) j += step;
        const uint32_t first = __shfl(incl, j) - __shfl(deg, j);
        const uint32_t base = __shfl(ob, j);
        const int32_t x = t < total ? load_idx<COH>(a.out_idx + base + (tt - first)) : -1;
        // the resident loop's class lists are short: claim at once instead of
        // looking first (one dependent access less)
        const uint32_t sx = x < 0 ? 0xFFFFFFFFu
                            : SPARSE && COH ? atomicMax(&a.stamp[x], sv) : ld<COH>(a.stamp + x);
        bool nw = false;
        if (sx < a.sbase) {
            if (SPARSE) nw = COH || atomicMax(&a.stamp[x], sv) < a.sbase;
            else st<COH>(a.stamp + x, sv);
        }
        if (SPARSE) {
            const int cls = nw ? class_of_id(a, x) : 0;
            append_to_bins<COH>(nw, x, cls, a.ctl, a.bins, a.n_stride, a.stage);
        }
    }
}

// Finish one row: Eq. 1, Delta r, writes; returns whether it must expand.
// The resident loop hands over the row's expansion stamp (`xs`), loaded with
// its other data: most rows of an iteration move by more than the frontier
// tolerance, and one dependent access less per iteration is 1-4% of a call
// (R-MAT scale 16 1.60 against 1.67 ms an update pair).  A launch per
// iteration, bound by its loads, looks only when the row has moved.
template <bool DF, bool F32, bool COH>
__device__ __forceinline__ bool finish_row(const IterArgs &a, int32_t v, uint32_t cnt, double s, double rc,
                                  uint32_t oc, uint32_t xs, Acc &acc)
{
    const double r = a.base_rank + a.alpha * s;
    const double dr = fabs(r - rc);
    st<COH>(a.Rn + v, r);
    if (F32) st<COH>(a.C32n + v, (float)(r / (double)oc));
    else st<COH>(a.Cn + v, r / (double)oc);
    acc.dr_max = fmax(acc.dr_max, dr);
    acc.r_max = fmax(acc.r_max, r);
    acc.c[0] += 1;
    acc.c[1] += cnt;
    if (DF && dr > acc.ftol && (COH ? xs : a.xstamp[v]) != a.sbase) {
        st<COH>(a.xstamp + v, a.sbase);
        acc.c[2] += 1;
        acc.c[3] += oc;
        return true;
    }
    return false;
}

// A lane's row of a wave unit: in-edges, out-degree, previous rank, the sum
// of Eq. 1, and whether this lane finishes it (the row's first lane).
struct UnitRow {
    int32_t v;
    uint32_t cnt, oc, xs;
    double rc, s;
    bool mine;
};

// One wave unit: 64/G rows (COH: at most `per` of them) of a class list (`list`), or of the id range
// starting at `id0` when `list` is NULL, G lanes per row.  LOOP (G = 1): the
// id range of rows whose only in-entry was the self-loop at load; few of
// them are marked, so their stamp is read first, and a row that has since
// gained in-edges is summed like any class-0 row.
template <int G, bool DF, bool F32, bool COH, bool LOOP = false>
__device__ __forceinline__ UnitRow wave_unit(const IterArgs &a, const Hub &hub, const int32_t *list,
                                          uint32_t id0, uint32_t count, uint32_t first, uint32_t per,
                                          bool check)
{
    const int lane = lane_id();
    const int sub = lane & (G - 1);
    if constexpr (COH) count = min(count, first + per);
    const uint32_t pos = first + lane / G;
    bool active = false;
    int32_t v = 0;
    uint32_t beg = 0, cnt = 0, oc = 1, xs = 0;
    double rc = 0.0;
    if (pos < count) {
        v = list ? ld<COH>(list + pos) : (int32_t)(id0 + pos);
        active = true;
        if (LOOP) {
            if (DF && check) {
                const uint32_t sx = ld<COH>(a.stamp + v);
                active = sx >= a.sbase && sx <= a.sbase + (uint32_t)a.it;
            }
            if (active) {
                cnt = a.in_cnt[v];
                beg = a.in_beg[v];
                rc = ld<COH>(a.Rc + v);
                oc = a.out_cnt[v];
                if (DF && COH) xs = ld<COH>(a.xstamp + v);
            }
        } else {
            // the row's start, length, rank and out-degree are loaded with
            // its stamp, not after it: on the full schedule (dense mode)
            // only marked rows are processed, but waiting for the stamp
            // first would add a dependent load to every row (1.6% per call
            // on R-MAT scale 22)
            beg = a.in_beg[v];
            cnt = a.in_cnt[v];
            if (sub == 0) {
                rc = ld<COH>(a.Rc + v);
                oc = a.out_cnt[v];
                if (DF && COH) xs = ld<COH>(a.xstamp + v);
            }
            if (DF && check) {
                const uint32_t sx = ld<COH>(a.stamp + v);
                active = sx >= a.sbase && sx <= a.sbase + (uint32_t)a.it;
            }
        }
    }
    double s = 0.0;
    if (active) {
        if (cnt == 1) {
            // the self-loop is the only in-edge
            if (sub == 0) s = F32 ? (double)ld<COH>(a.C32c + v) : ld<COH>(a.Cc + v);
        } else if (LOOP) {
            // a self-loop row that has gained in-edges since the load: rare,
            // summed in index order by its lane (as gather_sum with G = 1)
            if (F32) {
                float ks = 0.0f, kc = 0.0f;
                for (uint32_t k = 0; k < cnt; k++) {
                    const float y = ld<COH>(a.C32c + load_idx<COH>(a.in_idx + beg + k)) - kc;
                    const float t = ks + y;
                    kc = (t - ks) - y;
                    ks = t;
                }
                s = (double)ks - (double)kc;
            } else {
                for (uint32_t k = 0; k < cnt; k++)
                    s += ld<COH>(a.Cc + load_idx<COH>(a.in_idx + beg + k));
            }
        } else {
            s = gather_sum<F32, COH>(a, hub, a.in_idx + beg, sub, G, cnt);
        }
    }
#pragma unroll
    for (int off = G / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, G);
    return {v, cnt, oc, xs, rc, s, active && sub == 0};
}

// A wave unit of two rows a lane group, the one numbered as the group from
// `first` on and that 64 / G later (resident loop, FP64, full schedule).  A
// row's loads are a chain of three, and a wave whose units take one row a
// group waits each of them out between few instructions: on R-MAT scale 20
// the rows took 33 of their 65 us with the indices and the gathers left out.
// Two rows share the chain, four in-edges of each in flight.  LOOP as in
// wave_unit.  R-MAT with 1.5e6 vertices 11.05 -> 10.32 ms a call; see
// kPairUnits for where it is used.
template <int G, bool DF, bool LOOP = false>
__device__ __forceinline__ void wave_pair(const IterArgs &a, const Hub &hub, uint32_t id0, uint32_t count,
                                          uint32_t first, bool check, UnitRow (&row)[2])
{
    constexpr int U = kUnroll / 2;
    const int lane = lane_id();
    const int sub = lane & (G - 1);
    uint32_t beg[2], n[2];
    bool active[2];
#pragma unroll
    for (int p = 0; p < 2; p++) {
        const uint32_t pos = first + p * (kWave / G) + lane / G;
        UnitRow &r = row[p];
        r = {0, 0, 1, 0, 0.0, 0.0, false};
        beg[p] = n[p] = 0;
        active[p] = pos < count;
        r.v = (int32_t)(id0 + pos);
        if (DF && LOOP && check && active[p]) {
            const uint32_t sx = ld<true>(a.stamp + r.v);
            active[p] = sx >= a.sbase && sx <= a.sbase + (uint32_t)a.it;
        }
    }
#pragma unroll
    for (int p = 0; p < 2; p++) {
        UnitRow &r = row[p];
        if (!active[p]) continue;
        beg[p] = a.in_beg[r.v];
        r.cnt = a.in_cnt[r.v];
        if (sub == 0) {
            r.rc = ld<true>(a.Rc + r.v);
            r.oc = a.out_cnt[r.v];
            if (DF) r.xs = ld<true>(a.xstamp + r.v);
        }
        if (DF && !LOOP && check) {
            const uint32_t sx = ld<true>(a.stamp + r.v);
            active[p] = sx >= a.sbase && sx <= a.sbase + (uint32_t)a.it;
        }
    }
#pragma unroll
    for (int p = 0; p < 2; p++) {
        if (!active[p]) continue;
        // a self-loop as the only in-edge needs no index
        if (row[p].cnt == 1) row[p].s = sub == 0 ? ld<true>(a.Cc + row[p].v) : 0.0;
        else n[p] = row[p].cnt;
    }
    const uint32_t most = max(n[0], n[1]);
    for (uint32_t k0 = sub; k0 < most; k0 += G * U) {
        int32_t i[kUnroll];
#pragma unroll
        for (int j = 0; j < kUnroll; j++) {
            const uint32_t k = k0 + (j % U) * G;
            i[j] = k < n[j / U] ? a.in_idx[beg[j / U] + k] : -1;
        }
        double c[kUnroll];
        load_contribs<true>(hub.d, hub.n, a.Cc, i, c);
#pragma unroll
        for (int j = 0; j < kUnroll; j++)
            if (i[j] >= 0) row[j / U].s += c[j];
    }
#pragma unroll
    for (int p = 0; p < 2; p++) {
#pragma unroll
        for (int off = G / 2; off > 0; off >>= 1) row[p].s += __shfl_xor(row[p].s, off, G);
        row[p].mine = active[p] && sub == 0;
    }
}

// The rest of a wave unit, once its rows are summed.
template <bool DF, bool F32, bool COH>
__device__ __forceinline__ void finish_unit(const IterArgs &a, const UnitRow &row, bool sparse, Acc &acc)
{
    const int lane = lane_id();
    const int32_t v = row.v;
    const uint32_t oc = row.oc;
    bool expand = false;
    if (row.mine) expand = finish_row<DF, F32, COH>(a, v, row.cnt, row.s, row.rc, oc, row.xs, acc);
    // Rows with fewer out-edges than a wave has lanes expand together, one
    // out-edge per lane and round; longer rows one at a time with the whole
    // wave and kUnroll loads in flight per lane.
    if (DF && __ballot(expand)) {
        const uint32_t sv = a.sbase + (uint32_t)a.it + 1;
        const bool small = expand && oc < (uint32_t)kWave;
        if (__ballot(small)) {
            const uint32_t deg = small ? oc : 0u;
            const uint32_t ob = small ? a.out_beg[v] : 0u;
            uint32_t incl = deg;
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const uint32_t y = __shfl_up(incl, d);
                if (lane >= d) incl += y;
            }
            const uint32_t total = __shfl(incl, kWave - 1);
            if (sparse && !acc.plain) {
                expand_rows<true, COH>(a, incl, deg, ob, total, sv);
            } else {
                if (sparse && lane == 0) st<COH>(&a.ctl->force_dense, 1u);
                expand_rows<false, COH>(a, incl, deg, ob, total, sv);
            }
        }
        unsigned long long q = __ballot(expand && !small);
        while (q) {
            const int l = __ffsll((long long)q) - 1;
            const int32_t w = __shfl(v, l);
            const uint32_t wc = __shfl(oc, l);
            if (sparse && !acc.plain && !heavy_in_sparse(a, wc)) {
                mark_out_row<true, COH>(a, w, lane, kWave, sv);
            } else {
                if (sparse && lane == 0) st<COH>(&a.ctl->force_dense, 1u);
                mark_out_row<false, COH>(a, w, lane, kWave, sv);
            }
            q &= q - 1;
        }
    }
}

// Rows of more than 1024 in-edges (by their class).  The sum of such a row is
// that of strided parts, part p adding entries p, p + parts, ... in order: the
// parts of 64 neighbours fold with the butterfly of a wave, and the folds are
// added in order, or, the 16 of a long row, in pairs (one after the other they
// round 15 times at the size of the sum, where four folds round 3 times).  A
// row has kBlock parts, or, in FP64 with more than kLongRow in-edges,
// kLongParts.  The resident loop gives such a long row a workgroup
// of kLongParts threads, because one of 10^4 in-edges in 256 parts was the
// last thing every iteration waited for (13 us of 26 on R-MAT scale 18);
// kBlock threads take its parts in four passes, which sums the same bits.
// The line at 2048 against 1024 / 4096, per update pair: R-MAT scale 16
// 1.94 against 1.84 / 2.03 ms, scale 20 9.47 against 10.06 / 9.41, scale 22
// (launches) 29.97 against 30.80 / 30.03.
// The FP32 form keeps kBlock parts: with more, its Kahan sums would round
// differently.
// So does every row of a graph that is too large for the resident loop when it
// is loaded (dfpr_graph::long_row): in launches four passes are only slower.  The
// resident loop leaves the class to launches there, so that its own line is a
// constant (as a field it cost an update pair on R-MAT scale 16 0.7%).
// R-MAT with 2.5e6 vertices, 41.7M edges: a sweep 233.4 -> 231.3 us (228.8
// before there were long rows), Static 15.89 -> 15.76 ms; scale 22 24.16 ->
// 24.0 ms.
constexpr uint32_t kLongRow = 2048;
constexpr int kLongParts = 1024;
constexpr int kLongFolds = kLongParts / kWave;

// T threads per row, kBlock or kLongParts; a workgroup of more threads sums
// one row per T of them (its sub-blocks).  Every thread calls it, whether its
// sub-block has a row (`valid`) or not.
template <bool DF, bool F32, bool COH, int T>
__device__ __forceinline__ void block_row(const IterArgs &a, const Hub &hub, int32_t v, bool valid,
                                 bool check, bool sparse, Acc &acc, double *red, int *flag)
{
    const uint32_t t = threadIdx.x % T;
    bool active = valid;
    if (active && DF && check) {
        const uint32_t sx = ld<COH>(a.stamp + v);
        active = sx >= a.sbase && sx <= a.sbase + (uint32_t)a.it;
    }
    uint32_t cnt = 0;
    if (active) {
        cnt = a.in_cnt[v];
    }
    const bool lng = !F32 && cnt > (COH ? kLongRow : a.long_row);
    if (active) {
        const int32_t *idx = a.in_idx + a.in_beg[v];
        auto pass = [&](uint32_t q, auto step) {
            double s = gather_sum<F32, COH>(a, hub, idx, q * T + t, decltype(step)::value, cnt);
#pragma unroll
            for (int off = kWave / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, kWave);
            if (lane_id() == 0) red[q * (T / kWave) + t / kWave] = s;
        };
        if (!lng) {
            if (T == kBlock || t < kBlock) pass(0, std::integral_constant<uint32_t, kBlock>());
        } else {
#pragma unroll 1
            for (uint32_t q = 0; q < kLongParts / T; q++)
                pass(q, std::integral_constant<uint32_t, kLongParts>());
        }
    }
    __syncthreads();
    double r = 0.0;
    if (active && lng && t < kWave) {
        r = red[t % kLongFolds];
#pragma unroll
        for (int off = 1; off < kLongFolds; off *= 2) r += __shfl_xor(r, off, kWave);
    }
    if (t == 0) {
        *flag = 0;
        if (active) {
            if (!lng) r = ((red[0] + red[1]) + red[2]) + red[3];
            *flag = finish_row<DF, F32, COH>(a, v, cnt, r, ld<COH>(a.Rc + v), a.out_cnt[v],
                                             DF && COH ? ld<COH>(a.xstamp + v) : 0u, acc)
                        ? 1 : 0;
        }
    }
    __syncthreads();
    if (DF && *flag) {
        const uint32_t sv = a.sbase + (uint32_t)a.it + 1;
        if (sparse && !acc.plain && !heavy_in_sparse(a, a.out_cnt[v])) {
            mark_out_row<true, COH>(a, v, t, T, sv);
        } else {
            if (sparse && t == 0) st<COH>(&a.ctl->force_dense, 1u);
            mark_out_row<false, COH>(a, v, t, T, sv);
        }
    }
    __syncthreads();
}

// Fold a max and kCounters sums over a workgroup of W waves; thread 0 gets
// the result.  Waves fold with shuffles, then the wave results are combined
// in a fixed order.
template <int W = kWavesPerBlock>
__device__ __forceinline__ void block_fold(double &dr, double &rm, unsigned long long (&c)[kCounters],
                                  double *wdr, double *wrm, unsigned long long (*wc)[kCounters])
{
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        dr = fmax(dr, __shfl_xor(dr, off, kWave));
        rm = fmax(rm, __shfl_xor(rm, off, kWave));
#pragma unroll
        for (int j = 0; j < kCounters; j++) c[j] += __shfl_xor(c[j], off, kWave);
    }
    const int wave = threadIdx.x / kWave;
    if (lane_id() == 0) {
        wdr[wave] = dr;
        wrm[wave] = rm;
#pragma unroll
        for (int j = 0; j < kCounters; j++) wc[wave][j] = c[j];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < W; w++) {
            dr = fmax(dr, wdr[w]);
            rm = fmax(rm, wrm[w]);
#pragma unroll
            for (int j = 0; j < kCounters; j++) c[j] += wc[w][j];
        }
    }
    __syncthreads();
}

// Work of one iteration: per class, the list and its length; wave units
// of classes 5..0 and then of the self-loop-only rows (their own id
// range; class lists hold them in class 0), in that order; block units are
// the class-6 rows.
constexpr uint32_t kSkips = 16;
struct Plan {
    double ftol;                // frontier tolerance in effect
    uint32_t plain;             // Ctl::plain_marks
    uint32_t cnt[kBins];
    const int32_t *list[kBins]; // class lists (sparse), or NULL: the id range from id0
    uint32_t id0[kBins];
    uint32_t loop_cnt;          // the self-loop rows' id range (full schedule, DF)
    uint32_t loop_id0;
    uint32_t ustart[kBins];     // k < kBins - 1: class kBins - 2 - k; kBins - 1: loop rows
    uint32_t per[kBins];        // resident loop: rows of a wave unit of each class
    uint32_t lo[kSkips];        //   workgroups that sit out each of the first rounds
    uint32_t nwu, nbu;
    uint32_t nlong;             // resident loop: block rows after which none is long
};

// `snap`: the lengths of the class lists this iteration processes (sparse).
__device__ __forceinline__ void make_plan(const IterArgs &a, const Ctl *ctl, bool sparse, bool df,
                                          const uint32_t *snap, Plan &p)
{
    // a negative frontier tolerance asks for the call's adaptive choice
    p.ftol = a.ftol >= 0.0 ? a.ftol : ctl->ftol_used;
    p.plain = ctl->plain_marks;
    for (int b = 0; b < kBins; b++) {
        if (sparse) {
            p.cnt[b] = snap[b];
            p.list[b] = a.bins + (size_t)b * a.n_stride;
            p.id0[b] = 0;
        } else {
            // class b is the id range [cls[kBins - 1 - b], cls[kBins - b])
            p.cnt[b] = ctl->cls[kBins - b] - ctl->cls[kBins - 1 - b];
            p.list[b] = nullptr;
            p.id0[b] = ctl->cls[kBins - 1 - b];
        }
    }
    p.loop_cnt = sparse ? 0u : ctl->cls[kBins + 1] - ctl->cls[kBins];
    p.loop_id0 = ctl->cls[kBins];
    if (!df) {
        // every row is processed: class 0 and the self-loop rows are one
        // id range, walked as class 0
        p.cnt[0] += p.loop_cnt;
        p.loop_cnt = 0;
    }
    uint32_t acc = 0;
    for (int k = 0; k < kBins - 1; k++) {
        const int b = kBins - 2 - k;
        const uint32_t rows = kWave / group_of(b);
        p.ustart[k] = acc;
        acc += (p.cnt[b] + rows - 1) / rows;
    }
    p.ustart[kBins - 1] = acc;
    acc += (p.loop_cnt + kWave - 1) / kWave;
    p.nwu = acc;
    p.nbu = p.cnt[kBins - 1];
}

// log2 of the rows of a full wave unit of class b < kBins - 1.
__device__ __forceinline__ int lg_rows(int b)
{
    return b < 4 ? 6 - b : 5 - b;
}

// The same by one wave, for `waves` waves.  While the class lists hold fewer
// rows than the waves could take, a wave unit takes fewer rows: a wave's
// rows expand one round of out-edges after another, so a small frontier is
// done soonest when it is spread over all waves.  With `pairs` a unit of the
// full schedule takes twice the rows (wave_pair).  p.ftol and p.plain are
// left alone (they hold for the whole call).
// On the full schedule block rows follow decreasing in-degree too: workgroup
// b of G has long rows b, b + G, ..., and four of the others at a time, so the
// first ones are busy longest.  A long row takes about as long as
// 1 + in-edges / 16384 rounds of wave units (R-MAT scales 16 and 18), four of
// the others one.  In FP32 every row takes 256 threads, four rows at a time of
// which the first is the longest, and 1 + in-edges / 4096 rounds.  A workgroup
// sits out as many rounds as its rows take beyond those of the last workgroup.
__device__ __forceinline__ void make_plan_wave(const IterArgs &a, const Ctl *ctl, bool sparse, bool df,
                                               bool f32, bool pairs, const uint32_t *snap, uint32_t G,
                                               uint32_t waves, Plan &p)
{
    const int lane = (int)fresh((uint32_t)lane_id());
    const int b = lane < kBins ? lane : kBins - 1;
    uint32_t id0 = 0, cnt, loops = 0;
    if (sparse) {
        cnt = snap[b];
    } else {
        id0 = ctl->cls[kBins - 1 - b];
        cnt = ctl->cls[kBins - b] - id0;
        loops = ctl->cls[kBins + 1] - ctl->cls[kBins];
        if (!df && b == 0) cnt += loops;
        if (!df) loops = 0;
    }
    const bool unit = lane < kBins - 1;
    // full schedule, wave_pair: twice the rows
    const int two = pairs && !sparse ? 1 : 0;
    int lg = unit ? lg_rows(b) + two : 0;
    uint32_t n = unit ? (cnt + (1u << lg) - 1) >> lg : 0u;
    if (sparse) {
        uint32_t tot = n;
#pragma unroll
        for (int off = 4; off > 0; off >>= 1) tot += __shfl_xor(tot, off, 8);
        if (tot && tot < waves) {
            // the largest halving of the units that the waves take at once
            int s = __clz((int)tot) - __clz((int)waves);
            if (tot << s > waves) s--;
            lg = max(0, lg - s);
            n = unit ? (cnt + (1u << lg) - 1) >> lg : 0u;
        }
    }
    // units of the classes above this one come first
    uint32_t before = 0, tot = 0;
#pragma unroll
    for (int j = 0; j < kBins - 1; j++) {
        const uint32_t x = __shfl(n, j);
        tot += x;
        if (j > b) before += x;
    }
    if (lane < kBins) {
        p.cnt[b] = cnt;
        p.list[b] = sparse ? a.bins + (size_t)b * a.n_stride : nullptr;
        p.id0[b] = id0;
        p.per[b] = 1u << lg;
        p.ustart[unit ? kBins - 2 - b : kBins - 1] = unit ? before : tot;
        if (!unit) {
            p.loop_cnt = loops;
            if (!sparse) p.loop_id0 = ctl->cls[kBins];
            p.nwu = tot + ((loops + (kWave << two) - 1) >> (6 + two));
            p.nbu = cnt;
        }
    }
    const uint32_t nbu = __shfl(cnt, kBins - 1), first = __shfl(id0, kBins - 1);
    uint32_t lo[kSkips] = {0}, nlong = nbu;
    if (!sparse && nbu) {
        nlong = 0;
        for (uint32_t u0 = 0; u0 < nbu; u0 += kWave) {
            const unsigned long long m =
                __ballot(u0 + lane < nbu && a.in_cnt[first + u0 + lane] > kLongRow);
            if (m) nlong = u0 + kWave - __clzll((long long)m);
        }
        auto rounds = [&](uint32_t w) {
            uint32_t c = 0;
            if (f32) {
                for (uint32_t u = w; u < nbu; u += 4 * G) c += 1 + (a.in_cnt[first + u] >> 12);
                return c;
            }
            for (uint32_t u = w; u < nlong; u += G) c += 1 + (a.in_cnt[first + u] >> 14);
            for (uint32_t u = nlong + (w + G - nlong % G) % G * 4; u < nbu; u += 4 * G) c++;
            return c;
        };
        const uint32_t least = rounds(G - 1);
        for (uint32_t w0 = 0; w0 < G; w0 += kWave) {
            const uint32_t c = w0 + lane < G ? rounds(w0 + lane) : 0u;
#pragma unroll
            for (uint32_t r = 0; r < kSkips; r++) lo[r] += (uint32_t)__popcll(__ballot(c > least + r));
        }
    }
    if (lane == 0) p.nlong = nlong;
#pragma unroll
    for (uint32_t r = 0; r < kSkips; r++)
        if (lane == 0) p.lo[r] = min(lo[r], G - 1);
}

// Workgroups that have work in an iteration: 0 .. active-1.  With no work
// at all, workgroup 0 alone records the (empty) iteration.
template <int NW = kWavesPerBlock>
__device__ __forceinline__ uint32_t active_blocks(const Plan &p, uint32_t grid)
{
    constexpr uint32_t S = NW / kWavesPerBlock;    // rows of the block class at once
    const uint32_t wblocks = (p.nwu + NW - 1) / NW;
    return max(1u, max(min(grid, (p.nbu + S - 1) / S), min(grid, wblocks)));
}

// Shared memory of one workgroup of an iteration.
template <int NW = kWavesPerBlock>
struct IterSharedT {
    Plan plan;
    double red[NW / kWavesPerBlock * kLongFolds];
    int flag[NW / kWavesPerBlock];
    double wdr[NW], wrm[NW];
    unsigned long long wc[NW][kCounters];
};
using IterShared = IterSharedT<>;

// Threads of the per-iteration fold.  Its time is the launch and one round
// trip to the slots, not the fold: 1024 threads (one round of loads for a
// full grid) were no faster on R-MAT scale 22 and cost ~3 us per iteration
// more on small frontiers, and loading the control-block fields beside the
// slots left it at 4.3 us.
#ifndef DFPR_FINAL_THREADS
#define DFPR_FINAL_THREADS 256
#endif
constexpr int kFinalThreads = DFPR_FINAL_THREADS;
constexpr int kFinalWaves = kFinalThreads / kWave;

// Shared memory of the per-iteration fold.
struct FinalShared {
    int copy;
    double wdr[kFinalWaves], wrm[kFinalWaves];
    unsigned long long wc[kFinalWaves][kCounters];
};

// f with the lanes per row of class b < kBins - 1, and whether the unit is one of
// the self-loop rows.
template <class F>
__device__ __forceinline__ void by_class(int b, bool loop, F &&f)
{
    using std::integral_constant;
    if (loop) {
        f(integral_constant<int, group_of(0)>(), std::true_type());
        return;
    }
    switch (b) {
    case 0: f(integral_constant<int, group_of(0)>(), std::false_type()); break;
    case 1: f(integral_constant<int, group_of(1)>(), std::false_type()); break;
    case 2: f(integral_constant<int, group_of(2)>(), std::false_type()); break;
    case 3: f(integral_constant<int, group_of(3)>(), std::false_type()); break;
    case 4: f(integral_constant<int, group_of(4)>(), std::false_type()); break;
    default: f(integral_constant<int, group_of(5)>(), std::false_type());
    }
}

// Workgroup blk of G processes its share of the rows of the plan in sh.  A
// launch per iteration gives a workgroup NW neighbouring wave units at a
// time.  The resident loop (COH) deals the units out one workgroup after the
// other, so that a few long units, or a frontier of few units, are spread
// over all compute units.
template <bool DF, bool F32, int NW, bool COH, bool PAIRS = false>
__device__ __forceinline__ void iter_rows(const IterArgs &a, const Hub &hub, uint32_t blk, uint32_t G,
                                          IterSharedT<NW> &sh, bool check, bool sparse, Acc &acc)
{
    const uint32_t nbu = sh.plan.nbu, nwu = sh.plan.nwu;
    const int wave = threadIdx.x / kWave;
    const int32_t *blist = sh.plan.list[kBins - 1];
    // sub-blocks of T threads take rows from u0 on, one each and `apart` ids
    // from each other, up to n
    auto block_rows = [&](auto threads, uint32_t u0, uint32_t n, uint32_t apart = 1) {
        constexpr int T = decltype(threads)::value;
        constexpr uint32_t S = NW * kWave / T;
        const uint32_t sub = threadIdx.x / T;
        for (; u0 < n; u0 += G * S) {
            const uint32_t u = u0 + sub * apart;
            const bool valid = u < n;
            const int32_t v = !valid ? 0 : blist ? ld<COH>(blist + u)
                                                 : (int32_t)(sh.plan.id0[kBins - 1] + u);
            block_row<DF, F32, COH, T>(a, hub, v, valid, check, sparse, acc,
                                       sh.red + sub * kLongFolds, sh.flag + sub);
        }
    };
    constexpr std::integral_constant<int, kBlock> quarter{};
    if constexpr (COH && !F32) {
        // the long rows one per workgroup, then, from the next workgroup on,
        // the others four at a time
        const uint32_t nlong = sh.plan.nlong;
        block_rows(std::integral_constant<int, kLongParts>(), blk, nlong);
        block_rows(quarter, nlong + (blk + G - nlong % G) % G * (NW * kWave / kBlock), nbu);
    } else if constexpr (COH) {
        // The longest rows in workgroups of their own, which then sit out
        // units (make_plan_wave): with four rows in a row each, workgroup 0
        // was busy 113 us of an iteration and the others 85 (R-MAT, 1.5e6
        // vertices; the call 12.27 -> 10.63 ms).
        block_rows(quarter, blk, nbu, G);
    } else {
        block_rows(quarter, blk * (NW * kWave / kBlock), nbu);
    }
    auto run = [&](uint32_t u) {
        int k = 0;
        while (k + 1 < kBins && u >= sh.plan.ustart[k + 1]) k++;
        const bool loop = k == kBins - 1;
        const int b = loop ? 0 : kBins - 2 - k;
        const int32_t *list = loop ? nullptr : sh.plan.list[b];
        const uint32_t id0 = loop ? sh.plan.loop_id0 : sh.plan.id0[b];
        const uint32_t cnt = loop ? sh.plan.loop_cnt : sh.plan.cnt[b];
        // rows of a full unit of L lanes a row; resident loop: of this plan
        auto rows = [&](uint32_t L) {
            return !COH ? kWave / L : loop ? (uint32_t)kWave << (PAIRS && !sparse ? 1 : 0) : sh.plan.per[b];
        };
        auto unit = [&](auto lanes, auto self) -> UnitRow {
            constexpr int L = decltype(lanes)::value;
            const uint32_t per = rows(L);
            return wave_unit<L, DF, F32, COH, decltype(self)::value>(
                a, hub, list, id0, cnt, (u - sh.plan.ustart[k]) * per, per, check);
        };
        if constexpr (PAIRS) {
            if (!sparse) {
                UnitRow pair[2];
                by_class(b, loop, [&](auto lanes, auto self) {
                    wave_pair<decltype(lanes)::value, DF, decltype(self)::value>(
                        a, hub, id0, cnt, (u - sh.plan.ustart[k]) * rows(1), check, pair);
                });
#pragma unroll 1
                for (int p = 0; p < 2; p++)
                    finish_unit<DF, F32, COH>(a, p ? pair[1] : pair[0], sparse, acc);
                return;
            }
        }
        // The rest of a unit: one copy of its code for all classes, but with each
        // class where launches expand (one copy there: a Dynamic Frontier call
        // on a 2900 x 2900 grid 12.06 instead of 11.85 ms; one per class in a
        // sweep: R-MAT with 2.5e6 vertices, Static 15.76 instead of 15.60 ms).
        if constexpr (COH || !DF) {
            UnitRow row;
            by_class(b, loop, [&](auto lanes, auto self) { row = unit(lanes, self); });
            finish_unit<DF, F32, COH>(a, row, sparse, acc);
        } else {
            by_class(b, loop, [&](auto lanes, auto self) {
                finish_unit<DF, F32, COH>(a, unit(lanes, self), sparse, acc);
            });
        }
    };
    if constexpr (!COH) {
        for (uint32_t u = blk * NW + wave; u < nwu; u += G * NW) run(u);
    } else {
        // a round is one unit per wave of workgroups lo .. G - 1; those
        // before lo had longer block rows and sit it out
        uint32_t r = 0;
        for (uint32_t u0 = 0; u0 < nwu; r++) {
            const uint32_t lo = r < kSkips ? sh.plan.lo[r] : 0u;
            const uint32_t w = G - lo;
            const uint32_t u = u0 + (blk - lo) + wave * w;
            if (blk >= lo && u < nwu) run(u);
            u0 += w * NW;
        }
    }
}

// One workgroup's share of an iteration of one graph: workgroup blk of the
// G workgroups given to the graph.  Its results are folded into slot
// blk mod kFoldSlots.
template <bool DF, bool F32, int NW = kWavesPerBlock>
__device__ __forceinline__ void iter_body(const IterArgs &a, uint32_t blk, uint32_t G,
                                 IterSharedT<NW> &sh, double *hub_lds = nullptr)
{
    const Ctl *ctl = a.ctl;
    if (ctl->done || (F32 && ctl->phase_end)) return;
    const int par = a.it & 1;
    const bool sparse = DF && !ctl->dense;
    const bool check = DF && !sparse;
    if (threadIdx.x == 0) make_plan(a, ctl, sparse, DF, ctl->snap[par], sh.plan);
    __syncthreads();
    if (blk >= active_blocks<NW>(sh.plan, G)) return;
    // a sweep over the full schedule reads the hub contributions from LDS
    Hub hub{hub_lds, reinterpret_cast<const float *>(hub_lds), 0u};
    if (hub_lds && a.hub && !sparse) {
        hub.n = min(a.hub, (uint32_t)a.n);
        if (F32) {
            float *f = reinterpret_cast<float *>(hub_lds);
            for (uint32_t k = threadIdx.x; k < hub.n; k += NW * kWave) f[k] = a.C32c[k];
        } else {
            for (uint32_t k = threadIdx.x; k < hub.n; k += NW * kWave) hub_lds[k] = a.Cc[k];
        }
        __syncthreads();
    }

    Acc acc;
    acc.ftol = sh.plan.ftol;
    acc.plain = sh.plan.plain != 0;
    iter_rows<DF, F32, NW, false>(a, hub, blk, G, sh, check, sparse, acc);

    double dr = acc.dr_max, rm = acc.r_max;
    unsigned long long c[kCounters];
#pragma unroll
    for (int j = 0; j < kCounters; j++) c[j] = acc.c[j];
    block_fold<NW>(dr, rm, c, sh.wdr, sh.wrm, sh.wc);
    if (threadIdx.x == 0) {
        // non-negative doubles order like their bit patterns
        const uint32_t slot = blk % kFoldSlots;
        atomicMax(reinterpret_cast<unsigned long long *>(a.dr_part) + slot,
                  (unsigned long long)__double_as_longlong(dr));
        atomicMax(reinterpret_cast<unsigned long long *>(a.rmax_part) + slot,
                  (unsigned long long)__double_as_longlong(rm));
#pragma unroll
        for (int j = 0; j < kCounters; j++)
            if (c[j]) atomicAdd(&a.cnt_part[slot * kCounters + j], c[j]);
    }
}

// The state after iteration a.it, from its folded results: the control
// block's statistics, convergence or the cap, the next iteration's class
// lists and walk.  One thread.  In the FP32 phase of the precision form,
// reaching tol or the FP32 resolution of the ranks ends the phase instead of
// the call.  `lists`: the class lists' lengths and Ctl::force_dense.
__device__ __forceinline__ void final_step(const IterArgs &a, Ctl *ctl, const uint32_t *lists, bool sparse,
                                           bool f32, double dr, double rm)
{
    const int par = a.it & 1;
    ctl->iterations = a.it + 1;
    ctl->final_linf = dr;
    ctl->final_rmax = rm;
    if (sparse) {
        unsigned long long before = 0, after = 0;
#pragma unroll
        for (int b = 0; b < kBins; b++) {
            before += ctl->snap[par][b];
            after += lists[b];
            ctl->snap[par ^ 1][b] = lists[b];
        }
        ctl->marked += after - before;
        if (after > a.sparse_limit || lists[kBins]) ctl->dense = 1;
    }
    if (f32) {
        // FP32 contributions carry a relative rounding error of 2^-24;
        // changes below about 2^-22 of the largest rank are noise.  A
        // Delta R that stops falling counts as a stall only near that
        // floor (early on it can rise while the frontier grows).
        const double floor32 = rm * 0x1p-22;
        const bool stalled = ctl->phase_iters >= 3 && dr >= 0.97 * ctl->prev_linf &&
                             dr <= rm * 0x1p-16;
        ctl->phase_iters += 1;
        if (dr <= a.tol || dr <= floor32 || stalled) ctl->phase_end = 1;
        if (a.it + 1 >= a.max_iters) ctl->done = 1;
    } else {
        const bool conv = dr <= a.tol;
        if (conv) ctl->converged = 1;
        if (conv || a.it + 1 >= a.max_iters) ctl->done = 1;
    }
    ctl->prev_linf = dr;
}

// The control block to a host-visible copy by one wave of a workgroup whose
// thread 0 made the last updates, after a workgroup barrier.
__device__ __forceinline__ void ctl_to_mirror(const Ctl *ctl, Ctl *mirror)
{
    constexpr int words = (int)(sizeof(Ctl) / 4);
    const uint32_t *src = reinterpret_cast<const uint32_t *>(ctl);
    uint32_t *dst = reinterpret_cast<uint32_t *>(mirror);
    for (int i = threadIdx.x; i < words; i += kWave) dst[i] = ld<true>(src + i);
}

// After each iteration (one workgroup): fold the slots the iteration's
// workgroups left, decide convergence or the cap, and prepare the next
// iteration.  The launch boundary orders it after k_iter.
// The control block goes to the host mirror when `last` (the last launch
// the host queued before it next waits) or when this step ends the call or
// the phase: later launches then return at once.
__device__ __forceinline__ void final_body(const IterArgs &a, bool df, bool f32, FinalShared &sh, bool last)
{
    Ctl *ctl = a.ctl;
    if (ctl->done || (f32 && ctl->phase_end)) return;
    const bool sparse = df && !ctl->dense;
    double dr = 0.0, rm = 0.0;
    unsigned long long c[kCounters] = {0, 0, 0, 0};
    // each thread reads its slots and clears them for the next iteration
    for (uint32_t i = threadIdx.x; i < (uint32_t)kFoldSlots; i += kFinalThreads) {
        dr = fmax(dr, a.dr_part[i]);
        rm = fmax(rm, a.rmax_part[i]);
#pragma unroll
        for (int j = 0; j < kCounters; j++) c[j] += a.cnt_part[i * kCounters + j];
        a.dr_part[i] = 0.0;
        a.rmax_part[i] = 0.0;
#pragma unroll
        for (int j = 0; j < kCounters; j++) a.cnt_part[i * kCounters + j] = 0ull;
    }
    block_fold<kFinalWaves>(dr, rm, c, sh.wdr, sh.wrm, sh.wc);
    if (threadIdx.x == 0) {
        ctl->verts += c[0];
        ctl->edges += c[1];
        ctl->xverts += c[2];
        ctl->xedges += c[3];
        uint32_t lists[kBins + 1];
#pragma unroll
        for (int b = 0; b < kBins; b++) lists[b] = ctl->live[b];
        lists[kBins] = ctl->force_dense;
        final_step(a, ctl, lists, sparse, f32, dr, rm);
        sh.copy = a.mirror && (last || ctl->done || (f32 && ctl->phase_end));
    }
    __syncthreads();
    if (sh.copy && threadIdx.x < kWave) ctl_to_mirror(ctl, a.mirror);
}

}  // namespace dfpr
