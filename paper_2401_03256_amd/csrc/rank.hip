// Rank engines: Static, Naive-dynamic and Dynamic Frontier PageRank.
//
// One iteration of every engine is one launch of k_iter, which
//   - pulls Eq. 1 for the rows of the iteration: every vertex (Static,
//     Naive-dynamic) or the affected vertices (Dynamic Frontier);
//   - computes Delta r = |r - R[v]| and the L-inf maximum;
//   - (Dynamic Frontier) marks the out-neighbours of every row whose rank
//     moved by more than frontier_tol;
// followed by a one-workgroup launch of k_final that folds the slots the
// workgroups folded their results into and decides convergence
// (Delta R <= tol) or the iteration cap.
// The host enqueues iterations in chunks and reads the stop flag between
// chunks; launches issued after the stop flag is set return at once.  On
// small graphs, and while a frontier is small, the same iterations run inside
// one launch of k_resident instead (below).
//
// Work layout.  Rows are split by in-degree into classes; a class-b row is
// reduced by group_of(b) lanes of one wave (1, 2, 4, 8, 32 or 64 lanes) or,
// above 1024 in-edges, by a whole workgroup.  Internal ids follow
// decreasing in-degree at load, so each class is an id range, and a row
// keeps the class of its id for the life of the graph (Ctl::cls).
// Rows whose only in-entry was the self-loop form the last range.  Each
// lane loads kUnroll indices and then kUnroll contributions per round, so
// that many loads are in flight per wave.  Each lane sums its strided share
// of a row in order and the group folds the partial sums with a fixed
// butterfly, so the sum of a row depends on nothing but the row and its id.
//
// Marks.  stamp[v] holds the iteration, offset by a per-call base, from
// which v is affected: v is processed in iteration i iff
// base <= stamp[v] <= base + i.  Marks made in iteration i carry base+i+1,
// so they take effect from the next iteration (synchronous form), and a
// plain store suffices to make them.  Marks never go away within a call
// (Algorithm 1 has no unmarking step), and a vertex whose out-neighbours
// are all marked gains nothing from marking them again, so each vertex
// scans its out-row at most once per call (xstamp[v] == base afterwards).
//
// Two ways to walk the affected rows.  While few vertices are marked, the
// marking appends new vertices to per-class lists (sparse mode).  Once the
// lists pass a size limit, iterations walk every class's id range and skip
// rows whose stamp is out of range (dense mode, the "full schedule"); marks
// are then plain stores.  Expansions that would append more than the lists
// take (a row with a very long out-row, or a first frontier whose out-rows
// together pass the limit) also mark with plain stores, and the call walks
// the full schedule from the next iteration on.  Neither walk needs
// rebuilding when a batch changes in-degrees.
//
// Ranks are double-buffered (synchronous form, Section 4.2).  Both buffers
// hold identical values between calls; an iteration reads one and writes
// only its processed rows into the other.  Because marks only grow within a
// call, a row not processed in iteration i was not processed earlier in the
// call either, so the two buffers still agree there.  The contribution
// C[v] = R[v] / |out(v)| is stored beside each rank so the pull gathers one
// value per in-edge.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "common.h"
#include "engine.h"

namespace dfpr {


template <bool DF, bool F32>
__global__ __launch_bounds__(kBlock, DFPR_ITER_WAVES_PER_SIMD) void k_iter(IterArgs a)
{
    __shared__ IterShared sh;
#if DFPR_HUB
    __shared__ double hub[kHubRows];
    iter_body<DF, F32>(a, blockIdx.x, gridDim.x, sh, hub);
#else
    iter_body<DF, F32>(a, blockIdx.x, gridDim.x, sh);
#endif
}

// The full schedule in wide workgroups: more waves per workgroup, fewer
// workgroups per CU, the same 6 waves per SIMD as k_iter, and one larger
// LDS copy of the first contributions per workgroup instead of one of
// kHubRows per four waves.  Static and Naive-dynamic sweeps (Eq. 1 over
// every vertex) use 12 waves and 9216 entries (two workgroups per CU; about
// 34% of the gathers on R-MAT scale 22 read LDS instead of 18%, 4% less time
// per sweep).  Dynamic Frontier iterations on the full schedule use 8 waves
// and 6144 entries (three per CU; 12 waves left that kernel at the 80-VGPR
// cap with a spill and no gain, 8 give 1% per call), or 12288 FP32 entries
// in the FP32 phase of the precision form (2.5% per call at R-MAT scale 24).
// Results are bitwise those of k_iter: block-class rows keep their kBlock
// partition (see block_row).
#ifndef DFPR_WIDE
#define DFPR_WIDE 1
#endif
#ifndef DFPR_WIDE_HUB
#define DFPR_WIDE_HUB 9216
#endif
#ifndef DFPR_WIDE_F32_MUL
#define DFPR_WIDE_F32_MUL 2
#endif
#ifndef DFPR_WIDE_DF_HUB
#define DFPR_WIDE_DF_HUB 6144
#endif
constexpr int kWideWaves = 12, kWideDfWaves = 8;
constexpr uint32_t kWideHub = DFPR_WIDE_HUB, kWideDfHub = DFPR_WIDE_DF_HUB;

template <bool DF, bool F32, int NW, uint32_t HUB>
__global__ __launch_bounds__(NW * kWave, 6) void k_iter_wide(IterArgs a)
{
    __shared__ IterSharedT<NW> sh;
    __shared__ double hub[HUB];
    iter_body<DF, F32, NW>(a, blockIdx.x, gridDim.x, sh, hub);
}

// After each iteration (one workgroup): fold the slots the iteration's
// workgroups left, decide convergence or the cap, and prepare the next
// iteration.  The launch boundary orders it after k_iter.
__global__ __launch_bounds__(kFinalThreads) void k_final(IterArgs a, int df, int f32, int last)
{
    __shared__ FinalShared sh;
    final_body(a, df != 0, f32 != 0, sh, last != 0);
}

template <bool DF, bool F32, bool PAIRS>
__global__ __launch_bounds__(kResThreads) void k_resident(IterArgs a, ResArgs P)
{
    __shared__ ResLds lds;
    resident_body<DF, F32, PAIRS>(a, P, blockIdx.x, gridDim.x, lds);
}

// ---------------------------------------------------------------------------
// set-up kernels
// ---------------------------------------------------------------------------

// Clear the per-call loop state (not the batch-applier fields).  One thread.
__device__ inline void reset_ctl(Ctl *ctl)
{
    {
        for (int b = 0; b < kBins; b++) {
            ctl->live[b] = 0;
            ctl->snap[0][b] = ctl->snap[1][b] = 0;
        }
        ctl->done = 0;
        ctl->dense = 0;
        ctl->force_dense = 0;
        ctl->plain_marks = 0;
        ctl->phase_end = 0;
        ctl->phase_iters = 0;
        ctl->prev_linf = 0.0;
        ctl->renorm_scale = 1.0;
        ctl->iterations = 0;
        ctl->converged = 0;
        ctl->final_linf = 0.0;
        ctl->final_rmax = 0.0;
        ctl->edges = ctl->verts = 0;
        ctl->xverts = ctl->xedges = ctl->marked = 0;
        ctl->affected0 = ctl->affected = 0;
        ctl->err = 0;
        ctl->mk_light = ctl->mk_heavy = 0;
        ctl->reach = 0;
        for (int k = 0; k < 3; k++) ctl->qn[k] = ctl->qhn[k] = 0;
        ctl->loop_fail = 0;
        ctl->loop_closed = 0;
        ctl->reach0 = 0;
        ctl->ftol_used = 0.0;
    }
}

__global__ void k_reset(Ctl *ctl)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) reset_ctl(ctl);
}

// Adaptive frontier tolerance (the paper leaves the choice of tau_f by the
// nature of the batch to future work, Section 5.2.4 and the Conclusion).
// The initial marking measures how fast the frontier can grow: the mean
// out-degree g of the vertices it marked.  Mesh-like neighbourhoods (g <= 8)
// let the frontier creep outward over many iterations of changes far below
// tol, so expansion stops early (tau_f = tol/10); hub-rich ones (g > 64)
// reach most of the graph within a few iterations whatever tau_f is, so the
// accurate tol/1e5 costs little; the steps between take tol/100 ... tol/1e4.
// Integer comparisons only, so the choice is exact.
__host__ __device__ inline int adaptive_ftol_exponent(unsigned long long marked,
                                                      unsigned long long out_edges)
{
    if (marked == 0) return 5;
    return out_edges <= 8 * marked ? 1 : out_edges <= 16 * marked ? 2
         : out_edges <= 32 * marked ? 3 : out_edges <= 64 * marked ? 4 : 5;
}

// Freeze the lists built by the marking as iteration 0's snapshot and pick
// the walk of the first iteration.  One thread, after the marking (in the
// same launch with COH).
// `plain_limit`: entries the class lists may hold before an expansion that
// would append that many marks with plain stores instead.
template <bool COH>
__device__ inline void snap_ctl(Ctl *ctl, int32_t max_iters, uint32_t sparse_limit, uint32_t plain_limit,
                                int dense, double tol, double ftol)
{
    const unsigned long long marked = ld<COH>(&ctl->affected0), reach0 = ld<COH>(&ctl->reach0);
    if (ftol >= 0.0) {
        ctl->ftol_used = ftol;
    } else {
        const double p10[6] = {1.0, 1e1, 1e2, 1e3, 1e4, 1e5};
        ctl->ftol_used = tol / p10[adaptive_ftol_exponent(marked, reach0)];
    }
    unsigned long long tot = 0;
    for (int b = 0; b < kBins; b++) {
        const uint32_t l = ld<COH>(&ctl->live[b]);
        ctl->snap[0][b] = l;
        tot += l;
    }
    ctl->dense = (dense || ld<COH>(&ctl->dense) || tot > sparse_limit) ? 1 : 0;
    // a first frontier with more out-edges than the class lists take
    // would append most of them in its first expansions, one list
    // atomic per wave and round on counters that share a cache line;
    // its expansions mark with plain stores instead, and the call walks
    // the full schedule from the next iteration on
    ctl->plain_marks = reach0 > plain_limit ? 1 : 0;
    ctl->done = (ld<COH>(&ctl->err) || max_iters <= 0) ? 1 : 0;
}

__global__ void k_snap(Ctl *ctl, int32_t max_iters, uint32_t sparse_limit, int dense, Ctl *mirror,
                       double tol, double ftol)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        snap_ctl<false>(ctl, max_iters, sparse_limit, sparse_limit, dense, tol, ftol);
        if (mirror) __builtin_memcpy(mirror, ctl, sizeof(Ctl));
    }
}

__global__ void k_fill_u32(uint32_t *p, uint64_t len, uint32_t value)
{
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < len;
         i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = value;
}

// R[b][v] = (src ? src[v] : 1/n) and C[b][v] = R[b][v] / |out(v)|, b = 0, 1.
__global__ void k_init_ranks(int32_t n, const double *src, double *R0, double *R1, double *C0,
                             double *C1, const uint32_t *out_cnt)
{
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        const double r = src ? src[v] : 1.0 / (double)n;
        const double c = r / (double)out_cnt[v];
        R0[v] = r;
        R1[v] = r;
        C0[v] = c;
        C1[v] = c;
    }
}

__global__ void k_copy2(int32_t n, const double *a, double *a2, const double *b, double *b2)
{
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        a2[v] = a[v];
        b2[v] = b[v];
    }
}

// Flag (and abort the loop) if a batch id lies outside [0, n).
__global__ void k_validate(int32_t n, int64_t nd, const int32_t *ds, const int32_t *dd,
                           int64_t ni, const int32_t *is, const int32_t *id, Ctl *ctl)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= nd + ni) return;
    const int32_t s = i < nd ? ds[i] : is[i - nd];
    const int32_t d = i < nd ? dd[i] : id[i - nd];
    if (s < 0 || s >= n || d < 0 || d >= n) {
        atomicOr(&ctl->err, 1u);
        ctl->done = 1;
    }
}

// Initial marking (Section 4.1.1, Algorithm 1): every batch edge (u, v)
// marks G^t.out(u), and a deletion also marks v, which was in
// G^{t-1}.out(u).  Marks are stamps equal to the call's base.  A source
// whose out-row has been scanned gets its expansion stamp, so it never
// scans that row again in this call.
//
// Claim pass, one thread per batch entry: the first entry of each distinct
// source claims it through its expansion stamp; claimed sources go to a
// light list (out-row scanned by one wave) or a heavy list (scanned by the
// whole grid in workgroup-sized chunks), and their out-degrees are summed.
constexpr uint32_t kHeavyRow = 2048;   // out-rows longer than this use the grid
constexpr uint32_t kHeavySeg = 2048;   // heavy vertices whose chunk offsets sit in LDS at once

struct HeavyShared {
    uint32_t pre[kHeavySeg + 1];       // chunk offsets of a segment of heavy vertices
    uint32_t part[kBlock];
};

// Walk the out-rows of the heavy vertices list[0 .. nh) in chunks of kBlock
// out-edges: chunk c of the concatenated rows goes to workgroup
// c mod gridDim.x.  Each workgroup finds the vertex of a chunk by binary
// search over the chunk offsets, which it builds in LDS for up to
// kHeavySeg vertices at a time, so no workgroup walks the list serially.
// visit(x) is called by every thread of the workgroup with the same trip
// count (x < 0: no vertex).
template <class F>
__device__ inline void walk_heavy(const IterArgs &a, const int32_t *list, uint32_t nh,
                                  HeavyShared &sh, F &&visit)
{
    constexpr uint32_t per = kHeavySeg / kBlock;
    for (uint32_t h0 = 0; h0 < nh; h0 += kHeavySeg) {
        const uint32_t seg = min(kHeavySeg, nh - h0);
        // per thread: chunk counts of `per` consecutive vertices, then a scan
        // of the thread totals
        uint32_t cnt[per], tot = 0;
#pragma unroll
        for (uint32_t j = 0; j < per; j++) {
            const uint32_t i = threadIdx.x * per + j;
            cnt[j] = i < seg ? (a.out_cnt[list[h0 + i]] + kBlock - 1) / kBlock : 0u;
            tot += cnt[j];
        }
        sh.part[threadIdx.x] = tot;
        __syncthreads();
        for (int o = 1; o < kBlock; o <<= 1) {
            const uint32_t t = threadIdx.x >= (uint32_t)o ? sh.part[threadIdx.x - o] : 0u;
            __syncthreads();
            sh.part[threadIdx.x] += t;
            __syncthreads();
        }
        uint32_t run = sh.part[threadIdx.x] - tot;
#pragma unroll
        for (uint32_t j = 0; j < per; j++) {
            const uint32_t i = threadIdx.x * per + j;
            if (i < seg) sh.pre[i] = run;
            run += cnt[j];
        }
        if (threadIdx.x == kBlock - 1) sh.pre[seg] = sh.part[kBlock - 1];
        __syncthreads();
        const uint32_t total = sh.pre[seg];
        for (uint32_t c = blockIdx.x; c < total; c += gridDim.x) {
            uint32_t lo = 0, hi = seg;      // last h with pre[h] <= c
            while (hi - lo > 1) {
                const uint32_t mid = (lo + hi) / 2;
                if (sh.pre[mid] <= c) lo = mid;
                else hi = mid;
            }
            const int32_t u = list[h0 + lo];
            const uint32_t k = (c - sh.pre[lo]) * kBlock + threadIdx.x;
            const uint32_t oc = a.out_cnt[u];
            visit(k < oc ? a.out_idx[a.out_beg[u] + k] : -1);
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(kBlock) void k_mark_claim(IterArgs a, int64_t nd, const int32_t *ds,
                                                       int64_t ni, const int32_t *is,
                                                       int32_t *light, int32_t *heavy)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    int32_t u = -1;
    if (i < nd + ni) u = i < nd ? ds[i] : is[i - nd];
    bool take = false;
    uint32_t oc = 0;
    if (u >= 0 && u < a.n && a.xstamp[u] != a.sbase) {
        take = atomicMax(&a.xstamp[u], a.sbase) < a.sbase;
        if (take) oc = a.out_cnt[u];
    }
    const bool big = take && oc > kHeavyRow;
    const int lane = lane_id();
    const unsigned long long below = (1ull << lane) - 1ull;
    const unsigned long long ml = __ballot(take && !big), mh = __ballot(big);
    unsigned long long r = oc;
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) r += __shfl_xor(r, off, kWave);
    uint32_t bl = 0, bh = 0;
    if (lane == 0) {
        if (ml) bl = atomicAdd(&a.ctl->mk_light, (uint32_t)__popcll(ml));
        if (mh) bh = atomicAdd(&a.ctl->mk_heavy, (uint32_t)__popcll(mh));
        if (r) atomicAdd(&a.ctl->reach, r);
    }
    bl = __shfl(bl, 0);
    bh = __shfl(bh, 0);
    if (take && !big) light[bl + __popcll(ml & below)] = u;
    if (big) heavy[bh + __popcll(mh & below)] = u;
}

// Mark x (x < 0: no vertex).  Every lane of the wave calls it.  Lane 0
// counts the new marks in `mine` and, in `deg`, their out-edges.
__device__ inline void mark_one(const IterArgs &a, int32_t x, bool append,
                                unsigned long long &mine, unsigned long long &deg)
{
    bool nw = false;
    if (x >= 0 && a.stamp[x] < a.sbase) nw = atomicMax(&a.stamp[x], a.sbase) < a.sbase;
    const unsigned long long m = __ballot(nw);
    unsigned long long d = nw ? a.out_cnt[x] : 0u;
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) d += __shfl_xor(d, off, kWave);
    if (lane_id() == 0) {
        mine += __popcll(m);
        deg += d;
    }
    if (append) {
        const int cls = nw ? class_of_id(a, x) : 0;
        append_to_bins(nw, x, cls, a.ctl, a.bins, a.n_stride);
    }
}

// Marking pass: deletion targets, then light sources one wave each, then
// heavy sources in chunks of kBlock out-edges spread over the grid.  The
// class lists are filled (sparse mode) unless `dense` is set or the claimed
// sources reach more vertices than the sparse limit; the decision goes to
// the control block for the iterations.  Every loop bound is uniform
// within a wave.  With `snap` the last workgroup of the grid takes the
// snapshot of iteration 0.  A call that is over with it (an id outside [0, n),
// or no iteration allowed) has no iteration that would leave the control block
// in the host's copy, so it goes there from here.
// Bound by the latency of scattered stamps, so the waves in flight count.  A SIMD
// has 800 scalar registers and a wave gets 16 on top of its own for the trap
// handler: above 80 an eighth of the 2048 workgroups runs after the others.
// Capped at 80 against the 84 the snapshot's code brings it to: 2^22-vertex R-MAT,
// 694000 changes, 798 -> 567 us; 3000 x 3000 grid, 459000 changes, 384 -> 236 us.
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_num_sgpr(80)))
void k_mark_initial(IterArgs a, int64_t nd, const int32_t *dd, const int32_t *light,
                    const int32_t *heavy, int dense, int snap, uint32_t plain_limit)
{
    __shared__ unsigned long long s_new, s_deg;
    __shared__ HeavyShared hs;
    __shared__ int s_last, s_over;
    Ctl *ctl = a.ctl;
    const bool dn = dense || ctl->reach + (unsigned long long)nd > a.sparse_limit;
    const bool append = !dn;
    if (!ctl->err) {
        if (blockIdx.x == 0 && threadIdx.x == 0 && dn) st<true>(&ctl->dense, 1u);
        if (threadIdx.x == 0) s_new = s_deg = 0;
        __syncthreads();
        const int lane = lane_id();
        const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kWave;
        const int64_t waves = (int64_t)gridDim.x * kWavesPerBlock;
        unsigned long long mine = 0, mdeg = 0;
        for (int64_t b0 = wave * kWave; b0 < nd; b0 += waves * kWave) {
            const int64_t i = b0 + lane;
            mark_one(a, i < nd ? dd[i] : -1, append, mine, mdeg);
        }
        const uint32_t nl = ctl->mk_light, nh = ctl->mk_heavy;
        for (int64_t w = wave; w < nl; w += waves) {
            const int32_t u = light[w];
            const uint32_t ob = a.out_beg[u], oc = a.out_cnt[u];
            for (uint32_t kb = 0; kb < oc; kb += kWave) {
                const uint32_t k = kb + lane;
                mark_one(a, k < oc ? a.out_idx[ob + k] : -1, append, mine, mdeg);
            }
        }
        walk_heavy(a, heavy, nh, hs, [&](int32_t x) { mark_one(a, x, append, mine, mdeg); });
        if (lane == 0 && mine) {
            atomicAdd(&s_new, mine);
            atomicAdd(&s_deg, mdeg);
        }
        __syncthreads();
        if (threadIdx.x == 0 && s_new) {
            atomicAdd(&ctl->affected0, s_new);
            atomicAdd(&ctl->reach0, s_deg);
        }
    }
    if (!snap || !last_block(ctl->tick, &s_last)) return;
    if (threadIdx.x == 0) {
        snap_ctl<true>(ctl, a.max_iters, a.sparse_limit, plain_limit, dense, a.tol, a.ftol);
        s_over = ctl->done != 0;
        drain_stores();
    }
    __syncthreads();
    if (s_over && threadIdx.x < kWave) ctl_to_mirror(ctl, a.mirror);
}

// The start of a call in one launch: workgroup 0 clears the loop state and,
// for a batch of at most kSmallBatch entries, stages, checks and claims it
// (what k_map_ids4, k_validate and k_mark_claim do for larger ones); the other
// workgroups load the starting ranks.  Each of these kernels alone does
// nothing for most of its 2-5 us, and the dispatch between them costs as much
// again.
struct BeginArgs {
    int64_t nd, ni;             // the batch, 0 entries: none, or staged elsewhere
    const int32_t *src[4];      // its four arrays in the caller's ids
    const int32_t *ext2int, *int2ext;
    int32_t *staged;            // the four arrays in internal ids
    int32_t *light, *heavy;     // claimed sources
    int snap;                   // 1: no marking follows; take the snapshot here
    int dense;                  //   with the full schedule
    int ranks;                  // 1: from prev, 2: uniform, 0: as they are
    const double *prev;         // caller's order
    double *R0, *R1, *C0, *C1;
    const double *Ccur;         // contributions of the resident ranks
    float *A, *B;               // FP32 copies of the contributions (nullable)
};

constexpr int kBeginThreads = 1024;
static_assert(kSmallBatch <= kBeginThreads, "one batch entry per thread");

__global__ __launch_bounds__(kBeginThreads) void k_begin(IterArgs a, BeginArgs b)
{
    if (blockIdx.x > 0) {
        const int64_t step = (int64_t)(gridDim.x - 1) * kBeginThreads;
        for (int64_t v = (int64_t)(blockIdx.x - 1) * kBeginThreads + threadIdx.x; v < a.n; v += step) {
            double c;
            if (b.ranks) {
                const double r = b.ranks == 1 ? b.prev[b.int2ext[v]] : 1.0 / (double)a.n;
                c = r / (double)a.out_cnt[v];
                b.R0[v] = r;
                b.R1[v] = r;
                b.C0[v] = c;
                b.C1[v] = c;
            } else {
                c = b.Ccur[v];
            }
            if (b.A) {
                b.A[v] = (float)c;
                b.B[v] = (float)c;
            }
        }
        return;
    }
    __shared__ uint32_t s_light, s_heavy, s_err;
    __shared__ unsigned long long s_reach;
    if (threadIdx.x == 0) {
        reset_ctl(a.ctl);
        s_light = s_heavy = s_err = 0;
        s_reach = 0;
    }
    __syncthreads();
    const int64_t tot = b.nd + b.ni, i = threadIdx.x;
    if (i < tot) {
        const bool del = i < b.nd;
        const int64_t k = del ? i : i - b.nd;
        const int32_t s = (del ? b.src[0] : b.src[2])[k], d = (del ? b.src[1] : b.src[3])[k];
        const int32_t u = s >= 0 && s < a.n ? b.ext2int[s] : -1;
        const int32_t w = d >= 0 && d < a.n ? b.ext2int[d] : -1;
        int32_t *to = b.staged + (del ? 0 : 2 * b.nd);
        to[k] = u;
        to[k + (del ? b.nd : b.ni)] = w;
        if (u < 0 || w < 0) s_err = 1;
        if (u >= 0 && atomicMax(&a.xstamp[u], a.sbase) < a.sbase) {
            const uint32_t oc = a.out_cnt[u];
            atomicAdd(&s_reach, (unsigned long long)oc);
            if (oc > kHeavyRow) b.heavy[atomicAdd(&s_heavy, 1u)] = u;
            else b.light[atomicAdd(&s_light, 1u)] = u;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        Ctl *ctl = a.ctl;
        ctl->mk_light = s_light;
        ctl->mk_heavy = s_heavy;
        ctl->reach = s_reach;
        if (s_err) {
            ctl->err = 1;
            ctl->done = 1;
        }
        if (b.snap)
            snap_ctl<false>(ctl, a.max_iters, a.sparse_limit, a.sparse_limit, b.dense, a.tol, a.ftol);
    }
}

// Dynamic Traversal (Section 3.3.2): every vertex reachable from the
// source of a batch edge in G^{t-1} or in G^t is affected.  Every deleted
// edge leaves a batch source, so the vertices reachable in either graph are
// those reachable along G^t's out-edges from the batch sources and the
// deletion targets.  A level-synchronous breadth-first search claims each
// vertex once through its stamp (the call's base, so that it is processed
// from the first iteration) and appends it to the next level's queue (no class
// lists: the iterations walk the full schedule).  Vertices with more than kHeavyRow
// out-edges go to a separate queue whose out-rows the whole grid walks in
// workgroup-sized chunks; the others are walked by waves, 64 at a time.
// Three queues (of each kind) rotate: level L reads queue L mod 3, fills
// queue L+1 mod 3 and clears the lengths of queue L+2 mod 3.

struct BfsQueues {
    const int32_t *in, *hin;          // this level: light and heavy vertices
    const uint32_t *nin, *nhin;
    int32_t *out, *hout;              // next level
    uint32_t *nout, *nhout;
    uint32_t *clear, *hclear;         // the level after next
};

// Every lane of the wave calls it; x < 0 claims nothing.  `deg` sums this
// lane's claims' out-edges (REACH).
template <bool REACH>
__device__ inline void bfs_claim(const IterArgs &a, int32_t x, const BfsQueues &q,
                                 unsigned long long &mine, unsigned long long &deg)
{
    bool nw = false;
    if (x >= 0 && a.stamp[x] < a.sbase) nw = atomicMax(&a.stamp[x], a.sbase) < a.sbase;
    const uint32_t oc = nw ? a.out_cnt[x] : 0u;
    if (REACH) deg += oc;
    const bool big = oc > kHeavyRow;
    const unsigned long long ml = __ballot(nw && !big), mh = __ballot(big);
    const int lane = lane_id();
    const unsigned long long below = (1ull << lane) - 1ull;
    if (ml | mh) {
        uint32_t bl = 0, bh = 0;
        if (lane == 0) {
            if (ml) bl = atomicAdd(q.nout, (uint32_t)__popcll(ml));
            if (mh) bh = atomicAdd(q.nhout, (uint32_t)__popcll(mh));
            mine += __popcll(ml | mh);
        }
        bl = __shfl(bl, 0);
        bh = __shfl(bh, 0);
        if (nw && !big) q.out[bl + __popcll(ml & below)] = x;
        if (big) q.hout[bh + __popcll(mh & below)] = x;
    }
}

// A workgroup's claims (lane 0 of each wave holds `mine`) and, with REACH,
// their out-edges into the control block.  Every thread calls it.
template <bool REACH>
__device__ inline void bfs_totals(Ctl *ctl, unsigned long long mine, unsigned long long deg,
                                  unsigned long long &s_new, unsigned long long &s_reach)
{
    if (REACH)
        for (int off = kWave / 2; off > 0; off >>= 1) deg += __shfl_xor(deg, off, kWave);
    if (lane_id() == 0 && mine) {
        atomicAdd(&s_new, mine);
        if (REACH) atomicAdd(&s_reach, deg);
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_new) {
        atomicAdd(&ctl->affected0, s_new);
        if (REACH) atomicAdd(&ctl->reach, s_reach);
    }
}

__global__ __launch_bounds__(kBlock) void k_bfs_seed(IterArgs a, int64_t nd, const int32_t *ds,
                                                     const int32_t *dd, int64_t ni,
                                                     const int32_t *is, BfsQueues q)
{
    __shared__ unsigned long long s_new, s_reach;
    if (a.ctl->err) return;
    if (threadIdx.x == 0) s_new = s_reach = 0;
    __syncthreads();
    const int lane = lane_id();
    const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kWave;
    const int64_t waves = (int64_t)gridDim.x * kWavesPerBlock;
    unsigned long long mine = 0, deg = 0;
    for (int64_t b0 = wave * kWave; b0 < nd + ni; b0 += waves * kWave) {
        const int64_t i = b0 + lane;
        const int32_t u = i < nd + ni ? (i < nd ? ds[i] : is[i - nd]) : -1;
        bfs_claim<false>(a, u, q, mine, deg);
        bfs_claim<false>(a, i < nd ? dd[i] : -1, q, mine, deg);
    }
    bfs_totals<false>(a.ctl, mine, deg, s_new, s_reach);
}

// One level.  Light vertices: each wave takes 64 and walks their out-edges
// together, one out-edge per lane and round.  Heavy vertices: every
// workgroup takes chunks of kBlock out-edges of each of them.  REACH: the
// out-edges of its claims are summed too (the level before a look by the host;
// in each of the thousands of levels of a grid the sum cost 4% of a search).
template <bool REACH>
__global__ __launch_bounds__(kBlock) void k_bfs_level(IterArgs a, BfsQueues q)
{
    __shared__ unsigned long long s_new, s_reach;
    if (a.ctl->err) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *q.clear = 0;
        *q.hclear = 0;
    }
    const uint32_t nin = *q.nin, nh = *q.nhin;
    if (threadIdx.x == 0) s_new = s_reach = 0;
    __syncthreads();
    const int lane = lane_id();
    const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kWave;
    const int64_t waves = (int64_t)gridDim.x * kWavesPerBlock;
    unsigned long long mine = 0, claimed = 0;
    for (int64_t b0 = wave * kWave; b0 < nin; b0 += waves * kWave) {
        const int64_t i = b0 + lane;
        const int32_t x = i < nin ? q.in[i] : -1;
        const uint32_t deg = x >= 0 ? a.out_cnt[x] : 0u;
        const uint32_t ob = x >= 0 ? a.out_beg[x] : 0u;
        uint32_t incl = deg;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const uint32_t y = __shfl_up(incl, d);
            if (lane >= d) incl += y;
        }
        const uint32_t total = __shfl(incl, kWave - 1);
        for (uint32_t t0 = 0; t0 < total; t0 += kWave) {
            const uint32_t t = t0 + lane;
            const uint32_t tt = min(t, total - 1);
            int j = 0;
#pragma unroll
            for (int step = kWave / 2; step > 0; step >>= 1)
                if (__shfl(incl, j + step - 1) <= tt) j += step;
            const uint32_t first = __shfl(incl, j) - __shfl(deg, j);
            const uint32_t base = __shfl(ob, j);
            const int32_t y = t < total ? a.out_idx[base + (tt - first)] : -1;
            bfs_claim<REACH>(a, y, q, mine, claimed);
        }
    }
    __shared__ HeavyShared hs;
    walk_heavy(a, q.hin, nh, hs, [&](int32_t x) { bfs_claim<REACH>(a, x, q, mine, claimed); });
    bfs_totals<REACH>(a.ctl, mine, claimed, s_new, s_reach);
}

// A wide level.  Appending hundreds of thousands of vertices to the queues
// costs an atomic on one address per wave and round (13 ns each: 330 us a level
// on R-MAT scale 19, 2.3 ms a search), so wide levels keep no queue: a pass
// looks at every vertex and expands those marked but not expanded yet
// (expansion stamp), marking with plain stores; a mark made in the pass may be
// expanded by it too, which changes no result.  k_bfs_scan does the vertices of
// up to kHeavyRow out-edges and lists the others for k_bfs_heavy.  Waves take
// vertices a stride apart, since neighbouring ids have similar degrees.
// *nfresh and *nheavy count what the pass expanded; the search is over when
// that is nothing.
__global__ __launch_bounds__(kBlock) void k_bfs_scan(IterArgs a, int32_t *heavy, uint32_t *nfresh,
                                                     uint32_t *nheavy, uint32_t *clear, uint32_t *hclear)
{
    if (a.ctl->err) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *clear = 0;
        *hclear = 0;
    }
    __shared__ uint32_t s_fresh;
    if (threadIdx.x == 0) s_fresh = 0;
    __syncthreads();
    const int lane = lane_id();
    const int64_t waves = (int64_t)gridDim.x * kWavesPerBlock;
    const int64_t wave = blockIdx.x * (int64_t)kWavesPerBlock + threadIdx.x / kWave;
    uint32_t fresh = 0;
    for (int64_t v0 = 0; v0 < a.n; v0 += waves * kWave) {
        const int64_t v = v0 + lane * waves + wave;
        const bool take = v < a.n && a.stamp[v] == a.sbase && a.xstamp[v] != a.sbase;
        if (!__ballot(take)) continue;
        if (take) a.xstamp[v] = a.sbase;
        const uint32_t oc = take ? a.out_cnt[v] : 0u;
        const bool big = oc > kHeavyRow;
        const unsigned long long mh = __ballot(big);
        if (mh) {
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(nheavy, (uint32_t)__popcll(mh));
            at = __shfl(at, 0);
            if (big) heavy[at + __popcll(mh & ((1ull << lane) - 1ull))] = (int32_t)v;
        }
        fresh += (uint32_t)__popcll(__ballot(take && !big));
        // rows shorter than a wave together, the others one at a time
        const uint32_t deg = oc < (uint32_t)kWave ? oc : 0u;
        const uint32_t ob = deg ? a.out_beg[v] : 0u;
        uint32_t incl = deg;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const uint32_t y = __shfl_up(incl, d);
            if (lane >= d) incl += y;
        }
        expand_rows<false, false>(a, incl, deg, ob, __shfl(incl, kWave - 1), a.sbase);
        for (unsigned long long q = __ballot(oc >= (uint32_t)kWave && !big); q; q &= q - 1)
            mark_out_row<false, false>(a, __shfl((int32_t)v, __ffsll((long long)q) - 1), lane, kWave,
                                       a.sbase);
    }
    if (lane == 0 && fresh) atomicAdd(&s_fresh, fresh);
    __syncthreads();
    if (threadIdx.x == 0 && s_fresh) atomicAdd(nfresh, s_fresh);
}

__global__ __launch_bounds__(kBlock) void k_bfs_heavy(IterArgs a, const int32_t *heavy,
                                                      const uint32_t *nheavy)
{
    __shared__ HeavyShared hs;
    if (a.ctl->err) return;
    walk_heavy(a, heavy, *nheavy, hs, [&](int32_t x) {
        if (x >= 0 && a.stamp[x] < a.sbase) a.stamp[x] = a.sbase;
    });
}

// The vertices marked but not expanded into the queues of the next level.
__global__ __launch_bounds__(kBlock) void k_bfs_collect(IterArgs a, BfsQueues q)
{
    if (a.ctl->err) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *q.clear = 0;
        *q.hclear = 0;
    }
    const int lane = lane_id();
    const unsigned long long below = (1ull << lane) - 1ull;
    const int64_t step = (int64_t)gridDim.x * kBlock;
    for (int64_t v0 = blockIdx.x * (int64_t)kBlock + threadIdx.x - lane; v0 < a.n; v0 += step) {
        const int64_t v = v0 + lane;
        const bool take = v < a.n && a.stamp[v] == a.sbase && a.xstamp[v] != a.sbase;
        const bool big = take && a.out_cnt[v] > kHeavyRow;
        const unsigned long long ml = __ballot(take && !big), mh = __ballot(big);
        if (!(ml | mh)) continue;
        uint32_t bl = 0, bh = 0;
        if (lane == 0) {
            if (ml) bl = atomicAdd(q.nout, (uint32_t)__popcll(ml));
            if (mh) bh = atomicAdd(q.nhout, (uint32_t)__popcll(mh));
        }
        bl = __shfl(bl, 0);
        bh = __shfl(bh, 0);
        if (take && !big) q.out[bl + __popcll(ml & below)] = (int32_t)v;
        if (big) q.hout[bh + __popcll(mh & below)] = (int32_t)v;
    }
}

// The marks of a search that had wide levels.
__global__ __launch_bounds__(kBlock) void k_bfs_marked(IterArgs a)
{
    __shared__ unsigned long long s_cnt;
    if (threadIdx.x == 0) s_cnt = 0;
    __syncthreads();
    unsigned long long mine = 0;
    for (int64_t v = blockIdx.x * (int64_t)kBlock + threadIdx.x; v < a.n; v += (int64_t)gridDim.x * kBlock)
        mine += a.stamp[v] == a.sbase;
    for (int off = kWave / 2; off > 0; off >>= 1) mine += __shfl_xor(mine, off, kWave);
    if (lane_id() == 0 && mine) atomicAdd(&s_cnt, mine);
    __syncthreads();
    if (threadIdx.x == 0 && s_cnt) atomicAdd(&a.ctl->affected0, s_cnt);
}

// End of a Dynamic Frontier call: copy the rows processed in this call from
// the result buffer into the other buffer and count the marked vertices.
// A call that stayed on the class lists visits the listed vertices (every
// mark of the call was appended); otherwise all vertices by stamp.
__global__ __launch_bounds__(kBlock) void k_finish(int32_t n, const uint32_t *stamp, uint32_t lo,
                                                   uint32_t hi, const double *Rres, double *Roth,
                                                   const double *Cres, double *Coth, Ctl *ctl,
                                                   const int32_t *bins, int32_t n_stride)
{
    __shared__ unsigned long long s_cnt;
    if (threadIdx.x == 0) s_cnt = 0;
    __syncthreads();
    unsigned long long mine = 0;
    const int64_t t0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    if (!ctl->dense) {
        uint32_t len[kBins];
        int64_t tot = 0;
        for (int b = 0; b < kBins; b++) {
            len[b] = ctl->live[b];
            tot += len[b];
        }
        for (int64_t t = t0; t < tot; t += step) {
            int b = 0;
            int64_t r = t;
            while (r >= len[b]) r -= len[b++];
            const int32_t v = bins[(int64_t)b * n_stride + r];
            mine++;
            Roth[v] = Rres[v];
            Coth[v] = Cres[v];
        }
    } else {
        for (int64_t v = t0; v < n; v += step) {
            const uint32_t st = stamp[v];
            if (st >= lo && st <= hi) {
                mine++;
                Roth[v] = Rres[v];
                Coth[v] = Cres[v];
            }
        }
    }
    for (int off = kWave / 2; off > 0; off >>= 1) mine += __shfl_xor(mine, off, kWave);
    if (lane_id() == 0 && mine) atomicAdd(&s_cnt, mine);
    __syncthreads();
    if (threadIdx.x == 0 && s_cnt) atomicAdd(&ctl->affected, s_cnt);
}

// Sum of the ranks in FP64 with a fixed order: each workgroup folds a fixed
// range with a fixed tree, then one workgroup folds the partials in order.
constexpr int kSumBlocks = 1024;

__global__ __launch_bounds__(kBlock) void k_sum_part(int32_t n, const double *R, double *part)
{
    __shared__ double s[kBlock];
    const int64_t chunk = ((int64_t)n + gridDim.x - 1) / gridDim.x;
    const int64_t lo = blockIdx.x * chunk, hi = min<int64_t>(lo + chunk, n);
    double acc = 0.0;
    for (int64_t v = lo + threadIdx.x; v < hi; v += kBlock) acc += R[v];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int st = kBlock / 2; st > 0; st >>= 1) {
        if (threadIdx.x < st) s[threadIdx.x] += s[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = s[0];
}

__global__ __launch_bounds__(kBlock) void k_sum_final(const double *part, int nb, Ctl *ctl)
{
    __shared__ double s[kBlock];
    double acc = 0.0;
    for (int i = threadIdx.x; i < nb; i += kBlock) acc += part[i];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int st = kBlock / 2; st > 0; st >>= 1) {
        if (threadIdx.x < st) s[threadIdx.x] += s[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) ctl->renorm_scale = s[0] > 0.0 ? 1.0 / s[0] : 1.0;
}

// R <- R / sum(R) in both buffers and FP64 contributions rebuilt from it.
__global__ void k_renorm(int32_t n, double *Rres, double *Roth, double *C0, double *C1,
                         const uint32_t *out_cnt, const Ctl *ctl)
{
    const double scale = ctl->renorm_scale;
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        const double r = Rres[v] * scale;
        const double c = r / (double)out_cnt[v];
        Rres[v] = r;
        Roth[v] = r;
        C0[v] = c;
        C1[v] = c;
    }
}

static inline int blocks_for(int64_t items, int per_block = kBlock)
{
    const int64_t b = (items + per_block - 1) / per_block;
    return (int)std::max<int64_t>(1, std::min<int64_t>(b, 65535 * 16));
}

// Both passes of the initial marking on the graph's stream.  The batch
// arrays are staged in device memory; `lists` has room for the two source
// lists (2 (nd + ni) entries).
static void launch_initial_marking(dfpr_graph *g, const IterArgs &a, int64_t nd,
                                   const int32_t *ds, const int32_t *dd, int64_t ni,
                                   const int32_t *is, int dense, int32_t *lists, int snap,
                                   uint32_t plain_limit, bool claimed = false)
{
    int32_t *light = lists;
    int32_t *heavy = light + (nd + ni);
    if (!claimed)
        k_mark_claim<<<blocks_for(nd + ni), kBlock, 0, g->stream>>>(a, nd, ds, ni, is, light, heavy);
    const int64_t waves = std::max<int64_t>(nd + ni, 1024);
    k_mark_initial<<<(unsigned)std::min<int64_t>(blocks_for(waves * kWave), 2048), kBlock, 0,
                     g->stream>>>(a, nd, dd, light, heavy, dense, snap, plain_limit);
}


// The control block to its host copy (coherent pinned memory) by one wave.
// A copy-engine transfer of these few hundred bytes occupies the queue for
// ~20 us; a one-wave kernel takes a few.
__global__ __launch_bounds__(kWave) void k_ctl_to_host(const Ctl *ctl, Ctl *host)
{
    static_assert(sizeof(Ctl) % 4 == 0, "the control block is copied in 4-byte words");
    constexpr int words = (int)(sizeof(Ctl) / 4);
    const uint32_t *src = reinterpret_cast<const uint32_t *>(ctl);
    uint32_t *dst = reinterpret_cast<uint32_t *>(host);
    for (int i = threadIdx.x; i < words; i += kWave) dst[i] = src[i];
}

int ctl_to_host(dfpr_graph *g)
{
    k_ctl_to_host<<<1, kWave, 0, g->stream>>>(g->ctl, g->ctl_host);
    DFPR_HIP(hipGetLastError());
    return DFPR_OK;
}

int launch_fill_u32(dfpr_graph *g, uint32_t *p, uint64_t len, uint32_t value)
{
    k_fill_u32<<<std::min<int>(blocks_for((int64_t)len), 4096), kBlock, 0, g->stream>>>(p, len,
                                                                                       value);
    DFPR_HIP(hipGetLastError());
    return DFPR_OK;
}

// ---------------------------------------------------------------------------
// host drivers
// ---------------------------------------------------------------------------

struct BusyGuard {
    dfpr_graph *g;
    bool ok;
    explicit BusyGuard(dfpr_graph *g_) : g(g_)
    {
        ok = __atomic_exchange_n(&g->busy, 1, __ATOMIC_ACQ_REL) == 0;
    }
    ~BusyGuard()
    {
        if (ok) __atomic_store_n(&g->busy, 0, __ATOMIC_RELEASE);
    }
};

int check_params(const dfpr_params *p, dfpr_params &out)
{
    if (p) out = *p;
    else dfpr_params_default(&out);
    if (!(out.alpha >= 0.0 && out.alpha < 1.0) || !(out.tol >= 0.0) ||
        std::isnan(out.frontier_tol) || out.max_iters < 0 || out.max_iters > 100000 ||
        (out.precision != DFPR_FP64 && out.precision != DFPR_FP32_KAHAN) ||
        (out.mode != DFPR_SYNC && out.mode != DFPR_ASYNC) ||
        (out.loop != DFPR_LOOP_LAUNCHES && out.loop != DFPR_LOOP_DEVICE &&
         out.loop != DFPR_LOOP_ITERATION))
        return set_error(DFPR_E_ARG, "invalid parameters");
    return DFPR_OK;
}

IterArgs iter_args(dfpr_graph *g, const dfpr_params &p, uint32_t sbase)
{
    IterArgs a{};
    a.n = g->n;
    a.in_beg = g->csr[0].beg;
    a.in_cnt = g->csr[0].cnt;
    a.in_idx = g->csr[0].idx;
    a.out_beg = g->csr[1].beg;
    a.out_cnt = g->csr[1].cnt;
    a.out_idx = g->csr[1].idx;
    a.stamp = g->stamp;
    a.xstamp = g->xstamp;
    a.bins = g->bins;
    a.ctl = g->ctl;
    a.mirror = g->ctl_host;
    a.dr_part = g->it.dr_part;
    a.rmax_part = g->it.rmax_part;
    a.cnt_part = g->it.cnt_part;
    a.base_rank = (1.0 - p.alpha) / (double)g->n;
    a.alpha = p.alpha;
    a.tol = p.tol;
    a.ftol = p.frontier_tol;
    a.sbase = sbase;
    a.sparse_limit = g->sparse_limit;
    a.heavy = g->sparse_limit / 8;
    a.long_row = g->long_row;
    a.max_iters = p.max_iters;
    a.n_stride = g->n;
    // In the asynchronous form too: a copy taken when a workgroup starts
    // holds values the one rank vector had during this launch, which an
    // in-place sweep may read (on R-MAT scale 22 the same iterations and
    // error against the reference, 5% less time)
    a.hub = kHubRows;
    return a;
}

// Take a stamp base for a new call; stamps of earlier calls are all below it.
static int take_base(dfpr_graph *g, int32_t max_iters, uint32_t *base)
{
    const uint64_t span = (uint64_t)max_iters + 2;
    if ((uint64_t)g->next_base + span >= 0xF0000000ull) {
        int rc = launch_fill_u32(g, g->stamp, (uint64_t)g->n, 0);
        if (!rc) rc = launch_fill_u32(g, g->xstamp, (uint64_t)g->n, 0);
        if (!rc && g->mstamp) rc = launch_fill_u32(g, g->mstamp, (uint64_t)g->n, 0);
        if (!rc && g->mxstamp) rc = launch_fill_u32(g, g->mxstamp, (uint64_t)g->n, 0);
        if (rc) return rc;
        g->next_base = 1;
        g->last_iters = -1;           // the last update's marks are gone
    }
    *base = g->next_base;
    g->next_base += (uint32_t)span;
    return DFPR_OK;
}

// Run iterations it0, it0+1, ... until the device sets the stop flag (or,
// in the FP32 phase, the phase-end flag).  The phase starts on buffer
// `base`; iteration i reads buffer base ^ ((i - it0) & 1), or, in the
// asynchronous form (FP64 only), reads and writes buffer `base` in place.
// *res_buf receives the buffer holding the result.  Iterations are enqueued in
// chunks, up to two at a time; when a chunk completes the host reads the
// control block it left and sizes the next chunk from the observed
// geometric decay of Delta R, less what is still queued, so few launches
// run after convergence and the device does not wait for the host.
// Workgroups for the next chunk of a call still on the class lists: what
// the current lists need, times four and plus 64 for the frontier to grow
// within the chunk, at least one per CU.  Any grid gives the same result
// (the work is grid-strided); a small frontier just skips empty workgroups.
static uint32_t sparse_grid(const dfpr_graph *g, const Ctl &c)
{
    uint64_t nwu = 0;
    for (int b = 0; b < kBins - 1; b++) {
        const uint64_t rows = kWave / group_of(b);
        nwu += (c.live[b] + rows - 1) / rows;
    }
    const uint64_t need = std::max<uint64_t>(c.live[kBins - 1], (nwu + kWavesPerBlock - 1) /
                                                                     kWavesPerBlock);
    const uint64_t lo = std::min<uint64_t>(256, (uint64_t)g->grid);
    return (uint32_t)std::min<uint64_t>(g->grid, std::max<uint64_t>(lo, need * 4 + 64));
}

// Wave units of the full schedule (make_plan_wave).
static uint64_t wave_units(const dfpr_graph *g)
{
    const uint32_t *c = g->cls;
    uint64_t nwu = ((uint64_t)(c[kBins + 1] - c[kBins]) + kWave - 1) / kWave;
    for (int b = 0; b < kBins - 1; b++) {
        const uint64_t rows = kWave / group_of(b);
        nwu += ((uint64_t)(c[kBins - b] - c[kBins - 1 - b]) + rows - 1) / rows;
    }
    return nwu;
}

// Whether whole calls on the graph iterate in the resident loop (see kResEdges),
// and not only those on the class lists.
bool resident_whole(const dfpr_graph *g)
{
    return g->m <= kResEdges && g->long_row == kLongRow;
}

// Workgroups of a resident launch whose iterations walk the full schedule:
// enough waves for its wave units and enough sub-blocks for its long rows,
// one workgroup per compute unit at most.
uint32_t resident_grid(const dfpr_graph *g)
{
    const uint32_t *c = g->cls;
    const uint64_t nwu = wave_units(g);
    const uint64_t need = std::max<uint64_t>((nwu + kResWaves - 1) / kResWaves, (c[1] - c[0] + 3) / 4);
    return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(need, g->cus));
}

// Contributions a workgroup of a resident launch copies into LDS: the number
// that saves most.  A gather from L2 takes a compute unit about 1.1 ns beyond
// the 2 us that an iteration's chain of accesses takes anyway, a copied entry
// 0.21 ns (half that in FP32) and the copy itself 0.6 us; the share of the
// gathers that the first entries take is known from the load.  On R-MAT scale
// 18 that is all kResHub entries (4.1 us for 60% of 18 us of gathers), on a
// uniform graph or one of 10,000 vertices none.
uint32_t resident_hub(const dfpr_graph *g, bool f32, uint32_t G)
{
    const double gathers = 1.1e-3 * (double)g->m / G - 2.0;     // us per workgroup
    double best = 0.0;
    uint32_t hub = 0;
    for (int k = 0; k < kHubSteps; k++) {
        const uint32_t h = std::min<uint32_t>(1024u << k, (uint32_t)g->n);
        if (h > (f32 ? 2 * kResHub : kResHub)) break;
        const double gain = g->hub_share[k] * gathers - (f32 ? 1.05e-4 : 2.1e-4) * h - 0.6;
        if (gain > best) {
            best = gain;
            hub = h;
        }
    }
    return hub;
}

// Entries the class lists may hold in the resident loop.
uint32_t resident_lists(const dfpr_graph *g)
{
    return std::max<uint32_t>(g->sparse_limit, (uint32_t)(g->n / kResSparse));
}

// Arguments of a resident launch from iteration `it` of the phase that started
// at it0 on buffer `base`, with tags of its own.
int resident_args(dfpr_graph *g, int it0, int it, int base, bool full, uint32_t limit, ResArgs &P)
{
    if (g->res_tag > 0xFFFFFFFFu - 2 * kResTags) {
        // the tags start over: the words of earlier launches must not match
        DFPR_CHECK_RC(launch_fill_u32(g, reinterpret_cast<uint32_t *>(g->it.res),
                                      sizeof(ResWords) / 4, 0));
        g->res_tag = 0;
    }
    P = ResArgs{};
    for (int b = 0; b < 2; b++) {
        P.R[b] = g->R[b];
        P.C[b] = g->C[b];
        P.C32[b] = g->C32[b];
    }
    P.w = reinterpret_cast<ResWords *>(g->it.res);
    P.base = base;
    P.it0 = it0;
    P.it_start = it;
    P.full = full ? 1 : 0;
    P.limit = limit;
    P.blocks = g->long_row == kLongRow ? kNoLimit : 0u;
    P.spin = g->res_refuse ? 0u : kGoSpin;
    P.tag = g->res_tag + 1;
    P.ext2int = g->ext2int;
    g->res_tag += kResTags;
    return DFPR_OK;
}

// One launch of the resident loop from iteration `it` of the phase that
// started at it0 on buffer `base`.  *ran: the workgroups were all running
// and the control block's host copy is the state it left; otherwise nothing
// was changed.
static int launch_resident(dfpr_graph *g, IterArgs a, bool df, bool f32, int it0, int it, int base,
                           bool full, uint32_t limit, Close *close, bool *ran)
{
    *ran = false;
    ResArgs P;
    DFPR_CHECK_RC(resident_args(g, it0, it, base, full, limit, P));
    P.close = close ? 1 : 0;
    P.out = close ? close->out : nullptr;
    a.mirror = g->ctl_host;
    const uint32_t G = full ? resident_grid(g) : (uint32_t)g->cus;
    a.hub = full && a.hub ? resident_hub(g, f32, G) : 0u;
    if (limit == kNoLimit) a.sparse_limit = resident_lists(g);
    const bool pairs = full && !f32 && wave_units(g) >= (uint64_t)kPairUnits * kResWaves * G;
    auto *kernel = f32     ? k_resident<true, true, false>
                   : !df   ? pairs ? k_resident<false, false, true> : k_resident<false, false, false>
                   : pairs ? k_resident<true, false, true> : k_resident<true, false, false>;
    kernel<<<G, kResThreads, 0, g->stream>>>(a, P);
    DFPR_HIP(hipGetLastError());
    DFPR_HIP(hipEventRecord(g->ev1, g->stream));
    DFPR_HIP(hipStreamSynchronize(g->stream));
    if (g->ctl_host->loop_fail && g->ctl_host->loop_ran == P.tag) return set_error(DFPR_E_DEVICE, "resident loop: a barrier timed out");
    *ran = g->ctl_host->loop_ran == P.tag;
    if (close) close->done = *ran && g->ctl_host->loop_closed;
    return DFPR_OK;
}

// `lists`: the call is expected to iterate on the class lists (see first_lists;
// Dynamic Traversal is on the full schedule throughout).
static int run_loop(dfpr_graph *g, const dfpr_params &p, bool df, bool f32, uint32_t sbase,
                    int it0, int base, int *res_buf, Close *close, bool lists)
{
    IterArgs a = iter_args(g, p, sbase);
    const bool async = p.mode == DFPR_ASYNC && !f32;
    // Up to two chunks are in flight: while the host waits for the older
    // one and reads the control block it left in its own mirror, the newer
    // one keeps the device busy.  Chunk c uses mirror, completion event and
    // profiling events of slot c & 1.
    Ctl *const mirror[2] = {g->ctl_host, g->ctl_host + 1};
    struct Chunk {
        int k, slot;
    };
    Chunk q[2];
    int nq = 0, next_it = it0, nchunks = 0, chunk = 4, fin = 0;
    // iterations to keep queued beyond the last state read; until a state
    // is known, two chunks of four
    int target = 8, cap = 4;
    bool stop = false;
    uint32_t gsz = (uint32_t)g->grid;
    // walks of the full schedule run a wide kernel: Static and Naive-dynamic
    // from the start, Dynamic Frontier once a state shows the full schedule
    bool wide = DFPR_WIDE && !df;
    double prev_dr = -1.0;
    int prev_it = it0;
    *res_buf = base;
    // Iterations inside one launch (see kResEdges).  The asynchronous form,
    // DFPR_LOOP_ITERATION and, unless small frontiers are asked for, profiled
    // calls keep a launch per iteration.
    const bool device_loop = p.loop == DFPR_LOOP_DEVICE;
    const bool full = !device_loop && resident_whole(g);
    const bool resident = device_loop ? lists
                          : p.loop != DFPR_LOOP_ITERATION && !g->prof.enabled && (full || lists);
    if (!async && resident) {
        const uint32_t limit = device_loop ? kLoopRows : kNoLimit;
        while (next_it < p.max_iters) {
            bool ran = false;
            DFPR_CHECK_RC(launch_resident(g, a, df, f32, it0, next_it, base, full, limit,
                                           f32 ? nullptr : close, &ran));
            if (!ran) break;
            const Ctl &c = *g->ctl_host;
            const int steps = c.iterations - next_it;
            next_it = c.iterations;
            g->res_iters += steps;
            if (device_loop) g->loop_iters += steps;
            if (c.done || (f32 && c.phase_end)) {
                stop = true;
                break;
            }
            // a frontier with rows of the workgroup class is about to grow
            gsz = df && !c.dense && !c.live[kBins - 1] ? sparse_grid(g, c) : (uint32_t)g->grid;
            wide = DFPR_WIDE && (!df || c.dense);
            if (steps < kResSteps) break;     // handed over
        }
        if (g->prof.enabled && next_it > it0) {
            // not the iteration kernel's work
            const Ctl &c = *g->ctl_host;
            const unsigned long long ran[5] = {c.verts, c.edges, c.xverts, c.xedges, c.marked};
            for (int k = 0; k < 5; k++) g->prof_base[k] = (int64_t)ran[k];
        }
    }
    auto launch = [&](int k) -> int {
        const int slot = nchunks & 1;
        a.mirror = mirror[slot];
        hipEvent_t *ev = g->evk + slot * 2 * kLoopChunk;
        for (int j = 0; j < k; j++) {
            const int i = next_it + j;
            const int src = async ? base : base ^ ((i - it0) & 1);
            const int dst = async ? base : src ^ 1;
            a.Rc = g->R[src];
            a.Cc = g->C[src];
            a.Rn = g->R[dst];
            a.Cn = g->C[dst];
            a.C32c = g->C32[src];
            a.C32n = g->C32[src ^ 1];
            a.it = i;
            if (g->prof.enabled) DFPR_HIP(hipEventRecord(ev[2 * j], g->stream));
            if (wide) {
                IterArgs aw = a;
                if (!df) {
                    aw.hub = a.hub ? kWideHub : 0u;
                    k_iter_wide<false, false, kWideWaves, kWideHub>
                        <<<g->grid_wide, kWideWaves * kWave, 0, g->stream>>>(aw);
                } else if (f32) {
                    // FP32 contributions: the same LDS holds twice the entries
                    aw.hub = a.hub ? kWideDfHub * DFPR_WIDE_F32_MUL : 0u;
                    k_iter_wide<true, true, kWideDfWaves, kWideDfHub>
                        <<<g->grid_wide_df, kWideDfWaves * kWave, 0, g->stream>>>(aw);
                } else {
                    aw.hub = a.hub ? kWideDfHub : 0u;
                    k_iter_wide<true, false, kWideDfWaves, kWideDfHub>
                        <<<g->grid_wide_df, kWideDfWaves * kWave, 0, g->stream>>>(aw);
                }
            }
            else if (!df) k_iter<false, false><<<gsz, kBlock, 0, g->stream>>>(a);
            else if (f32) k_iter<true, true><<<gsz, kBlock, 0, g->stream>>>(a);
            else k_iter<true, false><<<gsz, kBlock, 0, g->stream>>>(a);
            if (g->prof.enabled) DFPR_HIP(hipEventRecord(ev[2 * j + 1], g->stream));
            k_final<<<1, kFinalThreads, 0, g->stream>>>(a, df ? 1 : 0, f32 ? 1 : 0,
                                                         j == k - 1 ? 1 : 0);
        }
        DFPR_HIP(hipGetLastError());
        DFPR_HIP(hipEventRecord(g->evc[slot], g->stream));
        q[nq++] = Chunk{k, slot};
        next_it += k;
        nchunks++;
        return DFPR_OK;
    };
    while (true) {
        int queued = 0;
        for (int t = 0; t < nq; t++) queued += q[t].k;
        while (!stop && nq < 2 && queued < target && next_it < p.max_iters) {
            const int k = std::min(std::min(target - queued, cap), p.max_iters - next_it);
            const int rc = launch(k);
            if (rc) return rc;
            queued += k;
        }
        if (nq == 0) break;
        const Chunk c = q[0];
        q[0] = q[1];
        nq--;
        // the chunk's last k_final, or the one that ended the call or the
        // phase, left the control block in the chunk's mirror
        DFPR_HIP(hipEventSynchronize(g->evc[c.slot]));
        if (g->prof.enabled) {
            // the iteration kernel alone, launch by launch
            const hipEvent_t *ev = g->evk + c.slot * 2 * kLoopChunk;
            for (int j = 0; j < c.k; j++) {
                float ms = 0.f;
                DFPR_HIP(hipEventElapsedTime(&ms, ev[2 * j], ev[2 * j + 1]));
                g->prof.ms += ms;
            }
            g->prof.launches += c.k;
        }
        if (stop) continue;             // later chunks return at once
        const Ctl &st = *mirror[c.slot];
        if (st.done || (f32 && st.phase_end)) {
            stop = true;
            fin = c.slot;
            continue;
        }
        // iterations still needed after this state, from the observed
        // geometric decay of Delta R
        gsz = df && !st.dense ? sparse_grid(g, st) : (uint32_t)g->grid;
        wide = DFPR_WIDE && (!df || st.dense);
        const double dr = st.final_linf;
        const int its = st.iterations;
        int need = std::min(chunk * 2, 32);
        // the FP32 phase ends at the larger of tol and its resolution
        // floor (see final_body); the FP64 loop at tol
        const double goal = f32 ? std::max(p.tol, st.final_rmax * 0x1p-22) : p.tol;
        if (prev_dr > 0.0 && dr > 0.0 && dr < prev_dr && its > prev_it && goal > 0.0) {
            const double rate = std::pow(dr / prev_dr, 1.0 / (its - prev_it));
            const double left = std::ceil(std::log(goal / dr) / std::log(rate));
            if (std::isfinite(left)) need = (int)std::min<double>(kLoopChunk, std::max(1.0, left));
        }
        prev_dr = dr;
        prev_it = its;
        chunk = need;
        cap = kLoopChunk;
        // at least one more iteration if nothing is queued: the call is not over
        target = std::max(need, nq > 0 ? 0 : 1);
    }
    if (fin == 1) *mirror[0] = *mirror[1];   // the final state goes to the main mirror
    if (p.max_iters <= it0) {
        DFPR_CHECK_RC(ctl_to_host(g));
        DFPR_HIP(hipStreamSynchronize(g->stream));
    }
    const Ctl &c = *g->ctl_host;
    *res_buf = async ? base : base ^ ((c.iterations - it0) & 1);
    if (g->prof.enabled) {
        const int64_t dv = (int64_t)c.verts - g->prof_base[0];
        const int64_t de = (int64_t)c.edges - g->prof_base[1];
        const int64_t dxv = (int64_t)c.xverts - g->prof_base[2];
        const int64_t dxe = (int64_t)c.xedges - g->prof_base[3];
        const int64_t dmk = (int64_t)c.marked - g->prof_base[4];
        g->prof.rows += dv;
        g->prof.edges += de;
        g->prof.exp_rows += dxv;
        g->prof.exp_edges += dxe;
        g->prof.marked += dmk;
        // per processed row: worklist entry 4 B, row start and length 8 B,
        // R[v] 8 B, |out(v)| 4 B, R'[v] and C'[v] written 16 B (12 B with an
        // FP32 contribution) (+ its mark 4 B and expansion stamp 4 B in
        // Dynamic Frontier); per in-edge: index 4 B and the gathered
        // contribution (8 B, or 4 B in FP32); per expanding row: out-row
        // start and length 8 B; per scanned out-edge: index 4 B and the
        // target's mark 4 B
        const double row_bytes = (df ? 48.0 : 40.0) - (f32 ? 4.0 : 0.0);
        const double edge_bytes = f32 ? 8.0 : 12.0;
        g->prof.bytes += row_bytes * dv + edge_bytes * de + 8.0 * dxv + 8.0 * dxe;
        g->prof_base[0] = (int64_t)c.verts;
        g->prof_base[1] = (int64_t)c.edges;
        g->prof_base[2] = (int64_t)c.xverts;
        g->prof_base[3] = (int64_t)c.xedges;
        g->prof_base[4] = (int64_t)c.marked;
    }
    return DFPR_OK;
}

static void fill_stats(dfpr_graph *g, dfpr_stats *st, bool df)
{
    if (!st) return;
    const Ctl &c = *g->ctl_host;
    st->iterations = c.iterations;
    st->converged = c.converged;
    st->refine_sweeps = g->refine_sweeps;
    st->loop_iterations = g->loop_iters;
    st->frontier_tol_used = df ? c.ftol_used : 0.0;
    st->final_linf = c.final_linf;
    float ms = 0.f, ms0 = 0.f, ms1 = 0.f;
    (void)hipEventElapsedTime(&ms, g->ev0, g->ev1);
    (void)hipEventElapsedTime(&ms0, g->ev0, g->ev_mid);
    (void)hipEventElapsedTime(&ms1, g->ev_mid, g->ev1);
    st->ms_device = ms;
    st->ms_mark = ms0;
    st->ms_iter = ms1;
    st->ms_apply = g->last_apply_ms;
    st->affected_initial = df ? (int64_t)c.affected0 : g->n;
    st->affected_final = df ? (int64_t)c.affected : g->n;
    st->vertices_processed = (int64_t)c.verts;
    st->edges_processed = (int64_t)c.edges;
}

// k_begin of a call: the loop state and the starting ranks (prev, host or
// device; uniform; or the resident ones), FP32 contributions with `f32`, and
// whatever `b` already asks for.
static int launch_begin(dfpr_graph *g, const IterArgs &a, BeginArgs b, const double *prev, int prev_dev,
                        bool uniform, bool f32)
{
    const int32_t n = g->n;
    if (prev && !prev_dev) {
        DFPR_HIP(hipMemcpyAsync(g->Rx, prev, (size_t)n * 8, hipMemcpyHostToDevice, g->stream));
        prev = g->Rx;
    }
    b.ext2int = g->ext2int;
    b.int2ext = g->int2ext;
    b.ranks = prev ? 1 : uniform ? 2 : 0;
    b.prev = prev;
    b.R0 = g->R[0];
    b.R1 = g->R[1];
    b.C0 = g->C[0];
    b.C1 = g->C[1];
    b.Ccur = g->C[g->cur];
    if (f32) {
        b.A = g->C32[0];
        b.B = g->C32[1];
    }
    // a vertex a thread (four: 17 us more on a 4096 x 4096 grid)
    const int64_t work = b.ranks || f32 ? ((int64_t)n + kBeginThreads - 1) / kBeginThreads : 0;
    k_begin<<<1 + (unsigned)std::min<int64_t>(work, 65536), kBeginThreads, 0, g->stream>>>(a, b);
    DFPR_HIP(hipGetLastError());
    g->refine_sweeps = 0;
    g->loop_iters = 0;
    std::memset(g->prof_base, 0, sizeof(g->prof_base));
    return DFPR_OK;
}

// Static (prev == NULL and !use_resident: uniform start) or Naive-dynamic
// (start from prev, or from the resident ranks).
static int full_sweeps(dfpr_graph *g, const dfpr_params *pp, const double *prev, int prev_dev,
                       bool use_resident, double *ranks_out, int out_dev, dfpr_stats *st)
{
    dfpr_params p;
    int rc = check_params(pp, p);
    if (rc) return rc;
    BusyGuard guard(g);
    if (!guard.ok) return set_error(DFPR_E_BUSY, "graph in use");
    const int32_t n = g->n;
    hipStream_t s = g->stream;
    DFPR_HIP(hipEventRecord(g->ev0, s));
    const int cur = g->cur;
    BeginArgs b{};
    b.snap = 1;
    b.dense = 1;
    DFPR_CHECK_RC(launch_begin(g, iter_args(g, p, 0), b, prev, prev_dev, !prev && !use_resident, false));
    int res = cur;
    DFPR_HIP(hipEventRecord(g->ev_mid, s));
    Close close;
    if (ranks_out) close.out = out_dev ? ranks_out : g->Rx;
    rc = run_loop(g, p, false, false, 0, 0, cur, &res, &close, false);
    if (rc) return rc;
    g->cur = res;
    if (!close.done) {
        k_copy2<<<blocks_for(n), kBlock, 0, s>>>(n, g->R[res], g->R[res ^ 1], g->C[res],
                                                 g->C[res ^ 1]);
        DFPR_HIP(hipEventRecord(g->ev1, s));
        if (ranks_out) DFPR_CHECK_RC(ranks_to_caller(g, g->R[res], ranks_out, out_dev));
    } else if (ranks_out && !out_dev) {
        DFPR_HIP(hipMemcpyAsync(ranks_out, g->Rx, (size_t)n * 8, hipMemcpyDeviceToHost, s));
    }
    DFPR_HIP(hipStreamSynchronize(s));
    fill_stats(g, st, false);
    return DFPR_OK;
}

// Everything of a Dynamic Frontier call before its iterations, enqueued on
// the graph's stream: the batch (host or device arrays) staged in `staging`
// (device arrays only) or in the graph's buffer, optional previous ranks (host
// or device, as the batch), a stamp base, the initial marking and the
// snapshot of iteration 0.  Returns the stamp base.
int df_begin(dfpr_graph *g, const dfpr_params &p, int64_t nd, const int32_t *ds,
             const int32_t *dd, int64_t ni, const int32_t *is, const int32_t *id, int on_device,
             const double *prev, uint32_t *sbase_out, int32_t *staging)
{
    const int64_t tot = nd + ni;
    const bool small = tot <= kSmallBatch;
    const int32_t *bds = nullptr, *bdd = nullptr, *bis = nullptr, *bid = nullptr;
    BeginArgs b{};
    if (small) {
        const int32_t *const in[4] = {ds, dd, is, id};
        for (int k = 0; k < 4; k++) b.src[k] = in[k];
        if (!staging) DFPR_CHECK_RC(stage_raw(g, nd, ds, dd, ni, is, id, on_device, b.src));
    } else if (staging) {
        DFPR_CHECK_RC(stage_batch_into(g, nd, ds, dd, ni, is, id, staging, &bds, &bdd, &bis, &bid));
    } else {
        DFPR_CHECK_RC(stage_batch(g, nd, ds, dd, ni, is, id, on_device, &bds, &bdd, &bis, &bid));
    }
    int32_t *const buf = staging ? staging : g->ap.batch_dev;
    int32_t *const lists = buf + 2 * tot;
    uint32_t sbase = 0;
    DFPR_CHECK_RC(take_base(g, p.max_iters, &sbase));
    // the initial marking decides on the device whether the batch's
    // sources reach enough vertices to start on the full schedule
    const int dense = 0;
    const IterArgs a = iter_args(g, p, sbase);
    // Expansions of iteration 0 append as long as the lists the iterations
    // keep can take it: where those are the resident loop's, from 1/64 to 1/8
    // of the vertices (2048 x 2048 grid, 256 scattered changes: a call
    // 3132 -> 2737 us; 10^6-vertex random graph: 4512 -> 4373 us).
    const bool resident = p.mode != DFPR_ASYNC && p.loop == DFPR_LOOP_LAUNCHES &&
                          !g->prof.enabled && resident_whole(g);
    const uint32_t plain_limit = resident ? resident_lists(g) : a.sparse_limit;
    if (small) {
        b.nd = nd;
        b.ni = ni;
        b.staged = buf;
        b.light = lists;
        b.heavy = lists + tot;
        bdd = buf + nd;
    }
    b.snap = tot == 0;
    DFPR_CHECK_RC(launch_begin(g, a, b, prev, on_device, false, p.precision == DFPR_FP32_KAHAN));
    if (tot > 0) {
        if (!small)
            k_validate<<<blocks_for(tot), kBlock, 0, g->stream>>>(g->n, nd, bds, bdd, ni, bis, bid,
                                                                 g->ctl);
        launch_initial_marking(g, a, nd, bds, bdd, ni, bis, dense, lists, 1, plain_limit, small);
    }
    DFPR_HIP(hipGetLastError());
    *sbase_out = sbase;
    return DFPR_OK;
}

// End of the FP32 phase (precision form).  If the call is over (the cap),
// rebuild the FP64 contributions from the ranks; otherwise renormalise the
// ranks to sum 1 in FP64 and rebuild the FP64 contributions, so FP64
// iterations can continue over the same marks from buffer `res`.
int df_phase_end(dfpr_graph *g, int res, bool call_done)
{
    const int32_t n = g->n;
    hipStream_t s = g->stream;
    if (call_done) {
        k_init_ranks<<<blocks_for(n), kBlock, 0, s>>>(n, g->R[res], g->R[0], g->R[1], g->C[0],
                                                      g->C[1], g->csr[1].cnt);
    } else {
        k_sum_part<<<kSumBlocks, kBlock, 0, s>>>(n, g->R[res], g->scratch_sum);
        k_sum_final<<<1, kBlock, 0, s>>>(g->scratch_sum, kSumBlocks, g->ctl);
        k_renorm<<<blocks_for(n), kBlock, 0, s>>>(n, g->R[res], g->R[res ^ 1], g->C[0], g->C[1],
                                                  g->csr[1].cnt, g->ctl);
    }
    DFPR_HIP(hipGetLastError());
    return DFPR_OK;
}

// After the last iteration (result in buffer `res`): bring the other buffer
// up to date on the processed rows, count the marks (unless the resident loop
// has `closed` the call), and make the result the resident ranks.
int df_finish(dfpr_graph *g, uint32_t sbase, int res, int32_t iters, bool closed)
{
    const int32_t n = g->n;
    if (!closed) {
        k_finish<<<std::min(blocks_for(n), 2048), kBlock, 0, g->stream>>>(
            n, g->stamp, sbase, sbase + (uint32_t)iters, g->R[res], g->R[res ^ 1], g->C[res],
            g->C[res ^ 1], g->ctl, g->bins, g->n);
        DFPR_HIP(hipGetLastError());
    }
    g->cur = res;
    g->last_base = sbase;
    g->last_iters = iters;
    return DFPR_OK;
}

// The end of a Dynamic Frontier or Traversal call, after its last iteration.
static int df_end(dfpr_graph *g, uint32_t sbase, int res, const Close &close, double *ranks_out,
                  int on_device, dfpr_stats *st)
{
    hipStream_t s = g->stream;
    if (g->ctl_host->err) return set_error(DFPR_E_RANGE, "vertex id outside [0, n) in the batch");
    DFPR_CHECK_RC(df_finish(g, sbase, res, g->ctl_host->iterations, close.done));
    if (!close.done) {
        DFPR_HIP(hipEventRecord(g->ev1, s));
        if (ranks_out) DFPR_CHECK_RC(ranks_to_caller(g, g->R[res], ranks_out, on_device));
        DFPR_CHECK_RC(ctl_to_host(g));
        DFPR_HIP(hipStreamSynchronize(s));
    } else if (ranks_out && !on_device) {
        DFPR_HIP(hipMemcpyAsync(ranks_out, g->Rx, (size_t)g->n * 8, hipMemcpyDeviceToHost, s));
        DFPR_HIP(hipStreamSynchronize(s));
    }
    fill_stats(g, st, true);
    return DFPR_OK;
}

// Whether a Dynamic Frontier call of `tot` batch entries on a graph above the
// resident loop's line is expected to stay on the class lists: the out-edges of
// a first frontier of mean out-degrees against half the limit above which its
// expansions mark with plain stores.  If not, the resident launch and the host's
// look after it only cost time.  Iterations with and without it:
//   4096 x 4096 grid, 9 / 855 / 8550 / 85000 changes: 0.14 / 0.48 / 4.74 / 8.26
//     and 0.23 / 1.54 / 4.42 / 8.09 ms; FP32 form, 8550: 5.9 and 5.3 ms
//   G(n, m), 3e6 vertices, 45e6 edges, 5 / 480 / 4800 changes: 0.26 / 3.06 /
//     3.57 and 0.62 / 2.94 / 3.52 ms; 6e6 vertices, 510: 14.0 and 14.6 ms
// With rows of the workgroup class, which a first frontier soon holds, it does
// not help (R-MAT scale 22, 7 changes, 8.49 and 8.51 ms), and they belong to the
// launches there (ResArgs::blocks).
static bool first_lists(const dfpr_graph *g, int64_t tot)
{
    if (g->cls[1] > 0) return false;
    const double mean = (double)g->m / g->n;
    return (double)tot * mean * mean <= (double)g->sparse_limit / 2;
}

// A Dynamic Frontier call.  `staging` (device arrays only): a caller-chosen
// buffer of 4 (nd + ni) ints for the staged batch and the marking's source
// lists, in place of the library's own; such a call allocates nothing.
static int df_impl(dfpr_graph *g, const dfpr_params *pp, int64_t nd, const int32_t *ds,
                   const int32_t *dd, int64_t ni, const int32_t *is, const int32_t *id,
                   int on_device, const double *prev, double *ranks_out, dfpr_stats *st,
                   int32_t *staging = nullptr)
{
    dfpr_params p;
    int rc = check_params(pp, p);
    if (rc) return rc;
    if (staging && !on_device) return set_error(DFPR_E_ARG, "staging needs device arrays");
    if (nd < 0 || ni < 0 || (nd && (!ds || !dd)) || (ni && (!is || !id)))
        return set_error(DFPR_E_ARG, "bad batch arrays");
    if (!on_device) {
        rc = check_ids_host(g->n, nd, ds, dd);
        if (!rc) rc = check_ids_host(g->n, ni, is, id);
        if (rc) return rc;
    }
    BusyGuard guard(g);
    if (!guard.ok) return set_error(DFPR_E_BUSY, "graph in use");
    hipStream_t s = g->stream;
    DFPR_HIP(hipEventRecord(g->ev0, s));
    const int cur = g->cur;
    uint32_t sbase = 0;
    rc = df_begin(g, p, nd, ds, dd, ni, is, id, on_device, prev, &sbase, staging);
    if (rc) return rc;
    Close close;
    if (ranks_out) close.out = on_device ? ranks_out : g->Rx;
    DFPR_HIP(hipEventRecord(g->ev_mid, s));
    int res = cur;
    const bool lists = p.loop == DFPR_LOOP_DEVICE || first_lists(g, nd + ni);
    if (p.precision == DFPR_FP32_KAHAN) {
        // FP32 phase on FP32 copies of the contributions
        rc = run_loop(g, p, true, true, sbase, 0, cur, &res, nullptr, lists);
        if (rc) return rc;
        if (g->ctl_host->err)
            return set_error(DFPR_E_RANGE, "vertex id outside [0, n) in the batch");
        const bool done = g->ctl_host->done != 0;
        rc = df_phase_end(g, res, done);
        if (rc) return rc;
        if (!done) {
            const int it0 = g->ctl_host->iterations;
            rc = run_loop(g, p, true, false, sbase, it0, res, &res, &close, !g->ctl_host->dense);
            if (rc) return rc;
            g->refine_sweeps = g->ctl_host->iterations - it0;
        }
    } else {
        rc = run_loop(g, p, true, false, sbase, 0, cur, &res, &close, lists);
        if (rc) return rc;
    }
    return df_end(g, sbase, res, close, ranks_out, on_device, st);
}

int df_device_staged(dfpr_graph *g, const dfpr_params *pp, int64_t nd, const int32_t *ds,
                     const int32_t *dd, int64_t ni, const int32_t *is, const int32_t *id,
                     const double *prev, double *ranks_out, dfpr_stats *st, int32_t *staging)
{
    return df_impl(g, pp, nd, ds, dd, ni, is, id, 1, prev, ranks_out, st, staging);
}

// Workgroups for a traversal level of `q` light vertices (a wave per 64),
// with room for the queue to grow sixteenfold within a chunk of levels; a
// level with heavy vertices gets the whole grid.
static uint32_t bfs_grid(const dfpr_graph *g, uint64_t q, uint64_t heavy)
{
    if (heavy) return (uint32_t)g->grid;
    const uint64_t blocks = (q + (uint64_t)kBlock - 1) / kBlock;
    return (uint32_t)std::min<uint64_t>(g->grid, std::max<uint64_t>(256, blocks * 16));
}

static BfsQueues bfs_queues(dfpr_graph *g, int64_t L)
{
    const size_t n = (size_t)g->n;
    int32_t *light = g->bfs_q, *heavy = g->bfs_q + 3 * n;
    uint32_t *qn = g->ctl->qn, *qhn = g->ctl->qhn;   // device addresses
    const int r0 = (int)(L % 3), r1 = (int)((L + 1) % 3), r2 = (int)((L + 2) % 3);
    BfsQueues q;
    q.in = light + r0 * n;
    q.hin = heavy + r0 * n;
    q.nin = qn + r0;
    q.nhin = qhn + r0;
    q.out = light + r1 * n;
    q.hout = heavy + r1 * n;
    q.nout = qn + r1;
    q.nhout = qhn + r1;
    q.clear = qn + r2;
    q.hclear = qhn + r2;
    return q;
}

// The traversal on the graph's stream: seed with the batch sources and
// deletion targets, then levels in chunks between host looks, until a
// level queues nothing.  Reached vertices end with stamp a.sbase.
static int traverse(dfpr_graph *g, const IterArgs &a, int64_t nd, const int32_t *bds,
                    const int32_t *bdd, int64_t ni, const int32_t *bis)
{
    const int32_t n = g->n;
    hipStream_t s = g->stream;
    if (!g->bfs_q) DFPR_HIP(hipMalloc(&g->bfs_q, (size_t)6 * n * sizeof(int32_t)));
    // the seed fills the queues that level 0 reads: those of a level -1
    // (which reads and clears nothing)
    BfsQueues q0 = bfs_queues(g, 2);
    k_bfs_seed<<<std::min(blocks_for(nd + ni), 2048), kBlock, 0, s>>>(a, nd, bds, bdd, ni, bis,
                                                                   q0);
    DFPR_HIP(hipGetLastError());
    uint32_t grid = (uint32_t)g->grid;
    int chunk = 1, walks = 2, looks = 0;
    // A small graph of few edges a vertex has many levels, and a wide one costs as
    // much as a narrow one there: 60 x 60 grid, a call 432 us with wide levels
    // and 375 without.  At 8 edges a vertex they
    // pay (G(n, m), 10^4 vertices: 191 us without and 155 with).
    const bool narrow = n < 16384 && g->m < 6 * (int64_t)n;
    bool wide = false, was_wide = false;
    unsigned long long reach = 0;       // Ctl::reach at the last look
    // every level, narrow or wide, reaches a vertex or is the last
    for (int64_t L = 0;;) {
        if (wide) {
            for (int j = 0; j < walks; j++, L++) {
                const BfsQueues q = bfs_queues(g, L);
                k_bfs_scan<<<std::min(blocks_for(n), 2048), kBlock, 0, s>>>(a, q.hout, q.nout, q.nhout,
                                                                          q.clear, q.hclear);
                k_bfs_heavy<<<1024, kBlock, 0, s>>>(a, q.hout, q.nhout);
            }
        } else {
            for (int j = 0; j < chunk; j++, L++) {
                auto *level = j == chunk - 1 ? k_bfs_level<true> : k_bfs_level<false>;
                level<<<grid, kBlock, 0, s>>>(a, bfs_queues(g, L));
            }
        }
        DFPR_HIP(hipGetLastError());
        DFPR_CHECK_RC(ctl_to_host(g));
        DFPR_HIP(hipStreamSynchronize(s));
        const Ctl &c = *g->ctl_host;
        const uint32_t next = c.qn[L % 3], nexth = c.qhn[L % 3];
        if (c.err || (next == 0 && nexth == 0)) break;
        if (wide) {
            if ((int64_t)next + nexth > n / 1024) {
                // two levels a look, and from the fourth look on, where the end is
                // seldom near, up to eight: 300 x 300 grid, 36 sources, 0.590 ->
                // 0.550 ms a call; 2048 x 2048, 1680 sources, 7.09 -> 6.91
                if (++looks > 3) walks = std::min(walks * 2, 8);
                continue;
            }
            // few are left: a narrow level costs less than a look at every vertex
            k_bfs_collect<<<std::min(blocks_for(n), 2048), kBlock, 0, s>>>(a, bfs_queues(g, L));
            L++;
            wide = false;
            grid = (uint32_t)g->grid;
            chunk = 1;
            walks = 2;
            looks = 0;
            continue;
        }
        // the levels to come are wide once the claims of one, the last, have
        // more out-edges than a quarter of the vertices (a grid of 2048 x 2048
        // vertices reaches that with the 16 levels of a chunk together: 24.5 ms
        // a call, and 26.0 with wide levels)
        wide = !narrow && c.reach - reach > (unsigned long long)n / 4;
        was_wide |= wide;
        reach = c.reach;
        grid = bfs_grid(g, next, nexth);
        chunk = std::min(chunk * 2, 16);
    }
    if (was_wide) {
        // wide levels do not count what they mark
        DFPR_CHECK_RC(launch_fill_u32(g, reinterpret_cast<uint32_t *>(&g->ctl->affected0), 2, 0));
        k_bfs_marked<<<std::min(blocks_for(n), 1024), kBlock, 0, s>>>(a);
        DFPR_HIP(hipGetLastError());
    }
    return DFPR_OK;
}

// Dynamic Traversal PageRank (Section 3.3.2): the reachable set is marked
// before the first iteration and never grows, so the iterations are those
// of Dynamic Frontier with no expansion.  Always FP64.
static int dt_impl(dfpr_graph *g, const dfpr_params *pp, int64_t nd, const int32_t *ds,
                   const int32_t *dd, int64_t ni, const int32_t *is, const int32_t *id,
                   int on_device, const double *prev, double *ranks_out, dfpr_stats *st)
{
    dfpr_params p;
    int rc = check_params(pp, p);
    if (rc) return rc;
    p.precision = DFPR_FP64;
    p.frontier_tol = INFINITY;   // no vertex joins during the iterations
    if (nd < 0 || ni < 0 || (nd && (!ds || !dd)) || (ni && (!is || !id)))
        return set_error(DFPR_E_ARG, "bad batch arrays");
    if (!on_device) {
        rc = check_ids_host(g->n, nd, ds, dd);
        if (!rc) rc = check_ids_host(g->n, ni, is, id);
        if (rc) return rc;
    }
    BusyGuard guard(g);
    if (!guard.ok) return set_error(DFPR_E_BUSY, "graph in use");
    const int32_t n = g->n;
    hipStream_t s = g->stream;
    DFPR_HIP(hipEventRecord(g->ev0, s));
    const int32_t *bds, *bdd, *bis, *bid;
    rc = stage_batch(g, nd, ds, dd, ni, is, id, on_device, &bds, &bdd, &bis, &bid);
    if (rc) return rc;
    const int cur = g->cur;
    uint32_t sbase = 0;
    rc = take_base(g, p.max_iters, &sbase);
    if (rc) return rc;
    IterArgs a = iter_args(g, p, sbase);
    DFPR_CHECK_RC(launch_begin(g, a, BeginArgs{}, prev, on_device, false, false));
    if (nd + ni > 0) {
        k_validate<<<blocks_for(nd + ni), kBlock, 0, s>>>(n, nd, bds, bdd, ni, bis, bid, g->ctl);
        rc = traverse(g, a, nd, bds, bdd, ni, bis);
        if (rc) return rc;
    }
    // the reachable set is usually most of the graph: the iterations walk
    // the full schedule and read the stamps, no class lists are built
    k_snap<<<1, 1, 0, s>>>(g->ctl, p.max_iters, g->sparse_limit, 1, g->ctl_host, p.tol,
                           p.frontier_tol);
    DFPR_HIP(hipGetLastError());
    DFPR_HIP(hipEventRecord(g->ev_mid, s));
    int res = cur;
    Close close;
    if (ranks_out) close.out = on_device ? ranks_out : g->Rx;
    rc = run_loop(g, p, true, false, sbase, 0, cur, &res, &close, false);
    if (rc) return rc;
    return df_end(g, sbase, res, close, ranks_out, on_device, st);
}

// Stamp arrays of the marking-only calls (dfpr_mark_affected,
// dfpr_mark_reachable), allocated on first use.  Keeping them apart from
// the iterations' stamps leaves the marks of the last update readable.
static int marking_stamps(dfpr_graph *g)
{
    if (g->mstamp) return DFPR_OK;
    const size_t bytes = (size_t)g->n * sizeof(uint32_t);
    DFPR_HIP(hipMalloc(&g->mstamp, bytes));
    hipError_t e = hipMalloc(&g->mxstamp, bytes);
    if (e != hipSuccess) {
        (void)hipFree(g->mstamp);
        g->mstamp = nullptr;
        return hip_fail(e, "hipMalloc(marking stamps)");
    }
    DFPR_CHECK_RC(launch_fill_u32(g, g->mstamp, (uint64_t)g->n, 0));
    DFPR_CHECK_RC(launch_fill_u32(g, g->mxstamp, (uint64_t)g->n, 0));
    return DFPR_OK;
}

}  // namespace dfpr

using namespace dfpr;

extern "C" {

int dfpr_set_ranks(dfpr_graph *g, const double *ranks, int on_device)
{
    if (!g) return set_error(DFPR_E_ARG, "graph is NULL");
    BusyGuard guard(g);
    if (!guard.ok) return set_error(DFPR_E_BUSY, "graph in use");
    const int32_t n = g->n;
    hipStream_t s = g->stream;
    if (ranks) {
        const int rc = ranks_from_caller(g, ranks, on_device, g->R[0]);
        if (rc) return rc;
    }
    k_init_ranks<<<blocks_for(n), kBlock, 0, s>>>(n, ranks ? g->R[0] : nullptr, g->R[0], g->R[1],
                                                  g->C[0], g->C[1], g->csr[1].cnt);
    DFPR_HIP(hipGetLastError());
    g->cur = 0;
    DFPR_HIP(hipStreamSynchronize(s));
    return DFPR_OK;
}

int dfpr_pagerank_static(dfpr_graph *g, const dfpr_params *p, double *ranks_out, dfpr_stats *st)
{
    if (!g) return set_error(DFPR_E_ARG, "graph is NULL");
    return full_sweeps(g, p, nullptr, 0, false, ranks_out, 0, st);
}

int dfpr_pagerank_naive_dynamic(dfpr_graph *g, const dfpr_params *p, const double *prev,
                                double *ranks_out, dfpr_stats *st)
{
    if (!g) return set_error(DFPR_E_ARG, "graph is NULL");
    return full_sweeps(g, p, prev, 0, true, ranks_out, 0, st);
}

int dfpr_pagerank_dynamic_frontier(dfpr_graph *g, const dfpr_params *p, int64_t n_del,
                                   const int32_t *del_src, const int32_t *del_dst, int64_t n_ins,
                                   const int32_t *ins_src, const int32_t *ins_dst,
                                   const double *prev, double *ranks_out, dfpr_stats *st)
{
    if (!g) return set_error(DFPR_E_ARG, "graph is NULL");
    return df_impl(g, p, n_del, del_src, del_dst, n_ins, ins_src, ins_dst, 0, prev, ranks_out, st);
}

int dfpr_pagerank_dynamic_frontier_device(dfpr_graph *g, const dfpr_params *p, int64_t n_del,
                                          const int32_t *del_src, const int32_t *del_dst,
                                          int64_t n_ins, const int32_t *ins_src,
                                          const int32_t *ins_dst, const double *prev,
                                          double *ranks_out, dfpr_stats *st)
{
    if (!g) return set_error(DFPR_E_ARG, "graph is NULL");
    return df_impl(g, p, n_del, del_src, del_dst, n_ins, ins_src, ins_dst, 1, prev, ranks_out, st);
}

int dfpr_pagerank_dynamic_traversal(dfpr_graph *g, const dfpr_params *p, int64_t n_del,
                                    const int32_t *del_src, const int32_t *del_dst,
                                    int64_t n_ins, const int32_t *ins_src,
                                    const int32_t *ins_dst, const double *prev,
                                    double *ranks_out, dfpr_stats *st)
{
    if (!g) return set_error(DFPR_E_ARG, "graph is NULL");
    return dt_impl(g, p, n_del, del_src, del_dst, n_ins, ins_src, ins_dst, 0, prev, ranks_out, st);
}

int dfpr_mark_reachable(dfpr_graph *g, int64_t n_del, const int32_t *del_src,
                        const int32_t *del_dst, int64_t n_ins, const int32_t *ins_src,
                        const int32_t *ins_dst, uint8_t *flags_out)
{
    if (!g || !flags_out) return set_error(DFPR_E_ARG, "NULL argument");
    if (n_del < 0 || n_ins < 0 || (n_del && (!del_src || !del_dst)) ||
        (n_ins && (!ins_src || !ins_dst)))
        return set_error(DFPR_E_ARG, "bad batch arrays");
    int rc = check_ids_host(g->n, n_del, del_src, del_dst);
    if (!rc) rc = check_ids_host(g->n, n_ins, ins_src, ins_dst);
    if (rc) return rc;
    BusyGuard guard(g);
    if (!guard.ok) return set_error(DFPR_E_BUSY, "graph in use");
    hipStream_t s = g->stream;
    const int32_t *bds, *bdd, *bis, *bid;
    rc = stage_batch(g, n_del, del_src, del_dst, n_ins, ins_src, ins_dst, 0, &bds, &bdd, &bis,
                     &bid);
    dfpr_params p;
    dfpr_params_default(&p);
    uint32_t sbase = 0;
    if (!rc) rc = marking_stamps(g);
    if (!rc) rc = take_base(g, 0, &sbase);
    if (rc) return rc;
    IterArgs a = iter_args(g, p, sbase);
    a.stamp = g->mstamp;
    a.xstamp = g->mxstamp;
    k_reset<<<1, 1, 0, s>>>(g->ctl);
    DFPR_HIP(hipGetLastError());
    if (n_del + n_ins > 0) {
        rc = traverse(g, a, n_del, bds, bdd, n_ins, bis);
        if (rc) return rc;
    }
    return flags_to_caller(g, g->mstamp, sbase, sbase, flags_out);
}

int dfpr_mark_affected(dfpr_graph *g, int64_t n_del, const int32_t *del_src,
                       const int32_t *del_dst, int64_t n_ins, const int32_t *ins_src,
                       const int32_t *ins_dst, uint8_t *flags_out)
{
    if (!g || !flags_out) return set_error(DFPR_E_ARG, "NULL argument");
    if (n_del < 0 || n_ins < 0 || (n_del && (!del_src || !del_dst)) ||
        (n_ins && (!ins_src || !ins_dst)))
        return set_error(DFPR_E_ARG, "bad batch arrays");
    int rc = check_ids_host(g->n, n_del, del_src, del_dst);
    if (!rc) rc = check_ids_host(g->n, n_ins, ins_src, ins_dst);
    if (rc) return rc;
    BusyGuard guard(g);
    if (!guard.ok) return set_error(DFPR_E_BUSY, "graph in use");
    hipStream_t s = g->stream;
    const int32_t *bds, *bdd, *bis, *bid;
    rc = stage_batch(g, n_del, del_src, del_dst, n_ins, ins_src, ins_dst, 0, &bds, &bdd, &bis,
                     &bid);
    dfpr_params p;
    dfpr_params_default(&p);
    uint32_t sbase = 0;
    if (!rc) rc = marking_stamps(g);
    if (!rc) rc = take_base(g, 0, &sbase);
    if (rc) return rc;
    IterArgs a = iter_args(g, p, sbase);
    a.stamp = g->mstamp;
    a.xstamp = g->mxstamp;
    k_reset<<<1, 1, 0, s>>>(g->ctl);
    if (n_del + n_ins > 0)
        launch_initial_marking(g, a, n_del, bds, bdd, n_ins, bis, 1,
                               g->ap.batch_dev + 2 * (n_del + n_ins), 0, a.sparse_limit);
    DFPR_HIP(hipGetLastError());
    return flags_to_caller(g, g->mstamp, sbase, sbase, flags_out);
}

int dfpr_get_affected(const dfpr_graph *g, uint8_t *flags_out)
{
    if (!g || !flags_out) return set_error(DFPR_E_ARG, "NULL argument");
    if (g->last_iters < 0) {
        std::memset(flags_out, 0, (size_t)g->n);
        return DFPR_OK;
    }
    return flags_to_caller(g, g->stamp, g->last_base, g->last_base + (uint32_t)g->last_iters, flags_out);
}

int dfpr_profile_reset(dfpr_graph *g, int enable)
{
    if (!g) return set_error(DFPR_E_ARG, "graph is NULL");
    // per-launch timing only, read after a stream synchronisation: no
    // system-scope fence (with it, each record stalls the queue ~6 us)
    if (enable)
        for (hipEvent_t &ev : g->evk)
            if (!ev) DFPR_HIP(hipEventCreateWithFlags(&ev, hipEventDisableSystemFence));
    g->prof = Profile{};
    g->prof.enabled = enable ? 1 : 0;
    return DFPR_OK;
}

int dfpr_profile_read(const dfpr_graph *g, dfpr_profile *out)
{
    if (!g || !out) return set_error(DFPR_E_ARG, "NULL argument");
    out->launches = g->prof.launches;
    out->ms = g->prof.ms;
    out->bytes = g->prof.bytes;
    out->rows = g->prof.rows;
    out->edges = g->prof.edges;
    out->expanded_rows = g->prof.exp_rows;
    out->expanded_edges = g->prof.exp_edges;
    out->marked = g->prof.marked;
    return DFPR_OK;
}

// For this library's tests, and in no header: whether resident launches of the
// graph are to end before they start, as they do when not all workgroups run;
// the last barrier tag handed out (0: as it is); and the number of iterations
// that ran in resident launches since the load, serving included.
int dfpr_test_resident(dfpr_graph *g, int refuse, uint32_t tag, int64_t *iterations)
{
    if (!g) return set_error(DFPR_E_ARG, "graph is NULL");
    g->res_refuse = refuse;
    if (tag) g->res_tag = tag;
    if (iterations) *iterations = g->res_iters;
    return DFPR_OK;
}

}  // extern "C"
