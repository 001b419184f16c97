// The resident loop: the iterations of Algorithm 1's loop inside one launch,
// for one graph (rank.hip) or for several side by side (serve.hip).
#pragma once

#include "iter.h"

namespace dfpr {

// Where an iteration's rows take less time than its two launches and the
// dispatch between them (about 20 us from one k_iter to the next on a small
// frontier), k_resident runs the iterations of Algorithm 1's loop inside one
// launch: one workgroup of 16 waves per compute unit at most, rows spread and
// summed exactly as in k_iter, and a barrier between iterations that carries
// the fold.
//
// What bounds it is the barrier and one chain of dependent accesses per
// iteration.  A barrier with agent-scope release and acquire fences took
// 9 us for 64 workgroups and 31 us for 256, because the fences write back
// and invalidate L2; so every access to data that another workgroup writes
// during the launch is a relaxed agent-scope one (COH, iter.h), each wave
// waits for its own stores to be acknowledged (s_waitcnt vmcnt(0)) before
// its workgroup arrives, and the barrier has no fence: 1.4 us for 64
// workgroups, 1.7 us for 256.
//
// Arrival: a workgroup stores its Delta R (and, in the FP32 phase, its largest
// rank) as two tagged words each.  One wave of workgroup 0 polls all of them,
// folds them, takes the decision of final_step on a copy of the control block
// in LDS, and publishes the state of the next iteration as eight tagged words,
// in eight copies so that an XCD's workgroups poll one of their own.  A word
// is 32 bits of value and a 32-bit tag that no other barrier of the graph
// uses, so a word is its own flag and nothing is cleared between launches.
// One wave instead of a thread per word saves the workgroup barriers around
// the fold, and lane moves instead of shuffles most of its latency: an
// iteration of a 10,000-vertex graph takes 9.5 us against 10.4.
//
// No cooperative launch: before anything is written, the workgroups wait a
// bounded time until all of them run, and one compare-and-swap decides for
// all whether they go or leave.  Other work on the device can so at worst
// send a call back to a launch per iteration.
//
// Where it is used.  Graphs of up to kResEdges in-edges run whole calls in
// it, because their full sweep is short next to the launches or gains from
// the larger LDS copy.  Static and a Dynamic Frontier call of 1e-5 of the edges,
// launches over resident loop: R-MAT with 16M / 25M / 33M / 39M edges 1.61 / 1.41
// / 1.31 / 1.14 and 1.52 / 1.32 / 1.22 / 1.16; grids with 20M / 29M / 39M 1.36 /
// 1.21 / 1.12 and 2.8; G(n, m) with 17M / 26M / 35M 1.05 / 1.00 / 1.00 and 1.12 /
// 1.07 / 1.06 at 13 edges a vertex, 1.26 / 1.02 / 0.99 and 0.99 / 0.93 / 0.98 at
// 24, where one iteration marks most vertices with stores that go past L2.  On
// R-MAT scale 22 (69M) its 16 waves per compute unit and gathers past the vector
// L1 lose to k_iter_wide (32.9 and 30.1 ms an update pair), so larger graphs use
// it only while a Dynamic Frontier call is on the class lists.
constexpr int64_t kResEdges = 40000000;
// In the resident loop a row goes to a class list by an LDS-staged append, so
// the lists may hold an eighth of the vertices before walking every id range
// with its stamp is quicker (a 64th with launches): 1.57 against 2.35 ms on
// uniform grid batches, no change on R-MAT.
constexpr int32_t kResSparse = 8;
// Wave units per wave of the full schedule from which FP64 sweeps take two rows
// a lane group (wave_pair).  Of a call on R-MAT scale 17 (2.2 units a wave) it
// takes 2134 instead of 2076 us, since waves are left without a unit; scale 18
// (4.4) 3009 instead of 3017, scale 20 (16) 8460 instead of 8742, a grid of
// 2048 x 2048 vertices (32) 5759 instead of 6889.  The FP32 form's sums are a
// longer chain of instructions and slower in pairs: 1.5e6 vertices 10.42
// instead of 10.25 ms.  On the class lists a unit has one row a lane group:
// pairs made a call on R-MAT scale 13 11% slower.
constexpr uint32_t kPairUnits = 4;
constexpr uint32_t kLoopRows = 16384;            // DFPR_LOOP_DEVICE: most rows of an iteration
constexpr uint32_t kNoLimit = 0xFFFFFFFFu;       //   ... of the other calls
constexpr int kResWaves = 16;
constexpr int kResThreads = kResWaves * kWave;
constexpr int kResMax = 256;                     // workgroups
constexpr uint32_t kResHub = 16384;              // contributions in LDS (twice as many FP32)
constexpr int kResSteps = 1024;                  // most iterations of one launch
constexpr uint32_t kResTags = kResSteps + 4;     // tags a launch takes
constexpr uint32_t kGoSpin = 256;                // polls before a launch gives up starting
constexpr uint32_t kSpinLimit = 1u << 24;        // polls of a barrier before it reports failure
constexpr int kResCopies = 8;                    // copies of the published state

constexpr int kResCounts = kCounters + 1;        // and the marks

// What the workgroups of a resident loop exchange (dfpr_graph::it.res).
struct ResWords {
    unsigned long long arrive[4][kResMax];           // Delta R (low, high half), largest rank
    unsigned long long state[kResCopies * 8];        // flags, class list lengths
    unsigned long long count[kResMax * kResCounts];  // counters of the launch, at its end
    unsigned long long go;                           // whether the launch of a tag runs
};

static_assert(sizeof(ResWords) <= kResBytes, "kResBytes holds the exchanged words");

struct ResArgs {
    double *R[2], *C[2];
    float *C32[2];
    ResWords *w;
    int base;           // buffer that iteration it0 reads
    int it0;            // first iteration of the phase (buffer parity)
    int it_start;       // first iteration of this launch
    int full;           // the launch keeps going on the full schedule
    uint32_t limit;     // class list rows of an iteration above which it hands over
    uint32_t blocks;    //   ... and rows of the workgroup class
    uint32_t spin;      // polls of workgroup 0 before the launch gives up starting
    uint32_t tag;       // first of its tags
    int close;          // end the call too, if it converges or reaches the cap
    double *out;        //   the ranks in the caller's order (nullable)
    const int32_t *ext2int;
    uint32_t budget;    // 10 ns ticks after which the launch hands over (0: none)
    uint32_t *stop;     // several graphs in one launch: set to stop_tag when one of
    uint32_t stop_tag;  //   them is over, so that the others hand over too
};

struct ResShared {
    Ctl ctl;                            // workgroup 0: the control block
    double wdr[kResWaves], wrm[kResWaves];
    unsigned long long wc[kResWaves][kCounters];
    uint32_t state[8];
    uint32_t lists[8];                  // class list lengths, and whether to leave the lists
    Stage stage;
    int go, fail;
};

struct ResLds {
    IterSharedT<kResWaves> sh;
    ResShared rs;
    double hub[kResHub];
};

__device__ __forceinline__ unsigned long long tagged(uint32_t value, uint32_t tag)
{
    return ((unsigned long long)value << 32) | tag;
}

// Poll a tagged word; false if its tag did not come within kSpinLimit polls.
__device__ __forceinline__ bool await_word(const unsigned long long *p, uint32_t tag, uint32_t &value)
{
    for (uint32_t n = 0; n < kSpinLimit; n++) {
        const unsigned long long x = ld<true>(p);
        if ((uint32_t)x == tag) {
            value = (uint32_t)(x >> 32);
            return true;
        }
    }
    return false;
}

// The value whose halves the G workgroups of a launch store in lo[] and hi[]
// under `tag`: the largest of those a lane of the polling wave takes.  All
// words of a round are loaded at once.
__device__ __forceinline__ bool await_all(const unsigned long long *lo, const unsigned long long *hi,
                                          uint32_t G, uint32_t tag, double &most)
{
    constexpr int K = kResMax / kWave;
    unsigned long long x[K], y[K];
    for (uint32_t n = 0; n < kSpinLimit; n++) {
        bool all = true;
#pragma unroll
        for (int k = 0; k < K; k++) {
            const uint32_t w = lane_id() + k * kWave;
            x[k] = w < G ? ld<true>(lo + w) : (unsigned long long)tag;
            y[k] = w < G ? ld<true>(hi + w) : (unsigned long long)tag;
        }
#pragma unroll
        for (int k = 0; k < K; k++) all = all && (uint32_t)x[k] == tag && (uint32_t)y[k] == tag;
        if (all) {
#pragma unroll
            for (int k = 0; k < K; k++)
                most = fmax(most, __hiloint2double((int)(y[k] >> 32), (int)(x[k] >> 32)));
            return true;
        }
    }
    return false;
}

// Whether every workgroup of the graph runs.  One compare-and-swap decides it
// for all of them: workgroup 0 makes it once all have arrived, any other that
// has waited too long makes it against.
__device__ inline bool resident_start(const ResArgs &P, uint32_t blk, uint32_t G, ResShared &rs)
{
    unsigned long long *const go = &P.w->go;
    // the decision of this launch: tag and 1 (go) or 0; anything else is an
    // earlier launch's
    auto decide = [&](uint32_t x) {
        unsigned long long was = ld<true>(go);
        while ((uint32_t)was != P.tag) {
            const unsigned long long seen = atomicCAS(go, was, tagged(x, P.tag));
            if (seen == was) return x;
            was = seen;
        }
        return (uint32_t)(was >> 32);
    };
    if (threadIdx.x == 0) {
        rs.go = 1;
        st<true>(&P.w->arrive[0][blk], tagged(0u, P.tag));
    }
    __syncthreads();
    if (blk == 0) {
        bool here = threadIdx.x >= G;
        for (uint32_t n = 0; n < P.spin && !here; n++)
            here = (uint32_t)ld<true>(&P.w->arrive[0][threadIdx.x]) == P.tag;
        if (!here) rs.go = 0;
        __syncthreads();
        if (threadIdx.x == 0) rs.go = (int)decide(rs.go ? 1u : 0u);
    } else if (threadIdx.x == 0) {
        unsigned long long x = 0;
        for (uint32_t n = 0; n < 2 * P.spin && (uint32_t)x != P.tag; n++) x = ld<true>(go);
        rs.go = (int)decide(0u);
    }
    __syncthreads();
    return rs.go != 0;
}

// Workgroup blk of the G that iterate one graph.
template <bool DF, bool F32, bool PAIRS>
__device__ __forceinline__ void resident_body(IterArgs a, const ResArgs &P, uint32_t blk, uint32_t G,
                                              ResLds &lds)
{
    IterSharedT<kResWaves> &sh = lds.sh;
    ResShared &rs = lds.rs;
    double *const hub_lds = lds.hub;
    if (!resident_start(P, blk, G, rs)) return;
    const unsigned long long t0_clock = P.budget ? wall_clock64() : 0ull;
    const int wave = threadIdx.x / kWave;
    // the state at the launch's start: the kernels before it left it
    bool dense = !DF || a.ctl->dense, stop = a.ctl->done || (F32 && a.ctl->phase_end);
    if (threadIdx.x < 8)
        rs.state[threadIdx.x] =
            threadIdx.x ? a.ctl->snap[P.it_start & 1][threadIdx.x - 1] : 0u;
    if (threadIdx.x == 0) {
        rs.fail = 0;
        // a negative frontier tolerance asks for the call's adaptive choice
        sh.plan.ftol = a.ftol >= 0.0 ? a.ftol : a.ctl->ftol_used;
        sh.plan.plain = a.ctl->plain_marks;
        rs.stage.item = reinterpret_cast<uint2 *>(hub_lds);
        rs.stage.cap = kResHub;
    }
    a.stage = &rs.stage;
    if (blk == 0) {
        constexpr int words = (int)(sizeof(Ctl) / 4);
        for (int i = threadIdx.x; i < words; i += kResThreads)
            reinterpret_cast<uint32_t *>(&rs.ctl)[i] = reinterpret_cast<const uint32_t *>(a.ctl)[i];
    }
    __syncthreads();
    unsigned long long tot[kCounters] = {0, 0, 0, 0};
    uint32_t tag = P.tag;
    bool planned = false;       // the full schedule's plan does not change
    bool over = false;          // the call has converged or reached the cap
    int k = 0;
    for (; k < kResSteps; k++) {
        const int it = P.it_start + k;
        const uint32_t tid = fresh(threadIdx.x);
        const int lane = tid % kWave;
        uint32_t rows = 0;
#pragma unroll
        for (int b = 0; b < kBins; b++) rows += rs.state[1 + b];
        if (stop || (dense ? !P.full : rows > P.limit || rs.state[kBins] > P.blocks))
            break;      // uniform over the launch
        const int src = P.base ^ ((it - P.it0) & 1);
        a.it = it;
        a.Rc = src ? P.R[1] : P.R[0];
        a.Cc = src ? P.C[1] : P.C[0];
        a.Rn = src ? P.R[0] : P.R[1];
        a.Cn = src ? P.C[0] : P.C[1];
        a.C32c = src ? P.C32[1] : P.C32[0];
        a.C32n = src ? P.C32[0] : P.C32[1];
        const bool sparse = DF && !dense;
        if (wave == 0 && !(dense && planned))
            make_plan_wave(a, a.ctl, sparse, DF, F32, PAIRS, rs.state + 1, G, G * kResWaves, sh.plan);
        planned = dense;
        if (sparse && tid <= kBins) (tid ? rs.stage.cnt[tid - 1] : rs.stage.n) = 0;
        Hub hub{hub_lds, reinterpret_cast<const float *>(hub_lds), 0u};
        if (!sparse && a.hub) {
            hub.n = a.hub;
            if (F32) {
                float *f = reinterpret_cast<float *>(hub_lds);
                for (uint32_t v = tid; v < hub.n; v += kResThreads) f[v] = ld<true>(a.C32c + v);
            } else {
                for (uint32_t v = tid; v < hub.n; v += kResThreads)
                    hub_lds[v] = ld<true>(a.Cc + v);
            }
        }
        __syncthreads();
        Acc acc;
        acc.ftol = sh.plan.ftol;
        acc.plain = sh.plan.plain != 0;
        iter_rows<DF, F32, kResWaves, true, PAIRS>(a, hub, blk, G, sh, DF && dense, sparse, acc);
#pragma unroll
        for (int j = 0; j < kCounters; j++) tot[j] += acc.c[j];
        if (sparse) {
            // the new list entries of the workgroup
            __syncthreads();
            const uint32_t n = min(rs.stage.n, rs.stage.cap);
            if (n) {
                if (tid < kBins && rs.stage.cnt[tid])
                    rs.stage.base[tid] =
                        atomicAdd(&a.ctl->live[tid], rs.stage.cnt[tid]);
                __syncthreads();
                for (uint32_t i = tid; i < n; i += kResThreads) {
                    const uint2 e = rs.stage.item[i];
                    const uint32_t c = e.y >> 28;
                    st<true>(&a.bins[(size_t)c * a.n_stride + rs.stage.base[c] + (e.y & 0xFFFFFFFu)],
                             (int32_t)e.x);
                }
            }
        }
        // arrive: Delta R and the largest rank of the workgroup
        const double wdr = wave_max<kWave>(acc.dr_max);
        const double wrm = F32 ? wave_max<kWave>(acc.r_max) : 0.0;
        if (lane == 0) {
            rs.wdr[wave] = wdr;
            if (F32) rs.wrm[wave] = wrm;
        }
        drain_stores();
        __syncthreads();
        tag++;
        if (wave == 0) {
            const double dr = wave_max<kResWaves>(rs.wdr[lane % kResWaves]);
            const double rm = F32 ? wave_max<kResWaves>(rs.wrm[lane % kResWaves]) : 0.0;
            const unsigned long long bits =
                (unsigned long long)__double_as_longlong(lane & 2 ? rm : dr);
            if (lane < (F32 ? 4 : 2))
                st<true>(&P.w->arrive[lane][blk],
                         tagged((uint32_t)(lane & 1 ? bits >> 32 : bits), tag));
        }
        if (blk == 0) {
            if (wave == 0) {
                double dr = 0.0, rm = 0.0;
                bool ok = await_all(P.w->arrive[0], P.w->arrive[1], G, tag, dr);
                if (F32) ok = await_all(P.w->arrive[2], P.w->arrive[3], G, tag, rm) && ok;
                if (__ballot(!ok)) rs.fail = 1;
                if (sparse && lane <= kBins)
                    rs.lists[lane] = lane < kBins ? ld<true>(&a.ctl->live[lane])
                                                  : ld<true>(&a.ctl->force_dense);
                dr = wave_max<kWave>(dr);
                if (F32) rm = wave_max<kWave>(rm);
                wave_fence();
                if (lane == 0) {
                    final_step(a, &rs.ctl, rs.lists, sparse, F32, dr, rm);
                    const bool end = rs.fail || rs.ctl.done || (F32 && rs.ctl.phase_end);
                    uint32_t out = (end ? 1u : 0u) | (rs.ctl.dense ? 2u : 0u) |
                                   (end && !rs.fail && rs.ctl.done ? 4u : 0u);
                    if (P.stop) {
                        if (end) st<true>(P.stop, P.stop_tag);
                        else if (ld<true>(P.stop) == P.stop_tag) out |= 1u;
                    }
                    if (P.budget && wall_clock64() - t0_clock > P.budget) out |= 1u;
                    rs.state[0] = out;
                }
                wave_fence();
                if (lane < kBins) rs.state[1 + lane] = rs.ctl.snap[(it & 1) ^ 1][lane];
                static_assert(kResCopies * 8 == kWave, "a lane per published word");
                wave_fence();
                st<true>(&P.w->state[lane], tagged(rs.state[lane & 7], tag));
            }
            __syncthreads();
        } else {
            if (tid < 8) {
                uint32_t v = 1u;
                if (!await_word(&P.w->state[(blk & (kResCopies - 1)) * 8 + tid], tag, v))
                    rs.fail = 1;
                rs.state[tid] = v;
            }
            __syncthreads();
        }
        stop = rs.fail || (rs.state[0] & 1u);
        dense = !DF || (rs.state[0] & 2u);
        over = rs.state[0] & 4u;
    }
    unsigned long long marks = 0;
    const bool close = !F32 && P.close && over && !rs.fail;
    if (close) {
        // the other buffer on the processed rows (k_finish, k_copy2), and
        // the ranks in the caller's order
        const int it = P.it_start + k, res = P.base ^ ((it - P.it0) & 1);
        const double *Rr = res ? P.R[1] : P.R[0], *Cr = res ? P.C[1] : P.C[0];
        double *Ro = res ? P.R[0] : P.R[1], *Co = res ? P.C[0] : P.C[1];
        const uint32_t t0 = blk * kResThreads + threadIdx.x, step = G * kResThreads;
        if (DF && !dense) {
            uint32_t tot = 0;
#pragma unroll
            for (int b = 0; b < kBins; b++) tot += rs.state[1 + b];
            for (uint32_t t = t0; t < tot; t += step) {
                uint32_t b = 0, r = t;
                while (r >= rs.state[1 + b]) r -= rs.state[1 + b++];
                const int32_t v = ld<true>(&a.bins[(size_t)b * a.n_stride + r]);
                marks++;
                Ro[v] = ld<true>(Rr + v);
                Co[v] = ld<true>(Cr + v);
            }
        } else {
            for (uint32_t v = t0; v < (uint32_t)a.n; v += step) {
                if (DF) {
                    const uint32_t sx = ld<true>(a.stamp + v);
                    if (sx < a.sbase || sx > a.sbase + (uint32_t)it) continue;
                    marks++;
                }
                Ro[v] = ld<true>(Rr + v);
                Co[v] = ld<true>(Cr + v);
            }
        }
        if (P.out)
            for (uint32_t v = t0; v < (uint32_t)a.n; v += step) P.out[v] = ld<true>(Rr + P.ext2int[v]);
    }
    // counters of the launch, and the control block back to memory and host
    double d0 = 0.0, d1 = 0.0;
    block_fold<kResWaves>(d0, d1, tot, rs.wdr, rs.wrm, rs.wc);
    unsigned long long mk[kCounters] = {marks, 0, 0, 0};
    if (DF) block_fold<kResWaves>(d0, d1, mk, rs.wdr, rs.wrm, rs.wc);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int j = 0; j < kCounters; j++) st<true>(&P.w->count[blk * kResCounts + j], tot[j]);
        st<true>(&P.w->count[blk * kResCounts + kCounters], mk[0]);
        drain_stores();
        st<true>(&P.w->arrive[0][blk], tagged(0u, P.tag + kResSteps + 1));
    }
    if (blk) return;
    uint32_t v = 0;
    if (threadIdx.x < G && !await_word(&P.w->arrive[0][threadIdx.x], P.tag + kResSteps + 1, v))
        rs.fail = 1;
#pragma unroll
    for (int j = 0; j < kCounters; j++)
        tot[j] = threadIdx.x < G ? ld<true>(&P.w->count[threadIdx.x * kResCounts + j]) : 0ull;
    block_fold<kResWaves>(d0, d1, tot, rs.wdr, rs.wrm, rs.wc);
    if (DF) {
        mk[0] = threadIdx.x < G ? ld<true>(&P.w->count[threadIdx.x * kResCounts + kCounters]) : 0ull;
        mk[1] = mk[2] = mk[3] = 0;
        block_fold<kResWaves>(d0, d1, mk, rs.wdr, rs.wrm, rs.wc);
    }
    if (threadIdx.x == 0) {
        Ctl *c = a.ctl;
        const Ctl &s = rs.ctl;
        c->verts = s.verts + tot[0];
        c->edges = s.edges + tot[1];
        c->xverts = s.xverts + tot[2];
        c->xedges = s.xedges + tot[3];
        c->marked = s.marked;
        c->affected = s.affected + mk[0];
        c->loop_closed = close && !rs.fail;
        c->iterations = s.iterations;
        c->final_linf = s.final_linf;
        c->final_rmax = s.final_rmax;
        c->prev_linf = s.prev_linf;
        c->phase_iters = s.phase_iters;
        c->phase_end = s.phase_end;
        c->converged = s.converged;
        c->dense = s.dense;
        c->done = rs.fail ? 1u : s.done;
        c->loop_fail = (uint32_t)rs.fail;
        c->loop_ran = P.tag;
        for (int b = 0; b < kBins; b++) {
            c->snap[0][b] = s.snap[0][b];
            c->snap[1][b] = s.snap[1][b];
        }
        drain_stores();
    }
    __syncthreads();
    if (threadIdx.x < kWave) ctl_to_mirror(a.ctl, a.mirror);
}

}  // namespace dfpr
