// The rank engines' host side (rank.hip), for the serving loop (serve.hip) and
// the entry point that allocates nothing (noalloc.hip).
#pragma once

#include "resident.h"

namespace dfpr {

// How a call ends, if its last iteration runs in the resident loop: that
// launch brings the other buffer up to date, counts the marks and writes the
// ranks in the caller's order.
struct Close {
    double *out = nullptr;      // device; NULL: not wanted
    bool done = false;          // the launch did it
};

IterArgs iter_args(dfpr_graph *g, const dfpr_params &p, uint32_t sbase);
int check_params(const dfpr_params *p, dfpr_params &out);
int df_begin(dfpr_graph *g, const dfpr_params &p, int64_t nd, const int32_t *ds,
             const int32_t *dd, int64_t ni, const int32_t *is, const int32_t *id, int on_device,
             const double *prev, uint32_t *sbase_out, int32_t *staging = nullptr);
// A Dynamic Frontier call on device arrays whose batch is staged in
// `staging` (4 (nd + ni) ints) instead of the library's buffer.
int df_device_staged(dfpr_graph *g, const dfpr_params *pp, int64_t nd, const int32_t *ds,
                     const int32_t *dd, int64_t ni, const int32_t *is, const int32_t *id,
                     const double *prev, double *ranks_out, dfpr_stats *st, int32_t *staging);
int df_phase_end(dfpr_graph *g, int res, bool call_done);
int df_finish(dfpr_graph *g, uint32_t sbase, int res, int32_t iters, bool closed = false);

// The resident loop's launches.
bool resident_whole(const dfpr_graph *g);
uint32_t resident_grid(const dfpr_graph *g);
uint32_t resident_hub(const dfpr_graph *g, bool f32, uint32_t G);
uint32_t resident_lists(const dfpr_graph *g);
int resident_args(dfpr_graph *g, int it0, int it, int base, bool full, uint32_t limit, ResArgs &P);

}  // namespace dfpr
