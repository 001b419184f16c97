// Graph store: loading, freeing, export, resident ranks, errors.
//
// A graph lives in device memory as two CSRs with per-row slack:
//   csr[0] (in-edges)  : row v lists G.in(v), used by the pull of Eq. 1;
//   csr[1] (out-edges) : row u lists G.out(u); its live count is |out(u)|.
// Loading (not timed by the paper, Section 5.1.5) copies the edge list up and
// builds both CSRs on the device with radix sorts.  Vertices get internal ids
// in order of decreasing in-degree (stable in the caller's ids); the maps
// between the two numberings are applied wherever ids or per-vertex values
// cross the C-ABI.
#include <algorithm>
#include <cstring>
#include <new>
#include <vector>

#include "common.h"
#include "launch.h"
#include "resident.h"

namespace dfpr {

// Iteration-kernel workgroups per CU.  The kernel fits five waves per SIMD,
// so most of the grid waits for a free slot; many small workgroups even
// out the uneven rows (32 per CU measured best on R-MAT scale 22, 5% over 8).
#ifndef DFPR_GRID_PER_CU
#define DFPR_GRID_PER_CU 32
#endif
constexpr int kGridPerCU = DFPR_GRID_PER_CU;
// Workgroups per CU of the wide full-schedule kernels: 12-wave sweeps (two
// resident per CU; 11 beat 8 and 16) and 8-wave Dynamic Frontier
// iterations (three resident per CU).
#ifndef DFPR_WIDE_GRID_PER_CU
#define DFPR_WIDE_GRID_PER_CU 11
#endif
#ifndef DFPR_WIDE_DF_GRID_PER_CU
#define DFPR_WIDE_DF_GRID_PER_CU 16
#endif
constexpr int kWideGridPerCU = DFPR_WIDE_GRID_PER_CU;
constexpr int kWideDfGridPerCU = DFPR_WIDE_DF_GRID_PER_CU;

static thread_local std::string g_last_error;

int set_error(int code, const std::string &msg)
{
    g_last_error = msg;
    return code;
}

int hip_fail(hipError_t e, const char *what)
{
    // reported here: the next look at the last error is not about it
    (void)hipGetLastError();
    return set_error(e == hipErrorOutOfMemory ? DFPR_E_NOMEM : DFPR_E_DEVICE,
                     std::string(what) + ": " + hipGetErrorString(e));
}

int check_ids_host(int32_t n, int64_t len, const int32_t *a, const int32_t *b)
{
    for (int64_t i = 0; i < len; i++)
        if (a[i] < 0 || a[i] >= n || b[i] < 0 || b[i] >= n)
            return set_error(DFPR_E_RANGE, "vertex id outside [0, n) at batch entry " +
                                                std::to_string(i));
    return DFPR_OK;
}

// Slack given to a row of `deg` live entries.
__host__ __device__ static inline uint64_t row_capacity(uint64_t deg)
{
    return deg + (deg / 8 > 2 ? deg / 8 : 2);
}

constexpr uint64_t kMaxEdgeSlots = 0xFFFFFFFFull;   // of an index array (32-bit offsets)

// Free slots kept after the packed rows for rows that outgrow their slack.
static inline uint64_t spill_reserve(uint64_t packed)
{
    return std::max<uint64_t>(packed / 16, 1 << 16);
}

static inline unsigned grid_of(int64_t items)
{
    return (unsigned)std::max<int64_t>(1, (items + kBlock - 1) / kBlock);
}

// ---------------------------------------------------------------------------
// building the graph on the device
// ---------------------------------------------------------------------------
// The edge list becomes 64-bit keys source << b | target (b bits per id) in
// internal ids, self-loops added; sorted and without repeats they are the
// out-rows one after the other, and a stable sort of them by target gives the
// in-rows.  Bound: the radix passes, each two reads and a write of the keys;
// on small graphs their launches.
// A load with its allocations, against the same on one host core: R-MAT scale
// 16 (1.1M keys) 1.2 and 22.9 ms, scale 20 9.4 and 572 ms, scale 22 34 and
// 2443 ms, of which the copy of the edge list takes 18.
// Memory: beside the graph, 16.5 bytes an input edge and 37 a vertex, on the
// device or, where that has no room for it, in pinned host memory, which the
// same kernels then work in over the bus.  What they update with atomics is in
// the graph's own arrays, so that the rest may be host memory.

// What the host needs back from the build.
struct LoadInfo {
    uint32_t err;               // an id outside [0, n)
    uint32_t dmax;              // largest in-degree as counted for the numbering
    uint32_t max_cap[2];        // largest row capacity, per orientation
    uint64_t edges;             // distinct edges, self-loops included
    uint64_t packed[2];         // slots of the packed rows
    uint64_t hub[kHubSteps];    // out-edges of the first 1024 << k vertices
    uint32_t cls[kBins + 2];
};

// In-degrees counted over the input edges (repeats and self-loops as given),
// plus one for the self-loop; deg starts at 1.
__global__ void k_load_degrees(int32_t n, int64_t m, const int32_t *src, const int32_t *dst,
                               uint32_t *deg, LoadInfo *info)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t u = src[i], v = dst[i];
        if (u < 0 || u >= n || v < 0 || v >= n) info->err = 1;
        else atomicAdd(&deg[v], 1u);
    }
}

__global__ __launch_bounds__(kBlock) void k_load_max(int32_t n, const uint32_t *deg, LoadInfo *info)
{
    uint32_t x = 0;
    for (int64_t v = blockIdx.x * (int64_t)kBlock + threadIdx.x; v < n; v += (int64_t)gridDim.x * kBlock)
        x = max(x, deg[v]);
    for (int off = kWave / 2; off > 0; off >>= 1) x = max(x, (uint32_t)__shfl_xor((int)x, off, kWave));
    if (threadIdx.x % kWave == 0) atomicMax(&info->dmax, x);
}

// Sort key of a vertex: decreasing degree, then the caller's id.
__global__ void k_load_vertex_keys(int32_t n, const uint32_t *deg, uint32_t dmax, uint64_t *key)
{
    const int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (v < n) key[v] = (uint64_t)(dmax - deg[v]) << 32 | (uint64_t)v;
}

// The two maps from the sorted vertex keys; one thread per class boundary
// finds the first id whose degree is at most the class's (see Ctl::cls).
__global__ void k_load_maps(int32_t n, const uint64_t *key, uint32_t dmax, int32_t *ext2int,
                            int32_t *int2ext, LoadInfo *info)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) {
        const int32_t v = (int32_t)(uint32_t)key[i];
        int2ext[i] = v;
        ext2int[v] = (int32_t)i;
    }
    if (blockIdx.x == 0 && threadIdx.x < kBins + 2) {
        // ids before cls[k] have a degree above most[k]
        const uint32_t most[kBins + 2] = {0xFFFFFFFFu, 1024, 128, 32, 16, 8, 4, 1, 0};
        uint32_t lo = 0, hi = (uint32_t)n;
        while (lo < hi) {
            const uint32_t mid = (lo + hi) / 2;
            if (dmax - (uint32_t)(key[mid] >> 32) > most[threadIdx.x]) lo = mid + 1;
            else hi = mid;
        }
        info->cls[threadIdx.x] = lo;
    }
}

__global__ void k_load_edge_keys(int32_t n, int64_t m, const int32_t *src, const int32_t *dst,
                                 const int32_t *ext2int, int b, uint64_t *key)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m + n;
         i += (int64_t)gridDim.x * blockDim.x)
        key[i] = i < m ? (uint64_t)ext2int[src[i]] << b | (uint64_t)ext2int[dst[i]]
                       : (uint64_t)(i - m) << b | (uint64_t)(i - m);
}

// One pass of a stable radix sort over digits of at most 8 bits.  A workgroup
// takes a tile of kSortTile keys, each wave a quarter of it in order.
constexpr int kSortRounds = 16;
constexpr int kSortTile = kBlock * kSortRounds;
constexpr int kDigits = 256;

// Lanes of the wave with the same digit (`bits` bits) among those with `ok`.
__device__ inline unsigned long long same_digit(uint32_t d, int bits, bool ok)
{
    unsigned long long m = __ballot(ok);
    for (int k = 0; k < bits; k++) {
        const unsigned long long one = __ballot(ok && ((d >> k) & 1u));
        m &= ((d >> k) & 1u) ? one : ~one;
    }
    return m;
}

// counts[digit * tiles + tile]
__global__ __launch_bounds__(kBlock) void k_sort_count(const uint64_t *key, uint64_t len, int shift,
                                                       int bits, uint64_t tiles, uint64_t *counts)
{
    __shared__ uint32_t s[kDigits];
    s[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t base = blockIdx.x * (uint64_t)kSortTile;
#pragma unroll 4
    for (int r = 0; r < kSortRounds; r++) {
        const uint64_t i = base + r * kBlock + threadIdx.x;
        if (i < len) atomicAdd(&s[(key[i] >> shift) & ((1u << bits) - 1)], 1u);
    }
    __syncthreads();
    if ((int)threadIdx.x < (1 << bits)) counts[threadIdx.x * tiles + blockIdx.x] = s[threadIdx.x];
}

__global__ __launch_bounds__(kBlock) void k_sort_scatter(const uint64_t *key, uint64_t len, int shift,
                                                         int bits, uint64_t tiles,
                                                         const uint64_t *offsets, uint64_t *out)
{
    __shared__ uint64_t at[kWavesPerBlock][kDigits];
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const uint64_t base = blockIdx.x * (uint64_t)kSortTile + wave * (kSortRounds * kWave);
    const uint32_t mask = (1u << bits) - 1;
    for (int k = threadIdx.x; k < kWavesPerBlock * kDigits; k += kBlock) (&at[0][0])[k] = 0;
    __syncthreads();
    uint64_t x[kSortRounds];
    uint32_t before[kSortRounds];       // keys of the wave with the same digit before this one
#pragma unroll
    for (int r = 0; r < kSortRounds; r++) {
        const uint64_t i = base + r * kWave + lane;
        x[r] = i < len ? key[i] : 0ull;
    }
#pragma unroll
    for (int r = 0; r < kSortRounds; r++) {
        const bool ok = base + r * kWave + lane < len;
        const uint32_t d = (uint32_t)(x[r] >> shift) & mask;
        const unsigned long long m = same_digit(d, bits, ok);
        const uint32_t rank = (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        // the wave runs in step: every lane reads the count before the first
        // lane of each digit adds to it
        const uint32_t c = ok ? (uint32_t)at[wave][d] : 0u;
        wave_fence();
        if (ok && rank == 0) at[wave][d] = c + (uint32_t)__popcll(m);
        wave_fence();
        before[r] = c + rank;
    }
    __syncthreads();
    if ((int)threadIdx.x <= (int)mask) {
        uint64_t o = offsets[threadIdx.x * tiles + blockIdx.x];
        for (int w = 0; w < kWavesPerBlock; w++) {
            const uint64_t c = at[w][threadIdx.x];
            at[w][threadIdx.x] = o;
            o += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortRounds; r++)
        if (base + r * kWave + lane < len)
            out[at[wave][(uint32_t)(x[r] >> shift) & mask] + before[r]] = x[r];
}

// Distinct keys of a tile, then their move to the front of `out`.
__global__ __launch_bounds__(kBlock) void k_load_distinct(const uint64_t *key, uint64_t len,
                                                          uint64_t *counts, uint64_t *out)
{
    __shared__ uint32_t s_wave[kSortRounds][kWavesPerBlock];
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const uint64_t base = blockIdx.x * (uint64_t)kSortTile;
    unsigned long long m[kSortRounds];
#pragma unroll
    for (int r = 0; r < kSortRounds; r++) {
        const uint64_t i = base + r * kBlock + threadIdx.x;
        m[r] = __ballot(i < len && (i == 0 || key[i] != key[i - 1]));
        if (lane == 0) s_wave[r][wave] = (uint32_t)__popcll(m[r]);
    }
    __syncthreads();
    uint64_t at = out ? counts[blockIdx.x] : 0;
#pragma unroll
    for (int r = 0; r < kSortRounds; r++)
        for (int w = 0; w < kWavesPerBlock; w++) {
            if (out && w == wave && ((m[r] >> lane) & 1ull))
                out[at + __popcll(m[r] & ((1ull << lane) - 1ull))] =
                    key[base + r * kBlock + threadIdx.x];
            at += s_wave[r][w];
        }
    if (!out && threadIdx.x == 0) counts[blockIdx.x] = at;
}

__global__ void k_load_swap(uint64_t len, int b, const uint64_t *key, uint64_t *out)
{
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < len;
         i += (uint64_t)gridDim.x * blockDim.x)
        out[i] = (key[i] & ((1ull << b) - 1)) << b | key[i] >> b;
}

// First key of every row (each row holds at least its self-loop).
__global__ void k_load_starts(uint64_t len, int b, int32_t n, const uint64_t *key, uint64_t *start)
{
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < len;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t r = key[i] >> b;
        if (i == 0 || (key[i - 1] >> b) != r) start[r] = i;
        if (i == 0) start[n] = len;
    }
}

__global__ void k_load_caps(int32_t n, const uint64_t *start, uint32_t *cnt, uint32_t *cap,
                            uint64_t *caps, int o, LoadInfo *info)
{
    const int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    uint32_t c = 0;
    if (r < n) {
        const uint32_t d = (uint32_t)(start[r + 1] - start[r]);
        c = (uint32_t)row_capacity(d);
        cnt[r] = d;
        cap[r] = c;
        caps[r] = c;
    } else if (r == n) {
        caps[r] = 0;
    }
    for (int off = kWave / 2; off > 0; off >>= 1) c = max(c, (uint32_t)__shfl_xor((int)c, off, kWave));
    if (threadIdx.x % kWave == 0 && c) atomicMax(&info->max_cap[o], c);
    if (o == 1 && blockIdx.x == 0 && threadIdx.x < kHubSteps)
        info->hub[threadIdx.x] = start[min((int64_t)1024 << threadIdx.x, (int64_t)n)];
}

// `at`: the scanned capacities, n + 1 of them.
__global__ void k_load_begs(int32_t n, const uint64_t *at, uint32_t *beg, int o, LoadInfo *info)
{
    const int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (r < n) beg[r] = (uint32_t)at[r];
    if (r == 0) info->packed[o] = at[n];
}

__global__ void k_load_rows(uint64_t len, int b, const uint64_t *key, const uint64_t *start,
                            const uint32_t *beg, int32_t *idx)
{
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < len;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t r = key[i] >> b;
        idx[(uint64_t)beg[r] + (i - start[r])] = (int32_t)(key[i] & ((1ull << b) - 1));
    }
}

// Memory of a scope, device or pinned host.
struct Scratch {
    void *p = nullptr;
    bool host = false;
    ~Scratch()
    {
        if (host) (void)hipHostFree(p);
        else (void)hipFree(p);
    }
    int take(size_t bytes, bool on_host)
    {
        host = on_host;
        if (host) DFPR_HIP(hipHostMalloc(&p, bytes, hipHostMallocDefault));
        else DFPR_HIP(hipMalloc(&p, bytes));
        return DFPR_OK;
    }
};

// Consecutive arrays of one allocation: sizes first (base NULL), then places.
struct Carve {
    char *base = nullptr;
    size_t at = 0;
    template <class T>
    void operator()(T *&p, uint64_t len)
    {
        if (base) p = reinterpret_cast<T *>(base + at);
        at += (size_t)((len * sizeof(T) + 255) / 256 * 256);
    }
};

// Stable sort of key[0 .. len) by bits [shift, shift + bits), in `key` and
// `tmp` in turn (swapped so that `key` ends up with the result).
static int sort_keys(hipStream_t s, uint64_t *&key, uint64_t *&tmp, uint64_t len, int shift, int bits,
                     uint64_t *counts, uint64_t *sums)
{
    const int passes = (bits + 7) / 8;
    const uint64_t tiles = (len + kSortTile - 1) / kSortTile;
    for (int p = 0; p < passes; p++) {
        const int lo = bits * p / passes, w = bits * (p + 1) / passes - lo;
        k_sort_count<<<(unsigned)tiles, kBlock, 0, s>>>(key, len, shift + lo, w, tiles, counts);
        scan_u64(s, counts, tiles << w, sums);
        k_sort_scatter<<<(unsigned)tiles, kBlock, 0, s>>>(key, len, shift + lo, w, tiles, counts, tmp);
        std::swap(key, tmp);
    }
    DFPR_HIP(hipGetLastError());
    return DFPR_OK;
}

// Workgroups of a kernel that strides over the edges.
static inline unsigned edge_grid(uint64_t items) { return stride_blocks(items, kBlock); }

// Build the numbering and both CSRs of g from m input edges (host arrays), on
// g->stream, with scratch on the device or in host memory.  top[o] receives the
// first free slot of each index array.
static int build_graph(dfpr_graph *g, int64_t m, const int32_t *src, const int32_t *dst, bool host_scratch,
                       uint32_t top[2])
{
    const int32_t n = g->n;
    hipStream_t s = g->stream;
    int b = 1;
    while ((int64_t(1) << b) < n) b++;
    const uint64_t len = (uint64_t)m + (uint64_t)n;
    const uint64_t tiles = (len + kSortTile - 1) / kSortTile;
    const uint64_t scan_len = std::max<uint64_t>(tiles * kDigits, (uint64_t)n + 1);
    // updated with atomics: in arrays of the graph that are set after the build
    static_assert(sizeof(LoadInfo) <= 4096 * sizeof(double), "scratch_sum holds it");
    LoadInfo *const info = reinterpret_cast<LoadInfo *>(g->scratch_sum);
    uint32_t *const deg = g->stamp;
    Scratch mem;
    uint64_t *key = nullptr, *tmp = nullptr, *counts = nullptr, *sums = nullptr;
    uint64_t *start = nullptr, *vertex = nullptr;
    for (int pass = 0; pass < 2; pass++) {
        Carve c{(char *)mem.p, 0};
        c(key, len);
        c(tmp, len);
        c(counts, scan_len);
        c(sums, scan_u64_sums(scan_len));
        c(start, (uint64_t)n + 1);
        c(vertex, n);
        if (pass == 0) DFPR_CHECK_RC(mem.take(c.at, host_scratch));
    }
    // the input edges, in tmp until they are keys
    int32_t *const es = reinterpret_cast<int32_t *>(tmp), *const ed = es + m;
    DFPR_HIP(hipMemsetAsync(info, 0, sizeof(LoadInfo), s));
    if (m) {
        DFPR_HIP(hipMemcpyAsync(es, src, (size_t)m * 4, hipMemcpyDefault, s));
        DFPR_HIP(hipMemcpyAsync(ed, dst, (size_t)m * 4, hipMemcpyDefault, s));
    }
    DFPR_CHECK_RC(launch_fill_u32(g, deg, (uint64_t)n, 1));
    if (m) k_load_degrees<<<edge_grid((uint64_t)m), kBlock, 0, s>>>(n, m, es, ed, deg, info);
    k_load_max<<<std::min(grid_of(n), 1024u), kBlock, 0, s>>>(n, deg, info);
    LoadInfo got;
    DFPR_HIP(hipMemcpyAsync(&got, info, sizeof(got), hipMemcpyDeviceToHost, s));
    DFPR_HIP(hipStreamSynchronize(s));
    if (got.err) return set_error(DFPR_E_RANGE, "vertex id outside [0, n)");
    // numbering
    uint64_t *vkey = vertex, *vtmp = start;
    k_load_vertex_keys<<<grid_of(n), kBlock, 0, s>>>(n, deg, got.dmax, vkey);
    int dbits = 1;
    while ((uint64_t)got.dmax >> dbits) dbits++;
    DFPR_CHECK_RC(sort_keys(s, vkey, vtmp, (uint64_t)n, 32, dbits, counts, sums));
    k_load_maps<<<grid_of(n), kBlock, 0, s>>>(n, vkey, got.dmax, g->ext2int, g->int2ext, info);
    // distinct edges by source, then target: the out-rows
    k_load_edge_keys<<<edge_grid(len), kBlock, 0, s>>>(n, m, es, ed, g->ext2int, b, key);
    DFPR_CHECK_RC(sort_keys(s, key, tmp, len, 0, 2 * b, counts, sums));
    k_load_distinct<<<(unsigned)tiles, kBlock, 0, s>>>(key, len, counts, nullptr);
    DFPR_HIP(hipMemsetAsync(counts + tiles, 0, 8, s));
    scan_u64(s, counts, tiles + 1, sums);
    k_load_distinct<<<(unsigned)tiles, kBlock, 0, s>>>(key, len, counts, tmp);
    DFPR_HIP(hipGetLastError());
    uint64_t edges = 0;
    DFPR_HIP(hipMemcpyAsync(&edges, counts + tiles, 8, hipMemcpyDefault, s));
    DFPR_HIP(hipStreamSynchronize(s));
    std::swap(key, tmp);
    for (int o = 1; o >= 0; o--) {
        if (o == 0) {
            // in-rows: a stable sort of the distinct edges by target
            k_load_swap<<<edge_grid(edges), kBlock, 0, s>>>(edges, b, key, tmp);
            std::swap(key, tmp);
            DFPR_CHECK_RC(sort_keys(s, key, tmp, edges, b, b, counts, sums));
        }
        Csr &c = g->csr[o];
        k_load_starts<<<edge_grid(edges), kBlock, 0, s>>>(edges, b, n, key, start);
        k_load_caps<<<grid_of((int64_t)n + 1), kBlock, 0, s>>>(n, start, c.cnt, c.cap, counts, o, info);
        scan_u64(s, counts, (uint64_t)n + 1, sums);
        k_load_begs<<<grid_of(n), kBlock, 0, s>>>(n, counts, c.beg, o, info);
        DFPR_HIP(hipGetLastError());
        DFPR_HIP(hipMemcpyAsync(&got, info, sizeof(got), hipMemcpyDeviceToHost, s));
        DFPR_HIP(hipStreamSynchronize(s));
        c.slots = got.packed[o] + spill_reserve(got.packed[o]);
        if (c.slots > kMaxEdgeSlots) return set_error(DFPR_E_LIMIT, "graph needs more than 2^32-1 edge slots");
        c.max_cap = got.max_cap[o];
        top[o] = (uint32_t)got.packed[o];
        DFPR_HIP(hipMalloc(&c.idx, c.slots * 4));
        k_load_rows<<<edge_grid(edges), kBlock, 0, s>>>(edges, b, key, start, c.beg, c.idx);
        DFPR_HIP(hipGetLastError());
    }
    DFPR_HIP(hipStreamSynchronize(s));
    g->m = (int64_t)edges;
    for (int k = 0; k < kBins + 2; k++) g->cls[k] = got.cls[k];
    for (int k = 0; k < kHubSteps; k++) g->hub_share[k] = (double)got.hub[k] / (double)edges;
    return DFPR_OK;
}

__global__ void k_map_ids(int32_t n, const int32_t *ext2int, const int32_t *in, int32_t *out,
                          int64_t len)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= len) return;
    const int32_t x = in[i];
    out[i] = (x >= 0 && x < n) ? ext2int[x] : -1;
}

// out[v] = Rint[ext2int[v]]: caller order from internal order
__global__ void k_to_caller(int32_t n, const int32_t *ext2int, const double *Rint, double *out)
{
    const int32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v < n) out[v] = Rint[ext2int[v]];
}

// Rint[i] = in[int2ext[i]]: internal order from caller order
__global__ void k_from_caller(int32_t n, const int32_t *int2ext, const double *in, double *Rint)
{
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) Rint[i] = in[int2ext[i]];
}

// Four arrays of lengths l0..l3 mapped into consecutive ranges of `out`.
__global__ void k_map_ids4(int32_t n, const int32_t *ext2int, const int32_t *i0,
                           const int32_t *i1, const int32_t *i2, const int32_t *i3, int64_t l0,
                           int64_t l1, int64_t l2, int64_t l3, int32_t *out)
{
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= l0 + l1 + l2 + l3) return;
    const int64_t k = i;
    const int32_t *src = i0;
    if (i >= l0) { i -= l0; src = i1;
        if (i >= l1) { i -= l1; src = i2;
            if (i >= l2) { i -= l2; src = i3; } } }
    const int32_t x = src[i];
    out[k] = (x >= 0 && x < n) ? ext2int[x] : -1;
}

int map_ids4(dfpr_graph *g, const int32_t *const in[4], const int64_t len[4], int32_t *out)
{
    const int64_t tot = len[0] + len[1] + len[2] + len[3];
    if (tot <= 0) return DFPR_OK;
    k_map_ids4<<<grid_of(tot), kBlock, 0, g->stream>>>(g->n, g->ext2int, in[0], in[1], in[2],
                                                       in[3], len[0], len[1], len[2], len[3], out);
    DFPR_HIP(hipGetLastError());
    return DFPR_OK;
}

// Ids outside [0, n) become -1, which every later check rejects.  `in` may
// equal `out`.
int map_ids(dfpr_graph *g, const int32_t *in, int32_t *out, int64_t len)
{
    if (len <= 0) return DFPR_OK;
    k_map_ids<<<grid_of(len), kBlock, 0, g->stream>>>(g->n, g->ext2int, in, out, len);
    DFPR_HIP(hipGetLastError());
    return DFPR_OK;
}

constexpr int32_t kFewFlags = 65536;

// out[v] = 1 if the stamp of v lies in [lo, hi] (caller order)
__global__ void k_flags(int32_t n, const int32_t *ext2int, const uint32_t *stamp, uint32_t lo,
                        uint32_t hi, uint8_t *out)
{
    const int32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    const uint32_t x = stamp[ext2int[v]];
    out[v] = x >= lo && x <= hi ? 1 : 0;
}

// Few flags go straight to the pinned block behind the mirrors; the copy that it
// saves costs more there (10^4 vertices: dfpr_get_affected 28 -> 14 us, at 65536
// 26 -> 17 us).
int flags_to_caller(const dfpr_graph *g, const uint32_t *stamp, uint32_t lo, uint32_t hi, uint8_t *out)
{
    const int32_t n = g->n;
    uint8_t *const few = reinterpret_cast<uint8_t *>(g->ctl_host + 2);
    uint8_t *dev = n <= kFewFlags ? few : reinterpret_cast<uint8_t *>(g->Rx);
    k_flags<<<grid_of(n), kBlock, 0, g->stream>>>(n, g->ext2int, stamp, lo, hi, dev);
    DFPR_HIP(hipGetLastError());
    if (dev != few) DFPR_HIP(hipMemcpyAsync(out, dev, (size_t)n, hipMemcpyDeviceToHost, g->stream));
    DFPR_HIP(hipStreamSynchronize(g->stream));
    if (dev == few) std::memcpy(out, few, (size_t)n);
    return DFPR_OK;
}

int ranks_to_caller(const dfpr_graph *g, const double *Rint, double *out, int out_dev)
{
    const int32_t n = g->n;
    k_to_caller<<<grid_of(n), kBlock, 0, g->stream>>>(n, g->ext2int, Rint, out_dev ? out : g->Rx);
    DFPR_HIP(hipGetLastError());
    if (!out_dev)
        DFPR_HIP(hipMemcpyAsync(out, g->Rx, (size_t)n * 8, hipMemcpyDeviceToHost, g->stream));
    return DFPR_OK;
}

int ranks_from_caller(const dfpr_graph *g, const double *in, int in_dev, double *Rint)
{
    const int32_t n = g->n;
    if (!in_dev) {
        DFPR_HIP(hipMemcpyAsync(g->Rx, in, (size_t)n * 8, hipMemcpyHostToDevice, g->stream));
        in = g->Rx;
    }
    k_from_caller<<<grid_of(n), kBlock, 0, g->stream>>>(n, g->int2ext, in, Rint);
    DFPR_HIP(hipGetLastError());
    return DFPR_OK;
}

}  // namespace dfpr

using namespace dfpr;

extern "C" {

const char *dfpr_last_error(void) { return g_last_error.c_str(); }

void dfpr_params_default(dfpr_params *p)
{
    if (!p) return;
    p->alpha = 0.85;
    p->tol = 1e-10;
    p->frontier_tol = 1e-10 / 1e5;
    p->max_iters = 500;
    p->precision = DFPR_FP64;
    p->mode = DFPR_SYNC;
    p->loop = DFPR_LOOP_LAUNCHES;
}

void dfpr_free_graph(dfpr_graph *g)
{
    if (!g) return;
    if (g->stream) (void)hipStreamSynchronize(g->stream);
    (void)hipFree(g->csr[0].idx);
    (void)hipFree(g->csr[1].idx);
    (void)hipFree(g->mstamp);
    (void)hipFree(g->mxstamp);
    (void)hipFree(g->bfs_q);
    (void)hipFree(g->arena);
    if (g->ctl_host) (void)hipHostFree(g->ctl_host);
    if (g->ap.batch_host) (void)hipHostFree(g->ap.batch_host);
    for (int o = 0; o < 2; o++) {
        for (int k = 0; k < 2; k++) (void)hipFree(g->ap.keys[o][k]);
        (void)hipFree(g->ap.tiny_list[o]);
        (void)hipFree(g->ap.small_list[o]);
        (void)hipFree(g->ap.big_list[o]);
        (void)hipFree(g->ap.ovf_list[o]);
        (void)hipFree(g->ap.ovf_need[o]);
    }
    (void)hipFree(g->ap.part);
    (void)hipFree(g->ap.slab);
    (void)hipFree(g->ap.batch_dev);
    for (hipEvent_t e : {g->ev0, g->ev1, g->ev_mid, g->ev_a0, g->ev_a1})
        if (e) (void)hipEventDestroy(e);
    for (hipEvent_t e : g->evk)
        if (e) (void)hipEventDestroy(e);
    for (hipEvent_t e : g->evc)
        if (e) (void)hipEventDestroy(e);
    if (g->own_stream) (void)hipStreamDestroy(g->own_stream);
    delete g;
}

int dfpr_load_graph(int32_t n, int64_t m, const int32_t *src, const int32_t *dst,
                    dfpr_graph **out)
{
    if (!out) return set_error(DFPR_E_ARG, "out is NULL");
    *out = nullptr;
    if (n <= 0 || m < 0 || (m > 0 && (!src || !dst)))
        return set_error(DFPR_E_ARG, "need n >= 1, m >= 0 and non-NULL edge arrays");
    // every vertex has its self-loop
    const uint64_t least = (uint64_t)n * row_capacity(1);
    if (least + spill_reserve(least) > kMaxEdgeSlots) {
        DFPR_CHECK_RC(check_ids_host(n, m, src, dst));
        return set_error(DFPR_E_LIMIT, "graph needs more than 2^32-1 edge slots");
    }
    dfpr_graph *g = new (std::nothrow) dfpr_graph();
    if (!g) return set_error(DFPR_E_NOMEM, "out of host memory");
    g->n = n;
    uint32_t top[2] = {0, 0};
    int rc = DFPR_OK;
    {
        hipError_t e = hipGetDevice(&g->device);
        if (e == hipSuccess) e = hipStreamCreateWithFlags(&g->own_stream, hipStreamNonBlocking);
        // two mirrors: the chunk in flight in each slot of the iteration loop;
        // behind them the flags of a small graph
        if (e == hipSuccess)
            e = hipHostMalloc((void **)&g->ctl_host, 2 * sizeof(Ctl) + kFewFlags, hipHostMallocCoherent);
        if (e == hipSuccess) std::memset(g->ctl_host, 0, 2 * sizeof(Ctl));
        if (e == hipSuccess) e = hipEventCreate(&g->ev0);
        if (e == hipSuccess) e = hipEventCreate(&g->ev1);
        // phase marks, read after the call's stream synchronisation
        for (hipEvent_t *ev : {&g->ev_mid, &g->ev_a0, &g->ev_a1})
            if (e == hipSuccess) e = hipEventCreateWithFlags(ev, hipEventDisableSystemFence);
        // waited on before the host reads a chunk's mirror: keep the fence
        for (hipEvent_t &ev : g->evc)
            if (e == hipSuccess) e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
        int cus = 0;
        if (e == hipSuccess)
            e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, g->device);
        if (e != hipSuccess) rc = hip_fail(e, "set-up of the graph");
        g->stream = g->own_stream;
        if (cus > 0) {
            g->grid = std::min(kMaxGrid, cus * kGridPerCU);
            g->grid_wide = std::min(kMaxGrid, cus * kWideGridPerCU);
            g->grid_wide_df = std::min(kMaxGrid, cus * kWideDfGridPerCU);
        }
        g->cus = std::max(1, std::min(256, cus));
    }
    // the arrays of fixed size, in one allocation
    for (int pass = 0; pass < 2 && !rc; pass++) {
        Carve c{(char *)g->arena, 0};
        c(g->ctl, 1);
        // the fold slots start cleared (every fold clears them again), and so
        // do the resident loop's words
        const size_t zero0 = c.at;
        c(g->it.dr_part, kFoldSlots);
        c(g->it.rmax_part, kFoldSlots);
        c(g->it.cnt_part, (uint64_t)kFoldSlots * kCounters);
        c(g->it.res, kResBytes / 8);
        const size_t zero1 = c.at;
        c(g->scratch_sum, 4096);
        for (int b = 0; b < 2; b++) {
            c(g->R[b], n);
            c(g->C[b], n);
            c(g->C32[b], n);
            c(g->csr[b].beg, n);
            c(g->csr[b].cnt, n);
            c(g->csr[b].cap, n);
        }
        c(g->stamp, n);
        c(g->xstamp, n);
        c(g->bins, (uint64_t)kBins * n);
        c(g->Rx, n);
        c(g->ext2int, n);
        c(g->int2ext, n);
        hipError_t e = hipSuccess;
        if (pass == 0) e = hipMalloc(&g->arena, c.at);
        else e = hipMemsetAsync((char *)g->arena + zero0, 0, zero1 - zero0, g->stream);
        if (e != hipSuccess) rc = hip_fail(e, "hipMalloc");
    }
    if (!rc) {
        rc = build_graph(g, m, src, dst, false, top);
        if (rc == DFPR_E_NOMEM) {
            // the graph may still fit without the scratch
            for (Csr &c : g->csr) {
                (void)hipFree(c.idx);
                c.idx = nullptr;
            }
            rc = build_graph(g, m, src, dst, true, top);
        }
    }
    if (!rc) {
        Ctl c0;
        std::memset(&c0, 0, sizeof(c0));
        for (int o = 0; o < 2; o++) {
            c0.top[o] = top[o];
            c0.max_cap[o] = g->csr[o].max_cap;
        }
        for (int k = 0; k < kBins + 2; k++) c0.cls[k] = g->cls[k];
        hipError_t e = hipMemcpyAsync(g->ctl, &c0, sizeof(Ctl), hipMemcpyHostToDevice, g->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(g->stream);
        if (e != hipSuccess) rc = hip_fail(e, "hipMemcpy");
        g->long_row = g->m > kResEdges ? 0xFFFFFFFFu : kLongRow;
        g->sparse_limit = (uint32_t)std::max<int64_t>(4096, n / 64);
    }
    if (!rc) rc = launch_fill_u32(g, g->stamp, (uint64_t)n, 0);
    if (!rc) rc = launch_fill_u32(g, g->xstamp, (uint64_t)n, 0);
    if (!rc) rc = dfpr_set_ranks(g, nullptr, 0);   // uniform 1/n
    if (!rc) {
        hipError_t e = hipStreamSynchronize(g->stream);
        if (e != hipSuccess) rc = hip_fail(e, "hipStreamSynchronize");
    }
    if (rc) {
        dfpr_free_graph(g);
        // a bad id is the error to report, and which one
        DFPR_CHECK_RC(check_ids_host(n, m, src, dst));
        return rc;
    }
    *out = g;
    return DFPR_OK;
}

int dfpr_set_stream(dfpr_graph *g, void *hip_stream)
{
    if (!g) return set_error(DFPR_E_ARG, "graph is NULL");
    DFPR_HIP(hipStreamSynchronize(g->stream));
    g->stream = hip_stream ? (hipStream_t)hip_stream : g->own_stream;
    return DFPR_OK;
}

int dfpr_graph_info(const dfpr_graph *g, int32_t *n, int64_t *m)
{
    if (!g) return set_error(DFPR_E_ARG, "graph is NULL");
    if (n) *n = g->n;
    if (m) *m = g->m;
    return DFPR_OK;
}

int dfpr_export_csr(const dfpr_graph *g, int out_orientation, int64_t *offsets, int32_t *idx)
{
    if (!g || !offsets || !idx) return set_error(DFPR_E_ARG, "NULL argument");
    const Csr &c = g->csr[out_orientation ? 1 : 0];
    int32_t n = g->n;
    std::vector<uint32_t> beg(n), cnt(n);
    std::vector<int32_t> slots(c.slots), ext2int(n), int2ext(n);
    DFPR_HIP(hipStreamSynchronize(g->stream));
    DFPR_HIP(hipMemcpy(ext2int.data(), g->ext2int, (size_t)n * 4, hipMemcpyDeviceToHost));
    DFPR_HIP(hipMemcpy(int2ext.data(), g->int2ext, (size_t)n * 4, hipMemcpyDeviceToHost));
    DFPR_HIP(hipMemcpy(beg.data(), c.beg, (size_t)n * 4, hipMemcpyDeviceToHost));
    DFPR_HIP(hipMemcpy(cnt.data(), c.cnt, (size_t)n * 4, hipMemcpyDeviceToHost));
    DFPR_HIP(hipMemcpy(slots.data(), c.idx, c.slots * 4, hipMemcpyDeviceToHost));
    // rows and entries in the caller's numbering, entries ascending
    int64_t pos = 0;
    for (int32_t v = 0; v < n; v++) {
        const int32_t r = ext2int[v];
        offsets[v] = pos;
        if (pos + cnt[r] > g->m)
            return set_error(DFPR_E_DEVICE, "device CSR holds more entries than m");
        if ((uint64_t)beg[r] + cnt[r] > (uint64_t)c.slots)
            return set_error(DFPR_E_DEVICE, "device CSR row runs past its slots");
        for (uint32_t k = 0; k < cnt[r]; k++) idx[pos + k] = int2ext[slots[beg[r] + k]];
        std::sort(idx + pos, idx + pos + cnt[r]);
        pos += cnt[r];
    }
    offsets[n] = pos;
    if (pos != g->m) return set_error(DFPR_E_DEVICE, "device CSR entry count differs from m");
    return DFPR_OK;
}

int dfpr_get_ranks(const dfpr_graph *g, double *ranks, int on_device)
{
    if (!g || !ranks) return set_error(DFPR_E_ARG, "NULL argument");
    const int rc = ranks_to_caller(g, g->R[g->cur], ranks, on_device);
    if (rc) return rc;
    DFPR_HIP(hipStreamSynchronize(g->stream));
    return DFPR_OK;
}

}  // extern "C"
