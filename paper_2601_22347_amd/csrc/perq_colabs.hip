// a_i = (1/M) sum_k |x[k,i]|  -- the sort key of Algorithm 1 -- as two deterministic passes; the
// same two passes with max in place of + give max_k |x[k,i]|, the statistic of the "absmax" and
// ZigZag permutations of the ablation (Appendix C).
//
// Pass 1: the M rows are cut into S slices; workgroup (column tile, slice) adds |x| over its rows:
// 32 lanes own 8 adjacent columns each (one 16-byte bf16 load per row), the eight groups of 32 take
// every eighth row, and their sums meet in LDS (in double).  It writes one partial sum per column
// and slice, in double.  Pass 2 adds a column's S partials in a fixed order and divides by M; a single
// slice (up to 128 rows, or d > 131072) writes the means itself, and up to 48 slices the last workgroup of a column
// tile may do it, in the same launch.  The only atomics count arrivals: the result is independent of scheduling.
// Rounding: fp32 is used inside a run of at most max_run(M, d) rows of one lane only, so a run's sum is off
// by less than max_run(M, d) - 1 roundings of non-negative terms, and the mean is rounded once more: the
// relative error of a_i is below (max_run(M, d) + 1) * 2^-24.
//   Bound by reading x, small inputs by the launch.  Eight row groups a workgroup instead of one
// (2048 columns each) make the partials a quarter as large (a quarter of the input at M <= 1024 before).
// Launches back to back: M = 16, d = 4096 4.1 -> 2.5 us, M = d = 32768 369 -> 319.
#include "perq.h"
#include "perq_launch.h"
#include "perq_schedule.h"

#include <mutex>
#include <type_traits>

namespace perq {
namespace {

constexpr int kColsPerLane = 8;
constexpr int kThreads = 256;
constexpr int kGroups = 8;                                    // row groups of a workgroup
constexpr int kTileCols = kColsPerLane * kThreads / kGroups;  // 256
static_assert(kTileCols == kThreads, "one lane per column adds the groups");

// Up to here a second launch costs more than the rows.  Their loads are all requested together; more rows take
// the loop, also where x is so wide that they are one slice (M = 4096, d = 200000: 261 against 299 us).
constexpr int kOneSlice = 128;
// Inputs past the last-level cache are read with streaming loads (M = 32768, d = 4096, three inputs in turn
// 49.8 -> 44.8 us; M = d = 32768 352 -> 319); smaller ones may be in it already and should stay (M = 4096, d = 28672
// again and again: 36.1 against 38.8).
constexpr int64_t kStreamBytes = (int64_t)256 << 20;

constexpr int kMostBlocks = 1024;                             // workgroups of a first pass of several slices

// One launch for both passes: whichever workgroup of a column tile is the last to leave its partials adds all of
// them up, in the second pass's order.  Arrivals are counted per tile and stream (a set belongs to one stream, whose
// launches do not overlap, and the last arrival puts the count back to zero); a stream without a set and a launch
// that is being captured take two launches.  Partials and counts go past the L2 of their XCD.
//   Up to 32 slices, which a lane of the last workgroup reads all at once, and of inputs that are read in about the
// time that the host takes for a second launch (2 - 3 us) up to 48, or 40 of few columns.  Two launches / one, us with the
// host ahead of the device (back to back):
//   M = 129, d = 8192 (3 slices) 5.0 / 4.1 (6.8 / 4.3), M = 2048, d = 4096 (32) 7.8 / 6.9 (7.6 / 6.6), M = 4096, d = 8192 (16)
//   16.0 / 15.3; M = 2500, d = 768 (40) 5.5 / 5.6 (6.2 / 5.4), M = 2900, d = 1568 (46) 6.1 / 6.2 (7.0 / 5.9), M = 2500,
//   d = 2304 (40) 6.7 / 6.6 (7.3 / 6.4), M = 2900, d = 2816 (46) 8.0 / 8.0 (7.8 / 7.8), M = 2500, d = 3072 (40) 7.6 / 7.4;
//   past these M = 3072, d = 768 (48) 5.6 / 6.0 (6.2 / 5.7), M = 4096, d = 1024 (64) 6.0 / 6.7 (7.1 / 6.4), M = 4096, d = 2304
//   (56) 8.7 / 9.4 (8.4 / 9.1), M = 3400, d = 2816 (46) 8.4 / 9.2 (8.1 / 8.8), M = 4096, d = 3584 (36) 10.5 / 10.8.
constexpr int kWays = 16;
constexpr int kOneLaunchTiles = 128;
int one_launch_slices(int64_t M, int32_t d) { return M * (int64_t)d > ((int64_t)1 << 23) ? 2 * kWays : d >= 1536 ? 48 : 40; }
__device__ uint32_t arrivals[schedule::kSets][kOneLaunchTiles][32];        // a count per cache line
// (apart from the row schedule's sets: a stream that only computes statistics takes none of those)
StreamSets arrival_sets;

struct ColabsPlan {
    int col_tiles;
    int slices;
    int rows_per_slice;
};

// Rows that one fp32 sum may take in (the bound that perq.h states).
int64_t max_run(int64_t M, int32_t d) {
    const int64_t tiles = ((int64_t)d + 2047) / 2048, slices = tiles < 512 ? 512 / tiles : 1;
    const int64_t run = (M + slices - 1) / slices;
    return run < 8 ? 8 : run;
}

ColabsPlan colabs_plan(int64_t M, int32_t d) {
    ColabsPlan pl;
    pl.col_tiles = (int)(((int64_t)d + kTileCols - 1) / kTileCols);
    const int64_t run = max_run(M, d);
    // 2 workgroups per CU (4: M = 32768, d = 4096 44.2 -> 46.3 us), or 4 where the slices of 2 would be longer than
    // `run` allows (M = 40000, d = 28672: 4 slices 334 us, 9 330; 5, which would do and leave the CUs uneven
    // shares, 384)
    int64_t want = kMostBlocks / 2 / pl.col_tiles;
    if (want == 0 || M > want * kGroups * run) want = kMostBlocks / pl.col_tiles;
    const int64_t most = (M + run - 1) / run / 2;       // no more bytes of partials than a float per run
    if (want > most) want = most;
    if (want < 1) want = 1;
    int64_t rps = (M + want - 1) / want;
    if (rps < 8 * kGroups) rps = 8 * kGroups;           // at least a few rows per lane
    if (M <= kOneSlice) rps = kOneSlice;
    pl.rows_per_slice = (int)rps;
    pl.slices = (int)((M + rps - 1) / rps);
    return pl;
}

// FEW: at most kOneSlice rows, workgroup = column tile.  STREAM: streaming loads.  part == nullptr: the only slice,
// which writes the result (m_rows: rows to divide by).
//   blocks: 0, or their number where rows are no multiple of 128 bytes.  Neighbours along a row then share a cache
// line.  Workgroups go round-robin to the 8 XCDs, each with an L2 of its own, so XCD x gets a contiguous share of
// the (slice, tile) pairs, tiles along the row first, and reads such a line once: M = 4045, d = 11096 19.4 -> 16.9 us,
// M = 40000, d = 8200 120 -> 107.  Rows of whole lines have nothing to share (M = 40000, d = 4096 52.8 -> 51.7, but
// d = 14336 168 -> 177).
template <bool MAXSTAT, bool FEW, bool STREAM>
__global__ void __launch_bounds__(kThreads)
colabs_partial_kernel(const uint16_t* __restrict__ x, int64_t M, int32_t d, int64_t ldx, int rows_per_slice,
                      uint32_t tiles, uint32_t blocks, double* __restrict__ part, float* __restrict__ out, float m_rows,
                      int slices, int set) {
    typedef typename std::conditional<MAXSTAT, float, double>::type sum_t;
    __shared__ sum_t red[kGroups][kTileCols];
    const int cl = threadIdx.x % (kThreads / kGroups), group = threadIdx.x / (kThreads / kGroups);
    uint32_t tile = blockIdx.x, slice = 0;
    if constexpr (!FEW) {
        const uint32_t xcd = blockIdx.x & 7u, share = blocks >> 3, more = blocks & 7u;
        const uint32_t pair = blocks == 0 ? blockIdx.x : xcd * share + (xcd < more ? xcd : more) + (blockIdx.x >> 3);
        slice = pair / tiles;
        tile = pair - slice * tiles;
    }
    const int64_t col0 = (int64_t)tile * kTileCols, col = col0 + cl * kColsPerLane;
    const int64_t r0 = (int64_t)slice * rows_per_slice;
    const int64_t r1 = r0 + rows_per_slice < M ? r0 + rows_per_slice : M;
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    auto add = [&](const uint4& w) {
        const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float lo = fabsf(bf16lo_to_f32(ww[q])), hi = fabsf(bf16hi_to_f32(ww[q]));
            acc[2 * q] = MAXSTAT ? fmaxf(acc[2 * q], lo) : acc[2 * q] + lo;
            acc[2 * q + 1] = MAXSTAT ? fmaxf(acc[2 * q + 1], hi) : acc[2 * q + 1] + hi;
        }
    };
    sum_t total[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (col < d) {
        const uint16_t* px = x + col;
        if constexpr (FEW) {
            // eight rows at a time, all requested together, their sums added up in double
            for (int64_t base = r0 + group; base < r1; base += 8 * kGroups) {
                uint4 w[8];
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    w[i] = base + i * kGroups < r1 ? *reinterpret_cast<const uint4*>(px + (base + i * kGroups) * ldx) : make_uint4(0, 0, 0, 0);
#pragma unroll
                for (int i = 0; i < 8; ++i) add(w[i]);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    total[e] = MAXSTAT ? (sum_t)acc[e] : total[e] + acc[e];
                    if constexpr (!MAXSTAT) acc[e] = 0.0f;
                }
            }
        } else {
#pragma unroll 8
            for (int64_t r = r0 + group; r < r1; r += kGroups)
                add(STREAM ? load_stream16(px + r * ldx) : *reinterpret_cast<const uint4*>(px + r * ldx));
#pragma unroll
            for (int e = 0; e < 8; ++e) total[e] = acc[e];
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) red[group][cl * kColsPerLane + e] = total[e];
    __syncthreads();
    const int64_t c = col0 + threadIdx.x;
    if (c < d) {
        double t = red[0][threadIdx.x];
#pragma unroll
        for (int g = 1; g < kGroups; ++g) {
            const double v = red[g][threadIdx.x];
            t = MAXSTAT ? (v > t ? v : t) : t + v;
        }
        if (FEW || part == nullptr) out[c] = MAXSTAT ? (float)t : (float)(t / (double)m_rows);
        else if (set < 0) part[(int64_t)slice * d + c] = t;
        else __hip_atomic_store(reinterpret_cast<unsigned long long*>(part) + ((int64_t)slice * d + c), (unsigned long long)__double_as_longlong(t),
                                __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if constexpr (!FEW) {
        if (set < 0) return;                                   // (the same for the whole launch)
        __shared__ uint32_t before;
        // Every partial is where the whole device sees it before the count says so: a store of device scope is written
        // through to there and counted out when it has arrived.  (A release fence would write the whole L2 of the XCD
        // back besides, once per wave: M = 4096, d = 8192 47 us.)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        uint32_t* const count = &arrivals[set][tile][0];
        if (threadIdx.x == 0) before = __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (before != (uint32_t)slices - 1u) return;
        // (read with device scope too: past the L2 of this XCD)
        if (threadIdx.x == 0) __hip_atomic_store(count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (c < d) {
            // the order of colabs_finish_kernel: 16 sums of every sixteenth slice, added up one after the other
            double way[kWays] = {};
            for (int k0 = 0; k0 < slices; k0 += 2 * kWays) {
                double v[2 * kWays];
#pragma unroll
                for (int k = 0; k < 2 * kWays; ++k) {
                    v[k] = 0.0;
                    if (k0 + k < slices)
                        v[k] = __longlong_as_double((long long)__hip_atomic_load(
                            reinterpret_cast<const unsigned long long*>(part) + ((int64_t)(k0 + k) * d + c), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                }
#pragma unroll
                for (int k = 0; k < 2 * kWays; ++k) way[k % kWays] = MAXSTAT ? (v[k] > way[k % kWays] ? v[k] : way[k % kWays]) : way[k % kWays] + v[k];
            }
            double t = way[0];
#pragma unroll
            for (int w = 1; w < kWays; ++w) t = MAXSTAT ? (way[w] > t ? way[w] : t) : t + way[w];
            out[c] = MAXSTAT ? (float)t : (float)(t / (double)m_rows);
        }
    }
}

// Pass 2: 16 columns per workgroup, 16 lanes per column.  Lane j of a column adds slices
// j, j+16, ...; the 16 sub-sums are then added in lane order.  Fixed order throughout.  Bound by latency: with 32
// columns M = 2048, d = 4096 5.9 us instead of 5.4, M = 4096, d = 8192 14.0 instead of 13.9.
constexpr int kFinishCols = 16;
constexpr int kFinishWays = kThreads / kFinishCols;
static_assert(kFinishWays == kWays, "both ways to the result add in one order");

template <bool MAXSTAT>
__global__ void __launch_bounds__(kThreads)
colabs_finish_kernel(const double* __restrict__ part, int slices, int32_t d, float m_rows,
                     float* __restrict__ out) {
    __shared__ double red[kFinishWays][kFinishCols];
    const int cl = threadIdx.x % kFinishCols, way = threadIdx.x / kFinishCols;
    const int col = blockIdx.x * kFinishCols + cl;
    double s = 0.0;
    if (col < d) {
#pragma unroll 8
        for (int k = way; k < slices; k += kFinishWays) {
            const double v = part[(int64_t)k * d + col];
            s = MAXSTAT ? (v > s ? v : s) : s + v;
        }
    }
    red[way][cl] = s;
    __syncthreads();
    if (way == 0 && col < d) {
        double t = red[0][cl];
#pragma unroll
        for (int j = 1; j < kFinishWays; ++j) t = MAXSTAT ? (red[j][cl] > t ? red[j][cl] : t) : t + red[j][cl];
        out[col] = MAXSTAT ? (float)t : (float)(t / (double)m_rows);
    }
}

__global__ void clear_arrivals_kernel(int set) { arrivals[set][threadIdx.x][0] = 0u; }

}  // namespace

// (of no other stream: a statistic may be running there, and a count that starts over never becomes full)
hipError_t clear_arrivals(hipStream_t stream) {
    const int set = arrival_sets.of(stream, false);
    if (set < 0) return hipSuccess;
    hipLaunchKernelGGL(clear_arrivals_kernel, dim3(1), dim3(kOneLaunchTiles), 0, stream, set);
    return hipGetLastError();
}

}  // namespace perq

extern "C" size_t perq_colabs_mean_workspace_bytes(int64_t M, int32_t d) {
    if (M <= 0 || d <= 0) return 0;
    const perq::ColabsPlan pl = perq::colabs_plan(M, d);
    // (a single slice writes the result itself; callers provide a row of floats all the same)
    return pl.slices == 1 ? (size_t)d * sizeof(float) : (size_t)pl.slices * (size_t)d * sizeof(double);
}

// Partial sums of perq_colabs_mean_static, for callers that cannot hand over device memory of their
// own.  In host code this name only stands for the array: its device address is looked up once per
// device (scratch_of_current_device) and that pointer is what kernels are given.
// Several slices never have more columns in all than kMostBlocks tiles.
static __device__ __align__(256) double scratch[perq::kMostBlocks * perq::kTileCols];
constexpr int32_t kStaticMostColumns = 1 << 20;

namespace perq {
namespace {
perq_status_t colabs_check(const uint16_t* x_bf16, int64_t M, int32_t d, int64_t ldx, const float* out) {
    if (x_bf16 == nullptr || out == nullptr) return PERQ_ERR_INVALID_ARG;
    if (M <= 0 || d <= 0 || ldx < d) return PERQ_ERR_INVALID_ARG;
    if (d % 8 != 0 || ldx % 8 != 0 || (reinterpret_cast<uintptr_t>(x_bf16) & 15u) != 0)
        return PERQ_ERR_UNSUPPORTED;
    return PERQ_OK;
}

template <bool MAXSTAT>
perq_status_t colabs_launch(const uint16_t* x_bf16, int64_t M, int32_t d, int64_t ldx, float* out, double* part,
                            void* hip_stream) {
    const ColabsPlan pl = colabs_plan(M, d);
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    auto kern = M <= kOneSlice                          ? colabs_partial_kernel<MAXSTAT, true, false>
                : M * (int64_t)d * 2 >= kStreamBytes ? colabs_partial_kernel<MAXSTAT, false, true>
                                                     : colabs_partial_kernel<MAXSTAT, false, false>;
    const uint32_t tiles = (uint32_t)pl.col_tiles, blocks = tiles * (uint32_t)pl.slices;
    const bool together = pl.slices > 1 && pl.slices <= one_launch_slices(M, d) && pl.col_tiles <= kOneLaunchTiles;
    const int set = together ? arrival_sets.of(stream) : -1;
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(kThreads), 0, stream, x_bf16, M, d, ldx, pl.rows_per_slice, tiles,
                       ldx % 64 != 0 ? blocks : 0u, pl.slices == 1 ? nullptr : part, out, (float)M, pl.slices, set);
    if (hipGetLastError() != hipSuccess) return PERQ_ERR_LAUNCH;
    if (pl.slices == 1 || set >= 0) return PERQ_OK;
    hipLaunchKernelGGL(colabs_finish_kernel<MAXSTAT>, dim3((d + kFinishCols - 1) / kFinishCols), dim3(kThreads), 0,
                       stream, part, pl.slices, d, (float)M, out);
    if (hipGetLastError() != hipSuccess) return PERQ_ERR_LAUNCH;
    return PERQ_OK;
}

template <bool MAXSTAT>
perq_status_t colabs_stat(const uint16_t* x_bf16, int64_t M, int32_t d, int64_t ldx, float* out, void* workspace,
                          size_t workspace_bytes, void* hip_stream) {
    const perq_status_t st = colabs_check(x_bf16, M, d, ldx, out);
    if (st != PERQ_OK) return st;
    const size_t need = perq_colabs_mean_workspace_bytes(M, d);
    if (workspace == nullptr || workspace_bytes < need) return PERQ_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(workspace) & 15u) != 0) return PERQ_ERR_INVALID_ARG;
    return colabs_launch<MAXSTAT>(x_bf16, M, d, ldx, out, static_cast<double*>(workspace), hip_stream);
}

// Device address of `scratch` on the current device: every device holds its own copy of the array
// at an address of its own, looked up at the first call with that device current.
perq_status_t scratch_of_current_device(double** out) {
    static std::mutex mu;
    static double* known[64] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return PERQ_ERR_LAUNCH;
    std::lock_guard<std::mutex> lock(mu);
    if (known[dev] == nullptr) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) {
            (void)hipGetLastError();
            return PERQ_ERR_LAUNCH;
        }
        known[dev] = static_cast<double*>(ptr);
    }
    *out = known[dev];
    return PERQ_OK;
}
}  // namespace
}  // namespace perq

extern "C" perq_status_t perq_colabs_mean(const uint16_t* x_bf16, int64_t M, int32_t d, int64_t ldx,
                                          float* out_mean, void* workspace, size_t workspace_bytes,
                                          void* hip_stream) {
    return perq::colabs_stat<false>(x_bf16, M, d, ldx, out_mean, workspace, workspace_bytes, hip_stream);
}

extern "C" perq_status_t perq_colabs_absmax(const uint16_t* x_bf16, int64_t M, int32_t d, int64_t ldx,
                                            float* out_max, void* workspace, size_t workspace_bytes,
                                            void* hip_stream) {
    return perq::colabs_stat<true>(x_bf16, M, d, ldx, out_max, workspace, workspace_bytes, hip_stream);
}

extern "C" perq_status_t perq_colabs_mean_static(const uint16_t* x_bf16, int64_t M, int32_t d, int64_t ldx,
                                                 float* out_mean, void* hip_stream) {
    const perq_status_t st = perq::colabs_check(x_bf16, M, d, ldx, out_mean);
    if (st != PERQ_OK) return st;
    if (d > kStaticMostColumns) return PERQ_ERR_UNSUPPORTED;
    double* part = nullptr;
    const perq_status_t sp = perq::scratch_of_current_device(&part);
    if (sp != PERQ_OK) return sp;
    return perq::colabs_launch<false>(x_bf16, M, d, ldx, out_mean, part, hip_stream);
}
