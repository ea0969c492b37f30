// Host-side launch plumbing shared by the kernel translation units.
#pragma once
#include <hip/hip_runtime.h>

#include <map>
#include <mutex>
#include <thread>
#include <tuple>

#include "perq_device.h"

namespace perq {

struct LaunchInfo {
    int num_cus;
    int lds_per_cu;   // bytes
};

// Properties of the current device (queried once per process and device).
const LaunchInfo& launch_info();

// Number of workgroups of `kern` (threads per workgroup, dynamic LDS bytes) that one CU keeps
// resident; on first use per device also raises the kernel's dynamic-LDS limit to lds_bytes.
// Asked of the runtime once per kernel, device and configuration, then remembered.
hipError_t resident_blocks(const void* kern, int threads, uint32_t lds_bytes, int* per_cu);

// Sets of device counters that belong to streams: the first `schedule::kSets` streams of a device get a set each
// and keep it for the life of the process.  The per-thread default stream is a different stream in every host
// thread and is told apart by the thread.
class StreamSets {
public:
    // The set of `stream` on the current device, or -1: the stream is being captured into a graph (which can be replayed
    // on any stream, beside anything), every set is taken, or (assign false) it has not been given one.
    int of(hipStream_t stream, bool assign = true);

private:
    std::mutex mu_;
    std::map<std::tuple<int, hipStream_t, std::thread::id>, int> sets_;
    int taken_[64] = {};          // sets handed out so far, per device
};

// Puts the arrival counts of the column statistics of `stream` back to zero.
hipError_t clear_arrivals(hipStream_t stream);

// Kernel families behind perq_permute_rotate_quant / perq_permute_rotate_f32.
hipError_t launch_butterfly(const ApplyParams& p, int out_kind, hipStream_t stream);
bool mfma_supports(const ApplyParams& p);
// The kernel that takes a call with a power-of-two block (b > 4096 on the chunked widths aside), and the one that a
// caller who asks for the matrix cores gets.
enum class Route { butterfly, block, mfma };
Route route_of(const ApplyParams& p, int out_kind);
Route matrix_core_route(const ApplyParams& p, int out_kind);
hipError_t launch_mfma(const ApplyParams& p, int out_kind, hipStream_t stream);
// Ticket counters of the row schedule for launches on `stream` (perq_schedule.h: kQueues, 256 bytes apart, all zero), or
// nullptr: the launch takes a fixed split.  The block statistics have counters of their own.
uint32_t* row_counters(hipStream_t stream, bool statistics);
// The matrix-core kernel of half the tile, b <= 2048: launches of few rows to a CU and rows that do not fill the tiles
// of the other one.
bool block_supports(const ApplyParams& p);
hipError_t launch_block(const ApplyParams& p, int out_kind, hipStream_t stream);
// Block sizes 2^k' * 4t, 4t = 12, 28 or 76 (non-power-of-two rotation), one family of kernels per base.
bool npo2_supports(const ApplyParams& p);
hipError_t launch_npo2(const ApplyParams& p, int out_kind, hipStream_t stream);
hipError_t launch_npo2_28(const ApplyParams& p, int out_kind, hipStream_t stream);
hipError_t launch_npo2_12(const ApplyParams& p, int out_kind, hipStream_t stream);
hipError_t launch_npo2_76(const ApplyParams& p, int out_kind, hipStream_t stream);
// The same chunked kernel with H_32 as base: power-of-two b > 4096 on d = 8192, 16384.
bool chunked_pow2_supports(const ApplyParams& p);
hipError_t launch_npo2_32(const ApplyParams& p, int out_kind, hipStream_t stream);

}  // namespace perq
