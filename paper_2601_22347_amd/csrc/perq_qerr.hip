// Per-token quantization error of the fused path's output (Section 3: the worst-case l2 error of a
// q-bit quantizer is sqrt(d) / (2^q - 2) times the row's largest magnitude, which is why suppressing
// outliers pays): from the pre-quantization values y (perq_permute_rotate_f32) and the codes and
// scales perq_permute_rotate_quant wrote for the same input,
//     out[t] = ( ||y_t - Q(y_t)||_2,  ||y_t||_2,  ||y_t||_inf )
// with Q(y) the value the codes stand for.  One workgroup per token; every thread adds its elements
// in index order and the 256 partial sums are added in a fixed tree, so the result does not depend on
// scheduling.  Sums are fp32.
//   Bound by reading y (4 bytes an element): a thread takes four elements at a time, one 16-byte load of
// y and two bytes of codes, and the sums of a wave meet in registers.  Against two elements a time, one
// byte of codes per load and a tree of eight barriers through LDS: T = 2048, d = 8192, INT4 13.1 -> 12.2 us,
// MXFP4 13.6 -> 12.3; T = 512, d = 14336 12.0 -> 4.8; T = 16, d = 4096 3.6 -> 2.3.
#include "perq.h"
#include "perq_device.h"
#include "perq_launch.h"

namespace perq {
namespace {

constexpr int kThreads = 256;

typedef float f32x4_a8 __attribute__((ext_vector_type(4), aligned(8)));       // (y is 8-byte aligned)
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// sum over the wave, a fixed tree
__device__ __forceinline__ float wave_sum(float v) {
    v += lane_xor<1>(v);
    v += lane_xor<2>(v);
    v += lane_xor<4>(v);
    v += lane_xor<8>(v);
    v += lane_xor<16>(v);
    v += lane_xor<32>(v);
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
    v = lane_max<1>(v);
    v = lane_max<2>(v);
    v = lane_max<4>(v);
    v = lane_max<8>(v);
    v = lane_max<16>(v);
    return lane_max<32>(v);
}

// four codes (element 0 in the low nibble of byte 0) without their scale
template <int FMT>
__device__ __forceinline__ void code_values(uint32_t w, float (&q)[4]) {
    if constexpr (FMT == PERQ_FMT_INT4_SYM_TOKEN) {
#pragma unroll
        for (int i = 0; i < 4; ++i) q[i] = (float)((int)(w << (28 - 4 * i)) >> 28);          // two's complement nibble
    } else if constexpr (FMT == PERQ_FMT_INT4_ASYM_TOKEN) {
#pragma unroll
        for (int i = 0; i < 4; ++i) q[i] = (float)((w >> (4 * i)) & 15u);
    } else {
        const f32x2_t lo = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w, 1.0f, 0), hi = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w, 1.0f, 1);
        q[0] = lo.x; q[1] = lo.y; q[2] = hi.x; q[3] = hi.y;
    }
}

template <int FMT>
__global__ void __launch_bounds__(kThreads)
quant_error_kernel(const float* __restrict__ y, int64_t T, int32_t d, const uint8_t* __restrict__ codes,
                   const void* __restrict__ scales, float* __restrict__ out) {
    __shared__ float red[3][kThreads / 64];
    const int64_t row = blockIdx.x;
    const float* yr = y + row * (int64_t)d;
    const uint8_t* cr = codes + row * (int64_t)(d >> 1);
    float step = 0.0f, zero = 0.0f;
    if constexpr (FMT == PERQ_FMT_INT4_SYM_TOKEN || FMT == PERQ_FMT_FP4_TOKEN) step = static_cast<const float*>(scales)[row];
    if constexpr (FMT == PERQ_FMT_INT4_ASYM_TOKEN) {
        step = static_cast<const float*>(scales)[2 * row];
        zero = static_cast<const float*>(scales)[2 * row + 1];
    }
    float err = 0.0f, nrm = 0.0f, amax = 0.0f;
#pragma unroll 4
    for (int k = threadIdx.x; k < (d >> 2); k += kThreads) {
        const f32x4_a8 v4 = *reinterpret_cast<const f32x4_a8*>(yr + 4 * k);
        uint16_t w;
        __builtin_memcpy(&w, cr + 2 * k, 2);                  // (codes need not be aligned)
        const float v[4] = {v4.x, v4.y, v4.z, v4.w};
        float q[4], s = step;
        code_values<FMT>(w, q);
        if constexpr (FMT == PERQ_FMT_MXFP4) {
            const uint32_t E = static_cast<const uint8_t*>(scales)[row * (int64_t)(d >> 5) + (k >> 3)];
            s = E == 0 ? 0x1p-127f : __uint_as_float(E << 23);         // 2^(E - 127)
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float e = v[i] - s * (FMT == PERQ_FMT_INT4_ASYM_TOKEN ? q[i] + zero : q[i]);
            err = __builtin_fmaf(e, e, err);
            nrm = __builtin_fmaf(v[i], v[i], nrm);
            amax = fmaxf(amax, fabsf(v[i]));
        }
    }
    err = wave_sum(err);
    nrm = wave_sum(nrm);
    amax = wave_max(amax);
    if ((threadIdx.x & 63) == 0) {
        const int w = threadIdx.x >> 6;
        red[0][w] = err;
        red[1][w] = nrm;
        red[2][w] = amax;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        out[3 * row] = sqrtf((red[0][0] + red[0][1]) + (red[0][2] + red[0][3]));
        out[3 * row + 1] = sqrtf((red[1][0] + red[1][1]) + (red[1][2] + red[1][3]));
        out[3 * row + 2] = fmaxf(fmaxf(red[2][0], red[2][1]), fmaxf(red[2][2], red[2][3]));
    }
}

}  // namespace
}  // namespace perq

extern "C" perq_status_t perq_quant_error(const float* y, int64_t T, int32_t d, const uint8_t* codes,
                                          const void* scales, perq_fmt_t fmt, float* out, void* hip_stream) {
    if (T < 0 || d <= 0 || d % 32 != 0) return PERQ_ERR_INVALID_ARG;
    if (fmt != PERQ_FMT_INT4_SYM_TOKEN && fmt != PERQ_FMT_MXFP4 && fmt != PERQ_FMT_INT4_ASYM_TOKEN &&
        fmt != PERQ_FMT_FP4_TOKEN && fmt != PERQ_FMT_FP4_TOKEN_AMAX7)
        return PERQ_ERR_INVALID_ARG;
    if (T == 0) return PERQ_OK;
    if (y == nullptr || codes == nullptr || scales == nullptr || out == nullptr) return PERQ_ERR_INVALID_ARG;
    if (T >= ((int64_t)1 << 31)) return PERQ_ERR_UNSUPPORTED;
    if ((reinterpret_cast<uintptr_t>(y) & 7u) != 0 || (reinterpret_cast<uintptr_t>(out) & 3u) != 0 ||
        (reinterpret_cast<uintptr_t>(scales) & (fmt == PERQ_FMT_MXFP4 ? 0u : 3u)) != 0)
        return PERQ_ERR_UNSUPPORTED;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const dim3 grid((unsigned)T), block(perq::kThreads);
    switch (fmt) {
        case PERQ_FMT_INT4_SYM_TOKEN:
            hipLaunchKernelGGL(perq::quant_error_kernel<PERQ_FMT_INT4_SYM_TOKEN>, grid, block, 0, stream, y, T, d, codes, scales, out);
            break;
        case PERQ_FMT_MXFP4:
            hipLaunchKernelGGL(perq::quant_error_kernel<PERQ_FMT_MXFP4>, grid, block, 0, stream, y, T, d, codes, scales, out);
            break;
        case PERQ_FMT_INT4_ASYM_TOKEN:
            hipLaunchKernelGGL(perq::quant_error_kernel<PERQ_FMT_INT4_ASYM_TOKEN>, grid, block, 0, stream, y, T, d, codes, scales, out);
            break;
        default:
            hipLaunchKernelGGL(perq::quant_error_kernel<PERQ_FMT_FP4_TOKEN>, grid, block, 0, stream, y, T, d, codes, scales, out);
            break;
    }
    return hipGetLastError() == hipSuccess ? PERQ_OK : PERQ_ERR_LAUNCH;
}
