// Consumers of the packed codes: out = A W^T for two operands in the layout the fused path writes,
// symmetric INT4 (one fp32 step per row) or MXFP4 (one e8m0 byte per 32 codes).
//
// Measured, T = 2048, N = d = 4096, INT4: 29.8 us; T = N = 2048, d = 8192, MXFP4: 23.9 us.  What bounds both is what the
// matrix unit draws: with random codes, registers only and nothing else running, it delivers 3.6 POP/s (int8) and 6.0
// PFLOP/s (fp4) on the whole chip, with zeros 4.7 and 9.4, and one workgroup alone runs its stages 1.4 times as fast
// as 256 do.  Past that, loads from L2: 32 KiB, a 128 x 128 stage of MXFP4, take a CU 0.31 us alone, its products 0.36.  LDS
// is not a bound since its reads have no bank conflicts (INT4 4.4 -> 2.3 M cycles, profiles/products_w4a4.txt).  Products
// of 16 x 16 (8 - 12 % more from the unit alone) gave nothing in INT4 and cost MXFP4 18 %: eight scale reads from LDS a stage
// instead of four.
//
// With P and the block rotation merged into the weights (Remark "Merging Permutations", Section 4:
// W~ = R~^T P^T W), the product of the two quantized operands stands for X W.
//
// Both formats run on the matrix cores, 32 codes (16 bytes, a "granule") per lane and operand:
//   INT4   v_mfma_i32_32x32x32_i8.  The nibbles of a packed byte become two signed bytes by masking:
//          w & 0xF0 is 16 times the high code, (w << 4) & 0xF0 is 16 times the low one, so a granule
//          is two A (or B) operands -- its even and its odd codes -- for three vector instructions a
//          dword.  The accumulated 256-fold sums stay below 64 * 256 * 32768 = 2^29 and are exact.
//   MXFP4  v_mfma_scale_f32_32x32x64_f8f6f4 takes a granule and its scale byte as they are: lane
//          (i, h), i = lane & 31, h = lane >> 5, supplies 32 codes of row i and the e8m0 byte of
//          exactly those 32.  The products are exact, the sums fp32.
// Which granules of a row meet in one product is free as long as both operands agree: a row is cut
// into stages of 8 granules (128 bytes, a cache line) and in step kc of a stage half-wave h takes
// granule 4 h + kc, so that the four scale bytes a lane needs are one dword, picked apart by the
// instruction's byte select.
// Accumulator j of lane (i, h) is row 8 (j >> 2) + 4 h + (j & 3), column i of the 32 x 32 tile.
#include "perq.h"
#include "perq_device.h"
#include "perq_launch.h"

#include <hip/hip_runtime.h>
#include <type_traits>

namespace perq {
namespace {

typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef int v8i_t __attribute__((ext_vector_type(8)));
typedef int v16i_t __attribute__((ext_vector_type(16)));
typedef float v16f_t __attribute__((ext_vector_type(16)));

constexpr uint32_t kStageBytes = 128;      // of one row's codes
constexpr uint32_t kHighNibbles = 0xF0F0F0F0u;

struct GemmParams {
    const uint8_t* a_codes;
    const void* a_scales;
    const uint8_t* w_codes;
    const void* w_scales;
    float* out;
    int64_t T, ldo;
    int32_t N, d;
    uint32_t tiles_t, tiles_n;
    int32_t stream_out;        // the tile kernels store their output with the streaming policy
};

__device__ __forceinline__ v4i_t high_codes(v4i_t w, int mask) { return w & mask; }
__device__ __forceinline__ v4i_t low_codes(v4i_t w, int mask) { return (w << 4) & mask; }

// 16 bytes per lane, global -> LDS (lane l to byte 16 l of `to`, the same in all lanes), as a buffer
// load: behind global_load_lds, a FLAT instruction that may touch LDS, the compiler waits for all of a
// wave's memory traffic at the next use of any load.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t buffer_of(const unsigned char* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(p), 0, bytes, 0x00020000);
}
__device__ __forceinline__ void load_to_lds16(rsrc_t from, uint32_t offset, uint32_t uniform_offset, unsigned char* to) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(from, (__attribute__((address_space(3))) void*)to, 16, (int)offset, (int)uniform_offset, 0, 0);
}

template <bool MX> using acc_t = typename std::conditional<MX, v16f_t, v16i_t>::type;

// one step: both operands' granules (A already cleared past the end of its row), scale dwords, byte kc
template <int KC>
__device__ __forceinline__ v16f_t mx_product(v4i_t a, v4i_t w, v16f_t acc, uint32_t sa, uint32_t sw) {
    const v8i_t va = {a[0], a[1], a[2], a[3], 0, 0, 0, 0};
    const v8i_t vw = {w[0], w[1], w[2], w[3], 0, 0, 0, 0};
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(va, vw, acc, 4 /* A: fp4 */, 4 /* B: fp4 */, KC, (int)sa, KC, (int)sw);
}

// Four scale bytes of a row from byte `at` on; bytes at or past nb (the row's number of them) are
// whatever: they meet codes that have been cleared.  at < nb + 4, nb >= 4.
__device__ __forceinline__ uint32_t scale_dword(const uint8_t* row, uint32_t at, uint32_t nb) {
    const uint32_t from = at + 4u <= nb ? at : nb - 4u;
    uint32_t v;
    __builtin_memcpy(&v, row + from, 4);             // (rows of scales need not be aligned)
    return v >> (8u * ((at - from) & 3u));
}

// Tile of this workgroup.  Workgroups go round-robin to the 8 XCDs, each with an L2 of its own: XCD x
// gets a contiguous share of the tiles in an order that walks columns of 8 tiles, so that its rows of
// A and W are read into its L2 once.
__device__ __forceinline__ void tile_of_block(const GemmParams& p, uint32_t& tt, uint32_t& tn) {
    const uint32_t total = p.tiles_t * p.tiles_n, x = blockIdx.x & 7u, idx = blockIdx.x >> 3;
    const uint32_t q = total >> 3, r = total & 7u;
    const uint32_t t = x * q + (x < r ? x : r) + idx;
    const uint32_t group = t / (8u * p.tiles_n), in = t - group * 8u * p.tiles_n;
    const uint32_t left = p.tiles_t - 8u * group, gh = left < 8u ? left : 8u;
    tt = 8u * group + in % gh;
    tn = in / gh;
}

// ---- tiles of 32 MT WM rows x 32 NT WN columns, WM x WN waves, operands staged in LDS --------------
// Stages go global -> LDS directly; NBUF stages are kept.  Place p of a row's 128-byte line holds
// granule p ^ ((r >> 1) & 7) of the stage: 16 rows a fragment read touches lie in 16 different places of the 64 banks.
//   Four stages make a superstage of 32 granules.  MXFP4: the 32 scale bytes that a row has in a superstage come into
// LDS as well, 1 KiB a load for 32 rows, and a lane picks the dword of each stage from there.  Loads of scales
// straight to the lanes that use them went to every row once per wave, and to spare some of them a stage took two halves
// of lines, which costs L2 twice the requests.  T = N = 2048, d = 8192 32.1 -> 23.9 us.
//   SHORT: rows of less than a superstage, whose scale bytes need a third of that LDS, so that a CU holds two workgroups and
// one stores its tile while the other multiplies (T = N = 4096, d = 256 15.4 us; one workgroup of four stages 19.4, of
// 128 x 256 19.7).
template <bool MX, int MT, int NT, int WM, int WN, int NBUF, int WGS, bool DWORDS, bool SHORT>
__global__ void __launch_bounds__(64 * WM * WN, WGS* WM* WN / 4)
gemm_tile_kernel(GemmParams p) {
    constexpr int kWaves = WM * WN, kBM = 32 * MT * WM, kBN = 32 * NT * WN;
    constexpr int kLoadA = kBM / 8 / kWaves, kLoadW = kBN / 8 / kWaves, kLoads = kLoadA + kLoadW;
    constexpr int kSc = MX ? MT + NT : 1, kRest = SHORT ? 0 : 2;         // scale bytes of the partial superstage
    constexpr int kScaleLoads = MX ? (kBM + kBN + 32 * kWaves - 1) / (32 * kWaves) : 1;      // of a wave and superstage
    constexpr uint32_t kBuf = (uint32_t)(kBM + kBN) * kStageBytes, kScaleBuf = (uint32_t)(kScaleLoads * kWaves) * 1024u;
    static_assert(kLoadA * 8 * kWaves == kBM && kLoadW * 8 * kWaves == kBN, "every wave loads whole pieces");
    static_assert(NBUF == 2 || NBUF == 4, "stage j of a superstage lies in buffer j % NBUF");
    extern __shared__ __align__(16) unsigned char lds[];
    const unsigned char* const scale_bytes_lds = lds + NBUF * kBuf;               // MXFP4: scale bytes of two superstages and of the partial one
    float* const scales_lds = reinterpret_cast<float*>(lds + NBUF * kBuf);        // INT4: steps of the rows, then of the columns

    const int lane = threadIdx.x & 63, i = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t tt, tn;
    tile_of_block(p, tt, tn);
    const int64_t t0 = (int64_t)tt * kBM;
    const int32_t n0 = (int32_t)tn * kBN;
    const uint32_t row_bytes = (uint32_t)p.d >> 1, granules = row_bytes >> 4;
    const int whole = SHORT ? 0 : (int)(granules >> 5);                             // whole superstages
    const uint32_t rest = granules & 31u;                                           // granules of the last, partial one
    // rows and columns past the end re-read the last one; their results are not stored
    const uint32_t last_t = (uint32_t)(p.T - t0 < kBM ? p.T - t0 : kBM) - 1u;
    const uint32_t last_n = (uint32_t)(p.N - n0 < kBN ? p.N - n0 : kBN) - 1u;

    if constexpr (!MX) {
        for (uint32_t r = threadIdx.x; r < (uint32_t)(kBM + kBN); r += 64u * kWaves) {
            const uint32_t c = r - kBM;
            scales_lds[r] = r < (uint32_t)kBM ? static_cast<const float*>(p.a_scales)[t0 + (r < last_t ? r : last_t)]
                                              : static_cast<const float*>(p.w_scales)[n0 + (int32_t)(c < last_n ? c : last_n)];
        }
    }

    // One load instruction fills 8 rows of a stage: lane l brings the granule of place l & 7 of row l >> 3.
    const uint32_t row8 = (uint32_t)lane >> 3, gran = ((uint32_t)lane & 7u) ^ ((row8 >> 1) + 4u * ((uint32_t)wave & 1u));
    const rsrc_t abuf = buffer_of(p.a_codes + t0 * row_bytes, (last_t + 1u) * row_bytes);
    const rsrc_t wbuf = buffer_of(p.w_codes + (int64_t)n0 * row_bytes, (last_n + 1u) * row_bytes);
    uint32_t off[kLoads];
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
        const uint32_t r = (uint32_t)((k < kLoadA ? k : k - kLoadA) * kWaves + wave) * 8u + row8;
        const uint32_t last = k < kLoadA ? last_t : last_n;
        off[k] = (r < last ? r : last) * row_bytes + 16u * gran;
    }
    // Requests the codes of stage j (0 .. 7) counted from superstage S.  Every call issues the same
    // number of loads, so that the waits below can count them.  `inner`: that superstage is a whole one.
    // Otherwise granules past the end of the row are clamped to it (cleared at use), and past the last
    // superstage all lanes load the same 16 bytes; no branches, which would keep the compiler from
    // leaving the products where they are put.
    auto request_codes = [&](int S, auto j_const, auto inner_const) {
        constexpr int jj = decltype(j_const)::value, j = jj & 3;
        constexpr bool inner = decltype(inner_const)::value;
        S += jj >> 2;
        const uint32_t g = gran + 8u * j, top = S < whole ? 31u : (rest != 0u ? rest - 1u : 0u);
        const uint32_t more = 16u * ((g < top ? g : top) - gran) + 512u * (uint32_t)S;
        const uint32_t keep = S < whole || (S == whole && rest != 0u) ? 0xFFFFFFFFu : 0u;
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            unsigned char* to = lds + (j % NBUF) * kBuf + (uint32_t)((k < kLoadA ? k * kWaves : kBM / 8 + (k - kLoadA) * kWaves) + wave) * 1024u;
            if constexpr (inner) load_to_lds16(k < kLoadA ? abuf : wbuf, off[k], 512u * (uint32_t)S + 128u * j, to);
            else load_to_lds16(k < kLoadA ? abuf : wbuf, (off[k] + more) & keep, 0u, to);
        }
    };

    // ---- MXFP4: scale bytes, 32 of every row and superstage, into LDS ---------------------------------
    // Lane l of piece q brings 16 bytes of row 32 q + (l >> 1): chunk (l & 1) ^ ((row >> 3) & 1) of its two.  Loads into
    // LDS, which ask for rows of whole dwords (DWORDS); through registers where the rows are not, and for the
    // superstage that the row's end cuts.
    const int wm = wave / WN, wn = wave % WN;
    const uint32_t nb = (uint32_t)p.d >> 5;
    const uint8_t* const a_bytes = static_cast<const uint8_t*>(p.a_scales) + (MX ? t0 * nb : 0);
    const uint8_t* const w_bytes = static_cast<const uint8_t*>(p.w_scales) + (MX ? (int64_t)n0 * nb : 0);
    const rsrc_t a_sbuf = buffer_of(a_bytes, (last_t + 1u) * nb), w_sbuf = buffer_of(w_bytes, (last_n + 1u) * nb);
    uint32_t soff[kScaleLoads];
    if constexpr (MX) {
#pragma unroll
        for (int k = 0; k < kScaleLoads; ++k) {
            const uint32_t row = (uint32_t)(k * kWaves + wave) * 32u + ((uint32_t)lane >> 1);
            const uint32_t r = row < (uint32_t)kBM ? row : row - kBM, last = row < (uint32_t)kBM ? last_t : last_n;
            soff[k] = (r < last ? r : last) * nb;
        }
    }
    const uint32_t chunk = 16u * (((uint32_t)lane & 1u) ^ (((uint32_t)lane >> 4) & 1u));      // (row >> 3 is lane >> 4 here)
    auto of_a = [&](int k) { return (k * kWaves + wave) * 32 < kBM; };
    auto piece_at = [&](int buffer, int k) { return NBUF * kBuf + (uint32_t)buffer * kScaleBuf + (uint32_t)(k * kWaves + wave) * 1024u; };
    struct Quad { uint32_t w[4]; } sreg[kScaleLoads], rest_sreg[kScaleLoads];
    auto request_scales = [&](int S) {
        if constexpr (MX) {
#pragma unroll
            for (int k = 0; k < kScaleLoads; ++k) {
                if constexpr (DWORDS) load_to_lds16(of_a(k) ? a_sbuf : w_sbuf, soff[k] + chunk, 32u * (uint32_t)S, lds + piece_at(S & 1, k));
                else __builtin_memcpy(sreg[k].w, (of_a(k) ? a_bytes : w_bytes) + (soff[k] + chunk + 32u * (uint32_t)S), 16);
            }
        }
    };
    auto keep_scales = [&](int buffer, const Quad (&from)[kScaleLoads]) {
#pragma unroll
        for (int k = 0; k < kScaleLoads; ++k) {
            const v4i_t v = {(int)from[k].w[0], (int)from[k].w[1], (int)from[k].w[2], (int)from[k].w[3]};
            const uint32_t to = piece_at(buffer, k) + 16u * (uint32_t)lane;
            // (an instruction: ahead of an LDS store that it knows, the compiler waits for every load into LDS)
            asm volatile("ds_write_b128 %0, %1" ::"v"(to), "v"(v) : "memory");
        }
    };
    // The partial superstage: dword q of a chunk; one that the row's end cuts is the row's last four bytes, shifted.
    auto rest_at = [&](uint32_t q) { return 32u * (uint32_t)whole + chunk + 4u * q; };
    auto request_rest_scales = [&]() {
#pragma unroll
        for (int k = 0; k < kScaleLoads; ++k) {
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q)
                __builtin_memcpy(&rest_sreg[k].w[q], (of_a(k) ? a_bytes : w_bytes) + (soff[k] + (rest_at(q) < nb - 4u ? rest_at(q) : nb - 4u)), 4);
        }
    };
    auto keep_rest_scales = [&]() {
#pragma unroll
        for (int k = 0; k < kScaleLoads; ++k) {
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) rest_sreg[k].w[q] >>= rest_at(q) < nb - 4u ? 0u : 8u * ((rest_at(q) - (nb - 4u)) & 3u);
        }
        keep_scales(kRest, rest_sreg);
    };
    // the four scale bytes of this lane's granules in each stage of superstage S
    struct Scales { uint32_t w[kSc][4]; };
    auto read_scales = [&](int buffer, Scales& to) {
        if constexpr (MX) {
            const unsigned char* base = scale_bytes_lds + (uint32_t)buffer * kScaleBuf + (uint32_t)i * 32u + 4u * (uint32_t)h;
            const uint32_t flip = 16u * (((uint32_t)i >> 3) & 1u);
#pragma unroll
            for (int m = 0; m < MT + NT; ++m) {
                const uint32_t row0 = (uint32_t)(m < MT ? (wm * MT + m) * 32 : kBM + (wn * NT + m - MT) * 32);
#pragma unroll
                for (int j = 0; j < 4; ++j) to.w[m][j] = *reinterpret_cast<const uint32_t*>(base + row0 * 32u + ((uint32_t)(16 * (j >> 1)) ^ flip) + 8 * (j & 1));
            }
        }
    };

    constexpr bool kEarly = !MX && MT * NT == 1;
    acc_t<MX> acc[MT][NT] = {};
    // byte offset of this lane's fragment rows inside a buffer; place of its granule in the line in step kc
    const uint32_t fa = (uint32_t)((wm * MT) * 32 + i) * kStageBytes, fw = (uint32_t)(kBM + (wn * NT) * 32 + i) * kStageBytes;
    uint32_t place[4];
#pragma unroll
    for (int kc = 0; kc < 4; ++kc) place[kc] = ((uint32_t)(4 * h + kc) ^ (((uint32_t)i >> 1) & 7u)) * 16u;
    struct Raw { v4i_t a[MT], w[NT]; };
    struct Ops { v4i_t ah[MT], al[MT], wh[NT], wl[NT]; };
    // step 0 .. 3: stage j; 4, 5: the first steps of the stage after it
    auto read = [&](int j, int step, Raw& f) {
        const unsigned char* base = lds + (uint32_t)((j + (step >> 2)) % NBUF) * kBuf + place[step & 3];
#pragma unroll
        for (int m = 0; m < MT; ++m) f.a[m] = *reinterpret_cast<const v4i_t*>(base + fa + m * 32 * kStageBytes);
#pragma unroll
        for (int n = 0; n < NT; ++n) f.w[n] = *reinterpret_cast<const v4i_t*>(base + fw + n * 32 * kStageBytes);
    };
    // -1, or 0 where the granule of stage j, step kc lies past the end of the row: the codes of A count as zero
    auto live = [&](int j, int kc) { return 8u * (uint32_t)j + 4u * (uint32_t)h + (uint32_t)kc < rest ? -1 : 0; };
    auto unpack = [&](const Raw& f, Ops& o, int keep) {
        const int am = (int)kHighNibbles & keep;
#pragma unroll
        for (int m = 0; m < MT; ++m) { o.ah[m] = high_codes(f.a[m], am); o.al[m] = low_codes(f.a[m], am); }
#pragma unroll
        for (int n = 0; n < NT; ++n) { o.wh[n] = high_codes(f.w[n], (int)kHighNibbles); o.wl[n] = low_codes(f.w[n], (int)kHighNibbles); }
    };
    auto multiply_i8 = [&](const Ops& o) {
#pragma unroll
        for (int n = 0; n < NT; ++n) {
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[m][n] = __builtin_amdgcn_mfma_i32_32x32x32_i8(o.ah[m], o.wh[n], acc[m][n], 0, 0, 0);
        }
#pragma unroll
        for (int n = 0; n < NT; ++n) {
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[m][n] = __builtin_amdgcn_mfma_i32_32x32x32_i8(o.al[m], o.wl[n], acc[m][n], 0, 0, 0);
        }
    };
    auto multiply_mx = [&](auto kc_const, const Raw& f, const uint32_t (&sw)[kSc], int keep) {
        constexpr int kc = decltype(kc_const)::value;
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const v4i_t a = f.a[m] & keep;
#pragma unroll
            for (int n = 0; n < NT; ++n) acc[m][n] = mx_product<kc>(a, f.w[n], acc[m][n], sw[m], sw[MT + n]);
        }
    };

    // The next stage is complete in LDS once this wave's loads of it have landed (younger ones may still
    // be on their way) and every wave has passed the barrier; by then every wave has read the whole of the
    // present stage, whose buffer is loaded next.
    Raw r0, r1;
    Ops u0, u1;
    Scales cur, nxt;
    auto advance = [&]() {
        // requested after the next stage's codes: those of NBUF - 2 stages (vmcnt: a six-bit count in bits 3:0
        // and 15:14).  Scales may have been requested among them and are not counted: those are loads like any
        // other, which the compiler takes out where nothing uses them, and a count of loads that are not there
        // lets the wait pass early.  A load into LDS stays where it was put.  (Counting them as well gains
        // 1.7 % at (2048, 4096, 4096) and nothing elsewhere.)
        constexpr int n = (NBUF - 2) * kLoads;
        static_assert(n < 64, "");
        __builtin_amdgcn_s_waitcnt(0x0F70 | (n & 15) | ((n >> 4) << 14));
        workgroup_barrier_lds();
    };
    // One stage.  INT4: the codes of a step are read two steps ahead of its products and unpacked while
    // the products of the step before run, a few vector instructions to a product (a wave issues in
    // order).  MXFP4: they are read one step ahead.
    auto stage = [&](int S, auto j_const, auto inner_const, auto tail_const) {
        constexpr int j = decltype(j_const)::value;
        constexpr bool tail = decltype(tail_const)::value, inner = decltype(inner_const)::value;
        if constexpr (MX) {
            uint32_t sw[kSc];
#pragma unroll
            for (int m = 0; m < kSc; ++m) sw[m] = cur.w[m][j];
            auto step = [&](auto kc_const, Raw& now, Raw& next) {
                constexpr int kc = decltype(kc_const)::value;
                constexpr bool kScalesNow = kc == 1 && j == 0 && inner;
                if constexpr (kc == 3) advance();
                read(j, kc + 1, next);
                if constexpr (kc == 3 && j == 3 && !tail) read_scales(inner ? (S + 1) & 1 : kRest, nxt);
                if constexpr (!DWORDS && kc == 1 && j == 3 && inner) keep_scales((S + 1) & 1, sreg);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (kc == 3) request_codes(S, std::integral_constant<int, j + NBUF>{}, inner_const);
                if constexpr (kScalesNow) request_scales(S + 1);
                multiply_mx(kc_const, now, sw, tail ? live(j, kc) : -1);
                if constexpr (kc == 3 || kScalesNow) {
#pragma unroll
                    for (int q = 0; q < MT * NT; ++q) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                  // one product
                        __builtin_amdgcn_sched_group_barrier(0x020, kc == 3 ? (kLoads + MT * NT - 1) / (MT * NT) : 1, 0);  // and its share of the loads
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            step(std::integral_constant<int, 0>{}, r0, r1);
            step(std::integral_constant<int, 1>{}, r1, r0);
            step(std::integral_constant<int, 2>{}, r0, r1);
            step(std::integral_constant<int, 3>{}, r1, r0);
        } else {
            auto step = [&](auto kc_const, const Ops& now, Ops& next, const Raw& raw_next, Raw& raw) {
                constexpr int kc = decltype(kc_const)::value;
                if constexpr (kc == 2) advance();
                if constexpr (kc == 2 && kEarly) {
                    request_codes(S, std::integral_constant<int, j + NBUF>{}, inner_const);
                    __builtin_amdgcn_sched_barrier(0);
                }
                read(j, kc + 2, raw);
                // (the step after the last one of a tail is never multiplied)
                unpack(raw_next, next, tail ? live(j + ((kc + 1) >> 2), (kc + 1) & 3) : -1);
                if constexpr (kc == 2 && !kEarly) request_codes(S, std::integral_constant<int, j + NBUF>{}, inner_const);
                multiply_i8(now);
                __builtin_amdgcn_sched_group_barrier(0x100, MT + NT, 0);                      // the reads
#pragma unroll
                for (int q = 0; q < 2 * MT * NT; ++q) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                        // one product
                    __builtin_amdgcn_sched_group_barrier(0x002, (12 * (MT + NT) + 2 * MT * NT - 1) / (2 * MT * NT), 0);
                    if constexpr (kc == 2 && !kEarly) __builtin_amdgcn_sched_group_barrier(0x020, (kLoads + 2 * MT * NT - 1) / (2 * MT * NT), 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            step(std::integral_constant<int, 0>{}, u0, u1, r1, r0);
            step(std::integral_constant<int, 1>{}, u1, u0, r0, r1);
            step(std::integral_constant<int, 2>{}, u0, u1, r1, r0);
            step(std::integral_constant<int, 3>{}, u1, u0, r0, r1);
        }
    };
    if constexpr (MX) {
        if (rest != 0u) request_rest_scales();
        if (whole > 0) request_scales(0);
    }
    __builtin_amdgcn_sched_barrier(0);
    request_codes(0, std::integral_constant<int, 0>{}, std::false_type{});
    __builtin_amdgcn_sched_barrier(0);
    request_codes(0, std::integral_constant<int, 1>{}, std::false_type{});
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (NBUF == 4) {
        request_codes(0, std::integral_constant<int, 2>{}, std::false_type{});
        __builtin_amdgcn_sched_barrier(0);
        request_codes(0, std::integral_constant<int, 3>{}, std::false_type{});
        __builtin_amdgcn_sched_barrier(0);
    }
    {
        constexpr int n = (NBUF - 1) * kLoads;
        if constexpr (MX) {
            if (!DWORDS && whole > 0) keep_scales(0, sreg);
            if (rest != 0u) keep_rest_scales();
        }
        __builtin_amdgcn_s_waitcnt(0x0F70 | (n & 15) | ((n >> 4) << 14));
        workgroup_barrier_lds();
        read(0, 0, r0);
        read_scales(whole > 0 ? 0 : kRest, cur);
        if constexpr (!MX) {
            read(0, 1, r1);
            unpack(r0, u0, whole > 0 ? -1 : live(0, 0));
        }
    }
    int S = 0;
    auto superstage = [&](auto inner_const) {
        stage(S, std::integral_constant<int, 0>{}, inner_const, std::false_type{});
        stage(S, std::integral_constant<int, 1>{}, inner_const, std::false_type{});
        stage(S, std::integral_constant<int, 2>{}, inner_const, std::false_type{});
        stage(S, std::integral_constant<int, 3>{}, inner_const, std::false_type{});
        cur = nxt;
    };
    for (; S + 1 < whole; ++S) superstage(std::true_type{});
    for (; S < whole; ++S) superstage(std::false_type{});
    if (rest != 0u) {
        // the first step was unpacked as if it were whole
        if (!MX && whole > 0) {
            const int keep = live(0, 0);
#pragma unroll
            for (int m = 0; m < MT; ++m) { u0.ah[m] &= keep; u0.al[m] &= keep; }
        }
        constexpr uint32_t kFrom = 8u;        // stage j holds something if rest > kFrom j
        stage(S, std::integral_constant<int, 0>{}, std::false_type{}, std::true_type{});
        if (rest > kFrom) stage(S, std::integral_constant<int, 1>{}, std::false_type{}, std::true_type{});
        if (rest > 2u * kFrom) stage(S, std::integral_constant<int, 2>{}, std::false_type{}, std::true_type{});
        if (rest > 3u * kFrom) stage(S, std::integral_constant<int, 3>{}, std::false_type{}, std::true_type{});
    }
    // no load may be on its way into LDS that another workgroup owns by then
    __builtin_amdgcn_s_waitcnt(0x0F70);

    auto store = [&](auto inner_const, auto whole_lines_const) {
        constexpr bool inner = decltype(inner_const)::value, whole_lines = decltype(whole_lines_const)::value;
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const uint32_t rt = (uint32_t)((wm * MT + m) * 32 + 4 * h);            // row of accumulator 0 in the tile
            float* o = p.out + (t0 + rt) * p.ldo + n0 + (wn * NT) * 32 + i;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float4 sa = make_float4(0, 0, 0, 0);
                if constexpr (!MX) sa = *reinterpret_cast<const float4*>(scales_lds + rt + 8 * q);
                const float sq[4] = {sa.x, sa.y, sa.z, sa.w};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    float* row = o + (8 * q + k) * p.ldo;
#pragma unroll
                    for (int n = 0; n < NT; ++n) {
                        const uint32_t c = (uint32_t)((wn * NT + n) * 32 + i);
                        float v;
                        if constexpr (MX) v = acc[m][n][4 * q + k];
                        else v = (float)acc[m][n][4 * q + k] * 0x1p-8f * sq[k] * scales_lds[kBM + c];      // (the sum is below 2^24: exact)
                        if constexpr (whole_lines) __builtin_nontemporal_store(v, row + n * 32);
                        else if (inner || (rt + 8 * q + k <= last_t && c <= last_n)) row[n * 32] = v;
                    }
                }
            }
        }
    };
    if (last_t + 1u == (uint32_t)kBM && last_n + 1u == (uint32_t)kBN) {
        if (p.stream_out) {
            // (the empty statements keep the compiler from making one store of the two, without the policy)
            asm volatile("" ::: "memory");
            store(std::true_type{}, std::true_type{});
            asm volatile("" ::: "memory");
        } else {
            store(std::true_type{}, std::false_type{});
        }
    } else {
        store(std::false_type{}, std::false_type{});
    }
}

// ---- few tiles: one 32 x 32 tile per workgroup, the contraction cut among its KW waves -------------
// Wave k takes the stages k, k + KW, ...: it brings a stage, a line of every row and column, into 8 KiB of LDS of its own
// with eight direct loads, reads its operands, asks for its next stage and multiplies; the partial tiles are added in
// wave order, the only barrier.
//   Bound by the loads.  Straight to registers, nothing is used twice either, but an instruction then meets 32 rows,
// which takes the address unit four times as long as eight rows of a line each, and that bound the kernel:
// INT4 / MXFP4 (3, 517, 28672) 18.8 / 25.2 -> 10.4 / 12.2 us, (64, 4096, 8192) 10.1 / 12.9 -> 6.1 / 7.0, (16, 4096, 4096)
// 5.0 / 5.4 -> 3.8 / 4.0 (registers, then LDS).  A second buffer per wave leaves one workgroup a CU instead of two:
// (123, 2665, 12288) INT4 14.4 instead of 11.4; sixteen waves: (64, 4096, 14336) 8.9 instead of 8.2.
template <bool MX, int KW>
__global__ void __launch_bounds__(64 * KW)
gemm_few_kernel(GemmParams p) {
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr uint32_t kStage = 64u * kStageBytes;
    const int lane = threadIdx.x & 63, i = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    unsigned char* const mine = lds + (uint32_t)wave * kStage;
    uint32_t tt, tn;
    tile_of_block(p, tt, tn);
    const int64_t t0 = (int64_t)tt * 32;
    const int32_t n0 = (int32_t)tn * 32;
    const uint32_t row_bytes = (uint32_t)p.d >> 1, granules = row_bytes >> 4, nb = (uint32_t)p.d >> 5;
    const uint32_t last_t = (uint32_t)(p.T - t0 < 32 ? p.T - t0 : 32) - 1u;
    const uint32_t last_n = (uint32_t)(p.N - n0 < 32 ? p.N - n0 : 32) - 1u;
    const rsrc_t abuf = buffer_of(p.a_codes + t0 * row_bytes, (last_t + 1u) * row_bytes);
    const rsrc_t wbuf = buffer_of(p.w_codes + (int64_t)n0 * row_bytes, (last_n + 1u) * row_bytes);
    const uint8_t* const as = static_cast<const uint8_t*>(p.a_scales) + (MX ? (t0 + ((uint32_t)i < last_t ? (uint32_t)i : last_t)) * nb : 0);
    const uint8_t* const ws = static_cast<const uint8_t*>(p.w_scales) + (MX ? (int64_t)(n0 + ((uint32_t)i < last_n ? (uint32_t)i : last_n)) * nb : 0);
    // a load fills 8 rows: lane l brings the granule of place l & 7 of row l >> 3 (place q of row r holds granule
    // q ^ ((r >> 1) & 7))
    uint32_t a_row[4], w_row[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t r = 8u * k + ((uint32_t)lane >> 3);
        a_row[k] = (r < last_t ? r : last_t) * row_bytes;
        w_row[k] = (r < last_n ? r : last_n) * row_bytes;
    }
    const uint32_t gran = ((uint32_t)lane & 7u) ^ ((uint32_t)lane >> 4);
    uint32_t sa_next = 0, sw_next = 0;
    // (granules past the end of a row are its last one, cleared in A at use)
    auto request = [&](int s) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t g = 8u * (uint32_t)s + (gran ^ (4u * (k & 1))), at = 16u * (g < granules ? g : granules - 1u);
            load_to_lds16(abuf, a_row[k] + at, 0u, mine + 1024 * k);
            load_to_lds16(wbuf, w_row[k] + at, 0u, mine + 1024 * (4 + k));
        }
        if constexpr (MX) {
            uint32_t at = 8u * (uint32_t)s + 4u * (uint32_t)h;
            at = at < nb ? at : nb - 1u;
            sa_next = scale_dword(as, at, nb);
            sw_next = scale_dword(ws, at, nb);
        }
    };
    acc_t<MX> acc = {};
    const int stages = (int)((granules + 7u) >> 3);
    if (wave < stages) request(wave);
    for (int s = wave; s < stages; s += KW) {
        __builtin_amdgcn_s_waitcnt(0x0F70);
        __builtin_amdgcn_sched_barrier(0);
        const unsigned char* const from = mine + (uint32_t)i * kStageBytes;
        v4i_t a[4], w[4];
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) {
            const uint32_t place = 16u * ((uint32_t)(4 * h + kc) ^ (((uint32_t)i >> 1) & 7u));
            a[kc] = *reinterpret_cast<const v4i_t*>(from + place);
            w[kc] = *reinterpret_cast<const v4i_t*>(from + 32u * kStageBytes + place);
        }
        const uint32_t sa = sa_next, sw = sw_next;
        // every read has landed before the buffer is loaded again
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3])::"memory");
        if (s + KW < stages) request(s + KW);
        if (8u * (uint32_t)s + 8u > granules) {
#pragma unroll
            for (int kc = 0; kc < 4; ++kc) {
                if (8u * (uint32_t)s + 4u * (uint32_t)h + (uint32_t)kc >= granules) a[kc] = v4i_t{0, 0, 0, 0};
            }
        }
        if constexpr (MX) {
            acc = mx_product<0>(a[0], w[0], acc, sa, sw);
            acc = mx_product<1>(a[1], w[1], acc, sa, sw);
            acc = mx_product<2>(a[2], w[2], acc, sa, sw);
            acc = mx_product<3>(a[3], w[3], acc, sa, sw);
        } else {
#pragma unroll
            for (int kc = 0; kc < 4; ++kc) {
                const int mk = (int)kHighNibbles;
                acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(high_codes(a[kc], mk), high_codes(w[kc], mk), acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(low_codes(a[kc], mk), low_codes(w[kc], mk), acc, 0, 0, 0);
            }
        }
    }
    // partial tiles into the waves' own buffers, which nothing is on its way to: [16][64]
    typedef typename std::conditional<MX, float, int>::type part_t;
    part_t* const part = reinterpret_cast<part_t*>(mine);
#pragma unroll
    for (int j = 0; j < 16; ++j) part[64 * j + lane] = acc[j];
    __syncthreads();
#pragma unroll
    for (int jj = 0; jj < 16 / KW; ++jj) {
        const int j = jj * KW + wave;
        part_t sum = 0;
#pragma unroll
        for (int k = 0; k < KW; ++k) sum += reinterpret_cast<const part_t*>(lds + (uint32_t)k * kStage)[64 * j + lane];
        const int64_t row = t0 + 8 * (j >> 2) + 4 * h + (j & 3);
        if (row < p.T && n0 + i < p.N) {
            float v;
            if constexpr (MX) v = sum;
            else v = (float)sum * 0x1p-8f * static_cast<const float*>(p.a_scales)[row] * static_cast<const float*>(p.w_scales)[n0 + i];
            p.out[row * p.ldo + n0 + i] = v;
        }
    }
}

// ---- rows of up to four granules (d <= 128): one 32 x 32 tile per wave, nothing but its operands -----
// Bound by the store.  Half-wave h takes granules h and 2 + h.
template <bool MX>
__global__ void __launch_bounds__(64)
gemm_short_kernel(GemmParams p) {
    const int lane = threadIdx.x, i = lane & 31, h = lane >> 5;
    uint32_t tt, tn;
    tile_of_block(p, tt, tn);
    const int64_t t0 = (int64_t)tt * 32, t = t0 + i < p.T ? t0 + i : p.T - 1;
    const int32_t n0 = (int32_t)tn * 32, n = n0 + i < p.N ? n0 + i : p.N - 1;
    const uint32_t row_bytes = (uint32_t)p.d >> 1, granules = row_bytes >> 4;
    acc_t<MX> acc = {};
    v4i_t a[2], w[2];
    uint32_t sa[2] = {0, 0}, sw[2] = {0, 0};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const uint32_t g = 2u * k + (uint32_t)h, gc = g < granules ? g : granules - 1u;
        a[k] = *reinterpret_cast<const v4i_t*>(p.a_codes + t * row_bytes + 16u * gc);
        w[k] = *reinterpret_cast<const v4i_t*>(p.w_codes + (int64_t)n * row_bytes + 16u * gc);
        if constexpr (MX) {
            sa[k] = static_cast<const uint8_t*>(p.a_scales)[t * granules + gc];
            sw[k] = static_cast<const uint8_t*>(p.w_scales)[(int64_t)n * granules + gc];
        }
        if (g >= granules) a[k] = v4i_t{0, 0, 0, 0};
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        if (2u * k >= granules) break;
        if constexpr (MX) {
            acc = mx_product<0>(a[k], w[k], acc, sa[k], sw[k]);
        } else {
            const int mk = (int)kHighNibbles;
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(high_codes(a[k], mk), high_codes(w[k], mk), acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(low_codes(a[k], mk), low_codes(w[k], mk), acc, 0, 0, 0);
        }
    }
    const float step_w = MX ? 1.0f : static_cast<const float*>(p.w_scales)[n];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const int64_t row = t0 + 8 * (j >> 2) + 4 * h + (j & 3);
        if (row < p.T && n0 + i < p.N) {
            float v;
            if constexpr (MX) v = acc[j];
            else v = (float)acc[j] * 0x1p-8f * static_cast<const float*>(p.a_scales)[row] * step_w;
            p.out[row * p.ldo + n0 + i] = v;
        }
    }
}

// Rows of the output begin and end with a 128-byte line.
bool whole_lines(const GemmParams& p) { return p.ldo % 32 == 0 && (reinterpret_cast<uintptr_t>(p.out) & 127u) == 0; }

template <bool MX, int MT, int NT, int WM, int WN, int NBUF, int WGS, bool DWORDS, bool SHORT = false>
hipError_t launch_tile_as(GemmParams p, hipStream_t stream) {
    constexpr uint32_t lds_bytes = (uint32_t)(32 * MT * WM + 32 * NT * WN) * (kStageBytes * NBUF + (MX ? 0u : 4u)) +
                                    (MX ? (SHORT ? 1u : 3u) * 1024u * WM * WN * ((MT * WM + NT * WN + WM * WN - 1) / (WM * WN)) : 0u);
    static_assert(WGS * lds_bytes <= 160u * 1024u, "LDS of a CU");
    p.tiles_t = (uint32_t)((p.T + 32 * MT * WM - 1) / (32 * MT * WM));
    p.tiles_n = (uint32_t)(((int64_t)p.N + 32 * NT * WN - 1) / (32 * NT * WN));
    // Whole lines of the output are stored with the streaming policy: all workgroups of a round store at the same time, and
    // what stays in L2 is written back at the end of the launch.  INT4 / MXFP4 (2048, 4096, 2048) 22.0 / 20.9 -> 18.8 / 15.2,
    // (2048, 14336, 4096) 112 / 111 -> 103 / 84, (2048, 2048, 1024) 9.5 / 8.8 -> 8.3 / 7.6.  Lines that two rows share:
    // (3000, 3500, 1024) 20.0 / 19.3 -> 22.9 / 22.2, so those keep the plain store.
    p.stream_out = whole_lines(p);
    auto kern = gemm_tile_kernel<MX, MT, NT, WM, WN, NBUF, WGS, DWORDS, SHORT>;
    int per_cu = 0;      // (raises the kernel's limit of dynamic LDS)
    const hipError_t e = resident_blocks(reinterpret_cast<const void*>(kern), 64 * WM * WN, lds_bytes, &per_cu);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(p.tiles_t * p.tiles_n), dim3(64 * WM * WN), lds_bytes, stream, p);
    return hipGetLastError();
}

template <bool MX, int MT, int NT, int WM, int WN, int NBUF, int WGS>
hipError_t launch_tile(const GemmParams& p, hipStream_t stream) {
    if constexpr (MX) {
        if (p.d % 128 != 0 || ((reinterpret_cast<uintptr_t>(p.a_scales) | reinterpret_cast<uintptr_t>(p.w_scales)) & 3u) != 0)
            return launch_tile_as<MX, MT, NT, WM, WN, NBUF, WGS, false>(p, stream);
    }
    return launch_tile_as<MX, MT, NT, WM, WN, NBUF, WGS, true>(p, stream);
}

// Rows of one launch of the kernel for short rows.  A grid takes less than 2^32 lanes, 64 to a tile of 32 x 32
// outputs: 2^36 outputs are more than that (and fit the card's memory).  The other kernels have a lane
// per 64 outputs, or few tiles.
constexpr int64_t rows_of_a_short_launch(int64_t tiles_n) {
    const int64_t most = ((int64_t)1 << 26) - 1;
    return 32 * (most / tiles_n > 0 ? most / tiles_n : 1);
}
static_assert(rows_of_a_short_launch(1) == 32 * (((int64_t)1 << 26) - 1), "one column of tiles: any T that is accepted");
static_assert(rows_of_a_short_launch(33000 / 32 + 1) < 2097120, "T = 2097120, N = 33000 (277 GB of output) takes two launches");
static_assert(rows_of_a_short_launch(33000 / 32 + 1) / 32 * (33000 / 32 + 1) * 64 < ((int64_t)1 << 32), "that fit");
static_assert(rows_of_a_short_launch(32768 / 32) >= 2097120, "T = 2097120, N = 32768 takes one");

template <bool MX>
hipError_t launch_short(const GemmParams& all, hipStream_t stream) {
    GemmParams p = all;
    p.tiles_n = (uint32_t)(((int64_t)p.N + 31) / 32);
    const int64_t rows = rows_of_a_short_launch(p.tiles_n), row_bytes = all.d >> 1, scale_bytes = MX ? all.d >> 5 : 4;
    for (int64_t t = 0; t < all.T; t += rows) {
        p.T = all.T - t < rows ? all.T - t : rows;
        p.a_codes = all.a_codes + t * row_bytes;
        p.a_scales = static_cast<const uint8_t*>(all.a_scales) + t * scale_bytes;
        p.out = all.out + t * all.ldo;
        p.tiles_t = (uint32_t)((p.T + 31) / 32);
        hipLaunchKernelGGL(gemm_short_kernel<MX>, dim3(p.tiles_t * p.tiles_n), dim3(64), 0, stream, p);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <bool MX, int KW>
hipError_t launch_few(GemmParams p, hipStream_t stream) {
    constexpr uint32_t lds_bytes = KW * 64u * kStageBytes;
    static_assert(lds_bytes <= 64u * 1024u, "what a kernel may ask for as it is");
    p.tiles_t = (uint32_t)((p.T + 31) / 32);
    p.tiles_n = (uint32_t)(((int64_t)p.N + 31) / 32);
    auto kern = gemm_few_kernel<MX, KW>;
    hipLaunchKernelGGL(kern, dim3(p.tiles_t * p.tiles_n), dim3(64 * KW), lds_bytes, stream, p);
    return hipGetLastError();
}

// Which kernel and tile.  Measured on both sides of every line, one GPU, launches back to back, us at (T, N, d): the
// kernel that a paragraph is about / the other one.
//   d < 128, MXFP4 also d = 128: no staging and no cut of the contraction, one wave per 32 x 32 tile.
//     INT4 (4096, 4096, 64) 14.7 / 19.1, MXFP4 12.2 / 15.6 against a trip of the tile through LDS; d = 128 against the tiles
//     below (4096, 4096) 15.9 / 16.3 and 13.2 / 14.4, (300, 14336) 7.7 / 8.2 and 6.7 / 7.6.
//   Few tiles of 32 x 32: the contraction cut among 8 waves, against 64 x 64 tiles.
//     INT4, up to 512 (64, 4096, 4096) 4.0 / 8.1, (300, 1500, 1088) 4.0 / 5.0; up to 768 (three workgroups on a CU) from
//     d = 2048 on (200, 3000, 2048) 5.3 / 5.9, (64, 12288, 4096) 8.7 / 9.2, past that (64, 13000, 4096) 10.4 / 9.6,
//     (128, 6400, 8192) 15.4 / 14.7; up to 900 where the 64 x 64 tiles are more than one a CU (96, 9568, 4096) 10.9 / 12.3.
//     MXFP4, up to 256 (64, 4096, 4096) 4.1 / 5.3, (64, 4096, 14336) 10.7 / 14.2, past that (96, 4096, 4096) 6.3 / 5.9; rows
//     of scale bytes that are no whole dwords, which tiles read through registers, up to 512 and d = 8192
//     (300, 1500, 1088) 3.7 / 4.6, d = 4000 6.7 / 7.0, (1848, 148, 7072) 9.6 / 11.5, past that (300, 1500, 8224) 13.6 / 13.2,
//     (128, 4000, 14368) 23.2 / 21.0.
//   One row of tiles, which fills half of a 64 x 64 tile or less: the same, any number of them.
//     INT4 (16, 65536, 4096) 30.1 / 36.0, (32, 65536, 8192) 59.5 / 63.1.
//     MXFP4 has half the products to a load, and all of A is loaded again every 32 columns, so it goes by T d:
//     (16, 65536, 4096) 32.1 / 32.6, (24, 65536, 4096) 34.7 / 34.1, (32, 65536, 2560) 21.0 / 19.9, (32, 65536, 8192) 74.9 /
//     60.9; below 65536 columns (32, 20480, 4096) 9.8 / 10.9, (32, 40960, 4096) 18.6 / 18.9, (24, 28672, 8192) 32.6 / 30.1,
//     (16, 20480, 14336) 39.5 / 38.3; 257 .. 384 tiles (32, 10000, 4096) 7.3 / 6.5, (1, 10000, 8192) 10.3 / 8.9,
//     d = 2048 4.7 / 4.7; no whole dwords (16, 65536, 2880) 22.9 / 22.8, (16, 65536, 4000) 36.5 / 33.0,
//     (16, 14336, 4000) 7.6 / 7.8, (32, 14336, 4000) 8.8 / 8.0.
//     Among 4 waves instead of 8 where there are more than 512 tiles and little to cut: (16, 65536, 2048) INT4
//     13.3 / 14.8, MXFP4 12.6 / 14.1, (16, 65536, 2880) INT4 20.7 / 22.1; no whole dwords, of which a wave then reads more,
//     MXFP4 d = 2400 19.2 / 19.7, d = 2880 24.3 / 22.9.
//   Up to 128 tiles of 128 x 128: 64 x 64 tiles, which two workgroups a CU hold at once up to there, against 128 x 128.
//     INT4 (512, 4096, 4096) 13.7 / 15.5, d = 1024 6.2 / 7.3, past that (640, 3328, 4096) 19.1 / 15.5; MXFP4 10.7 / 12.5,
//     5.4 / 6.5 and 13.7 / 12.1.
//   MXFP4, d < 1024: 128 x 128, two stages and two workgroups a CU, against 128 x 256 (/ four stages and one).
//     (4096, 4096) d = 160 15.6 / 20.0 / 19.4, d = 320 17.1 / 21.3 / 21.4, d = 640 18.4 / 25.4 / 26.4, d = 992 22.2 / 28.5 /
//     29.9; (3000, 3500, 256) 12.6 / 14.4 / 16.6, d = 768 15.9 / 18.0 / 19.9; (8192, 8192, 512) 57.6 / 68.0 / 88.4;
//     (2048, 2048, 256) 6.5 / 7.2 / 7.1, d = 992 7.8 / 8.8 / 8.6.  One round of 128 x 256 is as fast or faster up to d = 512:
//     (2048, 4096) d = 160 9.4 / 8.7, d = 512 10.6 / 10.0, d = 768 11.3 / 11.3; (300, 14336, 512) 7.7 / 7.2.
//   MXFP4, longer rows: 128 x 256, a sixth less to load per product, against 128 x 128, both one workgroup a CU, by rounds
//     of 256 tiles.  In eighths of a round of 128 x 128: a round that is not full 6 (fewer workgroups share L2 and power),
//     of 128 x 256 14 and 10.
//     One round for two (2177, 2177, 1024) 10.9 / 12.9, d = 8192 36.9 / 41.4, (2048, 4096, 4096) 25.7 / 29.7; two for three
//     (3000, 3500, 8192) 73.4 / 69.1, (2304, 4096, 8192) 68.1 / 60.3, (3072, 4096, 2048) 25.2 / 25.0; two for four
//     (4096, 4096, 2048) 33.5 / 34.3, d = 8192 84.3 / 92.4, (3968, 3969, 2880) 43.2 / 52.4; three for five
//     (4096, 5120, 2048) 37.1 / 39.6, but (4096, 4097, 8192) 109 / 107; four for seven (2048, 14336, 4096) 89.9 / 91.8;
//     (36000, 128, 4096), where half of every tile is empty, 43.9 / 24.9.
//   INT4: 128 x 256 against two workgroups of 128 x 128 a CU, which load less per product.
//     Where some CUs have one of those and some two; the more have two, the longer a row has to be: (2048, 2304, 4096)
//     23.7 / 28.7, (2048, 2560, 2880) 20.9 / 21.8, (2048, 3072, 4096) 26.5 / 29.5, d = 2880 21.9 / 22.1, d = 2048 17.7 / 17.1,
//     (2048, 3584, 4096) 29.1 / 29.2, (2048, 4096, 4096) 32.4 / 31.4, d = 5120 36.0 / 36.1, d = 14336 90.5 / 93.7; not for up
//     to 64 rows, (64, 65536, 8192) 77.6 / 72.4.
//     The longest rows, if the rounds are full: (4096, 4096, 4096) 62.2 / 59.8, d = 6144 82.2 / 82.5, d = 8192 107.2 /
//     107.9, d = 16384 199 / 204, (8192, 8192, 8192) 410 / 414; one round and a half (2048, 6144, 8192) 91 / 80.
//   128 x 128: MXFP4 four stages in LDS and one workgroup a CU, against two stages (2048, 2048, 8192) 23.9 / 27.8; INT4,
//     whose stages take twice as long, two and two workgroups, against four and one 30.6 / 33.0.
template <bool MX>
hipError_t launch_gemm(const GemmParams& p, hipStream_t stream) {
    auto tiles = [&](int64_t m, int64_t n) { return ((p.T + m - 1) / m) * (((int64_t)p.N + n - 1) / n); };
    if (p.d <= (MX ? 128 : 96)) return launch_short<MX>(p, stream);
    const int64_t small = tiles(32, 32), square = tiles(128, 128), wide = tiles(128, 256);
    const bool dwords = p.d % 128 == 0;                               // rows of scale bytes
    const bool one_row = p.T <= 32 && small <= (int64_t)1 << 22;      // (2^31 lanes; a grid takes less than 2^32)
    bool few = small <= 256;
    if (!MX) few = few || one_row || small <= 512 || (p.d >= 2048 && small <= (tiles(64, 64) > 256 ? 900 : 768));
    else if (!one_row) few = few || (small <= 512 && !dwords && p.d <= 8192);
    else if (!(dwords && small <= 384 && p.d >= 3072))
        few = few || p.T * p.d < (small >= 2048 ? (dwords ? 5 : 3) : (dwords ? 12 : 7)) << 14;
    if (few) return small > 512 && p.d < (!MX || dwords ? 4096 : 2560) ? launch_few<MX, 4>(p, stream) : launch_few<MX, 8>(p, stream);
    if (one_row || square <= 128) return launch_tile<MX, 1, 1, 2, 2, 4, 2>(p, stream);
    if constexpr (MX) {
        if (p.d < 1024 && !(p.d <= 512 && square > 256 && wide <= 256))
            return launch_tile_as<MX, 2, 2, 2, 2, 2, 2, false, true>(p, stream);
        auto eighths = [](int64_t n, int whole, int part) { return n / 256 * whole + (n % 256 != 0 ? part : 0); };
        if (eighths(wide, 14, 10) < eighths(square, 8, 6)) return launch_tile<MX, 2, 2, 2, 4, 2, 1>(p, stream);
        return launch_tile<MX, 2, 2, 2, 2, 4, 1>(p, stream);
    } else {
        const int64_t rounds = (wide + 255) / 256;
        if (square > 256 && (rounds == 1 ? p.T > 64 && p.d >= 9 * square : p.d >= 8192 && 16 * wide >= 15 * 256 * rounds))
            return launch_tile<MX, 2, 2, 2, 4, 2, 1>(p, stream);
        return launch_tile<MX, 2, 2, 2, 2, 2, 2>(p, stream);
    }
}

}  // namespace
}  // namespace perq

extern "C" perq_status_t perq_w4a4_mxfp4_gemm_ref(const uint8_t* a_codes, const uint8_t* a_scales, int64_t T,
                                                  const uint8_t* w_codes, const uint8_t* w_scales, int32_t N,
                                                  int32_t d, float* out, int64_t ldo, void* hip_stream) {
    if (T < 0 || N < 0 || d <= 0 || d % 32 != 0 || ldo < N) return PERQ_ERR_INVALID_ARG;
    if (d > PERQ_MAX_D) return PERQ_ERR_UNSUPPORTED;
    if (T == 0 || N == 0) return PERQ_OK;
    if (!a_codes || !a_scales || !w_codes || !w_scales || !out) return PERQ_ERR_INVALID_ARG;
    if (((reinterpret_cast<uintptr_t>(a_codes) | reinterpret_cast<uintptr_t>(w_codes)) & 15u) != 0 ||
        (reinterpret_cast<uintptr_t>(out) & 3u) != 0)
        return PERQ_ERR_UNSUPPORTED;
    if ((T + 31) / 32 > 65535) return PERQ_ERR_UNSUPPORTED;          // the documented reach
    const perq::GemmParams p = {a_codes, a_scales, w_codes, w_scales, out, T, ldo, N, d, 0, 0, 0};
    return perq::launch_gemm<true>(p, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? PERQ_OK : PERQ_ERR_LAUNCH;
}

extern "C" perq_status_t perq_w4a4_gemm_ref(const uint8_t* a_codes, const float* a_scales, int64_t T,
                                            const uint8_t* w_codes, const float* w_scales, int32_t N, int32_t d,
                                            float* out, int64_t ldo, void* hip_stream) {
    if (T < 0 || N < 0 || d <= 0 || d % 32 != 0 || ldo < N) return PERQ_ERR_INVALID_ARG;
    if (d > PERQ_MAX_D) return PERQ_ERR_UNSUPPORTED;
    if (T == 0 || N == 0) return PERQ_OK;
    if (!a_codes || !a_scales || !w_codes || !w_scales || !out) return PERQ_ERR_INVALID_ARG;
    if (((reinterpret_cast<uintptr_t>(a_codes) | reinterpret_cast<uintptr_t>(w_codes)) & 15u) != 0 ||
        ((reinterpret_cast<uintptr_t>(a_scales) | reinterpret_cast<uintptr_t>(w_scales) | reinterpret_cast<uintptr_t>(out)) & 3u) != 0)
        return PERQ_ERR_UNSUPPORTED;
    if ((T + 63) / 64 > 65535) return PERQ_ERR_UNSUPPORTED;          // the documented reach
    const perq::GemmParams p = {a_codes, a_scales, w_codes, w_scales, out, T, ldo, N, d, 0, 0, 0};
    return perq::launch_gemm<false>(p, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? PERQ_OK : PERQ_ERR_LAUNCH;
}
