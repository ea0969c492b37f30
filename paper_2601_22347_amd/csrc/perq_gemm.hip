// Consumers of the packed codes: out = A W^T for two operands in the layout the fused path writes,
// symmetric INT4 (one fp32 step per row) or MXFP4 (one e8m0 byte per 32 codes).
//
// Measured, T = 2048, N = d = 4096, INT4: 576 -> 30 - 32 us (2.2 POP/s; 8 codes per v_dot8_i32_i4 and no
// LDS before); T = N = 2048, d = 8192, MXFP4: 229 -> 32 - 34 us (2.1 PFLOP/s; one 32 x 32 tile per wave, both
// operands from memory for every product before).  The matrix unit alone would take 16 and 8 us.  Counters
// (profiles/products_w4a4.txt): INT4 keeps it 59 % busy and the vector ALU, which unpacks the nibbles, 61 %.  MXFP4
// keeps neither it (24 %) nor LDS (24 %) busy: a CU holds four waves of that tile, one a SIMD, and a wave issues
// its loads, its LDS reads and its products one after the other with nothing beside it.
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
// granule p ^ (r & 7) of the stage, so that the 32 rows a fragment read touches spread over all banks.
//   Four stages make a superstage of 32 granules.  MXFP4: in stage j half-wave h takes granules
// 16 h + 4 j + kc of the superstage, so that the scales of a lane's row for all four stages are 16
// consecutive bytes, one load; a load of a dword per row and stage took a third of the kernel's time
// (a load instruction that touches 32 rows occupies the address unit for as long as a product lasts).
template <bool MX, int MT, int NT, int WM, int WN, int NBUF, int WGS>
__global__ void __launch_bounds__(64 * WM * WN, WGS* WM* WN / 4)
gemm_tile_kernel(GemmParams p) {
    constexpr int kWaves = WM * WN, kBM = 32 * MT * WM, kBN = 32 * NT * WN;
    constexpr int kLoadA = kBM / 8 / kWaves, kLoadW = kBN / 8 / kWaves, kLoads = kLoadA + kLoadW;
    constexpr int kSc = MX ? MT + NT : 1;
    constexpr uint32_t kBuf = (uint32_t)(kBM + kBN) * kStageBytes;
    static_assert(kLoadA * 8 * kWaves == kBM && kLoadW * 8 * kWaves == kBN, "every wave loads whole pieces");
    static_assert(NBUF == 2 || NBUF == 4, "stage j of a superstage lies in buffer j % NBUF");
    extern __shared__ __align__(16) unsigned char lds[];
    float* const scales_lds = reinterpret_cast<float*>(lds + NBUF * kBuf);        // INT4: steps of the rows, then of the columns

    const int lane = threadIdx.x & 63, i = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t tt, tn;
    tile_of_block(p, tt, tn);
    const int64_t t0 = (int64_t)tt * kBM;
    const int32_t n0 = (int32_t)tn * kBN;
    const uint32_t row_bytes = (uint32_t)p.d >> 1, granules = row_bytes >> 4;
    const int whole = (int)(granules >> 5);                                         // whole superstages
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
    const uint32_t row8 = (uint32_t)lane >> 3, slot = ((uint32_t)lane & 7u) ^ row8;
    const uint32_t gran = MX ? 16u * (slot >> 2) + (slot & 3u) : slot;              // + 4 j (MXFP4) or 8 j in stage j
    constexpr uint32_t kPerStage = MX ? 4u : 8u;
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
        const uint32_t g = gran + kPerStage * j, top = S < whole ? 31u : (rest != 0u ? rest - 1u : 0u);
        const uint32_t more = 16u * ((g < top ? g : top) - gran) + 512u * (uint32_t)S;
        const uint32_t keep = S < whole || (S == whole && rest != 0u) ? 0xFFFFFFFFu : 0u;
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            unsigned char* to = lds + (j % NBUF) * kBuf + (uint32_t)((k < kLoadA ? k * kWaves : kBM / 8 + (k - kLoadA) * kWaves) + wave) * 1024u;
            if constexpr (inner) load_to_lds16(k < kLoadA ? abuf : wbuf, off[k], 512u * (uint32_t)S + 16u * kPerStage * j, to);
            else load_to_lds16(k < kLoadA ? abuf : wbuf, (off[k] + more) & keep, 0u, to);
        }
    };

    // ---- MXFP4: scale bytes of this lane's rows and columns, a superstage at a time -----------------
    const int wm = wave / WN, wn = wave % WN;
    const uint32_t nb = (uint32_t)p.d >> 5;
    const uint8_t* asc = static_cast<const uint8_t*>(p.a_scales) + (MX ? t0 * nb : 0);
    const uint8_t* wsc = static_cast<const uint8_t*>(p.w_scales) + (MX ? (int64_t)n0 * nb : 0);
    uint32_t soff[kSc];
    if constexpr (MX) {
#pragma unroll
        for (int m = 0; m < MT + NT; ++m) {
            const uint32_t r = (uint32_t)(m < MT ? (wm * MT + m) * 32 + i : (wn * NT + m - MT) * 32 + i);
            const uint32_t last = m < MT ? last_t : last_n;
            soff[m] = (r < last ? r : last) * nb;
        }
    }
    struct Scales { uint32_t w[kSc][4]; };
    // the four bytes of stage j of a partial superstage end with the row: where fewer are left, the
    // row's last four are loaded and shifted at use
    auto partial_at = [&](int j) { return 32u * (uint32_t)whole + 16u * (uint32_t)h + 4u * (uint32_t)j; };
    auto request_scales = [&](int S, Scales& to, auto inner_const) {
        if constexpr (MX) {
#pragma unroll
            for (int m = 0; m < MT + NT; ++m) {
                const uint8_t* from = (m < MT ? asc : wsc);
                const uint32_t at = 32u * (uint32_t)S + 16u * (uint32_t)h;
                if constexpr (decltype(inner_const)::value) {
                    __builtin_memcpy(to.w[m], from + (soff[m] + at), 16);
                } else {
#pragma unroll
                    for (uint32_t j = 0; j < 4; ++j)
                        __builtin_memcpy(&to.w[m][j], from + (soff[m] + (at + 4u * j < nb - 4u ? at + 4u * j : nb - 4u)), 4);
                }
            }
        }
    };

    acc_t<MX> acc[MT][NT] = {};
    // byte offset of this lane's fragment rows inside a buffer; place of its granule in the line in step kc
    const uint32_t fa = (uint32_t)((wm * MT) * 32 + i) * kStageBytes, fw = (uint32_t)(kBM + (wn * NT) * 32 + i) * kStageBytes;
    uint32_t place[4];
#pragma unroll
    for (int kc = 0; kc < 4; ++kc) place[kc] = ((uint32_t)(4 * h + kc) ^ ((uint32_t)lane & 7u)) * 16u;
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
    auto live = [&](int j, int kc) { return (MX ? 16u * (uint32_t)h + 4u * (uint32_t)j : 8u * (uint32_t)j + 4u * (uint32_t)h) + (uint32_t)kc < rest ? -1 : 0; };
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
    auto advance = [&](int S, auto j_const, auto inner_const, auto tail_const) {
        constexpr int j = decltype(j_const)::value;
        constexpr bool tail = decltype(tail_const)::value;
        // requested after the next stage's codes: those of NBUF - 2 stages (vmcnt: a six-bit count in bits 3:0
        // and 15:14).  Scales may have been requested among them and are not counted: those are loads like any
        // other, which the compiler takes out where nothing uses them, and a count of loads that are not there
        // lets the wait pass early.  A load into LDS stays where it was put.  (Counting them as well gains
        // 1.7 % at (2048, 4096, 4096) and nothing elsewhere.)
        constexpr int n = (NBUF - 2) * kLoads;
        static_assert(n < 64, "");
        __builtin_amdgcn_s_waitcnt(0x0F70 | (n & 15) | ((n >> 4) << 14));
        workgroup_barrier_lds();
        request_codes(S, std::integral_constant<int, j + NBUF>{}, inner_const);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (j == 0 && !tail) request_scales(S + 1, nxt, inner_const);
        __builtin_amdgcn_sched_barrier(0);
    };
    // One stage.  INT4: the codes of a step are read two steps ahead of its products and unpacked while
    // the products of the step before run, a few vector instructions to a product (a wave issues in
    // order).  MXFP4: they are read one step ahead.
    auto stage = [&](int S, auto j_const, auto inner_const, auto tail_const) {
        constexpr int j = decltype(j_const)::value;
        constexpr bool tail = decltype(tail_const)::value;
        if constexpr (MX) {
            uint32_t sw[kSc];
#pragma unroll
            for (int m = 0; m < kSc; ++m) {
                sw[m] = cur.w[m][j];
                if constexpr (tail) {
                    const uint32_t at = partial_at(j);
                    sw[m] >>= at > nb - 4u ? 8u * ((at - (nb - 4u)) & 3u) : 0u;
                }
            }
            auto step = [&](auto kc_const, Raw& now, Raw& next) {
                constexpr int kc = decltype(kc_const)::value;
                if constexpr (kc == 3) advance(S, j_const, inner_const, tail_const);
                read(j, kc + 1, next);
                __builtin_amdgcn_sched_barrier(0);
                multiply_mx(kc_const, now, sw, tail ? live(j, kc) : -1);
                __builtin_amdgcn_sched_barrier(0);
            };
            step(std::integral_constant<int, 0>{}, r0, r1);
            step(std::integral_constant<int, 1>{}, r1, r0);
            step(std::integral_constant<int, 2>{}, r0, r1);
            step(std::integral_constant<int, 3>{}, r1, r0);
        } else {
            auto step = [&](auto kc_const, const Ops& now, Ops& next, const Raw& raw_next, Raw& raw) {
                constexpr int kc = decltype(kc_const)::value;
                if constexpr (kc == 2) advance(S, j_const, inner_const, tail_const);
                read(j, kc + 2, raw);
                // (the step after the last one of a tail is never multiplied)
                unpack(raw_next, next, tail ? live(j + ((kc + 1) >> 2), (kc + 1) & 3) : -1);
                multiply_i8(now);
                __builtin_amdgcn_sched_group_barrier(0x100, MT + NT, 0);                      // the reads
#pragma unroll
                for (int q = 0; q < 2 * MT * NT; ++q) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                        // one product
                    __builtin_amdgcn_sched_group_barrier(0x002, (12 * (MT + NT) + 2 * MT * NT - 1) / (2 * MT * NT), 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            step(std::integral_constant<int, 0>{}, u0, u1, r1, r0);
            step(std::integral_constant<int, 1>{}, u1, u0, r0, r1);
            step(std::integral_constant<int, 2>{}, u0, u1, r1, r0);
            step(std::integral_constant<int, 3>{}, u1, u0, r0, r1);
        }
    };
    request_scales(0, cur, std::false_type{});
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
        __builtin_amdgcn_s_waitcnt(0x0F70 | (n & 15) | ((n >> 4) << 14));
        workgroup_barrier_lds();
        read(0, 0, r0);
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
        constexpr uint32_t kFrom = MX ? 4u : 8u;        // stage j holds something if rest > kFrom j
        stage(S, std::integral_constant<int, 0>{}, std::false_type{}, std::true_type{});
        if (rest > kFrom) stage(S, std::integral_constant<int, 1>{}, std::false_type{}, std::true_type{});
        if (rest > 2u * kFrom) stage(S, std::integral_constant<int, 2>{}, std::false_type{}, std::true_type{});
        if (rest > 3u * kFrom) stage(S, std::integral_constant<int, 3>{}, std::false_type{}, std::true_type{});
    }
    // no load may be on its way into LDS that another workgroup owns by then
    __builtin_amdgcn_s_waitcnt(0x0F70);

    auto store = [&](auto inner_const) {
        constexpr bool inner = decltype(inner_const)::value;
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
                        if (inner || (rt + 8 * q + k <= last_t && c <= last_n)) row[n * 32] = v;
                    }
                }
            }
        }
    };
    if (last_t + 1u == (uint32_t)kBM && last_n + 1u == (uint32_t)kBN) store(std::true_type{});
    else store(std::false_type{});
}

// ---- few rows: one 32 x 32 tile per workgroup, the contraction cut among its KW waves --------------
// Bound by the latency of the loads: nothing is used twice, so the granules go straight to registers,
// wave k takes the stages k, k + KW, ... and the partial tiles are added in LDS in wave order.  A stage's loads are
// all issued before its first product (left to itself the compiler puts some behind it: (64, 4096, 8000) INT4
// 10.4 -> 7.8 us, MXFP4 8.8 -> 8.1).
template <bool MX, int KW>
__global__ void __launch_bounds__(64 * KW)
gemm_skinny_kernel(GemmParams p) {
    __shared__ float part_f[KW][16][64];
    const int lane = threadIdx.x & 63, i = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t tt, tn;
    tile_of_block(p, tt, tn);
    const int64_t t0 = (int64_t)tt * 32, t = t0 + i < p.T ? t0 + i : p.T - 1;
    const int32_t n0 = (int32_t)tn * 32, n = n0 + i < p.N ? n0 + i : p.N - 1;
    const uint32_t row_bytes = (uint32_t)p.d >> 1, granules = row_bytes >> 4, nb = (uint32_t)p.d >> 5;
    const int stages = (int)((granules + 7u) >> 3);
    const uint8_t* ac = p.a_codes + t * row_bytes;
    const uint8_t* wc = p.w_codes + (int64_t)n * row_bytes;
    acc_t<MX> acc = {};
    for (int s = wave; s < stages; s += KW) {
        v4i_t a[4], w[4];
        uint32_t sa = 0, sw = 0;
        if constexpr (MX) {
            const uint8_t* as = static_cast<const uint8_t*>(p.a_scales) + t * nb;
            const uint8_t* ws = static_cast<const uint8_t*>(p.w_scales) + (int64_t)n * nb;
            uint32_t at = 8u * (uint32_t)s + 4u * (uint32_t)h;
            at = at < nb ? at : nb - 1u;
            sa = scale_dword(as, at, nb);
            sw = scale_dword(ws, at, nb);
        }
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) {
            const uint32_t g = 8u * (uint32_t)s + 4u * (uint32_t)h + kc, gc = g < granules ? g : granules - 1u;
            a[kc] = *reinterpret_cast<const v4i_t*>(ac + 16u * gc);
            w[kc] = *reinterpret_cast<const v4i_t*>(wc + 16u * gc);
            if (g >= granules) a[kc] = v4i_t{0, 0, 0, 0};
        }
        __builtin_amdgcn_sched_barrier(0);
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
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        if constexpr (MX) part_f[wave][j][lane] = acc[j];
        else part_f[wave][j][lane] = __int_as_float(acc[j]);
    }
    __syncthreads();
#pragma unroll
    for (int jj = 0; jj < 16 / KW; ++jj) {
        const int j = jj * KW + wave;
        acc_t<MX> sum = {};
#pragma unroll
        for (int k = 0; k < KW; ++k) {
            if constexpr (MX) sum[0] += part_f[k][j][lane];
            else sum[0] += __float_as_int(part_f[k][j][lane]);
        }
        const int64_t row = t0 + 8 * (j >> 2) + 4 * h + (j & 3);
        if (row < p.T && n0 + i < p.N) {
            float v;
            if constexpr (MX) v = sum[0];
            else v = (float)sum[0] * 0x1p-8f * static_cast<const float*>(p.a_scales)[row] * static_cast<const float*>(p.w_scales)[n0 + i];
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

template <bool MX, int MT, int NT, int WM, int WN, int NBUF, int WGS>
hipError_t launch_tile(GemmParams p, hipStream_t stream) {
    constexpr uint32_t lds_bytes = (uint32_t)(32 * MT * WM + 32 * NT * WN) * (kStageBytes * NBUF + (MX ? 0u : 4u));
    p.tiles_t = (uint32_t)((p.T + 32 * MT * WM - 1) / (32 * MT * WM));
    p.tiles_n = (uint32_t)(((int64_t)p.N + 32 * NT * WN - 1) / (32 * NT * WN));
    auto kern = gemm_tile_kernel<MX, MT, NT, WM, WN, NBUF, WGS>;
    int per_cu = 0;      // (raises the kernel's limit of dynamic LDS)
    const hipError_t e = resident_blocks(reinterpret_cast<const void*>(kern), 64 * WM * WN, lds_bytes, &per_cu);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(p.tiles_t * p.tiles_n), dim3(64 * WM * WN), lds_bytes, stream, p);
    return hipGetLastError();
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
hipError_t launch_skinny(GemmParams p, hipStream_t stream) {
    p.tiles_t = (uint32_t)((p.T + 31) / 32);
    p.tiles_n = (uint32_t)(((int64_t)p.N + 31) / 32);
    hipLaunchKernelGGL((gemm_skinny_kernel<MX, KW>), dim3(p.tiles_t * p.tiles_n), dim3(64 * KW), 0, stream, p);
    return hipGetLastError();
}

// Which kernel and tile.  Measured on both sides of every line, one GPU, launches back to back, INT4 / MXFP4
// us (T, N, d), the kernel that is taken first:
//   d < 128, MXFP4 also d = 128: no staging and no cut of the contraction, one wave per 32 x 32 tile.
//     (4096, 4096, 64) 14.7 / 12.2 against 19.1 / 15.6 with a trip of the tile through LDS, (16384, 512, 64)
//     9.3 / 7.5 against 12.4 / 10.6.  At d = 128 against the tiles below: (4096, 4096) 15.9 / 13.2 against 16.3 /
//     14.4, (16384, 512) 9.9 / 8.7 against 9.4 / 9.0, (300, 14336) 7.7 / 6.7 against 8.2 / 7.6.
//   up to 256 tiles of 32 x 32: the contraction cut among 8 waves, against 64 x 64 tiles.  256 tiles:
//     (64, 4096, 4096) 7.2 / 6.8 against 8.2 / 7.0, d = 6144 7.6 / 8.6 against 10.9 / 8.4, d = 8192 9.4 / 10.8 against
//     13.8 / 9.9 (MXFP4 has half the products per granule: not from d = 8192 on).  258 tiles: (96, 2752, 4096)
//     9.3 / 10.7 against 8.8 / 7.1.
//   up to 128 tiles of 128 x 128: 64 x 64 tiles, which two workgroups a CU hold at once up to there, against
//     128 x 128.  (512, 4096, 4096) 12.6 / 15.0 against 16.3 / 15.3, d = 1024 7.3 / 8.6 against 7.6 / 9.3; the other way
//     round with 130 tiles, (640, 3328, 4096) 16.5 / 15.5 against 17.9 / 20.7.
//   more than 256 tiles of 128 x 128: 128 x 256, a sixth less to load per product, for long rows, and only if the
//     rounds of 256 such tiles are full (or there is one: then a CU has two 128 x 128 tiles or one of these).
//     (4096, 4096): d = 2048 36.2 / 38.8 with 128 x 128 against 36.1 / 42.4, d = 2880 49.7 / 52.4 against 48.1 / 51.3,
//     d = 4096 61.0 / 61.5 against 57.0 / 62.5, d = 5120 72.7 / 76.1 against 68.1 / 73.0, d = 8192 110 / 110 against 102 / 103.
//     Rounds that are not full: (3000, 3500, 4096) 42.3 / 46.4 with 128 x 128 against 50.0 / 57.2, d = 8192 76.0 / 80.6
//     against 90.1 / 95.3; (2048, 14336, 4096), three and a half, 104 / 106 against 104 / 116.  One round: (2048, 4096,
//     4096) 29.9 / 33.0 against 29.8 / 33.0, (2177, 2177, 8192) 45.2 / 47.6 against 43.3 / 47.7.
//   MXFP4 with at most one 128 x 128 tile per CU: four stages in LDS instead of two and a second workgroup that
//     would not come, (2048, 2048, 4096) 19.5 against 20.6, (1280, 1664, 4096) 16.1 against 17.0, (1536, 1536, 1024) 9.6
//     against 9.5; INT4, whose stages take twice as long, is faster with two.
template <bool MX>
hipError_t launch_gemm(const GemmParams& p, hipStream_t stream) {
    auto tiles = [&](int64_t m, int64_t n) { return ((p.T + m - 1) / m) * (((int64_t)p.N + n - 1) / n); };
    if (p.d <= (MX ? 128 : 96)) return launch_short<MX>(p, stream);
    if (tiles(32, 32) <= 256 && !(MX && p.d >= 8192)) return launch_skinny<MX, 8>(p, stream);
    if (tiles(128, 128) <= 128) return launch_tile<MX, 1, 1, 2, 2, 4, 2>(p, stream);
    const int64_t wide = tiles(128, 256), rounds = (wide + 255) / 256;
    if (tiles(128, 128) > 256 && p.d >= (MX ? 5120 : 2880) && (rounds == 1 || 16 * wide >= 15 * 256 * rounds))
        return launch_tile<MX, 2, 2, 2, 4, 2, 1>(p, stream);
    if constexpr (MX) {
        if (tiles(128, 128) <= 256) return launch_tile<MX, 2, 2, 2, 2, 4, 1>(p, stream);
    }
    return launch_tile<MX, 2, 2, 2, 2, 2, 2>(p, stream);
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
    const perq::GemmParams p = {a_codes, a_scales, w_codes, w_scales, out, T, ldo, N, d, 0, 0};
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
    const perq::GemmParams p = {a_codes, a_scales, w_codes, w_scales, out, T, ldo, N, d, 0, 0};
    return perq::launch_gemm<false>(p, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? PERQ_OK : PERQ_ERR_LAUNCH;
}
