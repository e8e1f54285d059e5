// NHWC implicit-GEMM convolution with a 2:4-sparse (or, for the twin, dense) weight operand.
//
// Sec. 3.3: Y~ = (M (.) W) U(X) (Eq. 6).  The unfold U(X) (Eq. 5) is never materialised: every
// workgroup builds the [pixels x reduction-chunk] slice of it that it needs in LDS, straight from
// the NHWC activations, and multiplies it with weight tiles that are already stored in the
// register layout of the matrix instruction.
//
//   GEMM view:  D[o, p] = sum_k A[o, k] * B[k, p]
//     A = weights, rows o = output channels (the sparse operand of V_SMFMAC must be A),
//     B = unfolded activations, columns p = (n, ho, wo) flattened, k = reduction index in the
//         flattening the descriptor declares (blocks of 4 consecutive k form a 2:4 group).
//   One 32x32x32 sparse MFMA consumes, per lane l: 8 kept weights of row l%32 (+16 index bits)
//   and the 16 activations k = 16*(l/32) + [0,16) of pixel l%32; it leaves rows
//   8*(v/4) + 4*(l/32) + v%4, v = 0..15, of column l%32 in the lane's 16 accumulators, i.e. runs
//   of 4 consecutive output channels of one pixel.
//   The dense twin issues two 32x32x16 dense MFMAs on the same B registers instead.
//
// 8-bit operands (int8, FP8 E4M3) run through the same kernel: activations are staged as 2-byte units (pairs of
// channels), one 32x32x64 instruction then consumes the same 32 B of B and 16 B of A per lane as the 16-bit one
// and does twice the multiply-adds; sums are int32 (exact) or fp32, and the tail multiplies by a per-channel scale.
//
// All global reads of activations and weights are raw buffer loads: a lane whose element lies in
// the zero padding, past the last pixel or past the reduction length presents an offset beyond the
// buffer's size and the hardware returns 0 -- no branches, no selects.
//
// This header holds the kernel templates and their launch / tile-choice code.  It is included by one translation
// unit per (operand type, sparse | dense) pair, each of which instantiates its share (ss_conv_inst.h), so that the
// library's build runs in parallel.
#ifndef SS_CONV_KERNEL_H_
#define SS_CONV_KERNEL_H_
#include "ss_internal.h"
#include "ss_conv_params.h"
#include <atomic>
#include <type_traits>

namespace ss {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x16 __attribute__((ext_vector_type(16)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

// Accumulators of one 32x32 tile: fp32 for the floats (16-bit and FP8), int32 (exact) for 8-bit integers.
template <int DT> using Acc = typename std::conditional<DT == SS_I8, i32x16, f32x16>::type;
// Type of the 16-bit output (and of a residual): the operands' own, or binary16 for 8-bit operands.
template <int DT> constexpr int out_type() { return is_byte_type(DT) ? SS_F16 : DT; }

struct B32 {   // one lane's B fragment for a reduction step: 32 bytes (16 x 16-bit, or 32 x int8)
    u32x4 lo, hi;
};


// floor(n / d) by multiply + shift with the host-computed constants of fast_div_setup.
__device__ __forceinline__ int fast_div(int n, unsigned mul, unsigned sh)
{
    return (int)(((unsigned long long)(unsigned)n * mul) >> sh);
}

// The parameter block behind a launch's arguments (scalar arithmetic).  WINDOW: the window's size comes from the arguments, and not from KH x KW.
// SMALL: the few-pixel kernels' reading of m_mul and extra.
template <int DT, bool SPARSE, int KH, int KW, bool WINDOW, bool SMALL>
__device__ __forceinline__ ConvParams unpack_args(const ConvArgs &a)
{
    ConvParams p;
    p.x = a.x; p.a_vals = a.a_vals; p.bias = a.bias; p.y = a.y;
    p.residual = is_byte_type(DT) ? nullptr : static_cast<const uint16_t *>(a.tail);
    p.scale = is_byte_type(DT) ? static_cast<const float *>(a.tail) : nullptr;
    p.H = a.H; p.W = a.W; p.Cin = a.Cin; p.Cout = a.Cout; p.sh = a.sh; p.sw = a.sw; p.ph = a.ph; p.pw = a.pw;
    p.P = a.P; p.Ho = a.Ho; p.Wo = a.Wo;
    p.howo_mul = a.howo_mul; p.wo_mul = a.wo_mul;
    p.act = (int)(a.bits & 3u);
    p.howo_sh = a.bits >> 2 & 63u; p.wo_sh = a.bits >> 8 & 63u;
    (SMALL ? p.kw_mul : p.tm_mul) = a.m_mul;
    (SMALL ? p.kw_sh : p.tm_sh) = a.bits >> 14 & 63u;
    if constexpr (SMALL) { p.cin_mul = a.extra; p.cin_sh = a.bits >> 20 & 63u; }
    p.K = WINDOW ? a.window.K : a.Cin * KH * KW;
    p.kw = WINDOW ? a.window.kw : KW;
    p.nsplit = WINDOW || SMALL ? 1 : (int)a.extra;
    p.ws_part = WINDOW ? nullptr : a.ws_part;
    // The few-pixel kernels divide unsigned: signed, a division by a power of two is four scalar instructions instead of one, and these
    // stand before their first load.  (In the tiled kernels, which the same gives nothing to measure, a step count known to be positive
    // made the compiler unroll the 8-bit 2x2 loops until they spilled: 8.1 -> 12.1 us for an FP8 layer of 448 x 108 channels.)
    using Count = typename std::conditional<SMALL, unsigned, int>::type;
    p.Ks = (int)(((Count)p.K + 31) / 32);                 // (as tile_dims: K counts 2-byte units, for 8-bit operands an even number to the step)
    p.Kp = is_byte_type(DT) ? p.Ks : (int)(((Count)p.Ks + 1) / 2);
    p.Mt = (int)(((Count)p.Cout + 31) / 32);
    p.a_bytes = (unsigned)p.Mt * (unsigned)p.Ks * (SPARSE ? 1024u : 2048u);
    p.a_meta = reinterpret_cast<const uint32_t *>(p.a_vals + (SMALL ? (size_t)(SPARSE ? p.a_bytes : 0u) : (size_t)p.Mt * p.Ks * 1024));
    p.meta_bytes = SPARSE ? (unsigned)p.Mt * (unsigned)p.Kp * 256u : 4u;
    p.x_bytes = (unsigned)(fast_div(p.P, p.howo_mul, p.howo_sh) * p.H) * (unsigned)p.W * (unsigned)p.Cin * 2u;
    return p;
}

constexpr unsigned kOutOfRange = 0x80000000u;   // >= any buffer size used here: the load returns 0
constexpr int kRsrcFlags = 0x00020000;          // raw buffer, 32-bit data format (gfx9 family)

// The 8-bit instructions (32x32x64, integer and FP8 alike) pair slot s of A lane l (16 kept bytes, index field s of a full index
// word) with bytes 16*(l/32) + 4*((s%8)/2) + idx of the B lane of the same column in lane group s/8; B lane
// l holds the 32 reduction indices 32*(l/32) + [0,32) of pixel l%32.  Accumulators are laid out as above.
template <int DT>
__device__ __forceinline__ Acc<DT> mma_sparse(u32x4 a, const B32 &b, Acc<DT> c, uint32_t idx)
{
    if constexpr (DT == SS_I8)
        return __builtin_amdgcn_smfmac_i32_32x32x64_i8(__builtin_bit_cast(i32x4, a), __builtin_bit_cast(i32x8, b), c, (int)idx, 0, 0);
    else if constexpr (DT == SS_F8)
        return __builtin_amdgcn_smfmac_f32_32x32x64_fp8_fp8(__builtin_bit_cast(i32x4, a), __builtin_bit_cast(i32x8, b), c, (int)idx, 0, 0);
    else if constexpr (DT == SS_F16)
        return __builtin_amdgcn_smfmac_f32_32x32x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x16, b), c,
                                                         (int)idx, 0, 0);
    else
        return __builtin_amdgcn_smfmac_f32_32x32x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x16, b), c,
                                                          (int)idx, 0, 0);
}

// A 16-byte buffer store at a lane's offset plus a uniform one.  The sum is the lane's operand and not the instruction's scalar offset: without a scalar
// offset the compiler keeps the store's data registers unwritten for two wait states behind it, with one it takes none to be needed, and a vector
// instruction that followed at once has changed the stored words (a pixel's first dword was that instruction's result, now and then).
template <int POLICY = 0>
__device__ __forceinline__ void store_b128(const u32x4 &v, const __amdgpu_buffer_rsrc_t &r, int lane_off, int off)
{
    __builtin_amdgcn_raw_buffer_store_b128(v, r, lane_off + off, 0, POLICY);
}

// Workgroup barrier that orders LDS traffic only: the waves' outstanding global loads (weight ring, staging loads)
// and stores (output tile) stay in flight across it.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Which dense FP8 kernels use the 32x32x64 instruction (the others use pairs of 32x32x16, see mma_dense): the deep
// ones, which have the registers for its 8-register operands, and the short-chunk channels-last staging, whose shallow
// kernels are otherwise bound by the half-rate instruction (measured: 81 vs 69 us on the N=500 benchmark layer).
constexpr bool f8_wide(bool deep, int mode) { return deep || mode == 0 /* MODE_VEC */; }

// Dense FP8: one 32x32x64 instruction of the scaled-format family with both formats E4M3 and both block scales
// 2^0 (exponent byte 127); A and B slots s of lane l are k = 32*(l/32) + s.
__device__ __forceinline__ f32x16 mma_dense_f8(u32x4 a0, u32x4 a1, const B32 &b, f32x16 c)
{
    const i32x8 a = __builtin_shufflevector(__builtin_bit_cast(i32x4, a0), __builtin_bit_cast(i32x4, a1), 0, 1, 2, 3, 4, 5, 6, 7);
    const i32x8 bb = __builtin_shufflevector(__builtin_bit_cast(i32x4, b.lo), __builtin_bit_cast(i32x4, b.hi), 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, bb, c, 0, 0, 0, 0x7F7F7F7F, 0, 0x7F7F7F7F);
}

template <int DT>
__device__ __forceinline__ Acc<DT> mma_dense(u32x4 a, u32x4 b, Acc<DT> c)
{
    if constexpr (DT == SS_I8)      // 32x32x32: A lane l slot s <-> k = 16*(l/32) + s, B likewise
        return __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(i32x4, a), __builtin_bit_cast(i32x4, b), c, 0, 0, 0);
    else if constexpr (DT == SS_F8) {
        // Two 32x32x16 FP8 instructions on the low and high 8 bytes (A and B share the lane -> reduction-index map,
        // and the weight tile was laid out for these very bytes of B).  Half the rate of the 32x32x64 form, but its
        // operands are register pairs: used by the shallow kernels, which need the occupancy more than the rate.
        const unsigned long long a0 = a[0] | ((unsigned long long)a[1] << 32), a1 = a[2] | ((unsigned long long)a[3] << 32);
        const unsigned long long b0 = b[0] | ((unsigned long long)b[1] << 32), b1 = b[2] | ((unsigned long long)b[3] << 32);
        c = __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8((long)a0, (long)b0, c, 0, 0, 0);
        return __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8((long)a1, (long)b1, c, 0, 0, 0);
    } else if constexpr (DT == SS_F16)
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Two fp32 values to one dword of 16-bit floats, round to nearest even, in one instruction (V_CVT_PK_F16_F32 /
// V_CVT_PK_BF16_F32).
template <int DT>
__device__ __forceinline__ uint32_t cvt_pack2(float a, float b)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const f32x2 v = {a, b};
    if constexpr (DT == SS_F16)
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2));
    else
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// max(v, floor) that hands a NaN through (the IEEE 754-2019 maximum, one V_MAXIMUM3_F32): ReLU with floor = 0, the
// identity with floor = -inf.  (A sum of exactly -0 comes out as +0.)
__device__ __forceinline__ float floor_at(float v, float floor)
{
    return __builtin_elementwise_maximum(v, floor);
}

// Exact value of a 16-bit pattern as fp32.
template <int DT>
__device__ __forceinline__ float widen(uint16_t bits)
{
    if constexpr (DT == SS_F16)
        return (float)__builtin_bit_cast(_Float16, bits);
    else
        return __builtin_bit_cast(float, (uint32_t)bits << 16);
}

// GELU z * Phi(z) with the exact standard normal CDF.  With a = |z| and h = Phi(-a):
//     z >= 0:  z (1 - h) = z - a h        z < 0:  z h = -a h        i.e.  gelu(z) = max(z, 0) - a h,
// which needs no select.  log2 Phi(-a) is smooth and close to a parabola: a polynomial and one exp2.  Two fits, each as long as
// the values of its output type ODT ask for (a negative leading coefficient takes either to 0 behind its range):
//   binary16   a h rounds to 0 from a = 5.5 on: degree 8, fitted on [0, 6].  Ten full-rate instructions and one half-rate one
//              (48 clocks per wave: measured, a fused multiply-add takes 4 and exp2 8).
//   bfloat16   holds the whole lower tail: degree 10, fitted on [0, 12.95], where Phi reaches 2^-126, the least value exp2 gives
//              (56 clocks).
// Fitted for the smallest largest error of Phi (|error| < 1e-7 in fp32 arithmetic), and in the tail for relative errors: 6e-7 at
// a = 1, 2e-5 at 3, 3e-4 at 5; from there degree 8 loses the tail (6e-3 at 6.3, 8e-2 at 7, nothing is left at 10), degree 10 has
// 1e-3 at 6, 3e-3 at 8, 2.3e-2 at 10 and 3.5e-2 at 12.9.  The rational form 7.1.26 of Abramowitz & Stegun takes twelve and two
// instructions for 2e-7 absolute and 9e-4 at 4, 5e-3 at 6, 1.2e-2 at 8, 2.2e-2 at 10, 3.6e-2 at 12.5.  (A NaN stays a NaN.)
template <int ODT>
__device__ __forceinline__ float gelu_cdf(float z)
{
    const float a = fabsf(z);
    float q;
    if constexpr (ODT == SS_F16) {
        q = -8.120558493747162e-07f;
        q = __builtin_fmaf(q, a, 1.4290432782061204e-05f);
        q = __builtin_fmaf(q, a, -6.487764435589362e-05f);
        q = __builtin_fmaf(q, a, -0.0004287622419436152f);
        q = __builtin_fmaf(q, a, 0.007434012361791795f);
        q = __builtin_fmaf(q, a, -0.05273924310954606f);
        q = __builtin_fmaf(q, a, -0.4591337784121185f);
        q = __builtin_fmaf(q, a, -1.1511134917708818f);
        q = __builtin_fmaf(q, a, -0.9999998474115108f);
    } else {
        q = -3.325034692025497e-09f;
        q = __builtin_fmaf(q, a, 1.58049019205464e-07f);
        q = __builtin_fmaf(q, a, -3.0015255561011145e-06f);
        q = __builtin_fmaf(q, a, 2.81424345303094e-05f);
        q = __builtin_fmaf(q, a, -0.00011069921310991049f);
        q = __builtin_fmaf(q, a, -0.00034601808874867857f);
        q = __builtin_fmaf(q, a, 0.007352784276008606f);
        q = __builtin_fmaf(q, a, -0.052697665989398956f);
        q = __builtin_fmaf(q, a, -0.45914411544799805f);
        q = __builtin_fmaf(q, a, -1.1511123180389404f);
        q = __builtin_fmaf(q, a, -0.9999998807907104f);
    }
    // (the IEEE 754-2019 maximum: fmaxf takes a second instruction, which quiets a signalling NaN first)
    return __builtin_fmaf(-a, __builtin_amdgcn_exp2f(q), floor_at(z, 0.f));
}

// How the [pixels x reduction-chunk] slice of the unfolded input is built in LDS:
//   MODE_VEC    channels are contiguous inside every aligned run of 8 reduction indices (1x1
//               kernels, or the channels-last flattening, with cin % 8 == 0): 16-byte loads,
//               chunks of 64 reduction indices.
//   MODE_VEC8   the same with chunks of 256 reduction indices, for long reductions: a quarter of the barriers.
//   MODE_PW     MODE_VEC specialised for 1x1 kernels: a pixel's offset is fixed for the whole
//               reduction and the chunk's channel offset travels in the load's scalar offset.
//               Chunks of 128 reduction indices (MODE_PW) or 64 (MODE_PW2, for very short reductions).
//   MODE_GATHER any flattening / shape: one 16-bit load per element (slow, general fallback).
//   MODE_GATHER4 channels-last flattening with cin % 4 == 0 (e.g. an image padded from 3 to 4 channels, the
//               column-wise augmentation Sec. 3.3 suggests for reductions that are no multiple of 4): every
//               aligned run of 4 reduction indices is 8 contiguous, 8-byte aligned bytes of one pixel: one 8-byte
//               load per 2:4 block.
//   MODE_TAPS   the paper's flattening (channel slowest) with a KH x KW kernel and cin % 32 == 0:
//               a 2:4 block then holds 4 consecutive (channel, tap) pairs, i.e. activations of
//               different pixels.  A thread loads, for one output pixel and 8 channels, the
//               KH*KW taps as 16-byte channel vectors and transposes them in registers to
//               channel-major order before the LDS write, so the MFMA side still reads 16-byte
//               vectors.  A chunk is 32 channels = KH*KW reduction steps.  (8-bit operands: 16 channels per
//               vector, a byte transpose, chunks of 64 channels.)
//   MODE_TAPSR, MODE_PWR   MODE_TAPS and MODE_PW for channel counts that are multiples of 4 only: the last chunk's channel
//               octets past the end are out of range; an octet that straddles it (cin % 8 == 4) is loaded 8 bytes early, so that
//               no load reaches past its pixel, and moved into place on its way to LDS (cin >= 8).  (Modes of their own: the checks cost the plain
//               ones registers.  Against MODE_GATHER, which these shapes took before: 3x3 80 -> 136 on 6 x 45 x 61 pixels
//               51.4 -> 12.3 us; 212 -> 132 on 24 x 16 x 27: 60 -> 17 us.)
enum { MODE_VEC = 0, MODE_GATHER = 1, MODE_TAPS = 2, MODE_PW = 3, MODE_PW2 = 4, MODE_VEC8 = 5, MODE_GATHER4 = 6, MODE_TAPSR = 7, MODE_PWR = 8 };
constexpr bool is_vec(int mode) { return mode == MODE_VEC || mode == MODE_VEC8; }
constexpr bool is_taps(int mode) { return mode == MODE_TAPS || mode == MODE_TAPSR; }
constexpr bool is_pw(int mode) { return mode == MODE_PW || mode == MODE_PW2 || mode == MODE_PWR; }

// One 16-byte vector v of a tap-transposed unit: [tap][8 channels] -> [channel][tap] (8-bit operands: 16 channels), see MODE_TAPS.
template <bool Q8, bool RAG, int TAPS>
__device__ __forceinline__ u32x4 taps_vector(const u32x4 (&t)[TAPS], int v, bool half)
{
    u32x4 w;
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const int d = 4 * v + q;
        if constexpr (Q8) {
            uint32_t src[4], pick[4];
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const int h = 4 * d + e, c = h / TAPS, tp = h % TAPS;
                src[e] = t[tp][c >> 2];
                pick[e] = (uint32_t)(c & 3);
            }
            const uint32_t p01 = __builtin_amdgcn_perm(src[1], src[0], pick[0] | ((4u + pick[1]) << 8));
            const uint32_t p23 = __builtin_amdgcn_perm(src[3], src[2], pick[2] | ((4u + pick[3]) << 8));
            w[q] = __builtin_amdgcn_perm(p23, p01, 0x05040100u);
        } else {
            const int ha = 2 * d, hb = 2 * d + 1;
            const int ca = ha / TAPS, ta = ha % TAPS, cb = hb / TAPS, tb = hb % TAPS;
            uint32_t sa = t[ta][ca >> 1], sb = t[tb][cb >> 1];
            if constexpr (RAG) {
                sa = half ? (ca >= 4 ? 0u : t[ta][2 + (ca >> 1 & 1)]) : sa;
                sb = half ? (cb >= 4 ? 0u : t[tb][2 + (cb >> 1 & 1)]) : sb;
            }
            const uint32_t sel = (uint32_t)(2 * (ca & 1)) | ((uint32_t)(2 * (ca & 1) + 1) << 8) |
                                 ((uint32_t)(4 + 2 * (cb & 1)) << 16) | ((uint32_t)(5 + 2 * (cb & 1)) << 24);
            w[q] = __builtin_amdgcn_perm(sb, sa, sel);
        }
    }
    return w;
}

// Weight fragments of one 32-wide reduction step for the TM row tiles of a wave.
template <bool SPARSE, int TM>
struct AStep {
    u32x4 v[SPARSE ? 1 : 2][TM];
    uint32_t idx[TM];
};

template <int MODE, int KH, int KW, bool DEEP>
struct ChunkShape {
    static constexpr int TAPS = KH * KW;
    static constexpr int KSTEPS = is_taps(MODE) ? TAPS : (MODE == MODE_VEC8 ? 8 : (MODE == MODE_PW || MODE == MODE_PWR ? 4 : 2));   // 32-wide reduction steps per LDS chunk
    static constexpr int BK = KSTEPS * 32;
    // Bank-conflict-free layout of a pixel row in LDS.  Default: +16 bytes per row, so that the 16-byte fragment reads
    // of consecutive pixels hit distinct banks.  The 3x3 tap-transposing mode writes 16-byte vectors at a stride of 9
    // vectors (one 8-channel unit) from four threads per pixel, which collides with any such padding; there the row
    // is left unpadded (36 vectors) and the index of a 16-byte vector inside its row is XOR-ed with bits 2..3 of the
    // pixel row (SWZ): the vector stays inside its aligned group of four, and both the transposed writes (4 pixel
    // rows x 4 units per 16 lanes) and the fragment reads (16 consecutive pixel rows) cover all 64 banks exactly once.
    // Only in the deep variants: the swizzled addresses cost the shallow 128 x 64 kernel eight registers, which is the
    // step from four to three waves per SIMD (its fused form ran 35 -> 49 us with it); the deep variants run at one to
    // three waves per SIMD anyway.
    static constexpr bool SWZ = is_taps(MODE) && TAPS == 9 && DEEP;
    static constexpr int ROW = SWZ ? BK : BK + 8;
    // LDS copies of the chunk: double-buffered, so that the next chunk is written while this one is
    // multiplied -- except for the large unfolded 3x3 chunk in the shallow variant, which is kept once
    // (more workgroups per compute unit then hide the store phase instead).
    static constexpr int NBUF = (is_taps(MODE) && TAPS > 4 && !DEEP) ? 1 : 2;
};

constexpr int ring_size(int ksteps, int regs_per_step, int budget)
{
    int depth = budget / regs_per_step + 1;
    if (depth > 12) depth = 12;
    if (depth < 2) depth = 2;
    int best = 1;
    for (int r = 2; r <= depth; r++)
        if (ksteps % r == 0 || r % ksteps == 0) best = r;
    if (best >= 2) return best;
    for (int r = depth + 1;; r++)                    // nothing that shallow nests with the chunk: take the next that does
        if (ksteps % r == 0 || r % ksteps == 0) return r;
}

// LDS of a workgroup: the staging buffers, reused by the epilogue for the output tile (16-bit, or fp32 when a
// residual is added after it), followed by the tile's bias values (fp32).
// Fused second contraction: every wave owns a staging region of 32 pixels x (32 + 4) floats behind the 16-bit tile.
constexpr size_t kFuseRegion = 32 * kFuseRow * 4;

// Third contraction: 128 channels of the second one's finished output, [pixel][channel].
constexpr int kThirdRow = 128 + 8;

template <int BM, int BN, int MODE, int KH, int KW, bool DEEP>
constexpr size_t smem_body(bool with_residual, int fuse_waves = 0, bool third = false)
{
    using CS = ChunkShape<MODE, KH, KW, DEEP>;
    size_t stage = (size_t)CS::NBUF * BN * CS::ROW * 2;
    size_t epi = with_residual ? (size_t)BN * (BM + 4) * 4 : (size_t)BN * (BM * 2 + 8) + (size_t)fuse_waves * kFuseRegion + (third ? (size_t)BN * kThirdRow * 2 : 0);
    return stage > epi ? stage : epi;
}
template <int BM, int BN, int MODE, int KH, int KW, bool DEEP>
constexpr size_t smem_bytes(bool with_residual, int fuse_waves = 0, bool third = false)
{
    // (behind the body: the first layer's bias, later the third's, up to 128 channels)
    return smem_body<BM, BN, MODE, KH, KW, DEEP>(with_residual, fuse_waves, third) + (size_t)(third && BM < 128 ? 128 : BM) * 4;
}

// Waves per SIMD the register allocator must leave room for: small wave tiles are latency-bound
// and profit from 4 resident waves (128 VGPRs each); large ones need the registers.
constexpr int min_waves_per_simd(int tm, int tn, bool big_stage)
{
    return tm * tn <= 2 ? (big_stage ? 3 : 4) : (tm * tn <= 4 ? 2 : 1);   // the 3x3 transpose needs ~134 VGPRs: 4 waves would spill
}

// DEEP: for grids of at most about one workgroup per compute unit, where no other wave hides
// latency: weight fragments are prefetched 8+ steps ahead and activation fragments 3 steps ahead
// (instead of 1), at the price of registers, i.e. of the occupancy such a grid cannot use anyway.
// SPEC: four extra waves do nothing but build the activation chunks in LDS (loads two chunks ahead,
// transposes, LDS writes); the WAVES_M x WAVES_N waves only fetch weights, read LDS and multiply.
// A wave issues in order, so without this split every wait of the staging code also stalls the
// wave's matrix instructions.
// FUSE: the tile (all output channels of this convolution for BN pixels, bias and activation applied, rounded to
// 16 bit exactly as it would be stored) stays in LDS and is at once the activation operand of a following 1x1
// convolution, whose output (+ bias + residual, activation) is what the kernel writes: the 3x3 -> 1x1 expansion of a
// bottleneck without the intermediate tensor's round trip through memory.
// THIRD: that output is in turn the operand of one more 1x1 convolution, the channel reduction that opens the next bottleneck, which then
// does not read it back from memory (the number of 32 x 32 tiles of its output per wave; 0: there is none).
constexpr bool short_args(int mode, bool fuse) { return !fuse && mode != MODE_GATHER && mode != MODE_GATHER4; }      // (the others need more than ConvArgs holds)

template <int THIRD>
using kernel_params = typename std::conditional<(THIRD > 0), ChainParams, ConvParams>::type;

template <int DT, bool SPARSE, int WAVES_M, int WAVES_N, int TM, int TN, int MODE, int KH, int KW, bool DEEP, bool SPEC, bool FUSE = false, int THIRD = 0>
__global__ __launch_bounds__((WAVES_M * WAVES_N + (SPEC ? 4 : 0)) * 64)
__attribute__((amdgpu_waves_per_eu(DEEP ? 1 : (((DT == SS_F8 || FUSE) && !SPARSE && MODE == MODE_VEC && TM * TN == 2) ? 3 : min_waves_per_simd(TM, TN, is_taps(MODE) || MODE == MODE_VEC8)))))
void conv_kernel(typename std::conditional<short_args(MODE, FUSE), ConvArgs, kernel_params<THIRD>>::type args)
{
    kernel_params<THIRD> p;
    if constexpr (short_args(MODE, FUSE)) p = unpack_args<DT, SPARSE, KH, KW, is_vec(MODE), false>(args);
    else p = args;
    using CS = ChunkShape<MODE, KH, KW, DEEP>;
    static_assert(!SPEC || DEEP, "producer waves come with the deep variant only");
    constexpr bool Q8 = is_byte_type(DT);                 // 8-bit operands: staged as byte pairs, full index words, scaled tail
    constexpr int ODT = out_type<DT>();
    static_assert(!Q8 || (MODE != MODE_GATHER && MODE != MODE_GATHER4), "8-bit operands travel in 16-byte runs only");
    constexpr int NMATH = WAVES_M * WAVES_N * 64;         // threads that multiply
    constexpr int NT = NMATH + (SPEC ? 256 : 0);
    constexpr int BM = WAVES_M * TM * 32;
    constexpr int BN = WAVES_N * TN * 32;
    constexpr int TAPS = CS::TAPS;
    constexpr int KSTEPS = CS::KSTEPS;
    // Weight fragments are prefetched RING-1 reduction steps ahead into a register ring, as deep as
    // about 24 (48 when DEEP) VGPRs allow (deeper rings cost occupancy, which the bandwidth-bound layers need more); RING divides the chunk or is a multiple of it (then the chunk loop is
    // unrolled RING/KSTEPS times so that every ring slot is a compile-time register).
    constexpr int RING = ring_size(KSTEPS, TM * (SPARSE ? 5 : 8), SPEC ? 96 : (DEEP ? 48 : 24));
    constexpr int BD = DEEP ? 4 : 2;                      // activation-fragment ring depth
    constexpr int PF = RING - 1;
    constexpr int UNROLL = RING > KSTEPS ? RING / KSTEPS : 1;
    static_assert(KSTEPS % RING == 0 || RING % KSTEPS == 0, "ring and chunk must nest");
    constexpr int BK = CS::BK;
    constexpr int ROW = CS::ROW;
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    uint16_t *Bs0 = smem;
    constexpr int NBUF = CS::NBUF;
    uint16_t *Bs1 = smem + (NBUF - 1) * BN * ROW;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool producer = SPEC && wave >= NMATH / 64;     // wave-uniform
    const int wm = wave % WAVES_M;               // (producer waves: unused)
    const int wn = (wave / WAVES_M) % WAVES_N;
    // Workgroups are handed to the 8 XCDs round-robin, and each XCD has its own L2.  Renumber them so
    // that an XCD works on a contiguous run of tiles: both row tiles of a pixel tile, and pixel tiles
    // that share halo rows, then hit the same L2.
    constexpr bool CAN_SPLIT = !FUSE && !is_byte_type(DT) && !is_vec(MODE);
    const int nsplit = CAN_SPLIT ? p.nsplit : 1;
    const int tiles_m = (p.Cout + BM - 1) / BM;
    const int nb = tiles_m * ((p.P + BN - 1) / BN) * nsplit;      // (the grid; asking for its size would lengthen the launch's arguments)
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int lidx = xcd * (nb >> 3) + min(xcd, nb & 7) + slot;
    // Split reduction (p.nsplit > 1): nsplit workgroups share an output tile and each takes a contiguous share of the
    // reduction chunks; their fp32 partial sums meet in the workspace (see the epilogue).
    // (split-major numbering: neighbouring workgroups, which land on the same XCD, work on neighbouring tiles with the
    // same share of the reduction and so share that share's weights in their L2)
    // (A branch around all the divisions by runtime numbers: each is some 25 instructions ahead of the first load, and in a grid one tile
    // deep nothing hides them.  1x1 1024 -> 256 at batch 64: 10.30 -> 10.08 us, 400 layers drawn at random 0.984 of the time.)
    int ntiles = nb, split = 0, lid = lidx, c_first = 0;               // this workgroup's chunks: [c_first, c_first + nchunks)
    int nchunks = (p.Ks + KSTEPS - 1) / KSTEPS;
    if (nsplit > 1) {                                                  // uniform
        ntiles = nb / nsplit;
        split = lidx / ntiles;
        lid = lidx - split * ntiles;
        c_first = split * nchunks / nsplit;
        nchunks = (split + 1) * nchunks / nsplit - c_first;
    }
    const int tile_n = fast_div(lid, p.tm_mul, p.tm_sh);
    const int tile_m = lid - tile_n * tiles_m;
    const int m0 = tile_m * BM;
    const int n0 = tile_n * BN;
    const int HoWo = p.Ho * p.Wo;

    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(p.x), 0, (int)p.x_bytes, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(p.a_vals), 0, (int)p.a_bytes, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(p.a_meta), 0, (int)p.meta_bytes, kRsrcFlags);

    // The tile's bias values are fetched now and parked in LDS after the first staging store, so the
    // epilogue does not pay a global-memory round trip.
    static_assert(!FUSE || !Q8, "the fused second contraction is built for the 16-bit types");
    const bool with_res = !Q8 && !FUSE && p.residual != nullptr;     // uniform (fused: the residual belongs to the second layer)
    float *bias_s = reinterpret_cast<float *>(reinterpret_cast<char *>(smem) +
                                              (with_res ? smem_body<BM, BN, MODE, KH, KW, DEEP>(true)
                                                        : smem_body<BM, BN, MODE, KH, KW, DEEP>(false, FUSE ? NT / 64 : 0, THIRD > 0)));
    // (Loaded after the first activation / weight loads are on their way: issued first, its latency would
    // sit in front of everything else.)
    float *scale_s = bias_s + BM;                     // (8-bit operands only)
    float bias_r[(BM + NMATH - 1) / NMATH], scale_r[Q8 ? (BM + NMATH - 1) / NMATH : 1];
    auto load_bias = [&]() {
#pragma unroll
        for (int j = 0; j < (BM + NMATH - 1) / NMATH; j++) {
            const int o = m0 + tid + j * NMATH;
            const bool in = tid + j * NMATH < BM && o < p.Cout;
            bias_r[j] = (p.bias != nullptr && in) ? p.bias[o] : 0.f;
            if constexpr (Q8) scale_r[j] = (p.scale != nullptr && in) ? p.scale[o] : 1.f;
        }
    };

    // ------------------------------------------------------------------ activation staging state
    // per pixel row and chunk: 16-byte runs (VEC: 8, TAPS: 4 channel octets) or 4-element blocks (GATHER: 16)
    constexpr int UNITS = (MODE == MODE_GATHER || MODE == MODE_GATHER4) ? 16 : (is_taps(MODE) ? 4 : (MODE == MODE_VEC8 ? 32 : (MODE == MODE_PW || MODE == MODE_PWR ? 16 : 8)));
    // staging threads (whole waves); the rest only multiply
    constexpr int ST = SPEC ? 256 : (BN * UNITS % NT == 0 ? NT : (NT > 256 ? 256 : 128));
    constexpr int ITEMS = BN * UNITS / ST;
    constexpr int NSET = SPEC ? 2 : 1;                    // producer waves hold two chunks in registers
    static_assert(BN * UNITS % ST == 0 && ST % UNITS == 0 && ST % 64 == 0 && ITEMS >= 1, "tile/threads mismatch");
    const int stid = SPEC ? tid - NMATH : tid;            // index among the staging threads
    static_assert(!SPEC || ST == 256, "every producer thread stages");
    const bool stager = SPEC || ST == NT || wave < ST / 64;     // uniform (producer waves: only they call the staging code)
    // Thread -> (pixel row, unit): unit fastest, so consecutive lanes read consecutive 16-byte pieces of one
    // pixel (coalesced).  (Putting 16 pixel rows of one unit on consecutive lanes makes the transposed LDS
    // writes conflict-free but quadruples the cache lines per load instruction: measured 30-40 % slower.)
    const int unit = (stid & 0xFFFF) % UNITS;
    const int pr0 = ((stid & 0xFFFF) % ST) / UNITS;
    unsigned pixbyte[ITEMS];          // byte offset of x[n, ho*sh-ph, wo*sw-pw, 0] (wraps below 0 for padded pixels)
    int ih0[ITEMS], iw0[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; i++) {
        int pr = pr0 + i * (ST / UNITS);
        int pg = n0 + pr;
        if (pg < p.P) {
            int n = fast_div(pg, p.howo_mul, p.howo_sh);
            int rem = pg - n * HoWo;
            int ho = fast_div(rem, p.wo_mul, p.wo_sh);
            int wo = rem - ho * p.Wo;
            ih0[i] = ho * p.sh - p.ph;
            iw0[i] = wo * p.sw - p.pw;
            pixbyte[i] = (unsigned)(((n * p.H + ih0[i]) * p.W + iw0[i]) * p.Cin * 2);
        } else {
            ih0[i] = -(1 << 28);     // every bounds test fails -> zeros
            iw0[i] = -(1 << 28);
            pixbyte[i] = 0;
        }
    }

    // MODE_VEC: position of this thread's 8-element run in the (tap, channel) space, from the first chunk on (these modes never split the reduction)
    int vk = unit * 8, vc = 0, vr = 0, vt = 0;
    if constexpr (is_vec(MODE)) {
        vc = vk;
        if (p.Cin < UNITS * 8) {                          // uniform: else the first chunk lies in the first tap
            int tap = vk / p.Cin;
            vc = vk - tap * p.Cin;
            vr = tap / p.kw;
            vt = tap - vr * p.kw;
        }
    }
    // MODE_TAPS: per (pixel, tap) byte offsets, fixed for the whole reduction; the chunk's channel
    // offset travels in the scalar offset of the load.  Out-of-image taps are out of range for good.
    unsigned tapoff[is_taps(MODE) ? ITEMS : 1][is_taps(MODE) ? TAPS : 1];
    if constexpr (is_taps(MODE)) {
#pragma unroll
        for (int i = 0; i < ITEMS; i++)
#pragma unroll
            for (int tap = 0; tap < TAPS; tap++) {
                const int r = tap / KW, t = tap % KW;
                int ih = ih0[i] + r, iw = iw0[i] + t;
                bool ok = (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;
                tapoff[i][tap] = ok ? pixbyte[i] + (unsigned)(((r * p.W + t) * p.Cin + unit * 8) * 2) : kOutOfRange;
            }
    }

    // MODE_PW: per pixel byte offset of this thread's 16-byte run in the first chunk (out of range for pixels
    // past the end or in the padding)
    unsigned pwoff[is_pw(MODE) ? ITEMS : 1];
    if constexpr (is_pw(MODE)) {
#pragma unroll
        for (int i = 0; i < ITEMS; i++) {
            bool ok = (unsigned)ih0[i] < (unsigned)p.H && (unsigned)iw0[i] < (unsigned)p.W;
            pwoff[i] = ok ? pixbyte[i] + (unsigned)(unit * 16) : kOutOfRange;
        }
    }

    u32x4 stage_v_[NSET][(is_vec(MODE) || is_pw(MODE)) ? ITEMS : 1];
    uint16_t stage_g_[NSET][MODE == MODE_GATHER ? ITEMS : 1][4];
    uint2 stage_g4_[NSET][MODE == MODE_GATHER4 ? ITEMS : 1];
    u32x4 stage_t_[NSET][is_taps(MODE) ? ITEMS : 1][is_taps(MODE) ? TAPS : 1];
    bool half_[NSET];                 // MODE_TAPSR / MODE_PWR: the octet straddles the last channel and was loaded 8 bytes early

    auto stage_load = [&](int ci_rel, int set = 0) {      // set: compile time at every call site; chunk relative to c_first
        if (!stager) return;
        const int ci = ci_rel + c_first;
        auto &stage_v = stage_v_[set];
        auto &stage_g = stage_g_[set];
        auto &stage_t = stage_t_[set];
        if constexpr (is_vec(MODE)) {
            const unsigned koff = vk < p.K ? (unsigned)(((vr * p.W + vt) * p.Cin + vc) * 2) : kOutOfRange;
#pragma unroll
            for (int i = 0; i < ITEMS; i++) {
                int ih = ih0[i] + vr, iw = iw0[i] + vt;
                bool ok = (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W && koff != kOutOfRange;
                unsigned off = ok ? pixbyte[i] + koff : kOutOfRange;
                stage_v[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)off, 0, 0);
            }
            vk += BK;
            vc += BK;
            while (vc >= p.Cin) {
                vc -= p.Cin;
                if (++vt == p.kw) { vt = 0; ++vr; }
            }
        } else if constexpr (is_pw(MODE)) {
            int early = 0;
            if constexpr (MODE == MODE_PWR) {
                half_[set] = ci * BK + unit * 8 + 4 == p.K;
                early = half_[set] ? 8 : 0;
            }
            const bool kok = ci * BK + unit * 8 < p.K;      // the last chunk may reach past the reduction length
#pragma unroll
            for (int i = 0; i < ITEMS; i++)
                stage_v[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(kok ? pwoff[i] + (MODE == MODE_PWR ? ci * (BK * 2) - early : 0) : kOutOfRange), MODE == MODE_PWR ? 0 : ci * (BK * 2), 0);
        } else if constexpr (MODE == MODE_GATHER4) {
            // this thread's block of 4 reduction indices: one tap, 4 consecutive channels
            auto &stage_g4 = stage_g4_[set];
            const int k0 = ci * BK + unit * 4;
            const int tap = fast_div(k0, p.cin_mul, p.cin_sh);
            const int c = k0 - tap * p.Cin;
            const int r = fast_div(tap, p.kw_mul, p.kw_sh);
            const int t = tap - r * p.kw;
            const unsigned koff = k0 < p.K ? (unsigned)(((r * p.W + t) * p.Cin + c) * 2) : kOutOfRange;
#pragma unroll
            for (int i = 0; i < ITEMS; i++) {
                int ih = ih0[i] + r, iw = iw0[i] + t;
                bool ok = (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W && koff != kOutOfRange;
                stage_g4[i] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(rx, (int)(ok ? pixbyte[i] + koff : kOutOfRange), 0, 0));
            }
        } else if constexpr (MODE == MODE_GATHER) {
            unsigned off[4];
            int er[4], et[4];
#pragma unroll
            for (int e = 0; e < 4; e++) {
                int k = ci * BK + unit * 4 + e;
                int c, r, t;
                if (p.korder == SS_K_CRS) {
                    int khw = p.kh * p.kw;
                    c = k / khw;
                    int rem = k - c * khw;
                    r = rem / p.kw;
                    t = rem - r * p.kw;
                } else {
                    int tap = k / p.Cin;
                    c = k - tap * p.Cin;
                    r = tap / p.kw;
                    t = tap - r * p.kw;
                }
                er[e] = k < p.K ? r : (1 << 29);      // past the reduction length: fails the bounds test
                et[e] = t;
                off[e] = (unsigned)(((r * p.W + t) * p.Cin + c) * 2);
            }
#pragma unroll
            for (int i = 0; i < ITEMS; i++) {
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    int ih = ih0[i] + er[e], iw = iw0[i] + et[e];
                    bool ok = (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;
                    unsigned o = ok ? pixbyte[i] + off[e] : kOutOfRange;
                    stage_g[i][e] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rx, (int)o, 0, 0);
                }
            }
        } else {
            const unsigned soff = (unsigned)ci * 64;    // 32 channels per chunk
            unsigned past = 0, early = 0;               // kOutOfRange for an octet past the last channel
            if constexpr (MODE == MODE_TAPSR) {
                const int c = ci * 32 + unit * 8;
                past = c < p.Cin ? 0u : kOutOfRange;
                half_[set] = c + 4 == p.Cin;
                early = half_[set] ? 8u : 0u;           // (an out-of-image tap stays out of range: every buffer is 64 MiB short of 2 GiB)
            }
#pragma unroll
            for (int i = 0; i < ITEMS; i++)
#pragma unroll
                for (int tap = 0; tap < TAPS; tap++)
                    stage_t[i][tap] = MODE == MODE_TAPSR
                        ? __builtin_amdgcn_raw_buffer_load_b128(rx, (int)((tapoff[i][tap] | past) + (soff - early)), 0, 0)      // (one sum: the offset alone could go below 0)
                        : __builtin_amdgcn_raw_buffer_load_b128(rx, (int)tapoff[i][tap], soff, 0);
        }
    };
    // Writes slice j of n of the staged chunk to LDS (j, n are compile-time at every call site): a share of the
    // transposed 16-byte vectors (tap mode) or of the items (other modes).  stage_store = all of it.
    auto stage_store_slice = [&](uint16_t *Bs, int j, int n, int set = 0) {
        if (!stager) return;
        auto &stage_v = stage_v_[set];
        auto &stage_g = stage_g_[set];
        auto &stage_t = stage_t_[set];
#pragma unroll
        for (int i = 0; i < ITEMS; i++) {
            int pr = pr0 + i * (ST / UNITS);
            if constexpr (is_taps(MODE)) {
                // [tap][8 channels] -> [channel][tap]: output element h = c*TAPS + tap, two per dword, four dwords per vector
                u32x4 *rowp = reinterpret_cast<u32x4 *>(Bs + pr * ROW);
                const int vec0 = unit * TAPS, swz = CS::SWZ ? (pr >> 2) & 3 : 0;     // first vector of the unit; the row's XOR key
#pragma unroll
                for (int v = 0; v < TAPS; v++) {
                    if (v < j * TAPS / n || v >= (j + 1) * TAPS / n) continue;
                    rowp[(vec0 + v) ^ swz] = taps_vector<Q8, MODE == MODE_TAPSR, TAPS>(stage_t[i], v, MODE == MODE_TAPSR && half_[set]);
                }
            } else {
                if (i < j * ITEMS / n || i >= (j + 1) * ITEMS / n) continue;
                if constexpr (MODE == MODE_GATHER4) {
                    *reinterpret_cast<uint2 *>(Bs + pr * ROW + unit * 4) = stage_g4_[set][i];
                } else if constexpr (MODE == MODE_GATHER) {
                    uint2 v = make_uint2((uint32_t)stage_g[i][0] | ((uint32_t)stage_g[i][1] << 16),
                                         (uint32_t)stage_g[i][2] | ((uint32_t)stage_g[i][3] << 16));
                    *reinterpret_cast<uint2 *>(Bs + pr * ROW + unit * 4) = v;
                } else {
                    u32x4 v = stage_v[i];
                    if constexpr (MODE == MODE_PWR)
                        if (half_[set]) v = u32x4{v[2], v[3], 0u, 0u};
                    *reinterpret_cast<u32x4 *>(Bs + pr * ROW + unit * 8) = v;
                }
            }
        }
    };
    auto stage_store = [&](uint16_t *Bs, int set = 0) { stage_store_slice(Bs, 0, 1, set); };

    // ------------------------------------------------------------------ weight fragments
    // Row tiles past the last one are clamped to it (their rows are never stored); reduction steps
    // past the last one are clamped too: they only ever meet all-zero activations.
    unsigned a_voff[TM], m_voff[TM];
#pragma unroll
    for (int tm = 0; tm < TM; tm++) {
        int mt = min((m0 >> 5) + wm * TM + tm, p.Mt - 1);
        a_voff[tm] = (unsigned)((mt * p.Ks * (SPARSE ? 1 : 2)) * 64 + lane) * 16u;
        m_voff[tm] = (unsigned)(mt * p.Kp * 64 + lane) * 4u;
    }
    const int ks_first = c_first * KSTEPS;
    auto load_a = [&](AStep<SPARSE, TM> &a, int ks_rel) {       // step relative to this workgroup's first
        const int ks = min(ks_rel + ks_first, p.Ks - 1);
#pragma unroll
        for (int tm = 0; tm < TM; tm++) {
            if constexpr (SPARSE) {
                a.v[0][tm] = __builtin_amdgcn_raw_buffer_load_b128(ra, (int)a_voff[tm], ks * 1024, 0);
                // The index word of the step pair; the step's half is shifted down where it is used, steps later (a
                // shift here would have to wait for the load it follows and stall the wave at every step).
                a.idx[tm] = __builtin_amdgcn_raw_buffer_load_b32(rm, (int)m_voff[tm], (Q8 ? ks : (ks >> 1)) * 256, 0);
            } else {
                a.v[0][tm] = __builtin_amdgcn_raw_buffer_load_b128(ra, (int)a_voff[tm], ks * 2048, 0);
                a.v[1][tm] = __builtin_amdgcn_raw_buffer_load_b128(ra, (int)a_voff[tm], ks * 2048 + 1024, 0);
            }
        }
    };

    // This lane's two 16-byte vectors of a fragment inside the step's aligned group of four (in 16-bit units): lanes
    // 0..31 take vectors 0, 1 and lanes 32..63 vectors 2, 3, XOR-ed with the pixel row's key in the swizzled layout.
    const int frag_key = CS::SWZ ? (lane >> 2) & 3 : 0;
    const int frag_lo = ((2 * (lane >> 5)) ^ frag_key) * 8, frag_hi = ((2 * (lane >> 5) + 1) ^ frag_key) * 8;

    Acc<DT> acc[TM][TN];
#pragma unroll
    for (int tm = 0; tm < TM; tm++)
#pragma unroll
        for (int tn = 0; tn < TN; tn++)
#pragma unroll
            for (int v = 0; v < 16; v++) acc[tm][tn][v] = 0;

    // ------------------------------------------------------------------ main loop (double-buffered LDS, ring of weight steps)
    AStep<SPARSE, TM> a[RING];
    if constexpr (SPEC) {
        if (producer) {
            // ---- producer waves: chunk ci+1 is written to LDS while the others multiply chunk ci; its loads were
            // issued one chunk earlier.  One barrier per chunk, exactly as in the multiplying waves' loop below.
            // The steady-state loop issues its loads unconditionally: behind a condition, the compiler's wait before
            // the LDS writes must also cover the path without new loads, and so waits for the new loads as well
            // (a full memory latency per chunk).
            stage_load(0, 0);
            stage_store(Bs0, 0);
            if (nchunks > 1) stage_load(1, 1);
            __syncthreads();
            // the last two chunks: nothing left to load (set, buf: where chunk ci + 1 waits and where it goes)
            auto tail = [&](int ci, int set, uint16_t *buf) {
                if (ci + 1 < nchunks) {
                    stage_store(buf, set);
                    __syncthreads();
                    ci++;
                }
                if (ci < nchunks) __syncthreads();
            };
            for (int ci = 0;;) {
                if (ci + 2 >= nchunks) { tail(ci, 1, Bs1); break; }
                stage_load(ci + 2, 0);                      // set 0 held chunk ci, which is in LDS already
                stage_store(Bs1, 1);
                __syncthreads();
                ci++;
                if (ci + 2 >= nchunks) { tail(ci, 0, Bs0); break; }
                stage_load(ci + 2, 1);
                stage_store(Bs0, 0);
                __syncthreads();
                ci++;
            }
        }
    }
    if (!producer) {
    // With producer waves in the workgroup the multiplying waves set the pace (the producers wait for them at every
    // chunk's barrier): they get the issue slots first (measured 2-4 % on the 3x3 256 -> 256 layer at batch 32).
    if constexpr (SPEC) __builtin_amdgcn_s_setprio(3);
    if constexpr (!SPEC) stage_load(0);
    // (Issue order pinned: the loop's waits count loads in flight, and the compiler takes the weaker of the counts
    // that hold on entry and around the back edge; values and index words must interleave here as they do there.)
#pragma unroll
    for (int s = 0; s < PF; s++) {
        load_a(a[s], s);
        __builtin_amdgcn_sched_barrier(0);
    }
    load_bias();
    if constexpr (!SPEC) stage_store(Bs0);
#pragma unroll
    for (int j = 0; j < (BM + NMATH - 1) / NMATH; j++)
        if (tid + j * NMATH < BM) {
            bias_s[tid + j * NMATH] = bias_r[j];
            if constexpr (Q8) scale_s[tid + j * NMATH] = scale_r[j];
        }
    __syncthreads();
    for (int c0 = 0; c0 < nchunks; c0 += UNROLL) {
#pragma unroll
        for (int u = 0; u < UNROLL; u++) {
            const int ci = c0 + u;
            if (ci >= nchunks) break;                       // uniform
            const uint16_t *cur = (ci & 1) ? Bs1 : Bs0;
            uint16_t *nxt = (ci & 1) ? Bs0 : Bs1;
            const bool more = ci + 1 < nchunks;
            if constexpr (!SPEC)
                if (more) stage_load(ci + 1);
            __builtin_amdgcn_sched_barrier(0);
            B32 b[BD][TN];
            auto load_b = [&](B32 (&bf)[TN], int s) {
#pragma unroll
                for (int tn = 0; tn < TN; tn++) {
                    const uint16_t *src = cur + ((wn * TN + tn) * 32 + (lane & 31)) * ROW + s * 32;
                    bf[tn].lo = *reinterpret_cast<const u32x4 *>(src + frag_lo);
                    bf[tn].hi = *reinterpret_cast<const u32x4 *>(src + frag_hi);
                }
            };
#pragma unroll
            for (int s = 0; s < BD - 1 && s < KSTEPS; s++) load_b(b[s], s);
#pragma unroll
            for (int s = 0; s < KSTEPS; s++) {
                const int g = u * KSTEPS + s;               // position in the ring (compile time)
                load_a(a[(g + PF) % RING], ci * KSTEPS + s + PF);
                if (s + BD - 1 < KSTEPS) load_b(b[(s + BD - 1) % BD], s + BD - 1);   // later steps' activations while this step multiplies
                if constexpr (NBUF == 2 && !SPEC) {          // the next chunk's share of transposes / LDS writes rides along with the later steps
                    constexpr int S0 = KSTEPS / 2;
                    if (more && s >= S0) stage_store_slice(nxt, s - S0, KSTEPS - S0);
                }
                // (steps past the reduction length multiply clamped weights with all-zero activations:
                // cheaper than a branch, which would force copies of every accumulator)
                const AStep<SPARSE, TM> &as = a[g % RING];
                // the 16-bit instruction reads index bits [15:0]; the 8-bit one the whole word
                const int idx_shift = Q8 ? 0 : (min(ks_first + ci * KSTEPS + s, p.Ks - 1) & 1) * 16;
#pragma unroll
                for (int tm = 0; tm < TM; tm++)
#pragma unroll
                    for (int tn = 0; tn < TN; tn++) {
                        if constexpr (SPARSE) {
                            acc[tm][tn] = mma_sparse<DT>(as.v[0][tm], b[s % BD][tn], acc[tm][tn], as.idx[tm] >> idx_shift);
                        } else if constexpr (DT == SS_F8 && f8_wide(DEEP, MODE)) {
                            acc[tm][tn] = mma_dense_f8(as.v[0][tm], as.v[1][tm], b[s % BD][tn], acc[tm][tn]);
                        } else {
                            acc[tm][tn] = mma_dense<DT>(as.v[0][tm], b[s % BD][tn].lo, acc[tm][tn]);
                            acc[tm][tn] = mma_dense<DT>(as.v[1][tm], b[s % BD][tn].hi, acc[tm][tn]);
                        }
                    }
                // Scheduling: left alone, the compiler sinks every load to just before its first use and the
                // prefetch distance collapses to zero.  Pin this step's instructions to the step (barriers at both
                // ends) and interleave the loads for later steps between its matrix instructions.
                constexpr int NMMA = TM * TN * (SPARSE ? 1 : (DT == SS_F8 ? (f8_wide(DEEP, MODE) ? 1 : 4) : 2));
                constexpr int DSR = (2 * TN + NMMA - 1) / NMMA;
                constexpr int VMR = (TM * 2 + NMMA - 1) / NMMA;
#pragma unroll
                for (int i = 0; i < NMMA; i++) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // one MFMA
                    __builtin_amdgcn_sched_group_barrier(0x100, DSR, 0);    // LDS reads
                    __builtin_amdgcn_sched_group_barrier(0x020, VMR, 0);    // global reads
                    __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);      // transposes of the next chunk (when this step has any)
                    __builtin_amdgcn_sched_group_barrier(0x200, 2, 0);      // and their LDS writes
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (NBUF == 1) {
                __syncthreads();                            // everyone is done reading the only copy
                if (more) stage_store(nxt);
            }
            __syncthreads();
        }
    }
    }   // !producer

    // ------------------------------------------------------------------ epilogue
    // bias (+ residual) + activation in fp32, one rounding to the 16-bit type; the tile goes through LDS so that
    // every pixel's run of BM output channels leaves as 16-byte, fully coalesced NHWC stores.
    constexpr int RUNS = BM / 8;                  // 16-byte runs per pixel row
    const bool vec_ok = (p.Cout & 7) == 0;
    // The thread index again, from the wave number (scalar) and the lane count: keeping the launch-time register
    // alive across the main loop costs a spill in the variants that run at the register limit.
    const int etid = wave * 64 + (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    const float relu_floor = p.act == SS_ACT_RELU ? 0.f : -__builtin_inff();
    // ReLU when relu_floor = 0, identity when -inf (a NaN passes through); GELU = z * Phi(z) with the exact normal
    // CDF (gelu_cdf)
    auto relu_or_id = [&](float v) { return floor_at(v, relu_floor); };
    auto gelu = [](float v) { return gelu_cdf<ODT>(v); };
    if constexpr (CAN_SPLIT) {
        if (nsplit > 1) {
            // Every workgroup of the tile leaves its partial sums in the workspace, in register order (one 16-byte
            // vector per thread and accumulator quad: fully coalesced), and takes a ticket.  The last one to arrive adds
            // the partials in the order of the splits -- so the result does not depend on who arrived last --, hands the
            // ticket counter back at zero for the next launch, and runs the usual tail; the others are done.
            // The workgroups of a tile may run on different XCDs, whose L2 caches are not coherent with each other.  The
            // partial sums are therefore stored and loaded with the device-scope cache policy (sc1: written through to,
            // and read from, the level all XCDs share -- what a relaxed device-scope atomic store / load compiles to),
            // every wave waits for the acknowledgement of its stores before the workgroup takes its ticket, and the
            // ticket is a device-scope atomic.  Device-scope fences would do as well, but they write back (release) and
            // invalidate (acquire) the XCD's whole L2 under the workgroups still in their main loops: measured at
            // 3 us per doubling of the split with the release fence alone, 4-8 us per workgroup with both.
            constexpr int kDeviceScope = 16;            // cache-policy bit sc1 of the buffer instructions
            const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(p.ws_part + (size_t)lid * nsplit * (BM * BN), 0,
                                                                               nsplit * (BM * BN) * 4, kRsrcFlags);
            const int mtid = etid;                      // (multiplying threads are 0 .. NMATH-1)
            if (!producer) {
#pragma unroll
                for (int tm = 0; tm < TM; tm++)
#pragma unroll
                    for (int tn = 0; tn < TN; tn++)
#pragma unroll
                        for (int q = 0; q < 4; q++) {
                            const f32x4 fw = {(float)acc[tm][tn][4 * q + 0], (float)acc[tm][tn][4 * q + 1], (float)acc[tm][tn][4 * q + 2], (float)acc[tm][tn][4 * q + 3]};
                            store_b128<kDeviceScope>(__builtin_bit_cast(u32x4, fw), rp, (((tm * TN + tn) * 4 + q) * NMATH + mtid) * 16, split * (BM * BN * 4));
                        }
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // this wave's partial sums have been acknowledged
            __syncthreads();
            unsigned *ticket_s = reinterpret_cast<unsigned *>(smem);      // (the staging buffers are free)
            unsigned *const counter = reinterpret_cast<unsigned *>(reinterpret_cast<char *>(p.ws_part) - ticket_bytes(ntiles)) + lid;
            if (etid == 0) *ticket_s = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            const unsigned ticket = *ticket_s;
            if (ticket != (unsigned)(nsplit - 1)) return;                 // (uniform)
            if (etid == 0) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (!producer) {
#pragma unroll
                for (int tm = 0; tm < TM; tm++)
#pragma unroll
                    for (int tn = 0; tn < TN; tn++)
#pragma unroll
                        for (int v = 0; v < 16; v++) acc[tm][tn][v] = 0.f;
                for (int j = 0; j < nsplit; j++) {
#pragma unroll
                    for (int tm = 0; tm < TM; tm++)
#pragma unroll
                        for (int tn = 0; tn < TN; tn++)
#pragma unroll
                            for (int q = 0; q < 4; q++) {
                                // (the whole vector is reinterpreted at once: a bit cast of a single vector element reads element 0)
                                const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rp, (((tm * TN + tn) * 4 + q) * NMATH + mtid) * 16, j * (BM * BN * 4), kDeviceScope));
                                acc[tm][tn][4 * q + 0] += v[0]; acc[tm][tn][4 * q + 1] += v[1];
                                acc[tm][tn][4 * q + 2] += v[2]; acc[tm][tn][4 * q + 3] += v[3];
                            }
                }
            }
            __syncthreads();                            // the ticket word's LDS is about to hold the output tile
        }
    }
    if (!with_res) {
        constexpr int CROW = BM + 4;     // halfs per pixel row in LDS (+8 bytes: the 8-byte writes of 32 consecutive pixels spread over all banks)
        uint16_t *Cs = smem;             // the staging buffers are free: the loop ended with a barrier (every wave, producers included, ran the same number)
        auto to_lds = [&](auto actf) {
#pragma unroll
            for (int tm = 0; tm < TM; tm++) {
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int ol = (wm * TM + tm) * 32 + 8 * q + 4 * (lane >> 5);    // first of 4 consecutive output channels (tile-local)
                    const float4 bq = *reinterpret_cast<const float4 *>(bias_s + ol);
                    const float bv[4] = {bq.x, bq.y, bq.z, bq.w};
                    float sv[4] = {1.f, 1.f, 1.f, 1.f};
                    if constexpr (Q8) {
                        const float4 sq = *reinterpret_cast<const float4 *>(scale_s + ol);
                        sv[0] = sq.x; sv[1] = sq.y; sv[2] = sq.z; sv[3] = sq.w;
                    }
#pragma unroll
                    for (int tn = 0; tn < TN; tn++) {
                        float r[4];
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            if constexpr (Q8) r[e] = actf((float)acc[tm][tn][4 * q + e] * sv[e] + bv[e]);
                            else r[e] = actf(acc[tm][tn][4 * q + e] + bv[e]);
                        }
                        const int pl = (wn * TN + tn) * 32 + (lane & 31);
                        *reinterpret_cast<uint2 *>(Cs + pl * CROW + ol) = make_uint2(cvt_pack2<ODT>(r[0], r[1]), cvt_pack2<ODT>(r[2], r[3]));
                    }
                }
            }
        };
        float bias3 = 0.f;
        if constexpr (THIRD > 0)
            if (tid < p.Cout3 && p.bias3 != nullptr) bias3 = p.bias3[tid];      // (at most 128 channels)
        if (!producer) {
            if (p.act == SS_ACT_GELU) to_lds(gelu); else to_lds(relu_or_id);
        }
        __syncthreads();
        if constexpr (THIRD > 0) {
            if (tid < p.Cout3) bias_s[tid] = bias3;       // (the first layer's is done with; read behind the barriers below)
            // ---- second and third contraction, 128 channels of the second one's output at a time: each wave finishes one row tile of 32
            // (stored as in the pair below, and left in LDS), then multiplies the third one's weights with the 128 channels; its
            // accumulators stay in registers.  The weights and the residual of the next 128 are in flight meanwhile.
            static_assert(!SPEC && NT == 256 && BN == 64, "four waves, 64 pixels");
            constexpr int KS2 = BM / 32, ITEMS3 = THIRD;  // steps of the second reduction at most; 32 x 32 tiles of the third output per wave
            uint16_t *const Ts = reinterpret_cast<uint16_t *>(reinterpret_cast<char *>(smem) + (size_t)BN * (BM * 2 + 8) + (NT / 64) * kFuseRegion);
            float *const reg = reinterpret_cast<float *>(reinterpret_cast<char *>(smem) + (size_t)BN * (BM * 2 + 8)) + wave * (32 * kFuseRow);
            auto buffer = [](const void *base, unsigned bytes) {
                return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, base != nullptr ? (int)bytes : 0, kRsrcFlags);
            };
            const __amdgpu_buffer_rsrc_t ra2 = buffer(p.a2_vals, p.a2_bytes), rm2 = buffer(p.a2_meta, p.meta2_bytes);
            const __amdgpu_buffer_rsrc_t ra3 = buffer(p.a3_vals, p.a3_bytes), rm3 = buffer(p.a3_meta, p.meta3_bytes);
            const __amdgpu_buffer_rsrc_t rb2 = buffer(p.bias2, (unsigned)p.Cout2 * 4u);
            // outputs and residual of this workgroup's pixels: whatever lies behind the last one is out of range
            const unsigned px_here = (unsigned)min(BN, p.P - n0), row2 = (unsigned)p.Cout2 * 2u, row3 = (unsigned)p.Cout3 * 2u;
            const __amdgpu_buffer_rsrc_t rres = buffer(p.res2 != nullptr ? p.res2 + (size_t)n0 * p.Cout2 : nullptr, px_here * row2);
            const __amdgpu_buffer_rsrc_t ry2 = buffer(p.y2 + (size_t)n0 * p.Cout2, px_here * row2), ry3 = buffer(p.y3 + (size_t)n0 * p.Cout3, px_here * row3);
            const int l = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), g = l >> 5, c = l & 31;
            struct Rows {
                u32x4 v[SPARSE ? 1 : 2][4];
                uint32_t idx[4];
            };
            auto load_steps = [&](Rows &r, const __amdgpu_buffer_rsrc_t &rv, const __amdgpu_buffer_rsrc_t &ri, int mt, int Ks, int Kp, int ks0, int n) {
#pragma unroll
                for (int s = 0; s < 4; s++) {
                    if (s >= n) break;                    // uniform
                    const int ks = ks0 + s;
                    if constexpr (SPARSE) {
                        r.v[0][s] = __builtin_amdgcn_raw_buffer_load_b128(rv, l * 16, (mt * Ks + ks) * 1024, 0);
                        r.idx[s] = __builtin_amdgcn_raw_buffer_load_b32(ri, l * 4, (mt * Kp + (ks >> 1)) * 256, 0);
                    } else {
                        r.v[0][s] = __builtin_amdgcn_raw_buffer_load_b128(rv, l * 16, (mt * Ks + ks) * 2048, 0);
                        r.v[1][s] = __builtin_amdgcn_raw_buffer_load_b128(rv, l * 16, (mt * Ks + ks) * 2048 + 1024, 0);
                    }
                }
            };
            auto mma = [&](const Rows &r, int s, const B32 &b, f32x16 d) {
                if constexpr (SPARSE) return mma_sparse<DT>(r.v[0][s], b, d, r.idx[s] >> ((s & 1) * 16));
                else return mma_dense<DT>(r.v[1][s], b.hi, mma_dense<DT>(r.v[0][s], b.lo, d));
            };
            // The sums start from zero and the bias follows them, as in the pair and in the layer's own call: the bits are the same.  The second layer's bias
            // waits as one value per lane and crosses LDS behind the first rows of the wave's region: there are no registers for a lane's eight channels.
            auto clear = [](f32x16 &d) {
#pragma unroll
                for (int v = 0; v < 16; v++) d[v] = 0.f;
            };
            // a lane's 16-byte run number j of a 32 x 32 tile at pixel half tn: pixel and run of 8 channels
            auto run_px = [&](int tn, int j) { return tn * 32 + 16 * j + (l >> 2); };
            const int half3 = wave & 1;                   // tile i of this wave: row tile (wave >> 1) + 2 i on pixel half wave & 1
            auto row3_of = [&](int i) { return min((wave >> 1) + 2 * i, p.Mt3 - 1); };
            f32x16 acc3[ITEMS3];
#pragma unroll
            for (int i = 0; i < ITEMS3; i++) clear(acc3[i]);
            Rows w2, w3[ITEMS3];
            u32x4 res[2][2];
            load_steps(w2, ra2, rm2, wave, p.Ks2, p.Kp2, 0, p.Ks2);
            const float floor2 = p.act2 == SS_ACT_RELU ? 0.f : -__builtin_inff(), floor3 = p.act3 == SS_ACT_RELU ? 0.f : -__builtin_inff();
            auto put = [&](const f32x16 &d) {
#pragma unroll
                for (int q = 0; q < 4; q++) *reinterpret_cast<f32x4 *>(reg + c * kFuseRow + 8 * q + 4 * g) = f32x4{d[4 * q], d[4 * q + 1], d[4 * q + 2], d[4 * q + 3]};
            };
            auto get = [&](int j, const float *bias, int next, float (&v)[8]) {      // (a wave's LDS operations execute in order: it sees what put left)
                const float *src = reg + (16 * j + (l >> 2)) * kFuseRow + (l & 3) * 8;
                const f32x4 lo = *reinterpret_cast<const f32x4 *>(src), hi = *reinterpret_cast<const f32x4 *>(src + 4);
                const f32x4 bl = *reinterpret_cast<const f32x4 *>(bias), bh = *reinterpret_cast<const f32x4 *>(bias + next);
#pragma unroll
                for (int e = 0; e < 4; e++) { v[e] = lo[e] + bl[e]; v[4 + e] = hi[e] + bh[e]; }
            };
            auto finish = [&](float (&v)[8], int act, float floor) {
                if (act == SS_ACT_GELU) {
#pragma unroll
                    for (int e = 0; e < 8; e++) v[e] = gelu(v[e]);
                } else {
#pragma unroll
                    for (int e = 0; e < 8; e++) v[e] = floor_at(v[e], floor);
                }
                return u32x4{cvt_pack2<ODT>(v[0], v[1]), cvt_pack2<ODT>(v[2], v[3]), cvt_pack2<ODT>(v[4], v[5]), cvt_pack2<ODT>(v[6], v[7])};
            };
            constexpr int kNonTemporal = 2;               // cache-policy bit nt of the buffer instructions
            const int nparts = p.Cout2 / 128;
            // A residual is mostly the block's input at its last use, y2 what the next block reads as its own.  Where both together are about as large as the
            // 256 MB that the memory's cache holds, the residual's lines push y2 out before that: it is then read with the non-temporal hint.  (A hint: a
            // caller who reads the residual again finds it in memory.)  ResNet-50 trunk at 224 x 224, us without and with:
            //   residual of the 56 x 56 blocks, 64 channels: 40 images (61 MiB) 716 / 718, 48 (73) 907 / 883, 56 (86) 960 / 931, 64 (98) 1077 / 1038 (dense
            //   1241 / 1228), 72 (110) 1131 / 1096, 80 (122) 1215 / 1191, 88 (135) 1423 / 1412, 92 (141) 1460 / 1463; 96 (147) would be 1474 / 1486;
            //   of the 28 x 28 blocks, 128 channels: 100 images (77 MiB) 1524 / 1493, 128 (98) 1822 / 1788, 160 (122) 2099 / 2074, 184 (141) 2520 / 2507.
            // 200 images of 128 x 128 (100 MiB) 1089 / 1049, 48 of 256 x 256 (96) 1029 / 993, 64 (128) 1260 / 1224.
            const long long res_bytes = (long long)p.P * p.Cout2 * 2;
            const bool once = res_bytes >= (72ll << 20) && res_bytes < (144ll << 20);
            for (int part = 0; part < nparts; part++) {
                const int mt = part * 4 + wave;
#pragma unroll
                for (int tn = 0; tn < 2; tn++)
#pragma unroll
                    for (int j = 0; j < 2; j++)
                        res[tn][j] = once ? __builtin_amdgcn_raw_buffer_load_b128(rres, (int)(run_px(tn, j) * row2 + (l & 3) * 16), mt * 64, kNonTemporal)
                                          : __builtin_amdgcn_raw_buffer_load_b128(rres, (int)(run_px(tn, j) * row2 + (l & 3) * 16), mt * 64, 0);
                f32x16 acc2[2];
                clear(acc2[0]);
                clear(acc2[1]);
                const float bias2 = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rb2, c * 4, mt * 128, 0));
#pragma unroll
                for (int i = 0; i < ITEMS3; i++) load_steps(w3[i], ra3, rm3, row3_of(i), p.Ks3, p.Kp3, part * 4, 4);
#pragma unroll
                for (int s = 0; s < KS2; s++) {
                    if (s >= p.Ks2) break;                // uniform
#pragma unroll
                    for (int tn = 0; tn < 2; tn++) {
                        const uint16_t *src = Cs + (tn * 32 + c) * CROW + 32 * s + 16 * g;      // 8-byte aligned
                        const uint2 u0 = *reinterpret_cast<const uint2 *>(src), u1 = *reinterpret_cast<const uint2 *>(src + 4);
                        const uint2 u2 = *reinterpret_cast<const uint2 *>(src + 8), u3 = *reinterpret_cast<const uint2 *>(src + 12);
                        B32 b;
                        b.lo = u32x4{u0.x, u0.y, u1.x, u1.y};
                        b.hi = u32x4{u2.x, u2.y, u3.x, u3.y};
                        acc2[tn] = mma(w2, s, b, acc2[tn]);
                    }
                }
                load_steps(w2, ra2, rm2, min(mt + 4, p.Mt2 - 1), p.Ks2, p.Kp2, 0, p.Ks2);
                int at = l;
                asm volatile("" : "+v"(at));              // (addresses worked out in each part: kept over them, they would spill)
                reg[(at & 31) / 4 * kFuseRow + 32 + at % 4] = bias2;
                const float *const bias = reg + at % 4 * 2 * kFuseRow + 32;
#pragma unroll
                for (int tn = 0; tn < 2; tn++) {
                    put(acc2[tn]);
#pragma unroll
                    for (int j = 0; j < 2; j++) {
                        float v[8];
                        get(j, bias, kFuseRow, v);
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            v[2 * e] += widen<ODT>((uint16_t)(res[tn][j][e] & 0xFFFFu));
                            v[2 * e + 1] += widen<ODT>((uint16_t)(res[tn][j][e] >> 16));
                        }
                        const u32x4 w = finish(v, p.act2, floor2);
                        *reinterpret_cast<u32x4 *>(Ts + run_px(tn, j) * kThirdRow + wave * 32 + (l & 3) * 8) = w;
                        store_b128(w, ry2, (int)(run_px(tn, j) * row2 + (l & 3) * 16), mt * 64);
                    }
                }
                lds_barrier();
#pragma unroll
                for (int s = 0; s < 4; s++) {
                    const uint16_t *src = Ts + (half3 * 32 + c) * kThirdRow + 32 * s + 16 * g;
                    B32 b;
                    b.lo = *reinterpret_cast<const u32x4 *>(src);
                    b.hi = *reinterpret_cast<const u32x4 *>(src + 8);
#pragma unroll
                    for (int i = 0; i < ITEMS3; i++) acc3[i] = mma(w3[i], s, b, acc3[i]);
                }
                lds_barrier();                            // the next 128 channels may take their place
            }
#pragma unroll
            for (int i = 0; i < ITEMS3; i++) {
                if ((wave >> 1) + 2 * i >= p.Mt3) break;  // uniform
                put(acc3[i]);
#pragma unroll
                for (int j = 0; j < 2; j++) {
                    float v[8];
                    get(j, bias_s + row3_of(i) * 32 + (l & 3) * 8, 4, v);
                    store_b128(finish(v, p.act3, floor3), ry3, (int)(run_px(half3, j) * row3 + (l & 3) * 16), ((wave >> 1) + 2 * i) * 64);
                }
            }
            return;
        }
        if constexpr (FUSE) {
            // ---- second contraction: y2[pixel, o2] = act2( sum_c A2[o2, c] * tile[pixel, c] + bias2[o2] + residual[pixel, o2] )
            // Every wave (producers included) takes row tiles of 32 output channels in turn; its weights and bias for
            // the next row tile are fetched while the current one is multiplied.  The fp32 result of 32 pixels x 32
            // channels crosses the wave's own LDS region so that residual loads and stores are 16-byte runs.
            constexpr int NW = NT / 64;
            constexpr int KS2 = BM / 32;                  // upper bound of the second reduction's steps (its length is this convolution's cout)
            constexpr int TN2 = BN / 32;
            float *reg = reinterpret_cast<float *>(reinterpret_cast<char *>(smem) + (size_t)BN * (BM * 2 + 8)) + wave * (32 * kFuseRow);
            const __amdgpu_buffer_rsrc_t ra2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(p.a2_vals), 0, (int)p.a2_bytes, kRsrcFlags);
            const __amdgpu_buffer_rsrc_t rm2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(p.a2_meta), 0, (int)p.meta2_bytes, kRsrcFlags);
            const int lane2 = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
            const int g2 = lane2 >> 5, c2 = lane2 & 31;
            const float floor2 = p.act2 == SS_ACT_RELU ? 0.f : -__builtin_inff();
            struct Row2 {
                u32x4 v[SPARSE ? 1 : 2][KS2];
                uint32_t idx[KS2];
                float4 b[4];
            };
            auto load_row = [&](Row2 &r, int mt) {
#pragma unroll
                for (int s2 = 0; s2 < KS2; s2++) {
                    if (s2 >= p.Ks2) break;               // uniform
                    if constexpr (SPARSE) {
                        r.v[0][s2] = __builtin_amdgcn_raw_buffer_load_b128(ra2, (int)(((unsigned)(mt * p.Ks2 + s2) * 64 + lane2) * 16u), 0, 0);
                        r.idx[s2] = __builtin_amdgcn_raw_buffer_load_b32(rm2, (int)(((unsigned)(mt * p.Kp2 + (s2 >> 1)) * 64 + lane2) * 4u), 0, 0);
                    } else {
                        const unsigned off = ((unsigned)(mt * p.Ks2 + s2) * 128 + lane2) * 16u;
                        r.v[0][s2] = __builtin_amdgcn_raw_buffer_load_b128(ra2, (int)off, 0, 0);
                        r.v[1][s2] = __builtin_amdgcn_raw_buffer_load_b128(ra2, (int)off, 1024, 0);
                    }
                }
#pragma unroll
                for (int q = 0; q < 4; q++)
                    r.b[q] = p.bias2 ? *reinterpret_cast<const float4 *>(p.bias2 + mt * 32 + 8 * q + 4 * g2) : make_float4(0.f, 0.f, 0.f, 0.f);
            };
            Row2 cur, nxt;
            if (wave < p.Mt2) load_row(cur, wave);
            for (int mt = wave; mt < p.Mt2; mt += NW) {
                if (mt + NW < p.Mt2) load_row(nxt, mt + NW);
#pragma unroll
                for (int tn = 0; tn < TN2; tn++) {
                    f32x16 acc2;
#pragma unroll
                    for (int v = 0; v < 16; v++) acc2[v] = 0.f;
#pragma unroll
                    for (int s2 = 0; s2 < KS2; s2++) {
                        if (s2 >= p.Ks2) break;           // uniform
                        const uint16_t *src = Cs + (tn * 32 + c2) * CROW + 32 * s2 + 16 * g2;     // 8-byte aligned
                        const uint2 u0 = *reinterpret_cast<const uint2 *>(src), u1 = *reinterpret_cast<const uint2 *>(src + 4);
                        const uint2 u2 = *reinterpret_cast<const uint2 *>(src + 8), u3 = *reinterpret_cast<const uint2 *>(src + 12);
                        B32 bf;
                        bf.lo = u32x4{u0.x, u0.y, u1.x, u1.y};
                        bf.hi = u32x4{u2.x, u2.y, u3.x, u3.y};
                        if constexpr (SPARSE) {
                            acc2 = mma_sparse<DT>(cur.v[0][s2], bf, acc2, cur.idx[s2] >> ((s2 & 1) * 16));
                        } else {
                            acc2 = mma_dense<DT>(cur.v[0][s2], bf.lo, acc2);
                            acc2 = mma_dense<DT>(cur.v[1][s2], bf.hi, acc2);
                        }
                    }
#pragma unroll
                    for (int q = 0; q < 4; q++)
                        *reinterpret_cast<float4 *>(reg + c2 * kFuseRow + 8 * q + 4 * g2) =
                            make_float4(acc2[4 * q + 0] + cur.b[q].x, acc2[4 * q + 1] + cur.b[q].y, acc2[4 * q + 2] + cur.b[q].z, acc2[4 * q + 3] + cur.b[q].w);
                    // (a wave's LDS operations execute in order: the reads below see the writes above)
#pragma unroll
                    for (int j = 0; j < 2; j++) {
                        const int it = lane2 + 64 * j;
                        const int px = it >> 2, run = it & 3;
                        const int pg = n0 + tn * 32 + px, o = mt * 32 + run * 8;
                        const float4 lo = *reinterpret_cast<const float4 *>(reg + px * kFuseRow + run * 8);
                        const float4 hi = *reinterpret_cast<const float4 *>(reg + px * kFuseRow + run * 8 + 4);
                        if (pg >= p.P) continue;
                        float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
                        if (p.res2 != nullptr) {
                            const u32x4 rr = *reinterpret_cast<const u32x4 *>(p.res2 + (size_t)pg * p.Cout2 + o);
#pragma unroll
                            for (int e = 0; e < 4; e++) {
                                v[2 * e] += widen<ODT>((uint16_t)(rr[e] & 0xFFFFu));
                                v[2 * e + 1] += widen<ODT>((uint16_t)(rr[e] >> 16));
                            }
                        }
                        uint32_t w[4];
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            float a = v[2 * e], b = v[2 * e + 1];
                            if (p.act2 == SS_ACT_GELU) { a = gelu(a); b = gelu(b); }
                            else { a = a < floor2 ? 0.f : a; b = b < floor2 ? 0.f : b; }
                            w[e] = cvt_pack2<ODT>(a, b);
                        }
                        *reinterpret_cast<uint4 *>(p.y2 + (size_t)pg * p.Cout2 + o) = make_uint4(w[0], w[1], w[2], w[3]);
                    }
                }
                cur = nxt;
            }
            return;
        }
        if (vec_ok) {
            for (int it = etid; it < BN * RUNS; it += NT) {
                const int pl = it / RUNS, run = it % RUNS;
                const int pg = n0 + pl, o = m0 + run * 8;
                if (pg >= p.P || o >= p.Cout) continue;
                const uint2 lo = *reinterpret_cast<const uint2 *>(Cs + pl * CROW + run * 8);
                const uint2 hi = *reinterpret_cast<const uint2 *>(Cs + pl * CROW + run * 8 + 4);
                *reinterpret_cast<uint4 *>(p.y + (size_t)pg * p.Cout + o) = make_uint4(lo.x, lo.y, hi.x, hi.y);
            }
        } else {
            // Channel counts whose pixel rows are not 16-byte aligned: consecutive lanes write consecutive 8-, 4- or 2-byte
            // pieces of a pixel (contiguous per instruction; eight 2-byte stores per thread, 16 bytes apart from lane to
            // lane, before).
            auto pieces = [&](auto piece) {
                using T = decltype(piece);
                constexpr int E = (int)sizeof(T) / 2, PER = BM / E;
                for (int it = etid; it < BN * PER; it += NT) {
                    const int pl = it / PER, c = (it % PER) * E;
                    const int pg = n0 + pl, o = m0 + c;
                    if (pg >= p.P || o >= p.Cout) continue;
                    *reinterpret_cast<T *>(p.y + (size_t)pg * p.Cout + o) = *reinterpret_cast<const T *>(Cs + pl * CROW + c);
                }
            };
            if ((p.Cout & 3) == 0) pieces(uint2{});
            else if ((p.Cout & 1) == 0) pieces(uint32_t{});
            else pieces(uint16_t{});
        }
    } else if constexpr (!Q8) {
        // With a residual the tile crosses LDS in fp32 (conv + bias); the thread that stores a 16-byte run adds the
        // residual's run (fetched before the tile is written, so its latency hides behind the LDS phase), applies
        // the activation and rounds once.
        constexpr int CROW = BM + 4;     // floats per pixel row (+16 bytes: 16-byte writes of consecutive pixels spread over the banks)
        constexpr int ITERS = (BN * RUNS + NT - 1) / NT;
        float *Cf = reinterpret_cast<float *>(smem);
        u32x4 res[ITERS];
        auto load_res = [&]() {
            if (!vec_ok) return;
#pragma unroll
            for (int j = 0; j < ITERS; j++) {
                const int it = etid + j * NT;
                const int pl = it / RUNS, run = it % RUNS;
                const int pg = n0 + pl, o = m0 + run * 8;
                res[j] = u32x4{0u, 0u, 0u, 0u};
                if (it < BN * RUNS && pg < p.P && o < p.Cout)
                    res[j] = *reinterpret_cast<const u32x4 *>(p.residual + (size_t)pg * p.Cout + o);
            }
        };
        if constexpr (DEEP) load_res();      // (the shallow variants have no registers to spare next to the accumulators)
        if (!producer) {
#pragma unroll
            for (int tm = 0; tm < TM; tm++) {
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int ol = (wm * TM + tm) * 32 + 8 * q + 4 * (lane >> 5);
                    const float4 bq = *reinterpret_cast<const float4 *>(bias_s + ol);
#pragma unroll
                    for (int tn = 0; tn < TN; tn++) {
                        const int pl = (wn * TN + tn) * 32 + (lane & 31);
                        *reinterpret_cast<float4 *>(Cf + pl * CROW + ol) =
                            make_float4((float)acc[tm][tn][4 * q + 0] + bq.x, (float)acc[tm][tn][4 * q + 1] + bq.y,
                                        (float)acc[tm][tn][4 * q + 2] + bq.z, (float)acc[tm][tn][4 * q + 3] + bq.w);
                    }
                }
            }
        }
        if constexpr (!DEEP) load_res();
        __syncthreads();
        auto from_lds = [&](auto actf) {
#pragma unroll
            for (int j = 0; j < ITERS; j++) {
                const int it = etid + j * NT;
                const int pl = it / RUNS, run = it % RUNS;
                const int pg = n0 + pl, o = m0 + run * 8;
                if (it >= BN * RUNS || pg >= p.P || o >= p.Cout) continue;
                const float4 lo = *reinterpret_cast<const float4 *>(Cf + pl * CROW + run * 8);
                const float4 hi = *reinterpret_cast<const float4 *>(Cf + pl * CROW + run * 8 + 4);
                const float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
                uint32_t w[4];
#pragma unroll
                for (int e = 0; e < 4; e++)
                    w[e] = cvt_pack2<ODT>(actf(v[2 * e] + widen<ODT>((uint16_t)(res[j][e] & 0xFFFFu))),
                                          actf(v[2 * e + 1] + widen<ODT>((uint16_t)(res[j][e] >> 16))));
                *reinterpret_cast<uint4 *>(p.y + (size_t)pg * p.Cout + o) = make_uint4(w[0], w[1], w[2], w[3]);
            }
        };
        // (pixel rows that are not 16-byte aligned: as in the plain tail, one 4- or 2-byte piece per lane)
        auto from_lds_pieces = [&](auto actf, auto piece) {
            using T = decltype(piece);
            constexpr int E = (int)sizeof(T) / 2, PER = BM / E;
            for (int it = etid; it < BN * PER; it += NT) {
                const int pl = it / PER, c = (it % PER) * E;
                const int pg = n0 + pl, o = m0 + c;
                if (pg >= p.P || o >= p.Cout) continue;
                const size_t at = (size_t)pg * p.Cout + o;
                const T r = *reinterpret_cast<const T *>(p.residual + at);
                const float a = actf(Cf[pl * CROW + c] + widen<ODT>((uint16_t)(r & 0xFFFFu)));
                const float b = E == 2 ? actf(Cf[pl * CROW + c + E - 1] + widen<ODT>((uint16_t)((uint32_t)r >> 16))) : 0.f;
                *reinterpret_cast<T *>(p.y + at) = (T)cvt_pack2<ODT>(a, b);
            }
        };
        if (!vec_ok) {
            auto run = [&](auto actf) {
                if ((p.Cout & 1) == 0) from_lds_pieces(actf, uint32_t{}); else from_lds_pieces(actf, uint16_t{});
            };
            if (p.act == SS_ACT_GELU) run(gelu); else run(relu_or_id);
            return;
        }
        if (p.act == SS_ACT_GELU) from_lds(gelu); else from_lds(relu_or_id);
    }
}

// ---------------------------------------------------------------------------------------------
// 1x1 -> activation -> 1x1 (+ residual): the inverted bottleneck of a ConvNeXt block (narrow -> 4x wide -> narrow)
// in one kernel.  A workgroup owns 64 pixels.  Their input rows are staged in LDS once; the wide intermediate is
// produced 128 channels at a time (first contraction, bias, activation, rounding to 16 bit, LDS) and consumed at
// once by the second contraction, whose accumulators stay in registers across the chunks.  The intermediate, four
// times the size of the block's input and output, never reaches memory.
// ---------------------------------------------------------------------------------------------


// KS1: reduction steps of the first layer; TILES: output tiles per wave; GELU1: the first layer's activation is GELU (not a branch inside:
// where the two loops meet again, accumulators went through memory)
template <int DT, bool SPARSE, int KS1, int TILES, bool GELU1>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(SPARSE ? 4 : (TILES == 1 ? 3 : 2))))
void mlp_kernel(MlpParams p)
{
    constexpr int BN = 64, CH = 128;                      // pixels per workgroup, intermediate channels per chunk
    constexpr int CIN = KS1 * 32;
    constexpr int CROW = CH + 4;                          // halfs per pixel row of the intermediate chunk (8-byte aligned rows)
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    constexpr int XROW = CIN + 8;                         // halfs per pixel row of the input tile (16-byte aligned rows)
    uint16_t *Xs = smem;
    uint16_t *Cs = smem + BN * XROW;
    float *b1s = reinterpret_cast<float *>(Cs + BN * CROW);       // the first layer's bias, all Cmid values
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 5, c = lane & 31;
    const int n0 = blockIdx.x * BN, px_here = min(BN, p.P - n0);
    // weight tiles: values, then (sparse) index words
    constexpr int Kp1 = (KS1 + 1) / 2;
    const int Ks2 = p.Cmid / 32, Kp2 = (Ks2 + 1) / 2, Mt2 = p.Cout2 / 32;
    auto buffer = [](const void *base, unsigned bytes) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, base != nullptr ? (int)bytes : 0, kRsrcFlags);
    };
    const __amdgpu_buffer_rsrc_t r1 = buffer(p.a1_vals, (unsigned)(Ks2 * KS1) * (SPARSE ? 1024u : 2048u));
    const __amdgpu_buffer_rsrc_t r2 = buffer(p.a2_vals, (unsigned)(Mt2 * Ks2) * (SPARSE ? 1024u : 2048u));
    const __amdgpu_buffer_rsrc_t m1 = buffer(p.a1_vals + (size_t)(Ks2 * KS1) * 1024, SPARSE ? (unsigned)(Ks2 * Kp1) * 256u : 4u);
    const __amdgpu_buffer_rsrc_t m2 = buffer(p.a2_vals + (size_t)(Mt2 * Ks2) * 1024, SPARSE ? (unsigned)(Mt2 * Kp2) * 256u : 4u);
    // input, residual and output of this workgroup's pixels: whatever lies behind the last one is out of range
    const __amdgpu_buffer_rsrc_t rx = buffer(p.x + (size_t)n0 * CIN, (unsigned)px_here * (CIN * 2u));
    const unsigned out_bytes = (unsigned)px_here * (unsigned)p.Cout2 * 2u;
    const __amdgpu_buffer_rsrc_t rres = buffer(p.res2 != nullptr ? p.res2 + (size_t)n0 * p.Cout2 : nullptr, out_bytes);
    const __amdgpu_buffer_rsrc_t ry = buffer(p.y2 + (size_t)n0 * p.Cout2, out_bytes);
    const __amdgpu_buffer_rsrc_t rb1 = buffer(p.bias1, (unsigned)p.Cmid * 4u), rb2 = buffer(p.bias2, (unsigned)p.Cout2 * 4u);

    struct Row1 {                                         // one 32-row tile of the first layer: all its reduction steps
        u32x4 v[SPARSE ? 1 : 2][KS1];
        uint32_t idx[KS1];
    };
    auto load_row1 = [&](Row1 &r, int mt) {
#pragma unroll
        for (int s = 0; s < KS1; s++) {
            if constexpr (SPARSE) {
                r.v[0][s] = __builtin_amdgcn_raw_buffer_load_b128(r1, lane * 16, (mt * KS1 + s) * 1024, 0);
                r.idx[s] = __builtin_amdgcn_raw_buffer_load_b32(m1, lane * 4, (mt * Kp1 + (s >> 1)) * 256, 0);
            } else {
                r.v[0][s] = __builtin_amdgcn_raw_buffer_load_b128(r1, lane * 16, (mt * KS1 + s) * 2048, 0);
                r.v[1][s] = __builtin_amdgcn_raw_buffer_load_b128(r1, lane * 16, (mt * KS1 + s) * 2048 + 1024, 0);
            }
        }
    };
    // The second layer's weights for this wave's output tiles and the 4 reduction steps of one chunk.  Tile t = wave + 4 * ti is row tile t / 2
    // on pixel half t % 2, the same half for all of a wave's tiles.  (A wave without a last tile repeats the last one's loads and drops the result.)
    struct Row2 {
        u32x4 v[SPARSE ? 1 : 2][TILES][4];
        uint32_t idx[TILES][4];
    };
    const int half = wave & 1;
    auto row_tile = [&](int ti) { return min((wave + 4 * ti) >> 1, Mt2 - 1); };
    auto load_row2 = [&](Row2 &r, int mc) {
#pragma unroll
        for (int ti = 0; ti < TILES; ti++) {
            const int rt = row_tile(ti);
#pragma unroll
            for (int s = 0; s < 4; s++) {
                const int ks = mc * 4 + s;
                if constexpr (SPARSE) {
                    r.v[0][ti][s] = __builtin_amdgcn_raw_buffer_load_b128(r2, lane * 16, (rt * Ks2 + ks) * 1024, 0);
                    r.idx[ti][s] = __builtin_amdgcn_raw_buffer_load_b32(m2, lane * 4, (rt * Kp2 + (ks >> 1)) * 256, 0);
                } else {
                    r.v[0][ti][s] = __builtin_amdgcn_raw_buffer_load_b128(r2, lane * 16, (rt * Ks2 + ks) * 2048, 0);
                    r.v[1][ti][s] = __builtin_amdgcn_raw_buffer_load_b128(r2, lane * 16, (rt * Ks2 + ks) * 2048 + 1024, 0);
                }
            }
        }
    };

    // ---- the input tile: 64 pixel rows of Cin channels, four threads to a row, zeros past the last pixel (all loads on their way first)
    Row1 a1;
    Row2 a2;
    f32x16 acc2[TILES];                                   // the bias starts in the accumulators
    {
        u32x4 v[KS1];
        const int row = tid >> 2, q4 = tid & 3;
#pragma unroll
        for (int i = 0; i < KS1; i++) v[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, row * (CIN * 2) + q4 * 16, i * 64, 0);
        load_row1(a1, wave);
#pragma unroll
        for (int ti = 0; ti < TILES; ti++)
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const f32x4 b = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rb2, g * 16, (row_tile(ti) * 32 + 8 * q) * 4, 0));
#pragma unroll
                for (int e = 0; e < 4; e++) acc2[ti][4 * q + e] = b[e];
            }
        for (int i = tid; i < p.Cmid; i += 256) b1s[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rb1, i * 4, 0, 0));
#pragma unroll
        for (int i = 0; i < KS1; i++) *reinterpret_cast<u32x4 *>(Xs + row * XROW + q4 * 8 + i * 32) = v[i];
    }
    // the residual, in the output stage's lane -> (pixel, run of 8 channels) mapping
    // (The pixel is in the vector offset alone, which by itself passes the buffer's end behind the last one: that the check counts the scalar offset
    // in is nothing the intrinsic promises.  The scalar offset stays within a pixel's row.)
    auto out_lane = [&](int j) { return (half * 32 + 16 * j + (lane >> 2)) * p.Cout2 * 2 + (lane & 3) * 16; };
    auto out_row = [&](int ti) { return row_tile(ti) * 64; };
    u32x4 rres2[TILES][2];
    auto load_res = [&]() {
#pragma unroll
        for (int ti = 0; ti < TILES; ti++)
#pragma unroll
            for (int j = 0; j < 2; j++) rres2[ti][j] = __builtin_amdgcn_raw_buffer_load_b128(rres, out_lane(j), out_row(ti), 0);
    };
    const float floor1 = p.act1 == SS_ACT_RELU ? 0.f : -__builtin_inff();
    __syncthreads();

    const int nchunks = p.Cmid / CH;
    const uint16_t *const x_frag = Xs + c * XROW + 16 * g;
    uint16_t *const c_dst = Cs + c * CROW + wave * 32 + 4 * g;
    int c_at = BN * XROW + (half * 32 + c) * CROW + 16 * g;
    asm volatile("" : "+v"(c_at));                        // (an address of its own: as an offset from another one it is too large for the instruction, and an addition per read)
    const uint16_t *const c_frag = smem + c_at;
    // Bound by the vector ALU: 154 M GELUs on the ConvNeXt-T stage-1 block at batch 128 are 61 us of it (twelve full-rate instructions of 4
    // clocks and one of 8 per wave).  What else the vector ALU does is kept small: the activation is chosen outside the element loop, addresses
    // are scalar, biases start in accumulators, the residual is fetched behind the chunks (during the last one, behind a condition, its registers
    // travelled through copies in every chunk), and four waves per SIMD (128 registers) overlap one's matrix instructions with another's
    // GELUs: 113 -> 96 us (graph of 20; counters in profiles/block_kernel_counters.md).
    auto chunk = [&](auto act1, int mc) {
        // ---- first contraction: rows 128*mc + 32*wave + [0,32) of the intermediate, all 64 pixels
        f32x16 acc1[2];                                   // the bias starts in the accumulators
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const float4 bq1 = *reinterpret_cast<const float4 *>(b1s + (mc * 4 + wave) * 32 + 8 * q + 4 * g);
            const float bv[4] = {bq1.x, bq1.y, bq1.z, bq1.w};
#pragma unroll
            for (int tn = 0; tn < 2; tn++)
#pragma unroll
                for (int e = 0; e < 4; e++) acc1[tn][4 * q + e] = bv[e];
        }
#pragma unroll
        for (int s = 0; s < KS1; s++) {
#pragma unroll
            for (int tn = 0; tn < 2; tn++) {
                const uint16_t *src = x_frag + tn * 32 * XROW + 32 * s;
                B32 bf;
                bf.lo = *reinterpret_cast<const u32x4 *>(src);
                bf.hi = *reinterpret_cast<const u32x4 *>(src + 8);
                if constexpr (SPARSE) {
                    acc1[tn] = mma_sparse<DT>(a1.v[0][s], bf, acc1[tn], a1.idx[s] >> ((s & 1) * 16));
                } else {
                    acc1[tn] = mma_dense<DT>(a1.v[0][s], bf.lo, acc1[tn]);
                    acc1[tn] = mma_dense<DT>(a1.v[1][s], bf.hi, acc1[tn]);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 4; q++) {
#pragma unroll
            for (int tn = 0; tn < 2; tn++) {
                float r[4];
#pragma unroll
                for (int e = 0; e < 4; e++) r[e] = act1(acc1[tn][4 * q + e]);
                *reinterpret_cast<uint2 *>(c_dst + tn * 32 * CROW + 8 * q) = make_uint2(cvt_pack2<DT>(r[0], r[1]), cvt_pack2<DT>(r[2], r[3]));
            }
            __builtin_amdgcn_sched_barrier(0);            // eight evaluations overlap; more at once cost a wave per SIMD in registers
        }
        // (issued here, when the first contraction's accumulators are dead: four waves per SIMD hide the latency better than an
        // earlier issue at three)
        load_row2(a2, mc);
        load_row1(a1, min(mc + 1, nchunks - 1) * 4 + wave);      // in flight while the second contraction runs (behind the last chunk: not used)
        lds_barrier();
        // ---- second contraction: this chunk's 128 intermediate channels into the output accumulators
        B32 bf[2];
        auto load_frag = [&](B32 &f, int s) {
            const uint16_t *src = c_frag + 32 * s;        // 8-byte aligned
            const uint2 u0 = *reinterpret_cast<const uint2 *>(src), u1 = *reinterpret_cast<const uint2 *>(src + 4);
            const uint2 u2 = *reinterpret_cast<const uint2 *>(src + 8), u3 = *reinterpret_cast<const uint2 *>(src + 12);
            f.lo = u32x4{u0.x, u0.y, u1.x, u1.y};
            f.hi = u32x4{u2.x, u2.y, u3.x, u3.y};
        };
        load_frag(bf[0], 0);
#pragma unroll
        for (int s = 0; s < 4; s++) {
            if (s < 3) load_frag(bf[(s + 1) & 1], s + 1);
#pragma unroll
            for (int ti = 0; ti < TILES; ti++) {
                if constexpr (SPARSE) {
                    acc2[ti] = mma_sparse<DT>(a2.v[0][ti][s], bf[s & 1], acc2[ti], a2.idx[ti][s] >> ((s & 1) * 16));
                } else {
                    acc2[ti] = mma_dense<DT>(a2.v[0][ti][s], bf[s & 1].lo, acc2[ti]);
                    acc2[ti] = mma_dense<DT>(a2.v[1][ti][s], bf[s & 1].hi, acc2[ti]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);            // (all four steps' fragments at once would not fit the registers)
        }
        lds_barrier();                                    // the chunk buffer is free again
    };
    auto chunks = [&](auto act1) {
        for (int mc = 0; mc < nchunks; mc++) chunk(act1, mc);
    };
    if constexpr (GELU1) chunks([](float z) { return gelu_cdf<DT>(z); });
    else chunks([floor1](float z) { return floor_at(z, floor1); });
    load_res();

    // ---- output: residual + activation in fp32, one rounding; each 32 x 32 tile crosses the wave's own LDS region
    // (the input tile and the chunk buffer are dead: the loop ended with a barrier) and leaves as 16-byte runs
    float *reg = reinterpret_cast<float *>(smem) + wave * (32 * kFuseRow);
    auto finish = [&](auto act2) {
#pragma unroll
        for (int ti = 0; ti < TILES; ti++) {
            if (wave + 4 * ti >= Mt2 * 2) break;          // uniform
#pragma unroll
            for (int q = 0; q < 4; q++)
                *reinterpret_cast<f32x4 *>(reg + c * kFuseRow + 8 * q + 4 * g) = f32x4{acc2[ti][4 * q + 0], acc2[ti][4 * q + 1], acc2[ti][4 * q + 2], acc2[ti][4 * q + 3]};
#pragma unroll
            for (int j = 0; j < 2; j++) {
                const float *src = reg + ((lane >> 2) + 16 * j) * kFuseRow + (lane & 3) * 8;
                const f32x4 lo = *reinterpret_cast<const f32x4 *>(src), hi = *reinterpret_cast<const f32x4 *>(src + 4);
                const float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                u32x4 w;
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const uint32_t rr = rres2[ti][j][e];
                    w[e] = cvt_pack2<DT>(act2(v[2 * e] + widen<DT>((uint16_t)(rr & 0xFFFFu))), act2(v[2 * e + 1] + widen<DT>((uint16_t)(rr >> 16))));
                }
                store_b128(w, ry, out_lane(j), out_row(ti));
            }
        }
    };
    if (p.act2 == SS_ACT_GELU) finish([](float z) { return gelu_cdf<DT>(z); });
    else if (p.act2 == SS_ACT_RELU) finish([](float z) { return floor_at(z, 0.f); });
    else finish([](float z) { return z; });
}

// The same two layers, resident: a wave takes 32 pixels through both layers at a time, the intermediate in registers.  A lane's 16 accumulators of a row
// tile are four runs of four consecutive channels of its pixel, that is four whole 2:4 blocks of the second reduction; with the 16-bit
// blocks 0 1 | 2 3 | 4 5 | 6 7 of the two lane halves swapped to 0 4 | 1 5 | 2 6 | 3 7 (four V_PERMLANE32_SWAP) they are the second layer's operand.
// So the intermediate passes neither LDS nor a barrier.  The weights of both layers lie in LDS, one workgroup per compute unit walks over its pixel
// tiles, and a wave asks for its next tile's input while it works on this one.
// Bound by memory with ReLU (231 MB in 46 us), by the vector ALU with GELU (of 2880 vector instructions per tile of 96 -> 384 -> 96 in bf16, 2500 are
// the GELUs).  With the weights from memory for each wave the address unit took as long as the vector ALU; with an accumulator tile more, to
// multiply ahead of the activations, three waves per SIMD had no registers left for weights on their way, and each matrix instruction waited for LDS.
// 401408 pixels, 96 -> 384 -> 96, bf16, mlp_kernel against this one, us: ReLU sparse 69.0 -> 46.0, dense 88.9 -> 57.7; GELU dense 116.8 -> 98.6
// (f16 114.9 -> 94.0).  TILES: 32-channel tiles of the input and of the output; WAVES: per workgroup.
template <int DT, bool SPARSE, int TILES, int WAVES, bool GELU1>
__global__ __launch_bounds__(WAVES * 64)
void mlp_resident_kernel(MlpParams p)
{
    using L = MlpPair<SPARSE, TILES>;
    constexpr int BN = 32, CIN = TILES * 32, STEP = L::STEP, NT = WAVES * 64, HALVES = SPARSE ? 1 : 2;
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    uint8_t *const ws = reinterpret_cast<uint8_t *>(smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 5, c = lane & 31;
    const int Ks2 = p.Cmid / 32, pairs = Ks2 / 2;         // (Cmid is a multiple of 128)
    // a lane's 16 consecutive channels of a tile of channels, and the pixels of tile t (none behind the last): two 16-byte runs
    const int px_at = c * (CIN * 2) + g * 32;
    auto pixels = [&](const uint16_t *base, int t) {
        // (clamping to a range is a vector instruction: read back, or every load would be a loop over its lanes' descriptors)
        const int here = __builtin_amdgcn_readfirstlane(max(0, min(BN, p.P - t * BN)));
        uint16_t *const at = reinterpret_cast<uint16_t *>(reinterpret_cast<uintptr_t>(base) + (size_t)t * (BN * CIN * 2));
        return __builtin_amdgcn_make_buffer_rsrc(at, 0, base != nullptr ? here * (CIN * 2) : 0, kRsrcFlags);
    };
    auto load_runs = [&](B32 (&f)[TILES], const __amdgpu_buffer_rsrc_t &r) {
#pragma unroll
        for (int t = 0; t < TILES; t++) {
            f[t].lo = __builtin_amdgcn_raw_buffer_load_b128(r, px_at, t * 64, 0);
            f[t].hi = __builtin_amdgcn_raw_buffer_load_b128(r, px_at, t * 64 + 16, 0);
        }
    };
    // (the first tiles go to all compute units before any gets a second one)
    const int ntiles = (p.P + BN - 1) / BN, stride = p.blocks * WAVES;
    int tile = wave * p.blocks + blockIdx.x;
    B32 x[TILES], xn[TILES];
    load_runs(x, pixels(p.x, tile));

    // ---- weights and biases to LDS
    {
        // the weights: rows of 1024 bytes, one per wave at a time (all of this but the lane's place is scalar)
        constexpr int LAYER = 2 * TILES * HALVES, AHEAD = 8;      // rows of a layer per pair; loads under way at once
        const int rows = pairs * 2 * LAYER;
        for (int r0 = wave; r0 < rows; r0 += WAVES * AHEAD) {
            u32x4 v[AHEAD];
#pragma unroll
            for (int i = 0; i < AHEAD; i++) {
                const int r = min(r0 + i * WAVES, rows - 1), pm = r / (2 * LAYER), k = r % (2 * LAYER), k2 = k - LAYER;
                const uint8_t *const src = k < LAYER ? p.a1_vals + (pm * LAYER + k) * 1024
                                                     : p.a2_vals + (k2 / (2 * HALVES) * pairs + pm) * (2 * STEP) + k2 % (2 * HALVES) * 1024;
                v[i] = *reinterpret_cast<const u32x4 *>(src + lane * 16);
            }
#pragma unroll
            for (int i = 0; i < AHEAD; i++) {
                const int r = r0 + i * WAVES;
                if (r < rows) *reinterpret_cast<u32x4 *>(ws + r / (2 * LAYER) * L::BYTES + r % (2 * LAYER) * 1024 + lane * 16) = v[i];
            }
        }
        // the rest of each pair, 16 bytes per thread
        constexpr int UNITS = (L::BYTES - L::I1) / 16;
        const int vals = Ks2 * TILES * STEP;
        for (int u = tid; u < pairs * UNITS; u += NT) {
            const int pm = u / UNITS, at = L::I1 + u % UNITS * 16;
            const uint8_t *src = p.bias1 != nullptr ? reinterpret_cast<const uint8_t *>(p.bias1) + pm * 256 + (at - L::BIAS) : nullptr;
            if (at < L::I2) src = p.a1_vals + vals + pm * (2 * L::KP1 * 256) + (at - L::I1);
            else if (at < L::BIAS) src = p.a2_vals + vals + ((at - L::I2) / 256 * pairs + pm) * 256 + (at - L::I2) % 256;
            u32x4 v = {0, 0, 0, 0};
            if (src != nullptr) v = *reinterpret_cast<const u32x4 *>(src);
            *reinterpret_cast<u32x4 *>(ws + pm * L::BYTES + at) = v;
        }
        if (tid < CIN) reinterpret_cast<float *>(ws + pairs * L::BYTES)[tid] = p.bias2 != nullptr ? p.bias2[tid] : 0.f;
    }
    lds_barrier();
    if (tile >= ntiles) return;
    // a wave with one tile more than the others of its SIMD goes first: done last and alone, that tile would have nothing to overlap with
    if (ntiles > stride && tile < ntiles % stride) __builtin_amdgcn_s_setprio(1);

    auto start = [&](f32x16 &acc, const uint8_t *bias) {  // the bias starts in the accumulators (bias: the lane half's place)
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const f32x4 b = *reinterpret_cast<const f32x4 *>(bias + 32 * q);
#pragma unroll
            for (int e = 0; e < 4; e++) acc[4 * q + e] = b[e];
        }
    };
    struct Weights {
        u32x4 v[HALVES][TILES];
        uint32_t idx[TILES];
    };
    auto mma = [](const Weights &w, int t, const B32 &b, f32x16 acc) {
        if constexpr (SPARSE) {
            return mma_sparse<DT>(w.v[0][t], b, acc, w.idx[t]);
        } else {
            acc = mma_dense<DT>(w.v[0][t], b.lo, acc);
            return mma_dense<DT>(w.v[HALVES - 1][t], b.hi, acc);
        }
    };
    // Runs of four channels, two dwords each: lane half g has channels 8 q + 4 g .. of the tile in run q; as 16 consecutive channels 16 g .. , and back
    // (the swap is its own inverse).
    auto swap_halves = [](uint32_t (&d)[4][2]) {
#pragma unroll
        for (int q = 0; q < 2; q++)
#pragma unroll
            for (int e = 0; e < 2; e++) {
                const auto r = __builtin_amdgcn_permlane32_swap(d[q][e], d[q + 2][e], false, false);
                d[q][e] = r[0];
                d[q + 2][e] = r[1];
            }
    };
    const float floor1 = p.act1 == SS_ACT_RELU ? 0.f : -__builtin_inff();
    auto act1 = [floor1](float z) { return GELU1 ? gelu_cdf<DT>(z) : floor_at(z, floor1); };

    f32x16 acc1, acc2[TILES];
    Weights w;
    const int at16 = lane * 16, at4 = lane * 4, atg = g * 16;
    // a row tile of the first layer, and the reduction step of the second that belongs to it (index words: the half that is the step's)
    auto request1 = [&](int pair, int odd) {
        start(acc1, ws + atg + pair + (L::BIAS + odd * 128));
#pragma unroll
        for (int s = 0; s < TILES; s++) {
#pragma unroll
            for (int h = 0; h < HALVES; h++) w.v[h][s] = *reinterpret_cast<const u32x4 *>(ws + at16 + pair + ((odd * TILES + s) * STEP + h * 1024));
            if (SPARSE) w.idx[s] = *reinterpret_cast<const uint16_t *>(ws + at4 + pair + (L::I1 + (odd * L::KP1 + s / 2) * 256 + s % 2 * 2));
        }
    };
    auto request2 = [&](int pair, int odd) {
#pragma unroll
        for (int t = 0; t < TILES; t++) {
#pragma unroll
            for (int h = 0; h < HALVES; h++) w.v[h][t] = *reinterpret_cast<const u32x4 *>(ws + at16 + pair + (L::W2 + (2 * t + odd) * STEP + h * 1024));
            if (SPARSE) w.idx[t] = *reinterpret_cast<const uint16_t *>(ws + at4 + pair + (L::I2 + t * 256 + odd * 2));
        }
    };
    B32 res[TILES];
    // One row tile through both layers; `next`, `next_odd`: the one behind it.
    auto step = [&](int pair, int odd, int next, int next_odd, auto last) {
#pragma unroll
        for (int s = 0; s < TILES; s++) acc1 = mma(w, s, x[s], acc1);
        if constexpr (decltype(last)::value) load_runs(res, pixels(p.res2, tile));
        request2(pair, odd);
        __builtin_amdgcn_sched_barrier(0);
        uint32_t d[4][2];
#pragma unroll
        for (int q = 0; q < 4; q++) {
            float r[4];
#pragma unroll
            for (int e = 0; e < 4; e++) r[e] = act1(acc1[4 * q + e]);
            d[q][0] = cvt_pack2<DT>(r[0], r[1]);
            d[q][1] = cvt_pack2<DT>(r[2], r[3]);
            if (q % 2 == 1) __builtin_amdgcn_sched_barrier(0);
        }
        swap_halves(d);
        const B32 f = {u32x4{d[0][0], d[0][1], d[2][0], d[2][1]}, u32x4{d[1][0], d[1][1], d[3][0], d[3][1]}};
#pragma unroll
        for (int t = 0; t < TILES; t++) acc2[t] = mma(w, t, f, acc2[t]);
        request1(next, next_odd);
        __builtin_amdgcn_sched_barrier(0);
    };
    request1(0, 0);
    for (; tile < ntiles; tile += stride) {
        load_runs(xn, pixels(p.x, tile + stride));
#pragma unroll
        for (int t = 0; t < TILES; t++) start(acc2[t], ws + atg + pairs * L::BYTES + t * 128);
        int pair = 0;
        for (int i = 0; i + 1 < pairs; i++, pair += L::BYTES) {
            step(pair, 0, pair, 1, std::false_type{});
            step(pair, 1, pair + L::BYTES, 0, std::false_type{});
        }
        step(pair, 0, pair, 1, std::false_type{});
        step(pair, 1, 0, 0, std::true_type{});            // (behind the last tile: not used)
#pragma unroll
        for (int t = 0; t < TILES; t++) x[t] = xn[t];

        // ---- output: residual and activation in fp32, one rounding
        const __amdgpu_buffer_rsrc_t ry = pixels(p.y2, tile);
        auto finish = [&](auto act2) {
#pragma unroll
            for (int t = 0; t < TILES; t++) {
                uint32_t rr[4][2] = {{res[t].lo[0], res[t].lo[1]}, {res[t].hi[0], res[t].hi[1]}, {res[t].lo[2], res[t].lo[3]}, {res[t].hi[2], res[t].hi[3]}}, d[4][2];
                swap_halves(rr);
#pragma unroll
                for (int q = 0; q < 4; q++)
#pragma unroll
                    for (int e = 0; e < 2; e++)
                        d[q][e] = cvt_pack2<DT>(act2(acc2[t][4 * q + 2 * e] + widen<DT>((uint16_t)(rr[q][e] & 0xFFFFu))),
                                                act2(acc2[t][4 * q + 2 * e + 1] + widen<DT>((uint16_t)(rr[q][e] >> 16))));
                swap_halves(d);
                store_b128(u32x4{d[0][0], d[0][1], d[2][0], d[2][1]}, ry, px_at, t * 64);
                store_b128(u32x4{d[1][0], d[1][1], d[3][0], d[3][1]}, ry, px_at, t * 64 + 16);
            }
        };
        if (p.act2 == SS_ACT_GELU) finish([](float z) { return gelu_cdf<DT>(z); });
        else if (p.act2 == SS_ACT_RELU) finish([](float z) { return floor_at(z, 0.f); });
        else finish([](float z) { return z; });
    }
}

// The same two layers on few pixels.  mlp_kernel's four waves take the intermediate 128 channels at a time, so that a workgroup lives for
// four chunks of weights, matrix instructions, activations and barriers in a row, which nothing hides where there is one workgroup per
// compute unit.  Here a workgroup owns 32 pixels and has a wave for each 32 channels of the intermediate: every wave computes
// its row tile at once, the whole intermediate meets in LDS, and the waves share out the second layer's row tiles and its reduction;
// the partial sums are added in the order of the reduction.  Weights, input and residual are one memory latency.  What is left is mostly the
// activation: 32 x 384 GELUs of 56 clocks on four SIMDs are 1.1 us of the 3.9 us that 96 -> 384 -> 96 on 3136 pixels takes (7.6 -> 5.5 us with the launch).
constexpr int mlp_wide_smem(int cin, int waves)
{
    const int tiles = 32 * (cin + 8) * 2 + 32 * (32 * waves + 8) * 2, sums = waves * (int)kFuseRegion;      // (the partial sums take the place of both tiles)
    return tiles > sums ? tiles : sums;
}

template <int DT, bool SPARSE, int KS1, bool GELU1>
__global__ __launch_bounds__(1024)
void mlp_wide_kernel(MlpParams p)
{
    constexpr int BN = 32, CIN = KS1 * 32, XROW = CIN + 8, STEPS = 4;      // STEPS: a wave's steps of the second reduction, at most
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    uint16_t *const Xs = smem, *const Ts = smem + BN * XROW;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 5, c = lane & 31;
    const int n0 = blockIdx.x * BN, px_here = min(BN, p.P - n0);
    constexpr int Kp1 = (KS1 + 1) / 2;
    const unsigned Ks2 = (unsigned)p.Cmid / 32, Kp2 = (Ks2 + 1) / 2, Mt2 = (unsigned)p.Cout2 / 32, nwaves = Ks2;
    const int TROW = p.Cmid + 8;
    auto buffer = [](const void *base, unsigned bytes) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, base != nullptr ? (int)bytes : 0, kRsrcFlags);
    };
    const __amdgpu_buffer_rsrc_t r1 = buffer(p.a1_vals, Ks2 * KS1 * (SPARSE ? 1024u : 2048u));
    const __amdgpu_buffer_rsrc_t r2 = buffer(p.a2_vals, Mt2 * Ks2 * (SPARSE ? 1024u : 2048u));
    const __amdgpu_buffer_rsrc_t m1 = buffer(p.a1_vals + (size_t)(Ks2 * KS1) * 1024, SPARSE ? Ks2 * Kp1 * 256u : 4u);
    const __amdgpu_buffer_rsrc_t m2 = buffer(p.a2_vals + (size_t)(Mt2 * Ks2) * 1024, SPARSE ? Mt2 * Kp2 * 256u : 4u);
    const __amdgpu_buffer_rsrc_t rx = buffer(p.x + (size_t)n0 * CIN, (unsigned)px_here * (CIN * 2u));
    const unsigned out_bytes = (unsigned)px_here * (unsigned)p.Cout2 * 2u;
    const __amdgpu_buffer_rsrc_t rres = buffer(p.res2 != nullptr ? p.res2 + (size_t)n0 * p.Cout2 : nullptr, out_bytes);
    const __amdgpu_buffer_rsrc_t ry = buffer(p.y2 + (size_t)n0 * p.Cout2, out_bytes);
    const __amdgpu_buffer_rsrc_t rb1 = buffer(p.bias1, (unsigned)p.Cmid * 4u), rb2 = buffer(p.bias2, (unsigned)p.Cout2 * 4u);

    // ---- everything that comes from memory
    // the input tile: CIN / 8 vectors of 16 bytes per pixel, BN * CIN / 8 = 128 KS1 in all
    u32x4 xv[2];
    const int NT = (int)nwaves * 64;
#pragma unroll
    for (int i = 0; i < 2; i++) xv[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, (tid + i * NT) * 16, 0, 0);
    u32x4 a1[SPARSE ? 1 : 2][KS1], a2[SPARSE ? 1 : 2][STEPS];
    uint32_t i1[KS1], i2[STEPS];
#pragma unroll
    for (int s = 0; s < KS1; s++) {
        if constexpr (SPARSE) {
            a1[0][s] = __builtin_amdgcn_raw_buffer_load_b128(r1, lane * 16, (wave * KS1 + s) * 1024, 0);
            i1[s] = __builtin_amdgcn_raw_buffer_load_b32(m1, lane * 4, (wave * Kp1 + (s >> 1)) * 256, 0);
        } else {
            a1[0][s] = __builtin_amdgcn_raw_buffer_load_b128(r1, lane * 16, (wave * KS1 + s) * 2048, 0);
            a1[1][s] = __builtin_amdgcn_raw_buffer_load_b128(r1, lane * 16, (wave * KS1 + s) * 2048 + 1024, 0);
        }
    }
    f32x16 acc;                                           // the bias starts in the accumulators
    auto start = [&](const __amdgpu_buffer_rsrc_t &rb, int row) {
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const f32x4 b = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rb, g * 16, (row + 8 * q) * 4, 0));
#pragma unroll
            for (int e = 0; e < 4; e++) acc[4 * q + e] = b[e];
        }
    };
    start(rb1, wave * 32);
    // the second layer: row tile rt, share `split` of the reduction (a wave without one repeats the last share's loads and is told apart at the end)
    const unsigned nsplit = nwaves / Mt2, split = (unsigned)wave / Mt2, rt = (unsigned)wave - split * Mt2;
    const unsigned per = (Ks2 + nsplit - 1) / nsplit, k0 = split * per;
#pragma unroll
    for (int s = 0; s < STEPS; s++) {
        const unsigned ks = min(k0 + s, Ks2 - 1);
        if constexpr (SPARSE) {
            a2[0][s] = __builtin_amdgcn_raw_buffer_load_b128(r2, lane * 16, (int)(rt * Ks2 + ks) * 1024, 0);
            i2[s] = __builtin_amdgcn_raw_buffer_load_b32(m2, lane * 4, (int)(rt * Kp2 + (ks >> 1)) * 256, 0);
        } else {
            a2[0][s] = __builtin_amdgcn_raw_buffer_load_b128(r2, lane * 16, (int)(rt * Ks2 + ks) * 2048, 0);
            a2[1][s] = __builtin_amdgcn_raw_buffer_load_b128(r2, lane * 16, (int)(rt * Ks2 + ks) * 2048 + 1024, 0);
        }
    }
    // output run `it`: row tile it / 128, pixel it % 128 / 4, 8 channels
    auto out_at = [&](int it) { return (it >> 2 & 31) * p.Cout2 * 2 + (it >> 7) * 64 + (it & 3) * 16; };
    const int runs = (int)Mt2 * 128;
    u32x4 res[2];
#pragma unroll
    for (int i = 0; i < 2; i++) {
        const int it = tid + i * NT;
        res[i] = __builtin_amdgcn_raw_buffer_load_b128(rres, it < runs ? out_at(it) : (int)kOutOfRange, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 2; i++) {
        const int at = tid + i * NT;
        if (at < 128 * KS1) *reinterpret_cast<u32x4 *>(Xs + at / (4 * KS1) * XROW + at % (4 * KS1) * 8) = xv[i];
    }
    lds_barrier();

    // ---- first layer: rows 32 wave .. of the intermediate
    {
        const uint16_t *const src = Xs + c * XROW + 16 * g;
#pragma unroll
        for (int s = 0; s < KS1; s++) {
            B32 bf;
            bf.lo = *reinterpret_cast<const u32x4 *>(src + 32 * s);
            bf.hi = *reinterpret_cast<const u32x4 *>(src + 32 * s + 8);
            if constexpr (SPARSE) {
                acc = mma_sparse<DT>(a1[0][s], bf, acc, i1[s] >> ((s & 1) * 16));
            } else {
                acc = mma_dense<DT>(a1[0][s], bf.lo, acc);
                acc = mma_dense<DT>(a1[1][s], bf.hi, acc);
            }
        }
        uint16_t *const dst = Ts + c * TROW + wave * 32 + 4 * g;
        const float floor1 = p.act1 == SS_ACT_RELU ? 0.f : -__builtin_inff();
#pragma unroll
        for (int q = 0; q < 4; q++) {
            float r[4];
#pragma unroll
            for (int e = 0; e < 4; e++) r[e] = GELU1 ? gelu_cdf<DT>(acc[4 * q + e]) : floor_at(acc[4 * q + e], floor1);
            *reinterpret_cast<uint2 *>(dst + 8 * q) = make_uint2(cvt_pack2<DT>(r[0], r[1]), cvt_pack2<DT>(r[2], r[3]));
        }
    }
    lds_barrier();

    // ---- second layer
#pragma unroll
    for (int e = 0; e < 16; e++) acc[e] = 0.f;
    if (split < nsplit) {                                 // uniform
        const uint16_t *const src = Ts + c * TROW + 16 * g;
#pragma unroll
        for (int s = 0; s < STEPS; s++) {
            const unsigned ks = k0 + s;
            if ((unsigned)s >= per || ks >= Ks2) break;   // uniform
            B32 bf;
            bf.lo = *reinterpret_cast<const u32x4 *>(src + 32 * ks);
            bf.hi = *reinterpret_cast<const u32x4 *>(src + 32 * ks + 8);
            if constexpr (SPARSE) {
                acc = mma_sparse<DT>(a2[0][s], bf, acc, i2[s] >> ((ks & 1) * 16));
            } else {
                acc = mma_dense<DT>(a2[0][s], bf.lo, acc);
                acc = mma_dense<DT>(a2[1][s], bf.hi, acc);
            }
        }
    }
    lds_barrier();                                        // the tiles are dead: the partial sums take their place
    float *const sums = reinterpret_cast<float *>(smem);
    if (split < nsplit) {
        float *const dst = sums + wave * (32 * kFuseRow) + c * kFuseRow + 4 * g;
#pragma unroll
        for (int q = 0; q < 4; q++) *reinterpret_cast<f32x4 *>(dst + 8 * q) = f32x4{acc[4 * q + 0], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    }
    lds_barrier();

    // ---- output: the shares in their order, bias, residual and activation in fp32, one rounding, 16-byte runs
    auto finish = [&](auto act2) {
#pragma unroll
        for (int i = 0; i < 2; i++) {
            const int it = tid + i * NT;
            if (it >= runs) break;
            const float *src = sums + (it >> 7) * (32 * kFuseRow) + (it >> 2 & 31) * kFuseRow + (it & 3) * 8;
            f32x4 lo = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rb2, ((it >> 7) * 32 + (it & 3) * 8) * 4, 0, 0));
            f32x4 hi = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rb2, ((it >> 7) * 32 + (it & 3) * 8) * 4 + 16, 0, 0));
            for (unsigned j = 0; j < nsplit; j++) {
                lo += *reinterpret_cast<const f32x4 *>(src + j * Mt2 * (32 * kFuseRow));
                hi += *reinterpret_cast<const f32x4 *>(src + j * Mt2 * (32 * kFuseRow) + 4);
            }
            const float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            u32x4 w;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const uint32_t rr = res[i][e];
                w[e] = cvt_pack2<DT>(act2(v[2 * e] + widen<DT>((uint16_t)(rr & 0xFFFFu))), act2(v[2 * e + 1] + widen<DT>((uint16_t)(rr >> 16))));
            }
            __builtin_amdgcn_raw_buffer_store_b128(w, ry, out_at(it), 0, 0);
        }
    };
    if (p.act2 == SS_ACT_GELU) finish([](float z) { return gelu_cdf<DT>(z); });
    else if (p.act2 == SS_ACT_RELU) finish([](float z) { return floor_at(z, 0.f); });
    else finish([](float z) { return z; });
}

template <int DT, bool SPARSE>
static int launch_mlp_wide(const MlpParams &p, hipStream_t s)
{
    const int waves = p.Cmid / 32, smem = mlp_wide_smem(p.Cin, waves);
    const long long blocks = ((long long)p.P + 31) / 32;
    if (blocks <= 0 || blocks > 0x7FFFFFFFll || waves > kMlpWideWaves) return SS_ERR_UNSUPPORTED;
    auto go = [&](auto ks1) {
        constexpr int KS1 = decltype(ks1)::value;
        const auto kern = p.act1 == SS_ACT_GELU ? mlp_wide_kernel<DT, SPARSE, KS1, true> : mlp_wide_kernel<DT, SPARSE, KS1, false>;
        if (smem > 64 * 1024) {
            // (once per device and kernel; two threads racing here both set it: harmless)
            static std::atomic<unsigned long long> done_mask[2];
            std::atomic<unsigned long long> &done = done_mask[p.act1 == SS_ACT_GELU];
            int dev = 0;
            if (hipGetDevice(&dev) != hipSuccess) return (int)SS_ERR_HIP;
            const unsigned long long bit = 1ull << (dev & 63);
            if (dev >= 64 || !(done.load(std::memory_order_acquire) & bit)) {
                if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                        mlp_wide_smem(128, kMlpWideWaves)) != hipSuccess)
                    return (int)SS_ERR_HIP;
                if (dev < 64) done.fetch_or(bit, std::memory_order_release);
            }
        }
        kern<<<dim3((unsigned)blocks), dim3(waves * 64), smem, s>>>(p);
        return (int)(hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_HIP);
    };
    using std::integral_constant;
    switch (p.Cin / 32) {
        case 1: return go(integral_constant<int, 1>{});
        case 2: return go(integral_constant<int, 2>{});
        case 3: return go(integral_constant<int, 3>{});
        case 4: return go(integral_constant<int, 4>{});
        default: return SS_ERR_UNSUPPORTED;
    }
}

// The resident kernel on so many channels, if its weights fit the LDS.
template <int DT, bool SPARSE, int TILES>
static int launch_mlp_resident(const MlpParams &p0, int ncu, hipStream_t s)
{
    constexpr int WAVES = TILES <= 3 ? 12 : 8;            // three waves per SIMD, or the two that their registers leave room for
    MlpParams p = p0;
    const int tiles = (int)(((long long)p.P + 31) / 32), limit = block_limit();
    p.blocks = tiles < ncu ? tiles : ncu;
    if (limit > 0 && p.blocks > limit) p.blocks = limit;
    if (p.blocks <= 0) return SS_ERR_UNSUPPORTED;
    auto kern = mlp_resident_kernel<DT, SPARSE, TILES, WAVES, false>;
    if constexpr (!SPARSE) kern = p.act1 == SS_ACT_GELU ? mlp_resident_kernel<DT, SPARSE, TILES, WAVES, true> : kern;
    // (once per device and kernel; two threads racing here both set it: harmless)
    static std::atomic<unsigned long long> done_mask[2];
    std::atomic<unsigned long long> &done = done_mask[p.act1 == SS_ACT_GELU];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return SS_ERR_HIP;
    const unsigned long long bit = 1ull << (dev & 63);
    if (dev >= 64 || !(done.load(std::memory_order_acquire) & bit)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kMlpResidentSmem) != hipSuccess)
            return SS_ERR_HIP;
        if (dev < 64) done.fetch_or(bit, std::memory_order_release);
    }
    kern<<<dim3((unsigned)p.blocks), dim3(WAVES * 64), (MlpPair<SPARSE, TILES>::smem(p.Cmid)), s>>>(p);
    return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_HIP;
}

template <int DT, bool SPARSE>
static int launch_mlp(const MlpParams &p, hipStream_t s)
{
    const int forced = forced_tile(), ncu = compute_units();
    if (ncu <= 0) return SS_ERR_HIP;
    const int id = forced >= 40 && forced <= 42 && mlp_takes(p, SPARSE, forced) ? forced : choose_mlp(p, SPARSE, ncu);
    if (id == 41) return launch_mlp_wide<DT, SPARSE>(p, s);
    if (id == 42) {
        if constexpr (SPARSE) return p.Cin == 96 ? launch_mlp_resident<DT, SPARSE, 3>(p, ncu, s) : launch_mlp_resident<DT, SPARSE, 4>(p, ncu, s);
        else return launch_mlp_resident<DT, SPARSE, 3>(p, ncu, s);
    }
    const long long blocks = ((long long)p.P + 63) / 64;
    if (blocks <= 0 || blocks > 0x7FFFFFFFll) return SS_ERR_UNSUPPORTED;
    size_t smem = (size_t)64 * (p.Cin + 8) * 2 + (size_t)64 * (128 + 4) * 2 + (size_t)p.Cmid * 4;
    const size_t epi = 4 * kFuseRegion;
    if (smem < epi) smem = epi;
    auto go = [&](auto ks1) {
        constexpr int KS1 = decltype(ks1)::value;
        const bool gelu = p.act1 == SS_ACT_GELU;
        const auto kern = p.Cout2 <= 64 ? (gelu ? mlp_kernel<DT, SPARSE, KS1, 1, true> : mlp_kernel<DT, SPARSE, KS1, 1, false>)
                                        : (gelu ? mlp_kernel<DT, SPARSE, KS1, 2, true> : mlp_kernel<DT, SPARSE, KS1, 2, false>);
        kern<<<dim3((unsigned)blocks), dim3(256), smem, s>>>(p);
        return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_HIP;
    };
    using std::integral_constant;
    switch (p.Cin / 32) {
        case 1: return go(integral_constant<int, 1>{});
        case 2: return go(integral_constant<int, 2>{});
        case 3: return go(integral_constant<int, 3>{});
        case 4: return go(integral_constant<int, 4>{});
        default: return SS_ERR_UNSUPPORTED;
    }
}

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
template <int DT, bool SPARSE, int WAVES_M, int WAVES_N, int TM, int TN, int MODE, int KH, int KW, bool DEEP = false, bool SPEC = false, bool FUSE = false, int THIRD = 0>
static int launch(const kernel_params<THIRD> &p0, hipStream_t s)
{
    constexpr int BM = WAVES_M * TM * 32, BN = WAVES_N * TN * 32;
    constexpr int NWAVES = WAVES_M * WAVES_N + (SPEC ? 4 : 0);
    constexpr size_t scale_bytes = is_byte_type(DT) ? (size_t)BM * 4 : 0;      // the per-channel scales sit behind the bias values
    constexpr size_t smem_plain = smem_bytes<BM, BN, MODE, KH, KW, DEEP>(false, FUSE ? NWAVES : 0, THIRD > 0) + scale_bytes;
    constexpr size_t smem_res = (is_byte_type(DT) || FUSE) ? smem_plain : smem_bytes<BM, BN, MODE, KH, KW, DEEP>(true);
    static_assert(smem_plain <= 160 * 1024 && smem_res <= 160 * 1024, "LDS tile too large");
    const size_t smem = (p0.residual && !FUSE) ? smem_res : smem_plain;
    if (FUSE && (p0.Cout > BM || p0.Cout % 32 != 0)) return SS_ERR_UNSUPPORTED;      // the whole channel range must sit in one tile
    kernel_params<THIRD> p = p0;
    p.tiles_m = (p.Cout + BM - 1) / BM;
    fast_div_setup((unsigned)p.tiles_m, &p.tm_mul, &p.tm_sh);
    long long tiles_n = ((long long)p.P + BN - 1) / BN;
    long long blocks = (long long)p.tiles_m * tiles_n;
    if (FUSE || is_byte_type(DT) || p.nsplit < 1) p.nsplit = 1;
    if (p.nsplit > 1) {
        // the entry point planned the split for this very tile shape (plan_split) and sized the workspace for it
        if (p.ws_part == nullptr || p.plan_bm != BM || p.plan_bn != BN) return SS_ERR_WORKSPACE;
        blocks *= p.nsplit;
    }
    if (blocks <= 0 || blocks > 0x7FFFFFFFll) return SS_ERR_UNSUPPORTED;
    auto kern = conv_kernel<DT, SPARSE, WAVES_M, WAVES_N, TM, TN, MODE, KH, KW, DEEP, SPEC, FUSE, THIRD>;
    if (smem_res > 64 * 1024) {
        // Raises this kernel's dynamic-LDS limit, once per device (the attribute belongs to the device's copy of the
        // kernel).  Two threads racing here both set it: harmless.
        static std::atomic<unsigned long long> done_mask{0};
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) return SS_ERR_HIP;
        const unsigned long long bit = 1ull << (dev & 63);
        if (dev >= 64 || !(done_mask.load(std::memory_order_acquire) & bit)) {
            if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)smem_res) != hipSuccess)
                return SS_ERR_HIP;
            if (dev < 64) done_mask.fetch_or(bit, std::memory_order_release);
        }
    }
    const dim3 grid((unsigned)blocks), block((WAVES_M * WAVES_N + (SPEC ? 4 : 0)) * 64);
    if constexpr (short_args(MODE, FUSE)) kern<<<grid, block, smem, s>>>(conv_args(p, false, is_vec(MODE)));
    else kern<<<grid, block, smem, s>>>(p);
    return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_HIP;
}

// Staging modes with tiles of 96, 160 and 224 rows (choose_height).  1x1 layers gain nothing from them (over 1000 layers: 1 %), 2x2 ones 3 %.
constexpr bool any_height(int mode, int kh) { return (is_taps(mode) && kh == 3) || mode == MODE_VEC; }
constexpr bool dense_f8(int dt, bool sparse) { return dt == SS_F8 && !sparse; }

// Tile shapes (WAVES_M x WAVES_N multiplying waves, each TM x TN tiles of 32x32):
//   id 0:  64 x  64 (2x2 waves, 1x1)
//   id 1:  same, deep prefetch
//   id 2: 128 x  64 (4x1 waves, 1x2)
//   id 3: 256 x  64 (4x1 waves, 2x2), deep prefetch
//   id 4: 128 x  64 (4x1 waves, 1x2), deep prefetch, plus four producer waves
//   id 5: 256 x  64 (4x1 waves, 2x2), deep prefetch, plus four producer waves
//   ids 6, 7, 8: 96, 160, 224 x 64 (3, 5, 7 x 1 waves, 1x2), for output channels that fill the others badly
// Layouts with all four waves along the output channels fetch no weight tile twice inside a workgroup.
// Measured and dropped because they won nowhere: 2x2 layouts of the larger tiles, 128x128 and 256x128 tiles,
// deep 128x64 and shallow 256x64 without producer waves, and splitting a tile's reduction over two wave groups
// (halves the LDS reads per multiply, but the exchange of partial sums and the doubled first chunk cost more), and a
// 128x64 tile of two multiplying waves of 64x64 plus producers (half the LDS reads of id 4, same memory traffic:
// 11.2 vs 9.6 us on the 3x3 256 -> 256 layer at batch 32 -- two waves do not keep four SIMDs' worth of latency hidden).
template <int DT, bool SPARSE, int MODE, int KH, int KW>
static int launch_tile(int id, const ConvParams &p, hipStream_t s)
{
    if constexpr (MODE != MODE_VEC8) {       // (the long-chunk staging is only ever paired with the deep tiles)
        switch (id) {
            case 0: return launch<DT, SPARSE, 2, 2, 1, 1, MODE, KH, KW, false>(p, s);
            case 1: return launch<DT, SPARSE, 2, 2, 1, 1, MODE, KH, KW, true>(p, s);
            case 2: return launch<DT, SPARSE, 4, 1, 1, 2, MODE, KH, KW, false>(p, s);
            default: break;
        }
    }
    if constexpr (any_height(MODE, KH) && !(dense_f8(DT, SPARSE) && is_taps(MODE))) {
        if (id == 6) return launch<DT, SPARSE, 3, 1, 1, 2, MODE, KH, KW, false>(p, s);
    }
    if constexpr (any_height(MODE, KH) && !dense_f8(DT, SPARSE)) {
        if (id == 7) return launch<DT, SPARSE, 5, 1, 1, 2, MODE, KH, KW, false>(p, s);
        if (id == 8) return launch<DT, SPARSE, 7, 1, 1, 2, MODE, KH, KW, false>(p, s);
    }
    if constexpr (MODE != MODE_VEC8) {
        if (id == 3) return launch<DT, SPARSE, 4, 1, 2, 2, MODE, KH, KW, true>(p, s);
    }
    switch (id) {
        case 4: return launch<DT, SPARSE, 4, 1, 1, 2, MODE, KH, KW, true, true>(p, s);
        case 5: return launch<DT, SPARSE, 4, 1, 2, 2, MODE, KH, KW, true, true>(p, s);
        default: break;
    }
    return SS_ERR_INVALID_ARG;
}

template <int DT, bool SPARSE, int MODE, int KH, int KW>
static int pick_tile(const ConvParams &p, hipStream_t s)
{
    if (p.nsplit > 1) return launch_tile<DT, SPARSE, MODE, KH, KW>(p.plan_tile, p, s);     // planned by the entry point
    const int forced = forced_tile();                  // test hook (ss_debug.h): a tile shape by id, or -1
    if (forced >= 0) {
        int st = launch_tile<DT, SPARSE, MODE, KH, KW>(forced, p, s);
        if (st != SS_ERR_INVALID_ARG) return st;
    }
    constexpr bool pointwise = is_pw(MODE);
    constexpr bool bigchunk = (is_taps(MODE) && KH * KW > 4) || MODE == MODE_VEC8;
    int id = choose_tile(p, pointwise, bigchunk);
    if constexpr (is_taps(MODE) && KH == 3) {
        const int ncu = compute_units();
        if (ncu <= 0) return SS_ERR_HIP;
        id = choose_height(p, id, true, is_byte_type(DT), SPARSE, ncu, DT == SS_F8);
    }
    // The dense FP8 instruction of the deep kernels wants its 32-byte A operand in eight consecutive registers; the
    // 256x64 four-wave tile then runs at one wave per SIMD (measured 40 % slower than with producer waves).
    if (DT == SS_F8 && !SPARSE && id == 3) id = 5;
    return launch_tile<DT, SPARSE, MODE, KH, KW>(id, p, s);
}

// Channels-last flattening with taps (the choice: choose_vec).
template <int DT, bool SPARSE>
static int pick_vec(const ConvParams &p, hipStream_t s)
{
    const int forced = forced_tile(), ncu = compute_units();
    if (ncu <= 0) return SS_ERR_HIP;
    if (p.K < 512)
        return forced >= 0 ? pick_tile<DT, SPARSE, MODE_VEC, 1, 1>(p, s)
                           : launch_tile<DT, SPARSE, MODE_VEC, 1, 1>(choose_vec_short(p, is_byte_type(DT), SPARSE, DT == SS_F8, ncu), p, s);
    if (forced >= 0) return forced == 4 || forced == 5 ? pick_tile<DT, SPARSE, MODE_VEC8, 1, 1>(p, s) : pick_tile<DT, SPARSE, MODE_VEC, 1, 1>(p, s);
    int id = choose_height(p, choose_vec(p, is_byte_type(DT), SPARSE, ncu), false, is_byte_type(DT), SPARSE, ncu, DT == SS_F8);
    if (is_byte_type(DT) && SPARSE) id = choose_vec8_sparse(p, id, ncu);
    if (id == 4 || id == 5) return launch_tile<DT, SPARSE, MODE_VEC8, 1, 1>(id, p, s);
    return launch_tile<DT, SPARSE, MODE_VEC, 1, 1>(id, p, s);
}

template <int DT, bool SPARSE>
static int pick_mode(const ss_weight_desc *desc, const ConvParams &p, hipStream_t s)
{
    const int taps = desc->kh * desc->kw;
    if constexpr (is_byte_type(DT)) {    // validated by the entry point: byte pairs are contiguous in every 16-byte run
        if (taps == 1) return p.Ks <= 2 ? pick_tile<DT, SPARSE, MODE_PW2, 1, 1>(p, s) : pick_tile<DT, SPARSE, MODE_PW, 1, 1>(p, s);
        if (desc->korder == SS_K_RSC) return pick_vec<DT, SPARSE>(p, s);
        if (desc->kh == 3) return pick_tile<DT, SPARSE, MODE_TAPS, 3, 3>(p, s);
        return pick_tile<DT, SPARSE, MODE_TAPS, 2, 2>(p, s);
    } else {
    // channels contiguous inside every aligned run of 8 reduction indices?
    if (desc->cin % 8 == 0 && taps == 1)
        return p.Ks <= 2 ? pick_tile<DT, SPARSE, MODE_PW2, 1, 1>(p, s) : pick_tile<DT, SPARSE, MODE_PW, 1, 1>(p, s);
    if (desc->cin % 8 == 0 && desc->korder == SS_K_RSC) return pick_vec<DT, SPARSE>(p, s);
    if (desc->korder == SS_K_CRS && desc->cin % 32 == 0) {
        if (desc->kh == 3 && desc->kw == 3) return pick_tile<DT, SPARSE, MODE_TAPS, 3, 3>(p, s);
        if (desc->kh == 2 && desc->kw == 2) return pick_tile<DT, SPARSE, MODE_TAPS, 2, 2>(p, s);
    }
    if (desc->cin % 4 == 0 && desc->cin >= 8) {
        if (taps == 1 && p.Ks > 2) return pick_tile<DT, SPARSE, MODE_PWR, 1, 1>(p, s);
        if (desc->korder == SS_K_CRS && desc->kh == 3 && desc->kw == 3) return pick_tile<DT, SPARSE, MODE_TAPSR, 3, 3>(p, s);
        if (desc->korder == SS_K_CRS && desc->kh == 2 && desc->kw == 2) return pick_tile<DT, SPARSE, MODE_TAPSR, 2, 2>(p, s);
        if (taps == 1) return pick_tile<DT, SPARSE, MODE_GATHER4, 1, 1>(p, s);
    }
    if (desc->cin % 4 == 0 && desc->korder == SS_K_RSC) return pick_tile<DT, SPARSE, MODE_GATHER4, 1, 1>(p, s);
    return pick_tile<DT, SPARSE, MODE_GATHER, 1, 1>(p, s);
    }
}

// ---------------------------------------------------------------------------------------------
// 3x3 (or any k x k with a fast staging mode) convolution followed by a 1x1 convolution, fused
// ---------------------------------------------------------------------------------------------
template <int DT, bool SPARSE, int MODE, int KH, int KW>
static int launch_fused_tile(int id, const ConvParams &p, hipStream_t s)
{
    switch (id) {
        case 0: return launch<DT, SPARSE, 2, 2, 1, 1, MODE, KH, KW, false, false, true>(p, s);
        case 1: return launch<DT, SPARSE, 2, 2, 1, 1, MODE, KH, KW, true, false, true>(p, s);
        case 2: return launch<DT, SPARSE, 4, 1, 1, 2, MODE, KH, KW, false, false, true>(p, s);
        case 3: return launch<DT, SPARSE, 4, 1, 2, 2, MODE, KH, KW, true, false, true>(p, s);
        case 4: return launch<DT, SPARSE, 4, 1, 1, 2, MODE, KH, KW, true, true, true>(p, s);
        case 5: return launch<DT, SPARSE, 4, 1, 2, 2, MODE, KH, KW, true, true, true>(p, s);
        default: break;
    }
    return SS_ERR_INVALID_ARG;
}

// With a third contraction: the paper's flattening, tiles of 64 or 128 rows without producer waves.
template <int DT, bool SPARSE>
static int third_mode(const ss_weight_desc *d1, const ChainParams &p, hipStream_t s)
{
    if (d1->korder != SS_K_CRS || d1->kh != 3 || d1->kw != 3 || d1->cin % 32 != 0) return SS_ERR_UNSUPPORTED;
    if (p.Cout > 128 || p.Cout3 > 128) return SS_ERR_UNSUPPORTED;
    if (p.Cout > 64) return launch<DT, SPARSE, 4, 1, 1, 2, MODE_TAPS, 3, 3, false, false, true, 2>(p, s);
    return p.Cout3 <= 64 ? launch<DT, SPARSE, 2, 2, 1, 1, MODE_TAPS, 3, 3, false, false, true, 1>(p, s)
                         : launch<DT, SPARSE, 2, 2, 1, 1, MODE_TAPS, 3, 3, false, false, true, 2>(p, s);
}

template <int DT, bool SPARSE>
static int fused_mode(const ss_weight_desc *d1, const ChainParams &p, hipStream_t s)
{
    if (p.Cout3 > 0) return third_mode<DT, SPARSE>(d1, p, s);
    auto run = [&](int id) {
        if (d1->korder == SS_K_CRS && d1->kh == 3 && d1->kw == 3 && d1->cin % 32 == 0)
            return launch_fused_tile<DT, SPARSE, MODE_TAPS, 3, 3>(id, p, s);
        if (d1->korder == SS_K_RSC && d1->cin % 8 == 0) return launch_fused_tile<DT, SPARSE, MODE_VEC, 1, 1>(id, p, s);
        return (int)SS_ERR_UNSUPPORTED;
    };
    const int forced = forced_tile();      // test hook; a tile that cannot hold the first layer's channels falls back
    if (forced >= 0) {
        const int st = run(forced);
        if (st != SS_ERR_UNSUPPORTED && st != SS_ERR_INVALID_ARG) return st;
    }
    return run(choose_fused_tile(p));
}

}  // namespace ss

#endif
