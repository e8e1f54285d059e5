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
// This file holds the entry points: argument validation, the parameter block, and the hand-over to the translation
// unit that instantiates the kernels for the operand type (ss_conv_kernel.h, ss_conv_inst_*.hip).
#include "ss_conv_params.h"
#include "../../include/ss_debug.h"
#include <atomic>

namespace ss {

static std::atomic<int> g_forced_tile{-1};
int forced_tile() { return g_forced_tile.load(std::memory_order_relaxed); }
static std::atomic<int> g_block_limit{0};
int block_limit() { return g_block_limit.load(std::memory_order_relaxed); }
static std::atomic<int> g_forced_split{0};
int forced_split() { return g_forced_split.load(std::memory_order_relaxed); }

// Compute units the split heuristic plans for: those of the current device, or 256 (the MI355X count) when the runtime
// has no device to ask, so that the size query still answers on a build host.
static int planning_units()
{
    const int n = compute_units();
    return n > 0 ? n : 256;
}

int compute_units()
{
    static std::atomic<int> cached[64];                   // 0 = not asked yet
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return -1;
    if (dev >= 0 && dev < 64) {
        const int c = cached[dev].load(std::memory_order_relaxed);
        if (c > 0) return c;
    }
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return -1;
    if (dev >= 0 && dev < 64) cached[dev].store(n, std::memory_order_relaxed);
    return n;
}

// Offsets in the kernels are 32 bits, and "out of range" must stay above every real one.  (out_channels: of the widest output; asked by the calls and
// by their queries.)
static bool within_limits(const ss_weight_desc *d, int32_t N, int32_t H, int32_t Wd, int32_t ph, int32_t pw, int esize, long long P, long long out_channels)
{
    const long long xbytes = (long long)N * H * Wd * d->cin * esize;
    return xbytes < (1ll << 31) - (1ll << 26) && P * out_channels < (1ll << 31) && P < (1ll << 31) - 512 &&
           (long long)(ph + d->kh + 1) * (Wd + pw + d->kw) * d->cin * esize < (1ll << 26);
}

// q8: the call came through an 8-bit entry point (then `scale` may be given and the descriptor must say SS_I8 or
// SS_F8); the 16-bit entry points reject such descriptors.  pooled: where the 3x3 max pooling behind an image's first layer goes, in the same kernel.
template <bool SPARSE>
static int conv_entry(const ss_weight_desc *desc, const void *x, int32_t N, int32_t H, int32_t Wd, const void *wbuf,
                      const float *bias, const void *residual, int32_t sh, int32_t sw, int32_t ph, int32_t pw,
                      int32_t act, void *y, void *workspace, size_t ws_bytes, void *stream, bool q8 = false,
                      const float *scale = nullptr, void *pooled = nullptr)
{
    int st = check_desc(desc, SPARSE);
    if (st != SS_OK) return st;
    if (is_byte_type(desc->dtype) != q8) return q8 ? SS_ERR_INVALID_ARG : SS_ERR_UNSUPPORTED;
    const int esize = q8 ? 1 : 2;      // bytes per activation / weight element
    if (q8) {
        if (desc->cin % 16 != 0) return SS_ERR_UNSUPPORTED;
        if (desc->korder == SS_K_CRS && desc->kh * desc->kw != 1) {     // taps inside a block: the byte transpose
            const bool square = (desc->kh == 3 && desc->kw == 3) || (desc->kh == 2 && desc->kw == 2);
            if (!square || desc->cin % 64 != 0) return SS_ERR_UNSUPPORTED;
        }
        if (desc->dtype == SS_I8 && (long long)desc->cin * desc->kh * desc->kw > 131071) return SS_ERR_UNSUPPORTED;      // int32 sums
        if (scale && !aligned(scale, 4)) return SS_ERR_INVALID_ARG;
    }
    if (!x || !wbuf || !y) return SS_ERR_INVALID_ARG;
    if (N <= 0 || H <= 0 || Wd <= 0 || sh <= 0 || sw <= 0 || ph < 0 || pw < 0) return SS_ERR_INVALID_ARG;
    if (act != SS_ACT_NONE && act != SS_ACT_RELU && act != SS_ACT_GELU) return SS_ERR_INVALID_ARG;
    if (H + 2 * ph < desc->kh || Wd + 2 * pw < desc->kw) return SS_ERR_INVALID_ARG;
    if (!aligned(x, 16) || !aligned(wbuf, 16) || !aligned(y, 16) || (bias && !aligned(bias, 4)) ||
        (residual && !aligned(residual, 16)))
        return SS_ERR_INVALID_ARG;
    int Ho = (H + 2 * ph - desc->kh) / sh + 1;
    int Wo = (Wd + 2 * pw - desc->kw) / sw + 1;
    if (Ho <= 0 || Wo <= 0) return SS_ERR_INVALID_ARG;
    long long P = (long long)N * Ho * Wo;
    long long xbytes = (long long)N * H * Wd * desc->cin * esize;
    if (!within_limits(desc, N, H, Wd, ph, pw, esize, P, desc->cout)) return SS_ERR_UNSUPPORTED;

    TileDims t = tile_dims(desc);
    size_t wbytes = SPARSE ? packed_size(t) : dense_size(t);
    if (wbytes >= (1ull << 31)) return SS_ERR_UNSUPPORTED;
    ConvParams p{};
    p.x = static_cast<const uint16_t *>(x);
    p.a_vals = static_cast<const uint8_t *>(wbuf) + kHeaderBytes;
    p.a_meta = reinterpret_cast<const uint32_t *>(p.a_vals + (size_t)t.Mt * t.Ks * 1024);
    p.bias = bias;
    p.scale = scale;
    p.residual = static_cast<const uint16_t *>(residual);
    p.y = static_cast<uint16_t *>(y);
    // The kernel stages 2-byte units: for 8-bit operands a unit is a pair of channels, and Cin and K count pairs.
    p.N = N; p.H = H; p.W = Wd; p.Cin = desc->cin / (q8 ? 2 : 1); p.Cout = desc->cout; p.kh = desc->kh; p.kw = desc->kw;
    p.sh = sh; p.sw = sw; p.ph = ph; p.pw = pw; p.Ho = Ho; p.Wo = Wo; p.P = (int)P;
    p.K = t.K / (q8 ? 2 : 1); p.Ks = t.Ks; p.Kp = t.Kp; p.Mt = t.Mt; p.act = act; p.korder = desc->korder;
    p.tiles_m = 0;
    p.tm_mul = p.tm_sh = 0;
    fast_div_setup((unsigned)(Ho * Wo), &p.howo_mul, &p.howo_sh);
    fast_div_setup((unsigned)Wo, &p.wo_mul, &p.wo_sh);
    fast_div_setup((unsigned)p.Cin, &p.cin_mul, &p.cin_sh);
    fast_div_setup((unsigned)p.kw, &p.kw_mul, &p.kw_sh);
    p.x_bytes = (unsigned)xbytes;
    p.a_bytes = (unsigned)((size_t)t.Mt * t.Ks * (SPARSE ? 1024 : 2048));
    p.meta_bytes = SPARSE ? (unsigned)((size_t)t.Mt * t.Kp * 256) : 4u;
    // Split of the reduction over several workgroups per tile (16-bit operands, grids far below the chip's size): the
    // partial sums and ticket counters live in the caller's workspace, which ss_conv2d_workspace_bytes sized from
    // the same plan.  The few-pixel kernels, which dispatch asks first, do not split.
    p.nsplit = 1;
    p.plan_tile = -1;
    if (!q8 && !(forced_tile() < 0 && forced_split() == 0 && takes_small(desc, p, SPARSE, planning_units()))) {
        const SplitPlan pl = plan_split(desc, P, t.Ks, planning_units(), forced_tile(), forced_split());
        if (pl.nsplit > 1) {
            if (!workspace || ws_bytes < pl.ctr_bytes + pl.part_bytes) return SS_ERR_WORKSPACE;
            if (!aligned(workspace, 256)) return SS_ERR_INVALID_ARG;
            p.nsplit = pl.nsplit;
            p.plan_tile = pl.tile;
            p.plan_bm = pl.bm;
            p.plan_bn = pl.bn;
            p.ws_part = reinterpret_cast<float *>(static_cast<unsigned char *>(workspace) + pl.ctr_bytes);
        }
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (!SPARSE && pooled) {
        p.y2 = static_cast<uint16_t *>(pooled);
        const int pool_h = (Ho - 1) / 2 + 1, pool_w = (Wo - 1) / 2 + 1;      // window 3, stride 2, padding 1
        return desc->dtype == SS_F16 ? pooled_dispatch_f16_dense(desc, p, pool_h, pool_w, s) : pooled_dispatch_bf16_dense(desc, p, pool_h, pool_w, s);
    }
    switch (desc->dtype) {
        case SS_I8: return SPARSE ? conv_dispatch_i8_sparse(desc, p, s) : conv_dispatch_i8_dense(desc, p, s);
        case SS_F8: return SPARSE ? conv_dispatch_f8_sparse(desc, p, s) : conv_dispatch_f8_dense(desc, p, s);
        case SS_F16: return SPARSE ? conv_dispatch_f16_sparse(desc, p, s) : conv_dispatch_f16_dense(desc, p, s);
        default: return SPARSE ? conv_dispatch_bf16_sparse(desc, p, s) : conv_dispatch_bf16_dense(desc, p, s);
    }
}

// The 1x1 layer that follows a fused pair (d null: none).
struct ThirdLayer {
    const ss_weight_desc *d;
    const void *w;
    const float *bias;
    int32_t act;
    void *y;
};

// Can a third layer follow this pair?  (the conditions of the kernels: whole tiles everywhere, 128 channels of the second output at a time)
static bool third_fits(const ss_weight_desc *d1, const ss_weight_desc *d2, const ss_weight_desc *d3)
{
    return d1->korder == SS_K_CRS && d1->kh == 3 && d1->kw == 3 && d1->cin % 32 == 0 && d1->cout <= 128 && d2->cout % 128 == 0 &&
           d3->cout % 32 == 0 && d3->cout <= 128;
}

template <bool SPARSE>
static int fused_entry(const ss_weight_desc *d1, const void *x, int32_t N, int32_t H, int32_t Wd, const void *w1,
                       const float *bias1, int32_t sh, int32_t sw, int32_t ph, int32_t pw, int32_t act1,
                       const ss_weight_desc *d2, const void *w2, const float *bias2, const void *residual, int32_t act2,
                       void *y, void *stream, const ThirdLayer &third = {})
{
    int st = check_desc(d1, SPARSE);
    if (st != SS_OK) return st;
    st = check_desc(d2, SPARSE);
    if (st != SS_OK) return st;
    if (third.d) {
        st = check_desc(third.d, SPARSE);
        if (st != SS_OK) return st;
        if (third.d->dtype != d1->dtype) return SS_ERR_UNSUPPORTED;
        if (third.d->kh != 1 || third.d->kw != 1 || third.d->cin != d2->cout) return SS_ERR_INVALID_ARG;
        if (!third_fits(d1, d2, third.d)) return SS_ERR_UNSUPPORTED;
        if (!third.w || !third.y || !aligned(third.w, 16) || !aligned(third.y, 16) || (third.bias && !aligned(third.bias, 16))) return SS_ERR_INVALID_ARG;
        if (third.act != SS_ACT_NONE && third.act != SS_ACT_RELU && third.act != SS_ACT_GELU) return SS_ERR_INVALID_ARG;
    }
    if (is_byte_type(d1->dtype) || d2->dtype != d1->dtype) return SS_ERR_UNSUPPORTED;
    if (d2->kh != 1 || d2->kw != 1 || d2->cin != d1->cout) return SS_ERR_INVALID_ARG;
    const bool mlp = d1->kh * d1->kw == 1;        // 1x1 -> 1x1: the inverted-bottleneck kernel
    if (mlp) {
        if (d1->cin % 32 != 0 || d1->cin > 32 * kMlpKs1 || d1->cout % 128 != 0 || d2->cout % 32 != 0 ||
            d2->cout > 64 * kMlpTiles)
            return SS_ERR_UNSUPPORTED;
        // the kernel keeps the first layer's whole bias in LDS next to its two tiles: within the default 64 KiB
        if ((size_t)64 * (d1->cin + 8) * 2 + (size_t)64 * (128 + 4) * 2 + (size_t)d1->cout * 4 > 64 * 1024) return SS_ERR_UNSUPPORTED;
    } else if (d1->cout % 32 != 0 || d1->cout > 256 || d2->cout % 32 != 0) {
        return SS_ERR_UNSUPPORTED;
    }
    if (!x || !w1 || !w2 || !y) return SS_ERR_INVALID_ARG;
    if (N <= 0 || H <= 0 || Wd <= 0 || sh <= 0 || sw <= 0 || ph < 0 || pw < 0) return SS_ERR_INVALID_ARG;
    for (int a : {act1, act2})
        if (a != SS_ACT_NONE && a != SS_ACT_RELU && a != SS_ACT_GELU) return SS_ERR_INVALID_ARG;
    if (H + 2 * ph < d1->kh || Wd + 2 * pw < d1->kw) return SS_ERR_INVALID_ARG;
    if (!aligned(x, 16) || !aligned(w1, 16) || !aligned(w2, 16) || !aligned(y, 16) || (bias1 && !aligned(bias1, 4)) ||
        (bias2 && !aligned(bias2, 16)) || (residual && !aligned(residual, 16)))
        return SS_ERR_INVALID_ARG;
    const int Ho = (H + 2 * ph - d1->kh) / sh + 1, Wo = (Wd + 2 * pw - d1->kw) / sw + 1;
    if (Ho <= 0 || Wo <= 0) return SS_ERR_INVALID_ARG;
    const long long P = (long long)N * Ho * Wo, xbytes = (long long)N * H * Wd * d1->cin * 2;
    if (!within_limits(d1, N, H, Wd, ph, pw, 2, P, d2->cout)) return SS_ERR_UNSUPPORTED;
    const TileDims t1 = tile_dims(d1), t2 = tile_dims(d2);
    if ((SPARSE ? packed_size(t1) : dense_size(t1)) >= (1ull << 31) || (SPARSE ? packed_size(t2) : dense_size(t2)) >= (1ull << 31))
        return SS_ERR_UNSUPPORTED;
    if (mlp) {
        if (sh != 1 || sw != 1 || ph != 0 || pw != 0) return SS_ERR_UNSUPPORTED;
        if (bias1 && !aligned(bias1, 16)) return SS_ERR_INVALID_ARG;
        MlpParams m{};
        m.x = static_cast<const uint16_t *>(x);
        m.a1_vals = static_cast<const uint8_t *>(w1) + kHeaderBytes;
        m.a2_vals = static_cast<const uint8_t *>(w2) + kHeaderBytes;
        m.bias1 = bias1; m.bias2 = bias2;
        m.res2 = static_cast<const uint16_t *>(residual);
        m.y2 = static_cast<uint16_t *>(y);
        m.P = (int)P; m.Cin = d1->cin; m.Cmid = d1->cout; m.Cout2 = d2->cout;
        m.act1 = act1; m.act2 = act2;
        hipStream_t ms = static_cast<hipStream_t>(stream);
        if (d1->dtype == SS_F16) return SPARSE ? mlp_dispatch_f16_sparse(m, ms) : mlp_dispatch_f16_dense(m, ms);
        return SPARSE ? mlp_dispatch_bf16_sparse(m, ms) : mlp_dispatch_bf16_dense(m, ms);
    }
    ChainParams p{};
    p.x = static_cast<const uint16_t *>(x);
    p.a_vals = static_cast<const uint8_t *>(w1) + kHeaderBytes;
    p.a_meta = reinterpret_cast<const uint32_t *>(p.a_vals + (size_t)t1.Mt * t1.Ks * 1024);
    p.bias = bias1;
    p.scale = nullptr;
    p.residual = nullptr;
    p.y = nullptr;
    p.N = N; p.H = H; p.W = Wd; p.Cin = d1->cin; p.Cout = d1->cout; p.kh = d1->kh; p.kw = d1->kw;
    p.sh = sh; p.sw = sw; p.ph = ph; p.pw = pw; p.Ho = Ho; p.Wo = Wo; p.P = (int)P;
    p.K = t1.K; p.Ks = t1.Ks; p.Kp = t1.Kp; p.Mt = t1.Mt; p.act = act1; p.korder = d1->korder;
    p.tiles_m = 0;
    p.tm_mul = p.tm_sh = 0;
    fast_div_setup((unsigned)(Ho * Wo), &p.howo_mul, &p.howo_sh);
    fast_div_setup((unsigned)Wo, &p.wo_mul, &p.wo_sh);
    fast_div_setup((unsigned)p.Cin, &p.cin_mul, &p.cin_sh);
    fast_div_setup((unsigned)p.kw, &p.kw_mul, &p.kw_sh);
    p.x_bytes = (unsigned)xbytes;
    p.a_bytes = (unsigned)((size_t)t1.Mt * t1.Ks * (SPARSE ? 1024 : 2048));
    p.meta_bytes = SPARSE ? (unsigned)((size_t)t1.Mt * t1.Kp * 256) : 4u;
    p.a2_vals = static_cast<const uint8_t *>(w2) + kHeaderBytes;
    p.a2_meta = reinterpret_cast<const uint32_t *>(p.a2_vals + (size_t)t2.Mt * t2.Ks * 1024);
    p.bias2 = bias2;
    p.res2 = static_cast<const uint16_t *>(residual);
    p.y2 = static_cast<uint16_t *>(y);
    p.Cout2 = d2->cout; p.Ks2 = t2.Ks; p.Kp2 = t2.Kp; p.Mt2 = t2.Mt; p.act2 = act2;
    p.a2_bytes = (unsigned)((size_t)t2.Mt * t2.Ks * (SPARSE ? 1024 : 2048));
    p.meta2_bytes = SPARSE ? (unsigned)((size_t)t2.Mt * t2.Kp * 256) : 4u;
    if (third.d) {
        const TileDims t3 = tile_dims(third.d);
        p.a3_vals = static_cast<const uint8_t *>(third.w) + kHeaderBytes;
        p.a3_meta = reinterpret_cast<const uint32_t *>(p.a3_vals + (size_t)t3.Mt * t3.Ks * 1024);
        p.bias3 = third.bias;
        p.y3 = static_cast<uint16_t *>(third.y);
        p.Cout3 = third.d->cout; p.Ks3 = t3.Ks; p.Kp3 = t3.Kp; p.Mt3 = t3.Mt; p.act3 = third.act;
        p.a3_bytes = (unsigned)((size_t)t3.Mt * t3.Ks * (SPARSE ? 1024 : 2048));
        p.meta3_bytes = SPARSE ? (unsigned)((size_t)t3.Mt * t3.Kp * 256) : 4u;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (d1->dtype == SS_F16) return SPARSE ? fused_dispatch_f16_sparse(d1, p, s) : fused_dispatch_f16_dense(d1, p, s);
    return SPARSE ? fused_dispatch_bf16_sparse(d1, p, s) : fused_dispatch_bf16_dense(d1, p, s);
}

}  // namespace ss

using namespace ss;

extern "C" int ss_debug_force_tile(int32_t id)
{
    g_forced_tile.store(id < 0 ? -1 : id, std::memory_order_relaxed);
    return SS_OK;
}

extern "C" int ss_debug_force_split(int32_t n)
{
    g_forced_split.store(n < 0 ? 0 : n, std::memory_order_relaxed);
    return SS_OK;
}

extern "C" int ss_debug_limit_blocks(int32_t n)
{
    g_block_limit.store(n < 0 ? 0 : n, std::memory_order_relaxed);
    return SS_OK;
}

extern "C" int ss_conv2d_workspace_bytes(const ss_weight_desc *desc, int32_t N, int32_t H, int32_t Wd, int32_t stride_h,
                                         int32_t stride_w, int32_t pad_h, int32_t pad_w, size_t *bytes)
{
    if (!bytes) return SS_ERR_INVALID_ARG;
    int st = check_desc(desc, false);
    if (st != SS_OK) return st;
    if (N <= 0 || H <= 0 || Wd <= 0 || stride_h <= 0 || stride_w <= 0 || pad_h < 0 || pad_w < 0) return SS_ERR_INVALID_ARG;
    *bytes = 0;
    if (H + 2 * pad_h < desc->kh || Wd + 2 * pad_w < desc->kw) return SS_ERR_INVALID_ARG;
    const long long Ho = (H + 2 * pad_h - desc->kh) / stride_h + 1, Wo = (Wd + 2 * pad_w - desc->kw) / stride_w + 1;
    const long long P = (long long)N * Ho * Wo;
    if (P >= (1ll << 31) - 512) return SS_ERR_UNSUPPORTED;
    const TileDims t = tile_dims(desc);
    const int ncu = planning_units();
    const SplitPlan pl = plan_split(desc, P, t.Ks, ncu, forced_tile(), forced_split());
    if (pl.nsplit <= 1) return SS_OK;
    if (forced_tile() < 0 && forced_split() == 0) {       // as conv_entry; one answer for the sparse and the dense call
        ConvParams p{};
        p.Cin = desc->cin; p.Cout = desc->cout; p.P = (int)P; p.Ks = t.Ks; p.Mt = t.Mt;
        if (takes_small(desc, p, true, ncu) && takes_small(desc, p, false, ncu)) return SS_OK;
    }
    *bytes = pl.ctr_bytes + pl.part_bytes;
    return SS_OK;
}

extern "C" int ss_conv2d_fwd(const ss_weight_desc *desc, const void *x, int32_t N, int32_t H, int32_t Wd,
                             const void *packed, const float *bias, int32_t stride_h, int32_t stride_w, int32_t pad_h,
                             int32_t pad_w, int32_t act, void *y, void *workspace, size_t ws_bytes, void *stream)
{
    return conv_entry<true>(desc, x, N, H, Wd, packed, bias, nullptr, stride_h, stride_w, pad_h, pad_w, act, y,
                            workspace, ws_bytes, stream);
}

// ---------------------------------------------------------------------------------------------
// Entry point for callers that cannot provide a workspace: the split reduction's scratch lives in a device array
// that is part of the library's code object (one copy per GPU, held until the process ends).
// ---------------------------------------------------------------------------------------------
namespace {
// Largest workspace the library plans by itself: a split happens only while tiles x shares <= compute units (256),
// each share holds at most a 256 x 64 tile of fp32 partial sums (64 KiB), plus the ticket counters.
constexpr size_t kStaticWsBytes = ((size_t)16 << 20) + ((size_t)64 << 10);
__device__ __align__(256) unsigned char scratch[kStaticWsBytes];      // zero at load; every call hands its counters back at zero

// Device address of `scratch` on the current device (each GPU holds its own copy at its own address), looked up once
// per device.  In host code the array's name is only a handle for this lookup, never an address.
void *static_workspace()
{
    static std::atomic<void *> cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return nullptr;
    if (dev >= 0 && dev < 64) {
        void *p = cached[dev].load(std::memory_order_acquire);
        if (p) return p;
    }
    void *ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return nullptr;
    if (dev >= 0 && dev < 64) cached[dev].store(ptr, std::memory_order_release);
    return ptr;
}
}  // namespace

extern "C" int ss_conv2d_fwd_static_ws(const ss_weight_desc *desc, const void *x, int32_t N, int32_t H, int32_t Wd,
                                       const void *packed, const float *bias, int32_t stride_h, int32_t stride_w,
                                       int32_t pad_h, int32_t pad_w, int32_t act, void *y, void *stream)
{
    void *ws = static_workspace();
    if (!ws) return SS_ERR_HIP;
    // (a problem whose plan needs more than the array holds -- only a forced split can -- is rejected with
    // SS_ERR_WORKSPACE by the size check of the common entry)
    return conv_entry<true>(desc, x, N, H, Wd, packed, bias, nullptr, stride_h, stride_w, pad_h, pad_w, act, y, ws,
                            kStaticWsBytes, stream);
}

extern "C" int ss_conv2d_res_fwd(const ss_weight_desc *desc, const void *x, int32_t N, int32_t H, int32_t Wd,
                                 const void *packed, const float *bias, const void *residual, int32_t stride_h,
                                 int32_t stride_w, int32_t pad_h, int32_t pad_w, int32_t act, void *y, void *workspace,
                                 size_t ws_bytes, void *stream)
{
    return conv_entry<true>(desc, x, N, H, Wd, packed, bias, residual, stride_h, stride_w, pad_h, pad_w, act, y,
                            workspace, ws_bytes, stream);
}

extern "C" int ss_conv2d_dense_fwd(const ss_weight_desc *desc, const void *x, int32_t N, int32_t H, int32_t Wd,
                                   const void *dense, const float *bias, int32_t stride_h, int32_t stride_w,
                                   int32_t pad_h, int32_t pad_w, int32_t act, void *y, void *workspace, size_t ws_bytes,
                                   void *stream)
{
    return conv_entry<false>(desc, x, N, H, Wd, dense, bias, nullptr, stride_h, stride_w, pad_h, pad_w, act, y,
                             workspace, ws_bytes, stream);
}

extern "C" int ss_conv2d_dense_res_fwd(const ss_weight_desc *desc, const void *x, int32_t N, int32_t H, int32_t Wd,
                                       const void *dense, const float *bias, const void *residual, int32_t stride_h,
                                       int32_t stride_w, int32_t pad_h, int32_t pad_w, int32_t act, void *y,
                                       void *workspace, size_t ws_bytes, void *stream)
{
    return conv_entry<false>(desc, x, N, H, Wd, dense, bias, residual, stride_h, stride_w, pad_h, pad_w, act, y,
                             workspace, ws_bytes, stream);
}

extern "C" int ss_conv2d_maxpool_dense_fwd(const ss_weight_desc *desc, const void *x, int32_t N, int32_t H, int32_t Wd, const void *dense, const float *bias,
                                           int32_t stride_h, int32_t stride_w, int32_t pad_h, int32_t pad_w, int32_t act, void *y, void *pooled, void *stream)
{
    if (!pooled || !aligned(pooled, 16)) return SS_ERR_INVALID_ARG;
    if (act != SS_ACT_RELU) return act == SS_ACT_NONE || act == SS_ACT_GELU ? SS_ERR_UNSUPPORTED : SS_ERR_INVALID_ARG;
    return conv_entry<false>(desc, x, N, H, Wd, dense, bias, nullptr, stride_h, stride_w, pad_h, pad_w, act, y, nullptr, 0, stream, false, nullptr, pooled);
}

extern "C" int ss_conv2d_maxpool_dense_query(const ss_weight_desc *desc, int32_t N, int32_t H, int32_t Wd, int32_t stride_h, int32_t stride_w,
                                             int32_t pad_h, int32_t pad_w, int32_t act, int32_t *supported)
{
    if (!supported) return SS_ERR_INVALID_ARG;
    *supported = 0;
    const int st = check_desc(desc, false);
    if (st != SS_OK) return st == SS_ERR_INVALID_ARG ? st : (int)SS_OK;
    if (N <= 0 || H <= 0 || Wd <= 0 || stride_h <= 0 || stride_w <= 0 || pad_h < 0 || pad_w < 0) return SS_ERR_INVALID_ARG;
    if (H + 2 * pad_h < desc->kh || Wd + 2 * pad_w < desc->kw) return SS_ERR_INVALID_ARG;
    const long long P = (long long)N * ((H + 2 * pad_h - desc->kh) / stride_h + 1) * ((Wd + 2 * pad_w - desc->kw) / stride_w + 1);
    if (!within_limits(desc, N, H, Wd, pad_h, pad_w, 2, P, desc->cout) || dense_size(tile_dims(desc)) >= (1ull << 31)) return SS_OK;
    ConvParams p{};
    p.P = (int)P; p.Cout = desc->cout; p.sh = stride_h; p.sw = stride_w; p.nsplit = 1;
    *supported = act == SS_ACT_RELU && image_eligible(desc, p);
    return SS_OK;
}

extern "C" int ss_conv2d_q8_fwd(const ss_weight_desc *desc, const void *x, int32_t N, int32_t H, int32_t Wd,
                                const void *packed, const float *scale, const float *bias, int32_t stride_h,
                                int32_t stride_w, int32_t pad_h, int32_t pad_w, int32_t act, int32_t out_dtype, void *y,
                                void *workspace, size_t ws_bytes, void *stream)
{
    if (out_dtype != SS_F16) return out_dtype == SS_BF16 ? SS_ERR_UNSUPPORTED : SS_ERR_INVALID_ARG;
    return conv_entry<true>(desc, x, N, H, Wd, packed, bias, nullptr, stride_h, stride_w, pad_h, pad_w, act, y,
                            workspace, ws_bytes, stream, true, scale);
}

extern "C" int ss_conv2d_q8_dense_fwd(const ss_weight_desc *desc, const void *x, int32_t N, int32_t H, int32_t Wd,
                                      const void *dense, const float *scale, const float *bias, int32_t stride_h,
                                      int32_t stride_w, int32_t pad_h, int32_t pad_w, int32_t act, int32_t out_dtype,
                                      void *y, void *workspace, size_t ws_bytes, void *stream)
{
    if (out_dtype != SS_F16) return out_dtype == SS_BF16 ? SS_ERR_UNSUPPORTED : SS_ERR_INVALID_ARG;
    return conv_entry<false>(desc, x, N, H, Wd, dense, bias, nullptr, stride_h, stride_w, pad_h, pad_w, act, y,
                             workspace, ws_bytes, stream, true, scale);
}

extern "C" int ss_conv2d_pw_fused_query(const ss_weight_desc *d1, int32_t stride_h, int32_t stride_w, int32_t pad_h,
                                        int32_t pad_w, const ss_weight_desc *d2, int32_t sparse, int32_t *supported,
                                        int32_t *pays)
{
    if (!supported || !pays) return SS_ERR_INVALID_ARG;
    *supported = 0;
    *pays = 0;
    int st = check_desc(d1, sparse != 0);
    if (st == SS_OK) st = check_desc(d2, sparse != 0);
    if (st == SS_ERR_INVALID_ARG) return st;
    if (st != SS_OK) return SS_OK;                                        // (not supported, e.g. K % 4 != 0)
    if (stride_h <= 0 || stride_w <= 0 || pad_h < 0 || pad_w < 0) return SS_ERR_INVALID_ARG;
    if (is_byte_type(d1->dtype) || d2->dtype != d1->dtype) return SS_OK;
    if (d2->kh != 1 || d2->kw != 1 || d2->cin != d1->cout) return SS_ERR_INVALID_ARG;
    if (d1->kh * d1->kw == 1) {       // 1x1 -> 1x1: the inverted-bottleneck kernel (same conditions as fused_entry)
        if (d1->cin % 32 != 0 || d1->cin > 32 * kMlpKs1 || d1->cout % 128 != 0 || d2->cout % 32 != 0 || d2->cout > 64 * kMlpTiles ||
            (size_t)64 * (d1->cin + 8) * 2 + (size_t)64 * (128 + 4) * 2 + (size_t)d1->cout * 4 > 64 * 1024)
            return SS_OK;
        if (stride_h != 1 || stride_w != 1 || pad_h != 0 || pad_w != 0) return SS_OK;
        *supported = 1;
        *pays = 1;                    // measured 1.3-1.7x over the two calls: the 4x-wide intermediate never reaches memory
        return SS_OK;
    }
    if (d1->cout % 32 != 0 || d1->cout > 256 || d2->cout % 32 != 0) return SS_OK;
    const bool fast_first = (d1->korder == SS_K_CRS && d1->kh == 3 && d1->kw == 3 && d1->cin % 32 == 0) ||
                            (d1->korder == SS_K_RSC && d1->cin % 8 == 0);
    if (!fast_first) return SS_OK;
    *supported = 1;
    // Measured on the ResNet-50 bottlenecks (batch 64): the pair beats its two calls while the second contraction,
    // a plain loop over the tile held in LDS, is short: first-layer widths up to 128 on the sparse path (1.12-1.27x),
    // up to 64 on the dense twin; at 256 the two calls are faster (30.0 vs 31.1 us sparse, 35.7 vs 37.1 us dense).
    *pays = d1->cout <= (sparse ? 128 : 64);
    return SS_OK;
}

extern "C" int ss_conv2d_pw_fused_fwd(const ss_weight_desc *desc1, const void *x, int32_t N, int32_t H, int32_t Wd,
                                      const void *packed1, const float *bias1, int32_t stride_h, int32_t stride_w,
                                      int32_t pad_h, int32_t pad_w, int32_t act1, const ss_weight_desc *desc2,
                                      const void *packed2, const float *bias2, const void *residual, int32_t act2,
                                      void *y, void *stream)
{
    return fused_entry<true>(desc1, x, N, H, Wd, packed1, bias1, stride_h, stride_w, pad_h, pad_w, act1, desc2, packed2,
                             bias2, residual, act2, y, stream);
}

extern "C" int ss_conv2d_pw_fused_dense_fwd(const ss_weight_desc *desc1, const void *x, int32_t N, int32_t H, int32_t Wd,
                                            const void *dense1, const float *bias1, int32_t stride_h, int32_t stride_w,
                                            int32_t pad_h, int32_t pad_w, int32_t act1, const ss_weight_desc *desc2,
                                            const void *dense2, const float *bias2, const void *residual, int32_t act2,
                                            void *y, void *stream)
{
    return fused_entry<false>(desc1, x, N, H, Wd, dense1, bias1, stride_h, stride_w, pad_h, pad_w, act1, desc2, dense2,
                              bias2, residual, act2, y, stream);
}

extern "C" int ss_conv2d_pw2_fused_query(const ss_weight_desc *desc1, int32_t N, int32_t H, int32_t Wd, int32_t stride_h, int32_t stride_w,
                                         int32_t pad_h, int32_t pad_w, const ss_weight_desc *desc2, const ss_weight_desc *desc3, int32_t sparse,
                                         int32_t *supported, int32_t *pays)
{
    int st = ss_conv2d_pw_fused_query(desc1, stride_h, stride_w, pad_h, pad_w, desc2, sparse, supported, pays);
    if (st != SS_OK || !*supported) return st;
    if (N <= 0 || H <= 0 || Wd <= 0 || H + 2 * pad_h < desc1->kh || Wd + 2 * pad_w < desc1->kw) return SS_ERR_INVALID_ARG;
    const int32_t pair_pays = *pays;
    *supported = 0;
    *pays = 0;
    st = check_desc(desc3, sparse != 0);
    if (st == SS_ERR_INVALID_ARG) return st;
    if (st != SS_OK || desc3->dtype != desc1->dtype) return SS_OK;
    if (desc3->kh != 1 || desc3->kw != 1 || desc3->cin != desc2->cout) return SS_ERR_INVALID_ARG;
    const long long P = (long long)N * ((H + 2 * pad_h - desc1->kh) / stride_h + 1) * ((Wd + 2 * pad_w - desc1->kw) / stride_w + 1);
    if (!third_fits(desc1, desc2, desc3) || !within_limits(desc1, N, H, Wd, pad_h, pad_w, 2, P, desc2->cout)) return SS_OK;
    *supported = 1;
    // Few pixels: where their kernel takes all three layers, 0.61 to 0.91 of the pair's time and the third layer's.  Where it takes only the pair, the three
    // run in the tiled kernel, 64 pixels at a time, and lose (first layers of 32 and 96 channels up to 1.9, third layers of 32 up to 1.8, second ones of 1024
    // up to 3.2; 0.65 to 0.93 for sparse 32 -> 32 -> 128 alone).
    // Beyond: the ResNet-50 trunk at 224 x 224, us, no layer joined / all that can be: batch 32 726 / 677, 64 1115 / 1080.  Not
    // where it loses: 128 channels on one workgroup per compute unit, where the pair has producer waves (batch 16, 516 without, 528 with those three, 503
    // with the others), and dense layers whose third one has more than 64 channels (batch 64: 1290 / 1301; 1266 with those of 64).  Over 400 layers of 32 to
    // 128 channels by themselves 0.51 to 0.99 where it says so.
    const int px = pair_small_pixels(P, planning_units());
    if (px > 0) {
        *pays = pair_pays && (pair_small_fits(desc1, px, desc2->cout, desc3->cout) || (sparse && desc1->cout == 32 && desc2->cout == 128));
        return SS_OK;
    }
    ConvParams p{};
    p.P = (int)P; p.Cout = desc1->cout;
    *pays = pair_pays && (sparse ? choose_fused_tile(p) != 4 : desc3->cout <= 64);
    return SS_OK;
}

extern "C" int ss_conv2d_pw2_fused_fwd(const ss_weight_desc *desc1, const void *x, int32_t N, int32_t H, int32_t Wd,
                                       const void *packed1, const float *bias1, int32_t stride_h, int32_t stride_w,
                                       int32_t pad_h, int32_t pad_w, int32_t act1, const ss_weight_desc *desc2,
                                       const void *packed2, const float *bias2, const void *residual, int32_t act2,
                                       void *y2, const ss_weight_desc *desc3, const void *packed3, const float *bias3, int32_t act3,
                                       void *y3, void *stream)
{
    if (!desc3) return SS_ERR_INVALID_ARG;
    return fused_entry<true>(desc1, x, N, H, Wd, packed1, bias1, stride_h, stride_w, pad_h, pad_w, act1, desc2, packed2,
                             bias2, residual, act2, y2, stream, ThirdLayer{desc3, packed3, bias3, act3, y3});
}

extern "C" int ss_conv2d_pw2_fused_dense_fwd(const ss_weight_desc *desc1, const void *x, int32_t N, int32_t H, int32_t Wd,
                                             const void *dense1, const float *bias1, int32_t stride_h, int32_t stride_w,
                                             int32_t pad_h, int32_t pad_w, int32_t act1, const ss_weight_desc *desc2,
                                             const void *dense2, const float *bias2, const void *residual, int32_t act2,
                                             void *y2, const ss_weight_desc *desc3, const void *dense3, const float *bias3, int32_t act3,
                                             void *y3, void *stream)
{
    if (!desc3) return SS_ERR_INVALID_ARG;
    return fused_entry<false>(desc1, x, N, H, Wd, dense1, bias1, stride_h, stride_w, pad_h, pad_w, act1, desc2, dense2,
                              bias2, residual, act2, y2, stream, ThirdLayer{desc3, dense3, bias3, act3, y3});
}
