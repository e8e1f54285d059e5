// Max pooling over NHWC 16-bit activations: the one non-convolution step between the convolutions of a
// ResNet trunk (after the stem), so that a chained stack runs without leaving the library.
#include "ss_internal.h"

namespace ss {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

template <int DT>
__device__ __forceinline__ float widen16(uint32_t bits)
{
    if constexpr (DT == SS_F16)
        return (float)__builtin_bit_cast(_Float16, (uint16_t)bits);
    else
        return __builtin_bit_cast(float, bits << 16);
}

// One thread per (output pixel, run of 8 channels).  The result is one of the inputs (its bit pattern is copied); positions
// outside the image do not take part; a NaN wins.
//
// Memory-bound: the input is read once and a quarter of it written.  With K fixed (3, 2) all K*K loads are in flight together:
// a position outside the image is clamped to the nearest one inside, which is in the window too (2 * pad <= k), so it changes
// neither the maximum nor which of equal inputs comes first; a window with a NaN is left to the general loop.  The loop with
// its bounds tests and one load in flight took 46 us on the ResNet-50 stem's output at batch 64 (27 us here, 4.7 TB/s) and 9.4 us
// on one image, a chain of nine memory latencies (3.4 us back to back).  Workgroups are renumbered so that an XCD works on
// neighbouring rows, which share input rows.
template <int DT, int K>
__global__ __launch_bounds__(256) void maxpool_kernel(const uint16_t *__restrict__ x, uint16_t *__restrict__ y, int N,
                                                      int H, int W, int C, int k, int s, int pad, int Ho, int Wo)
{
    const unsigned runs = C >> 3;
    const long long total = (long long)N * Ho * Wo * runs;
    const unsigned nb = (unsigned)((total + 255) / 256), xcd = blockIdx.x & 7;
    const long long gid = (long long)(xcd * (nb >> 3) + min(xcd, nb & 7) + (blockIdx.x >> 3)) * 256 + threadIdx.x;
    if (gid >= total) return;
    int run, wo, ho, n;
    if (total < 1ll << 31) {                              // uniform
        unsigned rest = (unsigned)gid / runs;
        run = (int)((unsigned)gid - rest * runs);
        const unsigned row = rest / (unsigned)Wo;
        wo = (int)(rest - row * (unsigned)Wo);
        n = (int)(row / (unsigned)Ho);
        ho = (int)(row - (unsigned)n * (unsigned)Ho);
    } else {
        long long rest = gid / runs;
        run = (int)(gid % runs);
        wo = (int)(rest % Wo);
        rest /= Wo;
        ho = (int)(rest % Ho);
        n = (int)(rest / Ho);
    }
    uint16_t *const dst = y + (((size_t)n * Ho + ho) * Wo + wo) * C + run * 8;
    if constexpr (K > 0) {
        u32x4 v[K][K];
#pragma unroll
        for (int r = 0; r < K; r++) {
            const int ih = min(max(ho * s - pad + r, 0), H - 1);
#pragma unroll
            for (int t = 0; t < K; t++) {
                const int iw = min(max(wo * s - pad + t, 0), W - 1);
                v[r][t] = *reinterpret_cast<const u32x4 *>(x + (((size_t)n * H + ih) * W + iw) * C + run * 8);
            }
        }
        float best[8];
        u16x2 top[4];                                     // largest magnitude pattern: above infinity's where there is a NaN
#pragma unroll
        for (int i = 0; i < K * K; i++) {
            const u32x4 u = v[i / K][i % K];
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const float lo = widen16<DT>(u[e] & 0xFFFFu);
                const float hi = DT == SS_BF16 ? __builtin_bit_cast(float, u[e] & 0xFFFF0000u) : widen16<DT>(u[e] >> 16);
                const u16x2 mag = __builtin_bit_cast(u16x2, u[e] & 0x7FFF7FFFu);
                best[2 * e] = i == 0 || lo > best[2 * e] ? lo : best[2 * e];
                best[2 * e + 1] = i == 0 || hi > best[2 * e + 1] ? hi : best[2 * e + 1];
                top[e] = i == 0 ? mag : __builtin_elementwise_max(top[e], mag);
            }
        }
        const u16x2 m = __builtin_elementwise_max(__builtin_elementwise_max(top[0], top[1]), __builtin_elementwise_max(top[2], top[3]));
        const unsigned inf = DT == SS_BF16 ? 0x7F80u : 0x7C00u;
        if (m[0] <= inf && m[1] <= inf) {
            u32x4 out;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                if constexpr (DT == SS_BF16)
                    out[e] = (__builtin_bit_cast(uint32_t, best[2 * e]) >> 16) | (__builtin_bit_cast(uint32_t, best[2 * e + 1]) & 0xFFFF0000u);
                else                                      // (exact: the values came from binary16)
                    out[e] = (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)best[2 * e]) | ((uint32_t)__builtin_bit_cast(uint16_t, (_Float16)best[2 * e + 1]) << 16);
            }
            *reinterpret_cast<u32x4 *>(dst) = out;
            return;
        }
    }
    uint32_t best[8];
    float bestf[8];
    bool have = false;
    for (int r = 0; r < k; r++) {
        const int ih = ho * s - pad + r;
        if ((unsigned)ih >= (unsigned)H) continue;
        for (int t = 0; t < k; t++) {
            const int iw = wo * s - pad + t;
            if ((unsigned)iw >= (unsigned)W) continue;
            const u32x4 v = *reinterpret_cast<const u32x4 *>(x + (((size_t)n * H + ih) * W + iw) * C + run * 8);
#pragma unroll
            for (int e = 0; e < 8; e++) {
                const uint32_t b = (v[e >> 1] >> (16 * (e & 1))) & 0xFFFFu;
                const float f = widen16<DT>(b);
                if (!have || f > bestf[e] || f != f) {
                    if (!(have && bestf[e] != bestf[e])) {      // a NaN already there stays
                        best[e] = b;
                        bestf[e] = f;
                    }
                }
            }
            have = true;
        }
    }
    u32x4 out;
#pragma unroll
    for (int e = 0; e < 4; e++) out[e] = have ? (best[2 * e] | (best[2 * e + 1] << 16)) : 0u;
    *reinterpret_cast<u32x4 *>(dst) = out;
}

}  // namespace ss

using namespace ss;

extern "C" int ss_maxpool2d(const void *x, int32_t N, int32_t H, int32_t Wd, int32_t C, int32_t dtype, int32_t k,
                            int32_t stride, int32_t pad, void *y, void *stream)
{
    if (!x || !y) return SS_ERR_INVALID_ARG;
    if (N <= 0 || H <= 0 || Wd <= 0 || C <= 0 || k <= 0 || stride <= 0 || pad < 0 || 2 * pad > k) return SS_ERR_INVALID_ARG;
    if (dtype != SS_F16 && dtype != SS_BF16) return SS_ERR_INVALID_ARG;
    if (C % 8 != 0) return SS_ERR_UNSUPPORTED;
    if (((uintptr_t)x & 15) || ((uintptr_t)y & 15)) return SS_ERR_INVALID_ARG;
    if (H + 2 * pad < k || Wd + 2 * pad < k) return SS_ERR_INVALID_ARG;
    const int Ho = (H + 2 * pad - k) / stride + 1, Wo = (Wd + 2 * pad - k) / stride + 1;
    const long long total = (long long)N * Ho * Wo * (C / 8);
    if (total <= 0 || (total + 255) / 256 > 0x7FFFFFFFll) return SS_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)((total + 255) / 256)), block(256);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint16_t *xs = static_cast<const uint16_t *>(x);
    uint16_t *ys = static_cast<uint16_t *>(y);
    auto go = [&](auto kern) { kern<<<grid, block, 0, s>>>(xs, ys, N, H, Wd, C, k, stride, pad, Ho, Wo); };
    if (dtype == SS_F16)
        k == 3 ? go(maxpool_kernel<SS_F16, 3>) : k == 2 ? go(maxpool_kernel<SS_F16, 2>) : go(maxpool_kernel<SS_F16, 0>);
    else
        k == 3 ? go(maxpool_kernel<SS_BF16, 3>) : k == 2 ? go(maxpool_kernel<SS_BF16, 2>) : go(maxpool_kernel<SS_BF16, 0>);
    return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_HIP;
}
