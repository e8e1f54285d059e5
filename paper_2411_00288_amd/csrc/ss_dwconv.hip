// Depthwise convolution (one filter per channel), NHWC 16-bit, stride 1: the grouped convolutions that the paper
// leaves dense (Sec. 4, "Architectures"), e.g. the 7x7 of a ConvNeXt block.  Three kernels (choose_dw, ss_dwconv.h): square 5x5 and 7x7 filters
// with many outputs run on the matrix unit (dwconv_mfma_kernel), 3x3 and few outputs in one memory latency on the vector ALU (dwconv_few_kernel), the
// others on the vector ALU row by row, whose 49 multiply-adds per output bound the 7x7 at about 50 us for the 128 x 56 x 56 x 96 layer
// before any load or conversion (99 us measured).
#include "ss_internal.h"
#include "ss_conv_params.h"
#include "ss_dwconv.h"

namespace ss {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int DT>
__device__ __forceinline__ void widen8(const u32x4 &v, float (&f)[8])
{
#pragma unroll
    for (int e = 0; e < 4; e++) {
        if constexpr (DT == SS_F16) {
            f[2 * e] = (float)__builtin_bit_cast(_Float16, (uint16_t)(v[e] & 0xFFFFu));
            f[2 * e + 1] = (float)__builtin_bit_cast(_Float16, (uint16_t)(v[e] >> 16));
        } else {
            f[2 * e] = __builtin_bit_cast(float, v[e] << 16);
            f[2 * e + 1] = __builtin_bit_cast(float, v[e] & 0xFFFF0000u);
        }
    }
}

// Two fp32 values to one dword of 16-bit floats, round to nearest even, in one instruction.
template <int DT>
__device__ __forceinline__ uint32_t pack2(float a, float b)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const f32x2 v = {a, b};
    if constexpr (DT == SS_F16) return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2));
    else return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

constexpr int TW = 4;      // adjacent outputs along the image row per thread: a loaded input vector serves up to KW of them

// One thread: TW output pixels x 8 channels.  The filter taps sit in LDS ([kh][KW][C], 16-bit); input vectors come
// through raw buffer loads whose offset is out of range outside the image (the hardware returns zeros).
template <int DT, int KW>
__global__ __launch_bounds__(256) void dwconv_kernel(const uint16_t *__restrict__ x, const uint16_t *__restrict__ w,
                                                     const float *__restrict__ bias, uint16_t *__restrict__ y, int N, int H,
                                                     int W, int C, int kh, int ph, int pw, int Ho, int Wo, int act,
                                                     unsigned x_bytes)
{
    extern __shared__ __attribute__((aligned(16))) uint16_t w_s[];
    const int ntap = kh * KW * C;
    for (int i = threadIdx.x * 8; i < ntap; i += 256 * 8)
        *reinterpret_cast<u32x4 *>(w_s + i) = *reinterpret_cast<const u32x4 *>(w + i);
    __syncthreads();
    const int runs = C >> 3, wq = (Wo + TW - 1) / TW;
    const long long total = (long long)N * Ho * wq * runs;
    const long long gid = (long long)blockIdx.x * 256 + threadIdx.x;
    if (gid >= total) return;
    const int run = (int)(gid % runs);
    long long rest = gid / runs;
    const int wo0 = (int)(rest % wq) * TW;
    rest /= wq;
    const int ho = (int)(rest % Ho);
    const int n = (int)(rest / Ho);
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(x), 0, (int)x_bytes, 0x00020000);

    float acc[TW][8];
    {
        float b[8];
#pragma unroll
        for (int e = 0; e < 8; e++) b[e] = bias ? bias[run * 8 + e] : 0.f;
#pragma unroll
        for (int j = 0; j < TW; j++)
#pragma unroll
            for (int e = 0; e < 8; e++) acc[j][e] = b[e];
    }
    for (int r = 0; r < kh; r++) {
        const int ih = ho - ph + r;
        if ((unsigned)ih >= (unsigned)H) continue;
        float xf[KW + TW - 1][8];
#pragma unroll
        for (int j = 0; j < KW + TW - 1; j++) {
            const int iw = wo0 - pw + j;
            const unsigned off = (unsigned)iw < (unsigned)W ? (unsigned)((((size_t)n * H + ih) * W + iw) * C + run * 8) * 2u : 0x80000000u;
            widen8<DT>(__builtin_amdgcn_raw_buffer_load_b128(rx, (int)off, 0, 0), xf[j]);
        }
#pragma unroll
        for (int t = 0; t < KW; t++) {
            float wf[8];
            widen8<DT>(*reinterpret_cast<const u32x4 *>(w_s + ((size_t)r * KW + t) * C + run * 8), wf);
#pragma unroll
            for (int j = 0; j < TW; j++)
#pragma unroll
                for (int e = 0; e < 8; e++) acc[j][e] = __builtin_fmaf(wf[e], xf[j + t][e], acc[j][e]);
        }
    }
#pragma unroll
    for (int j = 0; j < TW; j++) {
        if (wo0 + j >= Wo) break;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const float z = acc[j][e];
            v[e] = act == SS_ACT_RELU ? (z < 0.f ? 0.f : z) : z;
        }
        u32x4 out = {pack2<DT>(v[0], v[1]), pack2<DT>(v[2], v[3]), pack2<DT>(v[4], v[5]), pack2<DT>(v[6], v[7])};
        *reinterpret_cast<u32x4 *>(y + ((((size_t)n * Ho + ho) * Wo + wo0 + j) * C + run * 8)) = out;
    }
}

// ---------------------------------------------------------------------------------------------
// Square filters on the matrix unit.
//
// For one channel and one filter row r, sixteen outputs along an image row are a banded Toeplitz matrix times the row's
// pixels: D[m, n] += sum_k T_r[m, k] X[k, n] with T_r[m, k] = w[r][k - m] (0 <= k - m < K) and X[k, n] = pixel w0 - pad + k of
// column n's input row.  The sixteen columns n of a V_MFMA_F32_16X16X32 are sixteen *strips* -- an image, a run of 16
// output columns, a segment of R output rows -- that all walk down their rows in step: an input row's fragment is read from LDS once and
// multiplied with the K matrices T_0 .. T_{K-1} into the K output rows it contributes to, whose accumulators rotate.  A fifth
// of the products are useful (K of 32), which the matrix unit's rate pays for many times over.
//
// A workgroup owns 16 strips x 16 channels, two channels per wave (their K matrices stay in registers).  Per input row: the rows
// two steps ahead are in flight to registers, the next one is transposed from channel-fastest to pixel-fastest (one
// v_perm per two elements) into the other LDS buffer, the current one is multiplied, and the finished output row crosses LDS back to
// channel-fastest order and is stored during the next step; one barrier per step.
//
// The zeros of T_r meet pixels outside an output's window, so a NaN or an infinity there reaches it as the NaN of 0 x inf: a
// workgroup that sees a non-finite output recomputes all of its outputs on the vector ALU, each from its own window.
// ---------------------------------------------------------------------------------------------
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

struct DwParams {
    const uint16_t *x, *w;
    const float *bias;
    uint16_t *y;
    int H, W, C, ph, pw, Ho, Wo, act;
    int per;                              // workgroups per group of channels (not from the grid's size: that would lengthen the launch's arguments to more than 112 bytes, which costs the host 0.6 us)
    int R, segs, wt, strips, groups;      // output rows per strip, segments per image, 16-wide tiles per row, strips in all, groups of 16 channels
    int rows, more;                       // rows of the blocks of 16 strips for each workgroup of a group: `rows`, and R or 1 (whole blocks or rows are
    int share;                            // dealt out: share) further ones for the first `more` of them
    unsigned x_bytes, w_bytes, y_bytes;
};
static_assert(sizeof(DwParams) <= 112, "a cheap launch");

template <int DT>
__device__ __forceinline__ f32x4 mma16(u32x4 a, u32x4 b, f32x4 c)
{
    if constexpr (DT == SS_F16)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// max(v, floor) that hands a NaN through: ReLU with floor = 0, the identity with floor = -inf.
__device__ __forceinline__ float max_nan(float v, float floor) { return __builtin_elementwise_maximum(v, floor); }

// Workgroup barrier that orders LDS traffic only: loads and output stores stay in flight across it.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

constexpr int kDwGroup = 16;              // channels of a workgroup
// 16-bit units of an input buffer: [channel][strip][32 pixels].  The four 16-byte vectors of a strip are XOR-ed with bits 2..3 of the strip's
// number, so that a fragment read (one vector of sixteen strips) covers all banks, and the upper eight channels, which the same lanes' neighbours
// write, lie 32 bytes further.
constexpr int kDwIn = 16 * 16 * 32 + 16;
__device__ __forceinline__ int dw_in_at(int channel, int strip, int vec) { return channel * 512 + (channel >> 3) * 16 + strip * 32 + ((vec ^ (strip >> 2)) & 3) * 8; }
constexpr int kDwPixel = 12;              // dwords per pixel of the output buffer (8 used) and
constexpr int kDwStrip = 16 * kDwPixel + 4;      // per strip: 16-byte aligned runs whose writes spread over the banks

// f(0), f(1), ... f(N - 1), each with its number as a constant
template <int N, int I = 0, class F>
__device__ __forceinline__ void each_below(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        each_below<N, I + 1>(f);
    }
}

template <int DT, int K>
__global__ __launch_bounds__(512) void dwconv_mfma_kernel(DwParams p)
{
    __shared__ __attribute__((aligned(16))) uint16_t in_s[2][kDwIn];
    __shared__ __attribute__((aligned(16))) uint32_t out_s[2][16 * kDwStrip];
    __shared__ int odd_s;                                 // a non-finite value was met
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // neighbouring workgroups, which share halo rows and the other channel groups' cache lines, on one XCD; a workgroup keeps its
    // channel group
    const int nb = p.per * p.groups, xcd = blockIdx.x & 7;
    const int lid = xcd * (nb >> 3) + min(xcd, nb & 7) + (blockIdx.x >> 3);
    const int c0 = (lid % p.groups) * kDwGroup, first = lid / p.groups;
    // This workgroup's share of the group's work, the rows of its blocks of 16 strips after each other: whole blocks, or (share = 1) rows dealt out
    // evenly.  A run of rows inside a block costs K - 1 input rows more than it has.
    const int lo = first * p.rows + min(first, p.more) * p.share, hi = lo + p.rows + (first < p.more ? p.share : 0);
    struct Run {
        int block, row, len;              // rows [row, row + len) of the block's strips
    };
    auto run_at = [&](int pos) {
        const int block = pos / p.R, row = pos - block * p.R;
        return Run{block, row, min(p.R - row, hi - pos)};
    };
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(p.x), 0, (int)p.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(p.w), 0, (int)p.w_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(p.y, 0, (int)p.y_bytes, 0x00020000);
    constexpr unsigned kOut = 0x80000000u;
    constexpr uint32_t kInf = DT == SS_BF16 ? 0x7F80u : 0x7C00u;

    struct Strip {
        int img, row, col;                                // first output row and column
        bool ok;
    };
    auto strip = [&](int block, int n) {
        const int s = block * 16 + n;
        const int rest = s / p.wt, img = rest / p.segs;
        return Strip{img, (rest - img * p.segs) * p.R, (s - rest * p.wt) * 16, s < p.strips};
    };
    // ---- staging: 384 threads, two neighbouring pixels x 8 channels each (the other 128 load nothing and write their zeros to
    // the unused pixels 24 .. 31, which must be finite: no branch, so that the compiler's waits count the loads in flight exactly)
    const bool stages = tid < 384;
    const int so = tid & 1, sp = stages ? (tid >> 1) % 12 : 12 + ((tid >> 1) & 3), sn = stages ? tid / 24 : (tid >> 3) & 15;
    const int sdst = dw_in_at(so * 8, sn, sp >> 2) / 2 + (sp & 3);
    const unsigned row_bytes = (unsigned)(p.W * p.C * 2);
    unsigned soff[2];                                     // byte offset of the thread's two pixels in the next row
    int srow = 0, lpos = lo, li = 0, lsteps = 0;          // next row to load: start of the run, input row of the run, input rows it has
    auto aim_loads = [&]() {
        const Run r = run_at(lpos);
        const Strip s = strip(r.block, sn);
        const bool ok = stages & s.ok & (c0 + so * 8 < p.C);
        srow = s.row + r.row - p.ph;
        lsteps = r.len + K - 1;
#pragma unroll
        for (int j = 0; j < 2; j++) {
            const int iw = s.col - p.pw + 2 * sp + j;
            const unsigned at = (unsigned)((((s.img * p.H + srow) * p.W + iw) * p.C + c0 + so * 8) * 2);
            soff[j] = (ok & ((unsigned)iw < (unsigned)p.W)) ? at : kOut;
        }
    };
    u32x4 st[K][2];                                       // input rows in flight: K, since the rotation of the accumulators unrolls the loop K times anyway
    u16x2 top = {0, 0};                                   // largest magnitude pattern of an output
    auto load_row = [&](u32x4 (&v)[2]) {
        // (arithmetic only: behind a branch the waits would lose count)
        const unsigned out = (unsigned)srow < (unsigned)p.H ? 0u : kOut;
#pragma unroll
        for (int j = 0; j < 2; j++) {
            v[j] = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(soff[j] | out), 0, 0);
            soff[j] += row_bytes;                         // (an offset out of range stays so: the launch sees to it)
        }
        srow++;
        if (++li == lsteps) {                             // uniform
            li = 0;
            lpos += lsteps - (K - 1);
            if (lpos < hi) aim_loads();                   // (some 150 instructions)
            else soff[0] = soff[1] = kOut;                // (nothing more to fetch: the K rows asked for behind the last one are never multiplied)
        }
    };
    auto store_row = [&](int buf, const u32x4 (&v)[2]) {
        uint32_t *dst = reinterpret_cast<uint32_t *>(in_s[buf]) + sdst;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            dst[(2 * e) * 256] = __builtin_amdgcn_perm(v[1][e], v[0][e], 0x05040100u);
            dst[(2 * e + 1) * 256] = __builtin_amdgcn_perm(v[1][e], v[0][e], 0x07060302u);
        }
    };
    // One tap of two channels per thread, ahead of the rows: asked for in turn, with the wait of each before the next, they were the longest part
    // of the set-up.
    static_assert(8 * K * K <= 512, "a thread loads at most one tap");
    const int tpair = tid / (K * K), tr = tid % (K * K) / K, tt = tid % K;      // (K * K is a multiple of K)
    const bool has_tap = tid < 8 * K * K;
    const uint32_t tap = __builtin_amdgcn_raw_buffer_load_b32(rw, (int)(has_tap && c0 + 2 * tpair < p.C ? (unsigned)(((tr * K + tt) * p.C + c0 + 2 * tpair) * 2) : kOut), 0, 0);
    aim_loads();
#pragma unroll
    for (int i = 0; i < K; i++) load_row(st[i]);
    // ---- the wave's two channels: K Toeplitz fragments each, from zero-padded rows of taps [channel pair][r][t + 15] in LDS
    const int m = lane & 15, kg = lane >> 4, cw = c0 + wave * 2;
    const int frag = dw_in_at(wave * 2, m, kg);           // (the pair's channels lie 512 apart)
    constexpr int TROW = 48;
    static_assert(8 * K * TROW <= 2 * 16 * kDwStrip, "the taps fit the output buffers");
    uint32_t *const taps = &out_s[0][0];
    static_assert(8 * K * TROW % 4 == 0, "whole vectors");
#pragma unroll
    for (int i = 0; i < (2 * K * TROW + 511) / 512; i++)
        if (tid + 512 * i < 2 * K * TROW) reinterpret_cast<u32x4 *>(taps)[tid + 512 * i] = u32x4{0u, 0u, 0u, 0u};
    lds_barrier();
    if (has_tap) taps[(tpair * K + tr) * TROW + 15 + tt] = tap;
    if (tid == 0) odd_s = 0;
    f32x4 b4[2];
#pragma unroll
    for (int j = 0; j < 2; j++) {
        const float b = p.bias && cw + j < p.C ? p.bias[cw + j] : 0.f;
        b4[j] = f32x4{b, b, b, b};
    }
    __syncthreads();
    u32x4 a[2][K];
#pragma unroll
    for (int r = 0; r < K; r++) {
        const uint32_t *src = taps + (wave * K + r) * TROW + 15 + 8 * kg - m;
        uint32_t d[8];
#pragma unroll
        for (int j = 0; j < 8; j++) d[j] = src[j];
#pragma unroll
        for (int q = 0; q < 4; q++) {
            a[0][r][q] = __builtin_amdgcn_perm(d[2 * q + 1], d[2 * q], 0x05040100u);
            a[1][r][q] = __builtin_amdgcn_perm(d[2 * q + 1], d[2 * q], 0x07060302u);
        }
    }
    // ---- output: one 16-byte run of a pixel per thread, range-checked
    const int oo = tid & 1, ow = (tid >> 1) & 15, on = tid >> 5;
    const unsigned yrow = (unsigned)(p.Wo * p.C * 2);
    int rows_left = 0, pos = lo, steps = 0;               // output rows of this thread's strip; start and input rows of the run
    unsigned yoff = 0;
    auto aim_stores = [&]() {
        const Run r = run_at(pos);
        const Strip s = strip(r.block, on);
        const bool ok = s.ok & (s.col + ow < p.Wo) & (c0 + oo * 8 < p.C);
        const int left = min(r.len, p.Ho - s.row - r.row);
        rows_left = ok ? left : 0;
        yoff = (unsigned)((((s.img * p.Ho + s.row + r.row) * p.Wo + s.col + ow) * p.C + c0 + oo * 8) * 2);
        steps = r.len + K - 1;
    };
    aim_stores();
    const float floor = p.act == SS_ACT_RELU ? 0.f : -__builtin_inff();
    // (The streaming cache policy, nt, would take the cold kernel alone from 65 to 51 us, but the layer behind it then reads
    // this output from memory instead of the memory-side cache and loses more: 215 against 196 us for the ConvNeXt block.)
    unsigned pending = kOut;                              // where the row written to LDS in the step before goes
    auto emit = [&](int buf) {
        const u32x4 v = *reinterpret_cast<const u32x4 *>(out_s[buf] + on * kDwStrip + ow * kDwPixel + oo * 4);
        __builtin_amdgcn_raw_buffer_store_b128(v, ry, (int)pending, 0, 0);
    };
    store_row(0, st[0]);
    load_row(st[0]);
    __syncthreads();                                      // (the taps have been read: the output buffers are free)
    f32x4 acc[2][K];
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
        for (int r = 0; r < K; r++) acc[j][r] = f32x4{0.f, 0.f, 0.f, 0.f};
    int par = 0, i = 0;
    auto step = [&](auto slot_of_step) {
        constexpr int u = decltype(slot_of_step)::value;  // (the slot of the rotation: a constant)
        // input row i of the block is in buffer par, the K rows after it are in or on their way to st[]
        const u32x4 bf[2] = {*reinterpret_cast<const u32x4 *>(in_s[par] + frag), *reinterpret_cast<const u32x4 *>(in_s[par] + frag + 512)};
        store_row(par ^ 1, st[(u + 1) % K]);
        load_row(st[(u + 1) % K]);
        emit(par ^ 1);
#pragma unroll
        for (int r = K - 1; r >= 0; r--)              // (the filter row that completes an output row first: its rounding overlaps with the others)
#pragma unroll
            for (int j = 0; j < 2; j++)
                acc[j][(u + K - r) % K] = mma16<DT>(a[j][r], bf[j], r == 0 ? b4[j] : acc[j][(u + K - r) % K]);
        {                                             // the last filter row completed output row i - (K - 1)
            const int slot = (u + 1) % K, h = i - (K - 1);
            uint32_t *dst = out_s[par] + m * kDwStrip + 4 * kg * kDwPixel + wave;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const uint32_t v = pack2<DT>(max_nan(acc[0][slot][e], floor), max_nan(acc[1][slot][e], floor));
                dst[e * kDwPixel] = v;
                top = __builtin_elementwise_max(top, __builtin_bit_cast(u16x2, v & 0x7FFF7FFFu));
            }
            pending = (yoff + (unsigned)h * yrow) | (h >= 0 && h < rows_left ? 0u : kOut);
        }
        lds_barrier();
        par ^= 1;
        if (++i == steps) {                               // uniform
            i = 0;
            pos += steps - (K - 1);
            if (pos < hi) aim_stores();
        }
    };
    // K steps at a time, and the rest after the loop: a loop that could be left from each of its K steps has those exits led through its head, where
    // the wait for a row loaded K steps ago would become one for the row loaded last, once every K steps (with that, taps fetched in turn and both
    // aims after the last run: 44.5 instead of 41.5 us for 128 x 56 x 56 x 96, 11.0 instead of 9.8 for 16 x 28 x 28 x 96).
    int total = hi - lo + K - 1;                          // input rows of all runs
    if (run_at(lo).len < hi - lo) total += ((hi - 1) / p.R - lo / p.R) * (K - 1);      // uniform: more than one
    for (int left = total / K; left > 0; left--) each_below<K>([&](auto u) { step(u); });
    const int rest = total % K;
    each_below<K - 1>([&](auto u) {
        if (decltype(u)::value < rest) step(u);           // uniform
    });
    emit(par ^ 1);
    if (top[0] >= kInf || top[1] >= kInf) odd_s = 1;
    __syncthreads();
    if (odd_s == 0) return;
    // ---- non-finite values: this workgroup's outputs again, each from its own window alone
    for (pos = lo; pos < hi; pos += steps - (K - 1)) {
        aim_stores();
        const Run run = run_at(pos);
        const Strip s = strip(run.block, on);
        const int c = c0 + oo * 8, wo = s.col + ow;
        for (int h = 0; h < rows_left; h++) {
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; e++) v[e] = p.bias ? p.bias[c + e] : 0.f;
            for (int r = 0; r < K; r++) {
                const int ih = s.row + run.row + h - p.ph + r;
                if ((unsigned)ih >= (unsigned)p.H) continue;
                for (int t = 0; t < K; t++) {
                    const int iw = wo - p.pw + t;
                    const unsigned off = (unsigned)iw < (unsigned)p.W ? (unsigned)((((s.img * p.H + ih) * p.W + iw) * p.C + c) * 2) : kOut;
                    float xf[8], wf[8];
                    widen8<DT>(__builtin_amdgcn_raw_buffer_load_b128(rx, (int)off, 0, 0), xf);
                    widen8<DT>(*reinterpret_cast<const u32x4 *>(p.w + ((size_t)r * K + t) * p.C + c), wf);
#pragma unroll
                    for (int e = 0; e < 8; e++) v[e] = __builtin_fmaf(wf[e], xf[e], v[e]);
                }
            }
#pragma unroll
            for (int e = 0; e < 8; e++) v[e] = max_nan(v[e], floor);
            *reinterpret_cast<u32x4 *>(reinterpret_cast<char *>(p.y) + yoff + (size_t)h * yrow) =
                u32x4{pack2<DT>(v[0], v[1]), pack2<DT>(v[2], v[3]), pack2<DT>(v[4], v[5]), pack2<DT>(v[6], v[7])};
        }
    }
}

// Segments per image and their shares: those for which the busiest workgroup walks over the fewest input rows (a run of R output rows needs
// R + K - 1).  Dealt out row by row, 32 blocks of 56 rows keep 42 workgroups of a channel group busy for 43 + 2 * 6 rows instead of 32 of them for
// 62 (128 x 56 x 56 x 96, 7x7: 46.5 -> 44.5 us then); where both walk over as many rows, whole blocks have fewer seams (64 images: 29.2 against 29.7 then).
template <int DT, int K>
static int launch_dw_mfma(DwParams p, int N, hipStream_t s)
{
    const int ncu = compute_units();
    if (ncu <= 0) return SS_ERR_HIP;
    p.wt = (p.Wo + 15) / 16;
    p.groups = (p.C + kDwGroup - 1) / kDwGroup;
    const long long per_group = ncu / p.groups > 0 ? ncu / p.groups : 1;
    long long best = -1;
    for (int segs = 1; segs <= p.Ho; segs++) {
        const int R = (p.Ho + segs - 1) / segs;
        if ((p.Ho + R - 1) / R != segs) continue;         // (no new length)
        const long long strips = (long long)N * segs * p.wt, blocks = (strips + 15) / 16;
        if (strips > 0x7FFFFFF0ll) break;
        const long long cost = (blocks + per_group - 1) / per_group * (R + K - 1);
        if (best < 0 || cost < best || (cost == best && p.share != p.R)) { best = cost; p.R = p.share = R; p.segs = segs; p.strips = (int)strips; }
        const long long rows = (blocks * R + per_group - 1) / per_group, even = rows + ((rows + R - 2) / R + 1) * (K - 1);      // (the most runs that so many rows can touch)
        if (blocks * R >= per_group && even < best) { best = even; p.R = R; p.share = 1; p.segs = segs; p.strips = (int)strips; }
    }
    if (best < 0) return SS_ERR_UNSUPPORTED;
    const long long units = (p.strips + 15ll) / 16 * (p.R / p.share);
    p.per = (int)(units < per_group ? units : per_group);
    p.rows = (int)(units / p.per) * p.share;
    p.more = (int)(units % p.per);
    dwconv_mfma_kernel<DT, K><<<dim3((unsigned)(p.per * p.groups)), dim3(512), 0, s>>>(p);
    return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_HIP;
}

// ---------------------------------------------------------------------------------------------
// Few outputs, square filters, on the vector ALU.
//
// A thread owns ROWS x TWF neighbouring outputs of two channels.  All of its inputs and the filter's taps are asked for before the first
// multiplication, so that there is one memory latency (dwconv_kernel has one per filter row, the matrix kernel a barrier per input row
// behind a set-up of 5 us); the taps wait in LDS as fp32, the threads' positions come from multiply-and-shift divisions.  Order of the sums and
// rounding are those of dwconv_kernel.  us, bf16, against the faster of those two before: 3x3 14 x 14 x 14 x 96 4.8 -> 3.7, 16 x 56 x 56 x 96 8.5 -> 6.3,
// 128 x 56 x 56 x 96 40.6 -> 32.1; 5x5 14 x 14 x 14 x 96 6.9 -> 3.8, 16 x 28 x 28 x 96 7.3 -> 4.7, 12 x 56 x 56 x 96 10.1 -> 7.7; 7x7 14 x 14 x 14 x 96
// 8.3 -> 3.9, 1 x 56 x 56 x 96 8.5 -> 4.4, 20 x 28 x 35 x 96 10.2 -> 7.6.  From there on the vector ALU bounds it: 49 multiply-adds and some 40
// other instructions per two 7x7 outputs (four rows of a thread share their inputs' conversion, but take registers and leave half of the chip idle
// where there are few).  Four channels per thread (twice the loads' width) are 1.1 to 1.6 times as slow, eight columns 1.0 to 1.3.
// ---------------------------------------------------------------------------------------------
struct DwFewParams {
    const uint16_t *x, *w;
    const float *bias;
    uint16_t *y;
    int H, W, C, ph, pw, Ho, Wo, act, total;
    unsigned x_bytes, w_bytes;
    unsigned run_mul, wq_mul, hq_mul, shifts;      // divisions by C / 2, ceil(Wo / TWF) and ceil(Ho / ROWS)
};
static_assert(sizeof(DwFewParams) <= 112, "a cheap launch");
template <int DT>
__device__ __forceinline__ void widen2(uint32_t v, float &a, float &b)
{
    if constexpr (DT == SS_F16) {
        a = (float)__builtin_bit_cast(_Float16, (uint16_t)(v & 0xFFFFu));
        b = (float)__builtin_bit_cast(_Float16, (uint16_t)(v >> 16));
    } else {
        a = __builtin_bit_cast(float, v << 16);
        b = __builtin_bit_cast(float, v & 0xFFFF0000u);
    }
}

template <int DT, int K, int TWF, int ROWS>
__global__ __launch_bounds__(256) void dwconv_few_kernel(DwFewParams p)
{
    constexpr int COLS = K + TWF - 1, INS = K + ROWS - 1;      // input columns and rows
    extern __shared__ __attribute__((aligned(16))) float taps_s[];      // [tap][C]
    const int tid = threadIdx.x;
    const unsigned gid = blockIdx.x * 256u + tid;
    const bool live = gid < (unsigned)p.total;
    auto div = [](unsigned n, unsigned mul, unsigned sh) { return (unsigned)(((unsigned long long)n * mul) >> sh); };
    const unsigned id = live ? gid : 0u;
    const int runs = p.C / 2, wq = (p.Wo + TWF - 1) / TWF;
    const unsigned r0 = div(id, p.run_mul, p.shifts & 63u), r1 = div(r0, p.wq_mul, p.shifts >> 6 & 63u), n = div(r1, p.hq_mul, p.shifts >> 12 & 63u);
    const int c = (int)(id - r0 * runs) * 2, wo0 = (int)(r0 - r1 * wq) * TWF, ho = (int)(r1 - n * ((p.Ho + ROWS - 1) / ROWS)) * ROWS;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(p.x), 0, (int)p.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(p.w), 0, (int)p.w_bytes, 0x00020000);

    // ---- the filter: at most TV vectors of 8 taps per thread
    constexpr int TV = kDwFewTaps / 2048;
    u32x4 wv[TV];
#pragma unroll
    for (int i = 0; i < TV; i++) wv[i] = __builtin_amdgcn_raw_buffer_load_b128(rw, (tid + 256 * i) * 16, 0, 0);
    // ---- the inputs (a column outside the image is out of range; rows outside it are loaded, from wherever in the buffer, and not used)
    unsigned off[COLS];
    const unsigned first = (unsigned)((((int)n * p.H + ho - p.ph) * p.W + wo0 - p.pw) * p.C + c) * 2u, row_bytes = (unsigned)(p.W * p.C) * 2u;
#pragma unroll
    for (int j = 0; j < COLS; j++) {
        const bool in = (unsigned)(wo0 - p.pw + j) < (unsigned)p.W;
        off[j] = in ? first + (unsigned)(j * p.C) * 2u : 0x80000000u;
    }
    uint32_t xv[INS][COLS];
#pragma unroll
    for (int r = 0; r < INS; r++)
#pragma unroll
        for (int j = 0; j < COLS; j++) xv[r][j] = __builtin_amdgcn_raw_buffer_load_b32(rx, (int)(off[j] + (unsigned)r * row_bytes), 0, 0);
    float acc[ROWS][TWF][2];
#pragma unroll
    for (int e = 0; e < 2; e++) {
        const float b = p.bias ? p.bias[c + e] : 0.f;
#pragma unroll
        for (int o = 0; o < ROWS; o++)
#pragma unroll
            for (int j = 0; j < TWF; j++) acc[o][j][e] = b;
    }
#pragma unroll
    for (int i = 0; i < TV; i++) {
        const int at = (tid + 256 * i) * 8;
        if (at < K * K * p.C) {
            float f[8];
            widen8<DT>(wv[i], f);
            *reinterpret_cast<f32x4 *>(taps_s + at) = f32x4{f[0], f[1], f[2], f[3]};
            *reinterpret_cast<f32x4 *>(taps_s + at + 4) = f32x4{f[4], f[5], f[6], f[7]};
        }
    }
    lds_barrier();
    if (!live) return;
    const float *const taps = taps_s + c;
#pragma unroll
    for (int r = 0; r < INS; r++) {
        if ((unsigned)(ho - p.ph + r) < (unsigned)p.H) {
            float xf[COLS][2];
#pragma unroll
            for (int j = 0; j < COLS; j++) widen2<DT>(xv[r][j], xf[j][0], xf[j][1]);
#pragma unroll
            for (int o = 0; o < ROWS; o++) {              // filter row r - o, for output row ho + o
                if (r - o < 0 || r - o >= K) continue;
#pragma unroll
                for (int t = 0; t < K; t++) {
                    float wf[2];
#pragma unroll
                    for (int e = 0; e < 2; e++) wf[e] = taps[((r - o) * K + t) * p.C + e];
#pragma unroll
                    for (int j = 0; j < TWF; j++)
#pragma unroll
                        for (int e = 0; e < 2; e++) acc[o][j][e] = __builtin_fmaf(wf[e], xf[j + t][e], acc[o][j][e]);
                }
            }
        }
    }
#pragma unroll
    for (int o = 0; o < ROWS; o++) {
        if (ho + o >= p.Ho) break;
        uint16_t *const dst = p.y + (((size_t)n * p.Ho + ho + o) * p.Wo + wo0) * p.C + c;
#pragma unroll
        for (int j = 0; j < TWF; j++) {
            if (wo0 + j >= p.Wo) break;
            float a = acc[o][j][0], b = acc[o][j][1];
            if (p.act == SS_ACT_RELU) { a = a < 0.f ? 0.f : a; b = b < 0.f ? 0.f : b; }
            *reinterpret_cast<uint32_t *>(dst + (size_t)j * p.C) = pack2<DT>(a, b);
        }
    }
}

// floor(n / d) for 0 <= n < 2^31 as (n * mul) >> sh (as fast_div_setup of the convolutions)
static inline unsigned div_setup(unsigned d, unsigned *mul)
{
    unsigned s = 0;
    while ((1ull << s) < d) s++;
    *mul = (unsigned)(((1ull << (31 + s)) + d - 1) / d);
    return 31 + s;
}

template <int DT, int K, int TWF, int ROWS>
static int launch_dw_few(const uint16_t *x, const uint16_t *w, const float *bias, uint16_t *y, int N, int H, int W, int C, int ph, int pw, int Ho, int Wo,
                         int act, unsigned x_bytes, hipStream_t s)
{
    DwFewParams p{};
    p.x = x; p.w = w; p.bias = bias; p.y = y;
    p.H = H; p.W = W; p.C = C; p.ph = ph; p.pw = pw; p.Ho = Ho; p.Wo = Wo; p.act = act;
    const int runs = C / 2, wq = (Wo + TWF - 1) / TWF;
    const int hq = (Ho + ROWS - 1) / ROWS;
    const long long total = (long long)N * hq * wq * runs;
    if (total <= 0 || total > 0x7FFFFF00ll) return SS_ERR_UNSUPPORTED;
    p.total = (int)total;
    p.x_bytes = x_bytes;
    p.w_bytes = (unsigned)(K * K * C * 2);
    p.shifts = div_setup((unsigned)runs, &p.run_mul);
    p.shifts |= div_setup((unsigned)wq, &p.wq_mul) << 6;
    p.shifts |= div_setup((unsigned)hq, &p.hq_mul) << 12;
    dwconv_few_kernel<DT, K, TWF, ROWS><<<dim3((unsigned)((total + 255) / 256)), dim3(256), (size_t)K * K * C * 4, s>>>(p);
    return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_HIP;
}

template <int DT>
static int launch_dw(const uint16_t *x, const uint16_t *w, const float *bias, uint16_t *y, int N, int H, int W, int C, int kh,
                     int kw, int ph, int pw, int Ho, int Wo, int act, unsigned x_bytes, hipStream_t s)
{
    const DwShape shape{N, H, W, C, kh, kw, ph, Ho, Wo};
    const int forced = forced_tile(), ncu = compute_units();      // test hook: the kernels by their ids
    if (ncu <= 0) return SS_ERR_HIP;
    const int id = forced >= DW_VECTOR && forced <= DW_FEW_4X4 && dw_fits(shape, forced) ? forced : choose_dw(shape, ncu);
#define SS_DW_FEW(K, TWF, ROWS) launch_dw_few<DT, K, TWF, ROWS>(x, w, bias, y, N, H, W, C, ph, pw, Ho, Wo, act, x_bytes, s)
    if (id >= DW_FEW_1X2) {
        if (kw == 3) return id == DW_FEW_1X4 ? SS_DW_FEW(3, 4, 1) : (id == DW_FEW_2X4 ? SS_DW_FEW(3, 4, 2) : SS_DW_FEW(3, 4, 4));
        if (kw == 5) return SS_DW_FEW(5, 4, 1);
        return id == DW_FEW_1X2 ? SS_DW_FEW(7, 2, 1) : (id == DW_FEW_2X4 ? SS_DW_FEW(7, 4, 2) : SS_DW_FEW(7, 4, 1));
    }
#undef SS_DW_FEW
    if (id == DW_MATRIX) {
        DwParams p{};
        p.x = x; p.w = w; p.bias = bias; p.y = y;
        p.H = H; p.W = W; p.C = C; p.ph = ph; p.pw = pw; p.Ho = Ho; p.Wo = Wo; p.act = act;
        p.x_bytes = x_bytes;
        p.w_bytes = (unsigned)(kh * kw * C * 2);
        p.y_bytes = (unsigned)((long long)N * Ho * Wo * C * 2);
        return kw == 5 ? launch_dw_mfma<DT, 5>(p, N, s) : launch_dw_mfma<DT, 7>(p, N, s);
    }
    const long long total = (long long)N * Ho * ((Wo + TW - 1) / TW) * (C / 8);
    if (total <= 0 || (total + 255) / 256 > 0x7FFFFFFFll) return SS_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)((total + 255) / 256)), block(256);
    const size_t smem = (size_t)kh * kw * C * 2;
    switch (kw) {
        case 3: dwconv_kernel<DT, 3><<<grid, block, smem, s>>>(x, w, bias, y, N, H, W, C, kh, ph, pw, Ho, Wo, act, x_bytes); break;
        case 5: dwconv_kernel<DT, 5><<<grid, block, smem, s>>>(x, w, bias, y, N, H, W, C, kh, ph, pw, Ho, Wo, act, x_bytes); break;
        case 7: dwconv_kernel<DT, 7><<<grid, block, smem, s>>>(x, w, bias, y, N, H, W, C, kh, ph, pw, Ho, Wo, act, x_bytes); break;
        default: return SS_ERR_UNSUPPORTED;
    }
    return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_HIP;
}

}  // namespace ss

using namespace ss;

extern "C" int ss_dwconv2d_fwd(const void *x, int32_t N, int32_t H, int32_t Wd, int32_t C, int32_t dtype, const void *w,
                               const float *bias, int32_t kh, int32_t kw, int32_t pad_h, int32_t pad_w, int32_t act,
                               void *y, void *stream)
{
    if (!x || !w || !y) return SS_ERR_INVALID_ARG;
    if (N <= 0 || H <= 0 || Wd <= 0 || C <= 0 || kh <= 0 || kw <= 0 || pad_h < 0 || pad_w < 0) return SS_ERR_INVALID_ARG;
    if (dtype != SS_F16 && dtype != SS_BF16) return SS_ERR_INVALID_ARG;
    if (act != SS_ACT_NONE && act != SS_ACT_RELU) return SS_ERR_INVALID_ARG;
    if (((uintptr_t)x & 15) || ((uintptr_t)w & 15) || ((uintptr_t)y & 15) || (bias && ((uintptr_t)bias & 3))) return SS_ERR_INVALID_ARG;
    if (H + 2 * pad_h < kh || Wd + 2 * pad_w < kw) return SS_ERR_INVALID_ARG;
    if (C % 8 != 0 || (kw != 3 && kw != 5 && kw != 7) || (long long)kh * kw * C * 2 > 64 * 1024) return SS_ERR_UNSUPPORTED;
    const long long xbytes = (long long)N * H * Wd * C * 2;
    if (xbytes >= (1ll << 31)) return SS_ERR_UNSUPPORTED;
    const int Ho = H + 2 * pad_h - kh + 1, Wo = Wd + 2 * pad_w - kw + 1;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint16_t *xs = static_cast<const uint16_t *>(x), *ws = static_cast<const uint16_t *>(w);
    uint16_t *ys = static_cast<uint16_t *>(y);
    return dtype == SS_F16 ? launch_dw<SS_F16>(xs, ws, bias, ys, N, H, Wd, C, kh, kw, pad_h, pad_w, Ho, Wo, act, (unsigned)xbytes, s)
                           : launch_dw<SS_BF16>(xs, ws, bias, ys, N, H, Wd, C, kh, kw, pad_h, pad_w, Ho, Wo, act, (unsigned)xbytes, s);
}
