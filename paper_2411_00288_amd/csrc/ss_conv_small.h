// Convolution on few output pixels (small-batch inference, the late stages of a network): one memory latency deep.
//
// A layer with a few hundred output pixels gives the tiled kernels a handful of workgroups, each of which walks through
// the whole reduction chunk by chunk: a chain of load -> LDS -> barrier -> multiply steps of about half a microsecond
// each on a chip that is otherwise idle (ResNet-50 at one image: 5-10 us per layer).  Here the output is cut into
// 32-channel x 32-pixel tiles, one per workgroup, and the workgroup's waves split the reduction: every wave issues all the loads
// of its share at once, multiplies, and the partial sums meet once in LDS, where they are added in wave order (a fixed
// order: the result does not depend on timing), rounded once and stored.  There is no barrier before that meeting.
//   * 1x1 kernels and the channels-last flattening (DIRECT): a lane's activation fragment, 16 consecutive reduction
//     indices of one pixel, is two aligned 16-byte runs in memory; it goes straight into the matrix instruction's
//     registers, no LDS.
//   * the paper's flattening with a KH x KW kernel: a wave takes whole chunks of 32 channels, transposes the taps in registers
//     as the tiled kernels do (stage_taps) into LDS of its own and reads the fragments back.
// The arithmetic is that of the tiled kernels up to the order of the fp32 additions.
// What bounds it: instructions in a row.  Nothing else runs beside a wave here, so each instruction costs its four to five clocks, and the
// time from the start to the first load and from the last product to the store counts in full (half of a kernel's 3 us).  Hence unsigned
// arithmetic ahead of the loads, weights asked for before the input's addresses are worked out, no choices where a wave's steps are all
// whole, and one branch for four activations: ResNet-50 at one image 212.7 -> 204.6 us over 53 layers, 250 layers of up to 3000
// pixels drawn at random 0.98 of the time.
#ifndef SS_CONV_SMALL_H_
#define SS_CONV_SMALL_H_
#include "ss_conv_kernel.h"

namespace ss {

// LDS of a wave: its staging area (taps), which later holds its partial sums
template <int MODE, int TAPS, int PX, int TM>
constexpr size_t small_wave_lds()
{
    const size_t stage = small_taps(MODE) ? (size_t)PX * TAPS * 64 : 0, part = (size_t)TM * 4096;
    return stage > part ? stage : part;
}

// PX: pixels of a tile (32, or 16: half of the matrix instruction's columns stay empty, and twice as many workgroups share
// the loads, which is what bounds a grid far below the chip's size).  NW: waves.  RING: reduction steps in flight per wave (direct modes).
template <int DT, bool SPARSE, int MODE, int KH, int KW, int PX, int TM, int NW, int RING>
__global__ __launch_bounds__(NW * 64) void conv_small_kernel(ConvArgs args)
{
    const ConvParams p = unpack_args<DT, SPARSE, KH, KW, MODE == SMALL_RSC || MODE == SMALL_RSCW, true>(args);
    constexpr bool Q8 = is_byte_type(DT);
    constexpr int ODT = out_type<DT>();
    constexpr int TAPS = KH * KW;
    constexpr bool SWZ = TAPS == 9;                       // LDS row layout of the tap modes (see ChunkShape::SWZ; 2x2 rows are 16 vectors, XOR-ed with the whole row number)
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 5, c = lane & 31;
    // Row tiles fastest: workgroups are dealt to the 8 XCDs round-robin, so with a multiple of 8 row tiles every XCD's L2
    // reads its own eighth of the weights only.
    const int mt = blockIdx.x * TM;                       // first row tile
    const int n0 = blockIdx.y * PX;
    const int HoWo = p.Ho * p.Wo;

    // What the finished quads need from memory, asked for right behind the first loads of the reduction: after it these loads would be
    // a second memory latency, ahead of it their addresses would delay the first.  Consecutive threads finish the tile's channels of a pixel.
    const float floor = p.act == SS_ACT_RELU ? 0.f : -__builtin_inff();
    const bool four = (p.Cout & 3) == 0;
    constexpr int QUADS = PX * 8 * TM, QIT = (QUADS + NW * 64 - 1) / (NW * 64);      // quads of channels in the tile, per thread
    struct Tail {
        unsigned bias[4], scale[4], res[4];               // (res: two pairs, or, where the channel count is no multiple of 4, four halves)
    };
    auto quad = [&](int t, int *pl, int *cq, int *pg, int *o) {
        *pl = t / (8 * TM);                               // pixel, quad of channels: accumulators 4*(cq/2).. of lane group cq%2
        *cq = t % (8 * TM);
        *pg = n0 + *pl;
        *o = mt * 32 + *cq * 4;
        return (QUADS % (NW * 64) == 0 || t < QUADS) && *pg < p.P && *o < p.Cout;
    };
    auto vector_of = [&](const void *v, size_t bytes) {  // (an absent vector: no bytes, every load gives zero)
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(v), 0, v != nullptr ? (int)bytes : 0, kRsrcFlags);
    };
    Tail tail[QIT];
    constexpr bool EARLY = !(small_taps(MODE) && TM == 2);      // (those hold 254 registers already: they fetch before the last barrier)
    auto fetch_tail = [&]() {
        const __amdgpu_buffer_rsrc_t rb = vector_of(p.bias, (size_t)p.Cout * 4), rs = vector_of(p.scale, (size_t)p.Cout * 4);
        const __amdgpu_buffer_rsrc_t rr = vector_of(p.residual, (size_t)p.P * p.Cout * 2);
#pragma unroll
        for (int i = 0; i < QIT; i++) {
            int pl, cq, pg, o;
            const bool in = quad(tid + i * NW * 64, &pl, &cq, &pg, &o);
            const unsigned vb = in ? (unsigned)o * 4u : kOutOfRange;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                tail[i].bias[e] = __builtin_amdgcn_raw_buffer_load_b32(rb, (int)(vb + 4u * e), 0, 0);
                if constexpr (Q8) tail[i].scale[e] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(vb + 4u * e), 0, 0);
            }
            if constexpr (!Q8) {
                const unsigned vr = in ? ((unsigned)pg * p.Cout + o) * 2u : kOutOfRange;      // (the launch keeps outputs below 2 GiB)
#pragma unroll
                for (int e = 0; e < 4; e++) tail[i].res[e] = 0u;
                if (p.residual != nullptr) {              // uniform
                    if (four) {
                        const auto u = __builtin_amdgcn_raw_buffer_load_b64(rr, (int)vr, 0, 0);
                        tail[i].res[0] = u[0]; tail[i].res[1] = u[1];
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; e++)       // (past the row's end: never used)
                            tail[i].res[e] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rr, (int)(vr + 2u * e), 0, 0);
                    }
                }
            }
        }
    };

    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(p.x), 0, (int)p.x_bytes, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(p.a_vals), 0, (int)p.a_bytes, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(p.a_meta), 0, (int)p.meta_bytes, kRsrcFlags);
    unsigned a_voff[TM], m_voff[TM];                      // (a row tile past the last one is clamped to it and not stored)
#pragma unroll
    for (int tm = 0; tm < TM; tm++) {
        const int m = min(mt + tm, p.Mt - 1);
        a_voff[tm] = (unsigned)(m * p.Ks * (SPARSE ? 1 : 2) * 64 + lane) * 16u;
        m_voff[tm] = (unsigned)(m * p.Kp * 64 + lane) * 4u;
    }
    using A = AStep<SPARSE, TM>;
    auto load_a = [&](A &a, int ks, unsigned out = 0u) {  // (out = bit 31: nothing is fetched, the weights are zero)
#pragma unroll
        for (int tm = 0; tm < TM; tm++) {
            if constexpr (SPARSE) {
                a.v[0][tm] = __builtin_amdgcn_raw_buffer_load_b128(ra, (int)(a_voff[tm] | out), ks * 1024, 0);
                a.idx[tm] = __builtin_amdgcn_raw_buffer_load_b32(rm, (int)(m_voff[tm] | out), (Q8 ? ks : (ks >> 1)) * 256, 0);
            } else {
                a.v[0][tm] = __builtin_amdgcn_raw_buffer_load_b128(ra, (int)(a_voff[tm] | out), ks * 2048, 0);
                a.v[1][tm] = __builtin_amdgcn_raw_buffer_load_b128(ra, (int)(a_voff[tm] | out), ks * 2048 + 1024, 0);
            }
        }
    };
    Acc<DT> acc[TM];
#pragma unroll
    for (int tm = 0; tm < TM; tm++)
#pragma unroll
        for (int v = 0; v < 16; v++) acc[tm][v] = 0;
    auto multiply = [&](const A &a, const B32 &b, int ks) {
        const int shift = Q8 ? 0 : (ks & 1) * 16;
#pragma unroll
        for (int tm = 0; tm < TM; tm++) {
            if constexpr (SPARSE) {
                acc[tm] = mma_sparse<DT>(a.v[0][tm], b, acc[tm], a.idx[tm] >> shift);
            } else {                                      // (dense FP8: pairs of the short instruction, whose operands are not tied to 8-register tuples)
                acc[tm] = mma_dense<DT>(a.v[0][tm], b.lo, acc[tm]);
                acc[tm] = mma_dense<DT>(a.v[1][tm], b.hi, acc[tm]);
            }
        }
    };
    // position of an output pixel's window
    struct Pixel {
        int ih, iw;
        unsigned byte;
    };
    auto pixel = [&](int pg) {
        Pixel q{-(1 << 28), -(1 << 28), 0u};              // past the last pixel: every bounds test fails
        if (pg < p.P) {
            const int n = fast_div(pg, p.howo_mul, p.howo_sh);
            const int rem = pg - n * HoWo;
            const int ho = fast_div(rem, p.wo_mul, p.wo_sh);
            q.ih = ho * p.sh - p.ph;
            q.iw = (rem - ho * p.Wo) * p.sw - p.pw;
            q.byte = (unsigned)(((n * p.H + q.ih) * p.W + q.iw) * p.Cin * 2);
        }
        return q;
    };

    if constexpr (!small_taps(MODE)) {
        // ------------------------------------------------------------ fragments straight from memory
        const int per = (int)(((unsigned)p.Ks + NW - 1) / NW);      // steps of a wave
        const int s0 = min(wave * per, p.Ks), s1 = min(s0 + per, p.Ks);
        const int rem = p.K - (p.Ks - 1) * 32;            // reduction indices of the last step
        const bool whole = rem == 32 && s1 - s0 >= RING;  // uniform: the first RING steps are all there and whole
        A a[RING];
        B32 b[RING];
        // Steps behind a share's end fetch nothing and multiply zeros.
        auto out = [&](int s) { return s < s1 ? 0u : kOutOfRange; };      // uniform
        // The weights' first steps before anything of the input's addresses, which take longer to work out.  Whole steps have nothing to
        // choose between: one address each for values and metadata, and constant offsets.
        if (whole) {
            constexpr int STEP = SPARSE ? 1024 : 2048;
#pragma unroll
            for (int j = 0; j < RING; j++)
#pragma unroll
                for (int tm = 0; tm < TM; tm++) {
                    a[j].v[0][tm] = __builtin_amdgcn_raw_buffer_load_b128(ra, (int)a_voff[tm], s0 * STEP + j * STEP, 0);
                    if constexpr (SPARSE) a[j].idx[tm] = __builtin_amdgcn_raw_buffer_load_b32(rm, (int)m_voff[tm], (Q8 ? s0 + j : ((s0 + j) >> 1)) * 256, 0);
                    else a[j].v[1][tm] = __builtin_amdgcn_raw_buffer_load_b128(ra, (int)a_voff[tm], s0 * STEP + j * STEP + 1024, 0);
                }
        } else {
#pragma unroll
            for (int j = 0; j < RING; j++) load_a(a[j], s0 + j, out(s0 + j));
        }
        __builtin_amdgcn_sched_barrier(0);
        const int pg = PX == 32 || c < PX ? n0 + c : p.P;
        Pixel px;
        if (MODE == SMALL_PW && p.sh == 1 && p.sw == 1 && (p.ph | p.pw) == 0) {      // uniform: pixels and positions in the input are the same thing
            px = Pixel{pg < p.P ? 0 : -(1 << 28), 0, (unsigned)pg * p.Cin * 2u};
        } else {
            px = pixel(pg);
        }
        // Byte offsets of a step's two octets of channels (bit 31: outside, reads as zero).
        const unsigned base = px.byte + 32u * g;
        const bool in0 = (unsigned)px.ih < (unsigned)p.H && (unsigned)px.iw < (unsigned)p.W;
        const unsigned pw0 = in0 ? base : kOutOfRange;
        const unsigned pw_lo = 16 * g < rem ? pw0 : kOutOfRange, pw_hi = 16 * g + 8 < rem ? pw0 : kOutOfRange;
        auto octet = [&](int k) -> u32x4 {                // RSC: 8 reduction indices from k
            const int tap = fast_div(k, p.cin_mul, p.cin_sh);
            const int r = fast_div(tap, p.kw_mul, p.kw_sh), t = tap - r * p.kw;
            const bool ok = (unsigned)(px.ih + r) < (unsigned)p.H && (unsigned)(px.iw + t) < (unsigned)p.W && k < p.K;
            return __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(ok ? px.byte + (unsigned)(((r * p.W + t) * p.Cin + k - tap * p.Cin) * 2) : kOutOfRange), 0, 0);
        };
        auto load_x = [&](B32 &b, int s) {
            if constexpr (MODE == SMALL_PW) {
                const bool last = s == p.Ks - 1;
                b.lo = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)((last ? pw_lo : pw0) | out(s)), s * 64, 0);
                b.hi = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(((last ? pw_hi : pw0) | out(s)) + 16u), s * 64, 0);
            } else if constexpr (MODE == SMALL_RSCW) {
                const int k = s * 32, tap = fast_div(k, p.cin_mul, p.cin_sh);
                const int r = fast_div(tap, p.kw_mul, p.kw_sh), t = tap - r * p.kw;
                const bool ok = (unsigned)(px.ih + r) < (unsigned)p.H && (unsigned)(px.iw + t) < (unsigned)p.W;
                const unsigned off = (ok ? base + (unsigned)(((r * p.W + t) * p.Cin + k - tap * p.Cin) * 2) : kOutOfRange) | out(s);
                b.lo = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)off, 0, 0);
                b.hi = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(off + 16u), 0, 0);
            } else {
                const int k = s < s1 ? s * 32 + 16 * g : 1 << 30;
                b.lo = octet(k);
                b.hi = octet(k + 8);
            }
        };
        if (MODE == SMALL_PW && whole) {
#pragma unroll
            for (int j = 0; j < RING; j++) {
                b[j].lo = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(pw0 + 64u * j), s0 * 64, 0);
                b[j].hi = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(pw0 + 64u * j + 16u), s0 * 64, 0);
                __builtin_amdgcn_sched_barrier(0);        // (in this order: the first step multiplies while the others are on their way)
            }
        } else {
#pragma unroll
            for (int j = 0; j < RING; j++) {
                load_x(b[j], s0 + j);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (EARLY) fetch_tail();
        int s = s0;
        for (; s + RING < s1; s += RING) {
#pragma unroll
            for (int j = 0; j < RING; j++) {
                multiply(a[j], b[j], s + j);
                load_a(a[j], s + RING + j, out(s + RING + j));
                load_x(b[j], s + RING + j);
            }
        }
#pragma unroll
        for (int j = 0; j < RING; j++) multiply(a[j], b[j], s + j);
    } else {
        // ------------------------------------------------------------ taps of whole channel chunks, transposed in the wave's own LDS
        constexpr int VPR = TAPS * 4;                     // 16-byte vectors per pixel row of a chunk (TAPS steps of 64 bytes)
        u32x4 *const mine = reinterpret_cast<u32x4 *>(smem) + wave * (PX * VPR);
        const int unit = lane & 3, nchunks = (p.Ks + TAPS - 1) / TAPS;
        constexpr int IT = PX / 16;                       // pixels per lane
        unsigned tapoff[IT][TAPS];
#pragma unroll
        for (int i = 0; i < IT; i++) {
            const Pixel px = pixel(n0 + (lane >> 2) + 16 * i);
#pragma unroll
            for (int tap = 0; tap < TAPS; tap++) {
                const int r = tap / KW, t = tap % KW;
                const bool ok = (unsigned)(px.ih + r) < (unsigned)p.H && (unsigned)(px.iw + t) < (unsigned)p.W;
                tapoff[i][tap] = ok ? px.byte + (unsigned)(((r * p.W + t) * p.Cin + unit * 8) * 2) : kOutOfRange;
            }
        }
        u32x4 x[IT][TAPS];
        A a[TAPS];
        bool half = false;
        auto load_x = [&](int ci) {
            const unsigned soff = (unsigned)ci * 64;
            if constexpr (MODE == SMALL_TAPSR) {
                const int ch = ci * 32 + unit * 8;
                half = ch + 4 == p.Cin;
                const unsigned past = ch < p.Cin ? 0u : kOutOfRange, early = half ? 8u : 0u;
#pragma unroll
                for (int i = 0; i < IT; i++)
#pragma unroll
                    for (int tap = 0; tap < TAPS; tap++)
                        x[i][tap] = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)((tapoff[i][tap] | past) + (soff - early)), 0, 0);
            } else {
#pragma unroll
                for (int i = 0; i < IT; i++)
#pragma unroll
                    for (int tap = 0; tap < TAPS; tap++)
                        x[i][tap] = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)tapoff[i][tap], soff, 0);
            }
        };
        if (wave < nchunks) load_x(wave);
        if constexpr (EARLY) fetch_tail();
        for (int ci = wave; ci < nchunks; ci += NW) {
#pragma unroll
            for (int s = 0; s < TAPS; s++) load_a(a[s], min(ci * TAPS + s, p.Ks - 1));      // (a ragged chunk's missing steps: LDS holds zeros for them)
#pragma unroll
            for (int i = 0; i < IT; i++) {
                const int pr = (lane >> 2) + 16 * i, key = SWZ ? (pr >> 2) & 3 : pr & 15;
#pragma unroll
                for (int v = 0; v < TAPS; v++) mine[pr * VPR + ((unit * TAPS + v) ^ key)] = taps_vector<Q8, MODE == SMALL_TAPSR, TAPS>(x[i], v, half);
            }
            if (ci + NW < nchunks) load_x(ci + NW);
            __builtin_amdgcn_wave_barrier();              // (a wave's LDS operations execute in order: the reads below see the writes above)
            const int cc = c & (PX - 1), key = SWZ ? (cc >> 2) & 3 : cc & 15;
#pragma unroll
            for (int s = 0; s < TAPS; s++) {
                B32 b;
                b.lo = mine[cc * VPR + ((s * 4 + 2 * g) ^ key)];
                b.hi = mine[cc * VPR + ((s * 4 + 2 * g + 1) ^ key)];
                multiply(a[s], b, ci * TAPS + s);
            }
            __builtin_amdgcn_wave_barrier();
        }
    }

    // ---------------------------------------------------------------- partial sums meet in LDS, in register order [wave][quad][lane]
    // (each wave's region lies inside its own staging area where there is one: no barrier before it)
    constexpr int RSTRIDE = (int)(small_wave_lds<MODE, TAPS, PX, TM>() / 16);       // 16-byte vectors from one wave's region to the next
    u32x4 *const part = reinterpret_cast<u32x4 *>(smem);
#pragma unroll
    for (int tm = 0; tm < TM; tm++)
#pragma unroll
        for (int q = 0; q < 4; q++) {
            u32x4 w;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const auto v = acc[tm][4 * q + e];
                w[e] = __builtin_bit_cast(uint32_t, v);
            }
            part[wave * RSTRIDE + (tm * 4 + q) * 64 + lane] = w;
        }
    // (FOUR: four whole channels, read and written at once.  One branch for the four activations: apart they run side by side)
    auto finish = [&](auto FOUR, int t, const Tail &f) {
        int pl, cq, pg, o;
        if (!quad(t, &pl, &cq, &pg, &o)) return;
        float v[4];
        const int from = (cq >> 1) * 64 + (cq & 1) * 32 + pl;
        using Quad = typename std::conditional<DT == SS_I8, i32x4, f32x4>::type;
        Quad sum = __builtin_bit_cast(Quad, part[from]);
#pragma unroll
        for (int w = 1; w < NW; w++) sum += __builtin_bit_cast(Quad, part[w * RSTRIDE + from]);
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const float bias = __builtin_bit_cast(float, f.bias[e]), scale = Q8 && p.scale != nullptr ? __builtin_bit_cast(float, f.scale[e]) : 1.f;
            const uint16_t res = FOUR ? (uint16_t)(f.res[e >> 1] >> (16 * (e & 1))) : (uint16_t)f.res[e];
            v[e] = Q8 ? (float)sum[e] * scale + bias : (float)sum[e] + bias + widen<ODT>(res);
        }
        if (p.act == SS_ACT_GELU) {
#pragma unroll
            for (int e = 0; e < 4; e++) v[e] = gelu_cdf<ODT>(v[e]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; e++) v[e] = floor_at(v[e], floor);
        }
        uint16_t *y = p.y + (size_t)pg * p.Cout + o;
        if constexpr (FOUR) {
            *reinterpret_cast<uint2 *>(y) = make_uint2(cvt_pack2<ODT>(v[0], v[1]), cvt_pack2<ODT>(v[2], v[3]));
        } else {
#pragma unroll
            for (int e = 0; e < 4; e++)
                if (o + e < p.Cout) y[e] = (uint16_t)(cvt_pack2<ODT>(v[e], 0.f) & 0xFFFFu);
        }
    };
    if constexpr (!EARLY) fetch_tail();
    __syncthreads();
    if (four) {
#pragma unroll
        for (int i = 0; i < QIT; i++) finish(std::true_type{}, tid + i * NW * 64, tail[i]);
    } else {
#pragma unroll
        for (int i = 0; i < QIT; i++) finish(std::false_type{}, tid + i * NW * 64, tail[i]);
    }
}

template <int DT, bool SPARSE, int MODE, int KH, int KW, int PX, int TM, int NW, int RING = 4>
static int launch_small_waves(const ConvParams &p, hipStream_t s)
{
    constexpr size_t smem = NW * small_wave_lds<MODE, KH * KW, PX, TM>();
    static_assert(smem <= 160 * 1024, "LDS");
    const long long rows = (p.Mt + TM - 1) / TM, cols = ((long long)p.P + PX - 1) / PX;
    if (rows <= 0 || cols <= 0 || cols > 65535) return SS_ERR_INVALID_ARG;      // (the grid's second dimension; only a forced variant gets here)
    auto kern = conv_small_kernel<DT, SPARSE, MODE, KH, KW, PX, TM, NW, RING>;
    if (smem > 64 * 1024) {
        static std::atomic<unsigned long long> done_mask{0};      // as in launch(): once per device
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) return SS_ERR_HIP;
        const unsigned long long bit = 1ull << (dev & 63);
        if (dev >= 64 || !(done_mask.load(std::memory_order_acquire) & bit)) {
            if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem) != hipSuccess)
                return SS_ERR_HIP;
            if (dev < 64) done_mask.fetch_or(bit, std::memory_order_release);
        }
    }
    kern<<<dim3((unsigned)rows, (unsigned)cols), dim3(NW * 64), smem, s>>>(conv_args(p, true, MODE == SMALL_RSC || MODE == SMALL_RSCW));
    return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_HIP;
}

template <int DT, bool SPARSE, int MODE, int KH, int KW>
static int launch_small(const ConvParams &p, int variant, hipStream_t s)
{
    constexpr int taps = small_taps(MODE) ? KH * KW : 0;
    if (variant < 0) {                                    // the library decides
        const int ncu = compute_units();
        if (ncu <= 0) return SS_ERR_HIP;
        variant = small_variant(p, taps, SPARSE, ncu);
        if (variant < 0) return SS_ERR_INVALID_ARG;
    }
    auto waves = [&](auto px, auto tm) -> int {
        constexpr int PX = decltype(px)::value, TM = decltype(tm)::value;
        switch (small_waves(p, taps, PX == 16)) {
            case 2: return launch_small_waves<DT, SPARSE, MODE, KH, KW, PX, TM, 2>(p, s);
            case 4: return launch_small_waves<DT, SPARSE, MODE, KH, KW, PX, TM, 4>(p, s);
            case 8:
                if constexpr (taps == 0)                  // shares of more than four steps
                    if (p.Ks > 32) return launch_small_waves<DT, SPARSE, MODE, KH, KW, PX, TM, 8, 8>(p, s);
                return launch_small_waves<DT, SPARSE, MODE, KH, KW, PX, TM, 8>(p, s);
            default: break;
        }
        if constexpr (PX == 16 && taps == 0) return launch_small_waves<DT, SPARSE, MODE, KH, KW, PX, TM, 16>(p, s);
        return SS_ERR_INVALID_ARG;
    };
    using std::integral_constant;
    if (variant == SMALL_16) return waves(integral_constant<int, 16>{}, integral_constant<int, 1>{});
    if (variant == SMALL_32) return waves(integral_constant<int, 32>{}, integral_constant<int, 1>{});
    return waves(integral_constant<int, 32>{}, integral_constant<int, 2>{});
}

// Returns SS_ERR_INVALID_ARG where no mode fits, or (variant < 0: the library decides) where the tiled kernels are the better choice.
template <int DT, bool SPARSE>
static int small_mode(const ss_weight_desc *desc, const ConvParams &p, int variant, hipStream_t s)
{
    switch (small_staging(desc, p)) {
        case SMALL_PW: return launch_small<DT, SPARSE, SMALL_PW, 1, 1>(p, variant, s);
        case SMALL_RSCW: return launch_small<DT, SPARSE, SMALL_RSCW, 1, 1>(p, variant, s);
        case SMALL_RSC: return launch_small<DT, SPARSE, SMALL_RSC, 1, 1>(p, variant, s);
        case SMALL_TAPS:
            return desc->kh == 3 ? launch_small<DT, SPARSE, SMALL_TAPS, 3, 3>(p, variant, s) : launch_small<DT, SPARSE, SMALL_TAPS, 2, 2>(p, variant, s);
        case SMALL_TAPSR:
            if constexpr (!is_byte_type(DT))
                return desc->kh == 3 ? launch_small<DT, SPARSE, SMALL_TAPSR, 3, 3>(p, variant, s) : launch_small<DT, SPARSE, SMALL_TAPSR, 2, 2>(p, variant, s);
            return SS_ERR_INVALID_ARG;
        default: return SS_ERR_INVALID_ARG;
    }
}

// ---------------------------------------------------------------------------------------------
// The fused pair (3x3 in the paper's flattening -> 1x1 + residual, see conv_kernel's FUSE) on few output pixels: a workgroup of eight
// waves owns PX pixels through both layers.  All chunks of the first layer's unfolded input are staged in LDS at once (one
// memory latency, the weights of both layers in flight with it); the waves then split rows x reduction of the first layer, the
// partial sums meet in LDS, the finished 16-bit tile stays there, and the waves take the second layer's row tiles in turn.
// Measured against the tiled fused kernel, whose 64-pixel workgroups are 49 and 13 on one image: 64 -> 64 -> 256 at 56x56
// 9.2 -> 5.8 us, 128 -> 128 -> 512 at 28x28 11.5 -> 8.3 (bound by the weights each workgroup fetches: a ring of 18 instead of 9
// steps in flight measured 8.6); past one workgroup per compute unit the tiled kernel shares them over more pixels and wins.
// ---------------------------------------------------------------------------------------------
// THIRD: as in conv_kernel.  The second layer's output stays in LDS as well, and the waves split the third one's rows and reduction.  Its sums are those of
// its own call, share for share (pw_shares), so that both give the same bits: a wave has one share; or two, where there are more of them than
// waves to a row tile; or begins or ends one that is longer than the eight steps a wave holds weights for, the second taking the sums over
// through LDS.  (A kernel each: with the three in one, decided at run time, the 64- and 128-channel ones took 0.74 and 0.96 us longer on one image.)
enum { THIRD_NONE = 0, THIRD_SHARE = 1, THIRD_TWO = 2, THIRD_HANDED = 3 };
// MT: the first layer's row tiles (2 or 4: a bottleneck of 64 or 128 channels), or 0 where they are known at run time only.  Known, the
// waves' shares and the loops over them are constants, and every LDS read of a phase is under way before the first is needed.
template <int DT, bool SPARSE, int PX, int MT, int THIRD>
__global__ __launch_bounds__(kPairWaves * 64) void pair_small_kernel(kernel_params<THIRD> p)
{
    ThirdParams p3{};
    if constexpr (THIRD != THIRD_NONE) p3 = p;
    if constexpr (MT > 0) { p.Mt = p.Ks2 = MT; p.Cout = 32 * MT; }
    constexpr int TAPS = 9, VPR = 36, NT = kPairWaves * 64, RING = 9, KS2 = MT > 0 ? MT : 8;
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 5, c = lane & 31, cc = c & (PX - 1);
    const int n0 = blockIdx.x * PX;
    const int HoWo = p.Ho * p.Wo;
    const int nchunks = (int)((unsigned)p.Ks / TAPS);     // cin % 32 == 0
    const PairShape sh = pair_shape(PX, nchunks, p.Cout, THIRD != THIRD_NONE ? p.Cout2 : 0);
    u32x4 *const stage = reinterpret_cast<u32x4 *>(smem);
    u32x4 *const part = reinterpret_cast<u32x4 *>(reinterpret_cast<char *>(smem) + sh.stage);
    uint16_t *const tile = reinterpret_cast<uint16_t *>(reinterpret_cast<char *>(smem) + sh.stage + sh.part);
    const int TROW = p.Cout + 8;                          // 16-bit units per pixel row of the tile
    uint16_t *const out2 = reinterpret_cast<uint16_t *>(reinterpret_cast<char *>(smem) + sh.stage + sh.part + sh.tile);
    const int T2ROW = p.Cout2 + 8;
    float *const bias1 = reinterpret_cast<float *>(reinterpret_cast<char *>(smem) + sh.stage + sh.part + sh.tile + sh.third);
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(p.x), 0, (int)p.x_bytes, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(p.a_vals), 0, (int)p.a_bytes, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(p.a_meta), 0, (int)p.meta_bytes, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t ra2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(p.a2_vals), 0, (int)p.a2_bytes, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t rm2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(p.a2_meta), 0, (int)p.meta2_bytes, kRsrcFlags);

    // ---- first layer: this wave's row tile and share of the reduction steps
    // (a division by a runtime number is some 25 instructions ahead of the first load: 8 / Mt is a power of two, the other comes as a product)
    const int lg = p.Mt == 1 ? 3 : p.Mt == 2 ? 2 : p.Mt <= 4 ? 1 : 0, groups = 1 << lg;      // waves per row tile (Mt <= 8)
    const int kg = MT > 0 ? wave / MT : fast_div(wave, p.tm_mul, p.tm_sh), rt = wave - kg * p.Mt;
    const bool works = kg < groups;
    const int s0 = works ? kg * p.Ks >> lg : 0, s1 = works ? (kg + 1) * p.Ks >> lg : 0;
    using A = AStep<SPARSE, 1>;
    auto load_w = [&](A &a, __amdgpu_buffer_rsrc_t rv, __amdgpu_buffer_rsrc_t ri, int mt, int Ks, int Kp, int ks) {
        if constexpr (SPARSE) {
            a.v[0][0] = __builtin_amdgcn_raw_buffer_load_b128(rv, lane * 16, (mt * Ks + ks) * 1024, 0);
            a.idx[0] = __builtin_amdgcn_raw_buffer_load_b32(ri, lane * 4, (mt * Kp + (ks >> 1)) * 256, 0);
        } else {
            a.v[0][0] = __builtin_amdgcn_raw_buffer_load_b128(rv, lane * 16, (mt * Ks + ks) * 2048, 0);
            a.v[1][0] = __builtin_amdgcn_raw_buffer_load_b128(rv, lane * 16, (mt * Ks + ks) * 2048 + 1024, 0);
        }
    };
    auto mma = [&](const A &a, const B32 &b, f32x16 acc, int ks) {
        if constexpr (SPARSE) return mma_sparse<DT>(a.v[0][0], b, acc, a.idx[0] >> ((ks & 1) * 16));
        else return mma_dense<DT>(a.v[1][0], b.hi, mma_dense<DT>(a.v[0][0], b.lo, acc));
    };
    // ---- activations: item = (chunk, pixel, octet of channels), nine taps each
    auto stage_item = [&](int it, u32x4 (&x)[TAPS]) {
        const int unit = it & 3, pr = (it >> 2) & (PX - 1), ci = it / (PX * 4);
        const int pg = n0 + pr;
        int ih = -(1 << 28), iw = -(1 << 28);
        unsigned byte = 0;
        if (pg < p.P) {
            const int n = fast_div(pg, p.howo_mul, p.howo_sh);
            const int rem = pg - n * HoWo;
            const int ho = fast_div(rem, p.wo_mul, p.wo_sh);
            ih = ho * p.sh - p.ph;
            iw = (rem - ho * p.Wo) * p.sw - p.pw;
            byte = (unsigned)((((n * p.H + ih) * p.W + iw) * p.Cin + ci * 32 + unit * 8) * 2);
        }
#pragma unroll
        for (int tap = 0; tap < TAPS; tap++) {
            const int r = tap / 3, t = tap % 3;
            const bool ok = (unsigned)(ih + r) < (unsigned)p.H && (unsigned)(iw + t) < (unsigned)p.W;
            x[tap] = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(ok ? byte + (unsigned)((r * p.W + t) * p.Cin * 2) : kOutOfRange), 0, 0);
        }
    };
    auto store_item = [&](int it, const u32x4 (&x)[TAPS]) {
        const int unit = it & 3, pr = (it >> 2) & (PX - 1), ci = it / (PX * 4), key = (pr >> 2) & 3;
#pragma unroll
        for (int v = 0; v < TAPS; v++) stage[(ci * PX + pr) * VPR + ((unit * TAPS + v) ^ key)] = taps_vector<false, false, TAPS>(x, v, false);
    };
    const int items = nchunks * PX * 4;
    const float bias_mine = tid < p.Cout && p.bias != nullptr ? p.bias[tid] : 0.f;      // (at most 256 channels)
    A a[RING];
    {
        u32x4 x[TAPS];
        if (tid < items) stage_item(tid, x);
#pragma unroll
        for (int j = 0; j < RING; j++)
            if (s0 + j < s1) load_w(a[j], ra, rm, rt, p.Ks, p.Kp, s0 + j);      // uniform
        if (tid < items) store_item(tid, x);
    }
    for (int it = tid + NT; it < items; it += NT) {
        u32x4 x[TAPS];
        stage_item(it, x);
        store_item(it, x);
    }
    if (tid < p.Cout) bias1[tid] = bias_mine;
    struct Row2 {
        A a[KS2];
        float4 b[4];
    };
    constexpr int IT = PX * 4 / 64;                       // 16-byte runs of an output row tile per lane
    auto load_res = [&](u32x4 (&res)[IT], int mt) {
#pragma unroll
        for (int j = 0; j < IT; j++) {
            const int it = lane + 64 * j, pg = n0 + (it >> 2);
            res[j] = u32x4{0u, 0u, 0u, 0u};
            if (p.res2 != nullptr && pg < p.P) res[j] = *reinterpret_cast<const u32x4 *>(p.res2 + (size_t)pg * p.Cout2 + mt * 32 + (it & 3) * 8);
        }
    };
    auto load_row2 = [&](Row2 &r, int mt) {
#pragma unroll
        for (int s = 0; s < KS2; s++)
            if (s < p.Ks2) load_w(r.a[s], ra2, rm2, mt, p.Ks2, p.Kp2, s);      // uniform
#pragma unroll
        for (int q = 0; q < 4; q++)
            r.b[q] = p.bias2 ? *reinterpret_cast<const float4 *>(p.bias2 + mt * 32 + 8 * q + 4 * g) : make_float4(0.f, 0.f, 0.f, 0.f);
    };
    Row2 r2;
    u32x4 res[IT], res_next[IT];
    if (wave < p.Mt2) {                                   // in flight while the first layer is multiplied
        load_row2(r2, wave);
        load_res(res_next, wave);
    }
    lds_barrier();
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; v++) acc[v] = 0.f;
    {
        const int key = (cc >> 2) & 3;
        for (int s = s0; s < s1; s += RING) {
#pragma unroll
            for (int j = 0; j < RING; j++) {
                if (s + j < s1) {                         // uniform
                    const int ci = (s + j) * 7282 >> 16, st = s + j - ci * TAPS;      // chunk and step inside it (7282 = ceil(2^16 / 9), exact below 2^13)
                    const u32x4 *row = stage + (ci * PX + cc) * VPR;
                    B32 b;
                    b.lo = row[(st * 4 + 2 * g) ^ key];
                    b.hi = row[(st * 4 + 2 * g + 1) ^ key];
                    acc = mma(a[j], b, acc, s + j);
                    if (s + RING + j < s1) load_w(a[j], ra, rm, rt, p.Ks, p.Kp, s + RING + j);
                }
            }
        }
    }
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const f32x4 w = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
        part[wave * 256 + q * 64 + lane] = __builtin_bit_cast(u32x4, w);
    }
    lds_barrier();
    const float floor1 = p.act == SS_ACT_RELU ? 0.f : -__builtin_inff();
    for (int t = tid; t < PX * 8 * p.Mt; t += NT) {       // quads of channels, pixel fastest: (row tile, quad, pixel)
        const int pl = t & (PX - 1), q = t / PX, m = q >> 3, cq = q & 7;
        float v[4] = {0.f, 0.f, 0.f, 0.f};
        auto add = [&](int k) {
            const f32x4 u = __builtin_bit_cast(f32x4, part[(k * p.Mt + m) * 256 + (cq >> 1) * 64 + (cq & 1) * 32 + pl]);
#pragma unroll
            for (int e = 0; e < 4; e++) v[e] += u[e];
        };
        if constexpr (MT > 0) {
#pragma unroll
            for (int k = 0; k < kPairWaves / MT; k++) add(k);
        } else {
            for (int k = 0; k < groups; k++) add(k);
        }
        const int o = m * 32 + cq * 4;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            v[e] += bias1[o + e];
        }
        if (p.act == SS_ACT_GELU) {
#pragma unroll
            for (int e = 0; e < 4; e++) v[e] = gelu_cdf<DT>(v[e]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; e++) v[e] = floor_at(v[e], floor1);
        }
        *reinterpret_cast<uint2 *>(tile + pl * TROW + o) = make_uint2(cvt_pack2<DT>(v[0], v[1]), cvt_pack2<DT>(v[2], v[3]));
    }
    lds_barrier();
    // ---- the third layer's weights: in flight while the second one is multiplied
    constexpr int KS3 = THIRD ? 8 : 1;
    const int kg3 = THIRD ? (p3.Mt3 == 2 ? wave >> 1 : p3.Mt3 == 3 ? wave * 11 >> 5 : wave >> 2) : 0, rt3 = wave - kg3 * p3.Mt3;      // (2 <= Mt3 <= 4)
    const int span3 = THIRD == THIRD_SHARE ? p3.per3 : THIRD == THIRD_TWO ? 2 * p3.per3 : KS3;      // (a multiple of 4 steps in all, 16 at most)
    const int t0 = THIRD ? min(kg3 * span3, p3.Ks3) : 0, t1 = THIRD ? min(t0 + span3, p3.Ks3) : 0;
    A a3[KS3];
    if constexpr (THIRD) {
        const __amdgpu_buffer_rsrc_t ra3 = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(p3.a3_vals), 0, (int)p3.a3_bytes, kRsrcFlags);
        const __amdgpu_buffer_rsrc_t rm3 = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(p3.a3_meta), 0, (int)p3.meta3_bytes, kRsrcFlags);
#pragma unroll
        for (int j = 0; j < KS3; j++)
            if (t0 + j < t1) load_w(a3[j], ra3, rm3, rt3, p3.Ks3, p3.Kp3, t0 + j);      // uniform
    }
    // ... and the bias of the quads of channels that this thread will finish
    constexpr int Q3 = THIRD ? PX * 32 / NT : 1;          // (at most four row tiles)
    f32x4 bias3[Q3];
    auto quad3 = [&](int i, int *pl) {                    // quad of channels, the fastest; pixel
        const int t = tid + i * NT, n = p3.Mt3 * 8;
        *pl = p3.Mt3 == 4 ? t >> 5 : p3.Mt3 == 2 ? t >> 4 : t * 2731 >> 16;      // (2731 = ceil(2^16 / 24), exact below 2^12)
        return t - *pl * n;
    };
    if constexpr (THIRD) {
        const __amdgpu_buffer_rsrc_t rb3 = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p3.bias3), 0, p3.bias3 != nullptr ? p3.Cout3 * 4 : 0, kRsrcFlags);
#pragma unroll
        for (int i = 0; i < Q3; i++) {
            int pl;
            bias3[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rb3, quad3(i, &pl) * 16, 0, 0));
        }
    }
    // ---- second layer
    const float floor2 = p.act2 == SS_ACT_RELU ? 0.f : -__builtin_inff();
    float *const slab = reinterpret_cast<float *>(smem) + wave * (PX * kFuseRow);
    for (int mt = wave; mt < p.Mt2; mt += kPairWaves) {
#pragma unroll
        for (int j = 0; j < IT; j++) res[j] = res_next[j];
        f32x16 acc2;
#pragma unroll
        for (int v = 0; v < 16; v++) acc2[v] = 0.f;
        auto fragment = [&](int s) {
            const uint16_t *src = tile + cc * TROW + 32 * s + 16 * g;
            return B32{*reinterpret_cast<const u32x4 *>(src), *reinterpret_cast<const u32x4 *>(src + 8)};
        };
        if constexpr (MT > 0) {
            B32 b[KS2];
#pragma unroll
            for (int s = 0; s < KS2; s++) b[s] = fragment(s);
#pragma unroll
            for (int s = 0; s < KS2; s++) acc2 = mma(r2.a[s], b[s], acc2, s);
        } else {
#pragma unroll
            for (int s = 0; s < KS2; s++) {
                if (s >= p.Ks2) break;                    // uniform
                acc2 = mma(r2.a[s], fragment(s), acc2, s);
            }
        }
        if (PX == 32 || c < PX) {
#pragma unroll
            for (int q = 0; q < 4; q++)
                *reinterpret_cast<float4 *>(slab + cc * kFuseRow + 8 * q + 4 * g) =
                    make_float4(acc2[4 * q] + r2.b[q].x, acc2[4 * q + 1] + r2.b[q].y, acc2[4 * q + 2] + r2.b[q].z, acc2[4 * q + 3] + r2.b[q].w);
        }
        if (mt + kPairWaves < p.Mt2) {
            load_row2(r2, mt + kPairWaves);
            load_res(res_next, mt + kPairWaves);
        }
        __builtin_amdgcn_wave_barrier();                  // (a wave's LDS operations execute in order: the reads below see the writes above)
#pragma unroll
        for (int j = 0; j < IT; j++) {
            const int it = lane + 64 * j, px = it >> 2, run = it & 3, pg = n0 + px;
            const float4 lo = *reinterpret_cast<const float4 *>(slab + px * kFuseRow + run * 8);
            const float4 hi = *reinterpret_cast<const float4 *>(slab + px * kFuseRow + run * 8 + 4);
            if (pg >= p.P) continue;
            float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
            for (int e = 0; e < 8; e++) v[e] += widen<DT>((uint16_t)(res[j][e >> 1] >> (16 * (e & 1))));
            if (p.act2 == SS_ACT_GELU) {
#pragma unroll
                for (int e = 0; e < 8; e++) v[e] = gelu_cdf<DT>(v[e]);
            } else {
#pragma unroll
                for (int e = 0; e < 8; e++) v[e] = floor_at(v[e], floor2);
            }
            uint32_t w[4];
#pragma unroll
            for (int e = 0; e < 4; e++) w[e] = cvt_pack2<DT>(v[2 * e], v[2 * e + 1]);
            *reinterpret_cast<uint4 *>(p.y2 + (size_t)pg * p.Cout2 + mt * 32 + run * 8) = make_uint4(w[0], w[1], w[2], w[3]);
            if constexpr (THIRD) *reinterpret_cast<uint4 *>(out2 + px * T2ROW + mt * 32 + run * 8) = make_uint4(w[0], w[1], w[2], w[3]);
        }
        __builtin_amdgcn_wave_barrier();
    }
    if constexpr (THIRD) {
        // ---- third layer (pixels behind the last one hold whatever LDS held: their columns are not stored)
        lds_barrier();
        f32x16 acc3;
#pragma unroll
        for (int v = 0; v < 16; v++) acc3[v] = 0.f;
        B32 b3[KS3];
#pragma unroll
        for (int j = 0; j < KS3; j++) {                   // (all on their way first; a step past the share's end is read and not used)
            const uint16_t *src = out2 + cc * T2ROW + 32 * min(t0 + j, p3.Ks3 - 1) + 16 * g;
            b3[j].lo = *reinterpret_cast<const u32x4 *>(src);
            b3[j].hi = *reinterpret_cast<const u32x4 *>(src + 8);
        }
        // Partial sums: a row tile's pixels of one quad of channels in a row, turned by the quad's number, so that the threads below, which go over the
        // channels first, find them in different banks (not turned, each of their reads took 0.2 us).
        auto place = [&](int m, int cq, int pl) { return (cq >> 1) * 64 + (cq & 1) * 32 + ((pl + cq + 8 * m) & (PX - 1)); };
        auto keep = [&](u32x4 *to, const f32x16 &sums) {
#pragma unroll
            for (int q = 0; q < 4; q++) to[place(rt3, 2 * q + g, cc)] = __builtin_bit_cast(u32x4, f32x4{sums[4 * q], sums[4 * q + 1], sums[4 * q + 2], sums[4 * q + 3]});
        };
        // A wave's second share: with 16 pixels behind the first one's, from the lanes that repeat its columns; else where the staged input was.
        u32x4 *const part2 = PX == 16 ? part + 16 : stage;
        auto multiply = [&]() {
#pragma unroll
            for (int j = 0; j < KS3; j++)
                if (t0 + j < t1) acc3 = mma(a3[j], b3[j], acc3, t0 + j);      // uniform
            keep(part + wave * 256, acc3);
        };
        if constexpr (THIRD == THIRD_TWO) {
            f32x16 second = acc3;
            constexpr int PER = KS3 / 2;                  // steps of a share: four, or three of twelve in all
#pragma unroll
            for (int j = 0; j < PER; j++) {
                if (j == PER - 1 && p3.per3 < PER) break;  // uniform
                acc3 = mma(a3[j], b3[j], acc3, t0 + j);
            }
            if (p3.per3 < PER) second = mma(a3[PER - 1], b3[PER - 1], second, t0 + PER - 1);
#pragma unroll
            for (int j = PER; j < KS3; j++)
                if (t0 + j < t1) second = mma(a3[j], b3[j], second, t0 + j);
            // (waves without a row tile have multiplied nothing of use: their places are not read)
            if constexpr (PX == 16) {
#pragma unroll
                for (int v = 0; v < 16; v++) acc3[v] = c < PX ? acc3[v] : second[v];
                keep(part + wave * 256 + (c & 16), acc3);
            } else {
                keep(part + wave * 256, acc3);
                keep(part2 + wave * 256, second);
            }
        } else if constexpr (THIRD == THIRD_HANDED) {
            if (kg3 == 0) multiply();
            lds_barrier();
            if (kg3 == 1) {
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const f32x4 u = __builtin_bit_cast(f32x4, part[rt3 * 256 + place(rt3, 2 * q + g, cc)]);
#pragma unroll
                    for (int e = 0; e < 4; e++) acc3[4 * q + e] = u[e];
                }
                multiply();
            }
        } else {
            multiply();
        }
        lds_barrier();
        const float floor3 = p3.act3 == SS_ACT_RELU ? 0.f : -__builtin_inff();
#pragma unroll
        for (int i = 0; i < Q3; i++) {
            int pl;
            const int q = quad3(i, &pl), m = q >> 3, cq = q & 7, o = q * 4;
            if (pl >= PX) break;                          // (fewer than four row tiles)
            float v[4] = {0.f, 0.f, 0.f, 0.f};
            const u32x4 *const from = part + m * 256 + place(m, cq, pl);
            auto add = [&](int at) {
                const f32x4 u = __builtin_bit_cast(f32x4, from[at]);
#pragma unroll
                for (int e = 0; e < 4; e++) v[e] += u[e];
            };
            const int next = p3.Mt3 * 256, other = (int)(part2 - part);      // from a row tile's wave to its next one, from a share to the wave's second
            if constexpr (THIRD == THIRD_TWO) {
                add(0);
                add(other);
                add(next);
                add(next + other);
            } else if constexpr (THIRD == THIRD_HANDED) {
                add(next);
            } else {
                add(0);
                if (p3.shares3 > 1) add(next);             // uniform
                if (p3.shares3 > 2) {
                    add(2 * next);
                    add(3 * next);
                }
            }
#pragma unroll
            for (int e = 0; e < 4; e++) v[e] += bias3[i][e];
            if (p3.act3 == SS_ACT_GELU) {
#pragma unroll
                for (int e = 0; e < 4; e++) v[e] = gelu_cdf<DT>(v[e]);
            } else {
#pragma unroll
                for (int e = 0; e < 4; e++) v[e] = floor_at(v[e], floor3);
            }
            if (n0 + pl < p.P)
                *reinterpret_cast<uint2 *>(p3.y3 + (size_t)(n0 + pl) * p3.Cout3 + o) = make_uint2(cvt_pack2<DT>(v[0], v[1]), cvt_pack2<DT>(v[2], v[3]));
        }
    }
}

template <int DT, bool SPARSE, int PX, int MT, int THIRD>
static int launch_pair_small(kernel_params<THIRD> p, hipStream_t s)
{
    fast_div_setup((unsigned)p.Mt, &p.tm_mul, &p.tm_sh);      // (the kernel deals its waves out over the row tiles)
    const size_t smem = pair_shape(PX, p.Ks / 9, p.Cout, THIRD != THIRD_NONE ? p.Cout2 : 0).total;
    auto kern = pair_small_kernel<DT, SPARSE, PX, MT, THIRD>;
    if (smem > 64 * 1024) {
        static std::atomic<unsigned long long> done_mask{0};      // as in launch(): once per device
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) return SS_ERR_HIP;
        const unsigned long long bit = 1ull << (dev & 63);
        if (dev >= 64 || !(done_mask.load(std::memory_order_acquire) & bit)) {
            if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
                return SS_ERR_HIP;
            if (dev < 64) done_mask.fetch_or(bit, std::memory_order_release);
        }
    }
    kern<<<dim3((unsigned)(((long long)p.P + PX - 1) / PX)), dim3(kPairWaves * 64), smem, s>>>(p);
    return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_HIP;
}

// The fused pair on few pixels: PX = 16 or 32 as given, or chosen (px = 0) while one workgroup per compute unit holds them
// all.  SS_ERR_INVALID_ARG where it does not fit or the tiled kernel is the better choice.
template <int DT, bool SPARSE>
static int pair_small(const ss_weight_desc *d1, const ChainParams &p, int px, hipStream_t s)
{
    const int ncu = compute_units();
    if (ncu <= 0) return SS_ERR_HIP;
    const bool third = p.Cout3 > 0;
    if (px == 0) px = pair_small_pixels(p.P, ncu);
    if (px == 0 || !pair_small_fits(d1, px, third ? p.Cout2 : 0, p.Cout3)) return SS_ERR_INVALID_ARG;
    ChainParams q = p;
    int plan = THIRD_NONE;
    if (third) {
        q.shares3 = pw_shares(p.P, p.Ks3, p.Mt3, SPARSE, ncu);
        q.per3 = p.Ks3 / q.shares3;
        plan = q.per3 > 8 ? THIRD_HANDED : (q.shares3 > 2 && p.Mt3 > 2 ? THIRD_TWO : THIRD_SHARE);
    }
    auto go = [&](auto mt) -> int {
        constexpr int MT = decltype(mt)::value;
        auto pixels = [&](auto t) -> int {
            constexpr int THIRD = decltype(t)::value;
            // (a chain of products is the layer's own form from more pixels on than workgroups of 16 hold)
            if constexpr (THIRD == THIRD_HANDED) return px == 16 ? (int)SS_ERR_INVALID_ARG : launch_pair_small<DT, SPARSE, 32, MT, THIRD>(q, s);
            else return px == 16 ? launch_pair_small<DT, SPARSE, 16, MT, THIRD>(q, s) : launch_pair_small<DT, SPARSE, 32, MT, THIRD>(q, s);
        };
        using std::integral_constant;
        if constexpr (MT > 0) {
            if (plan == THIRD_SHARE) return pixels(integral_constant<int, THIRD_SHARE>{});
            if (plan == THIRD_TWO) return pixels(integral_constant<int, THIRD_TWO>{});
            if (plan == THIRD_HANDED) return pixels(integral_constant<int, THIRD_HANDED>{});
        }
        return third ? (int)SS_ERR_INVALID_ARG : pixels(integral_constant<int, THIRD_NONE>{});
    };
    using std::integral_constant;
    return p.Mt == 2 ? go(integral_constant<int, 2>{}) : p.Mt == 4 ? go(integral_constant<int, 4>{}) : go(integral_constant<int, 0>{});
}

}  // namespace ss

#endif
