// Parameter blocks of the convolution kernels and the per-type dispatch functions that connect the entry points
// (ss_conv.hip) with the translation units that instantiate the kernels (ss_conv_inst_*.hip).
#ifndef SS_CONV_PARAMS_H_
#define SS_CONV_PARAMS_H_
#include "ss_internal.h"

namespace ss {

struct ConvParams {
    const uint16_t *x;
    const uint8_t *a_vals;    // first value tile (after the header)
    const uint32_t *a_meta;   // first metadata tile (sparse only)
    const float *bias;
    const float *scale;       // 8-bit operands: per-output-channel factor of the sum, or nullptr (= 1)
    const uint16_t *residual; // [P][Cout] like y, or nullptr
    uint16_t *y;
    int N, H, W, Cin, Cout, kh, kw, sh, sw, ph, pw, Ho, Wo, P, K, Ks, Kp, Mt, act, korder;
    int tiles_m;
    unsigned x_bytes, a_bytes, meta_bytes;
    // division by Ho*Wo, Wo and tiles_m as multiply + shift (see fast_div)
    unsigned howo_mul, howo_sh, wo_mul, wo_sh, tm_mul, tm_sh, cin_mul, cin_sh, kw_mul, kw_sh;
    // fused second contraction (a 1x1 convolution on this convolution's output tile)
    const uint8_t *a2_vals;
    const uint32_t *a2_meta;
    const float *bias2;
    const uint16_t *res2;     // [P][Cout2] or nullptr
    uint16_t *y2;             // [P][Cout2]
    int Cout2, Ks2, Kp2, Mt2, act2;
    unsigned a2_bytes, meta2_bytes;
    // split reduction: workgroups per output tile (1 = none), fp32 partial sums [tile][split][BM*BN] and one ticket
    // counter per tile, both in the caller's workspace
    int nsplit, plan_tile, plan_bm, plan_bn;      // plan_*: the tile the split was planned (and the workspace sized) for
    float *ws_part;
};

// With a third contraction, a 1x1 convolution on the second one's output, which is written too (apart from ConvParams: every other call would clear
// these fields, and the kernels that take all of it carry them).
struct ThirdParams {
    const uint8_t *a3_vals;
    const uint32_t *a3_meta;
    const float *bias3;
    uint16_t *y3;             // [P][Cout3]
    int Cout3, Ks3, Kp3, Mt3, act3;      // Cout3 = 0: there is none
    unsigned a3_bytes, meta3_bytes;
    int shares3, per3;        // few pixels: the shares in which this reduction is added up (pw_shares), and the steps of one
};
struct ChainParams : ConvParams, ThirdParams {};
static_assert(sizeof(ConvParams) <= 288, "what every call clears");

// What a launch carries to the kernels of the short calls; the rest of ConvParams follows from it (unpack_args).  A launch whose arguments
// take more than 112 bytes costs the host 3.65 to 3.8 us, up to 112 bytes 3.0 (none at all: 1.5), whatever the kernel: as long as all of a
// small layer's work on the GPU (profiles/launch_and_packing_waits.md).  (ConvParams has some 300 bytes, and a kernel that asks for its
// grid's size another 256.)
struct ConvArgs {
    const uint16_t *x;
    const uint8_t *a_vals;
    const float *bias;
    const void *tail;         // 16-bit operands: the residual; 8-bit: the scale
    uint16_t *y;
    union {
        float *ws_part;       // split reduction: partial sums (the ticket counters end where they begin)
        struct {
            int K, kw;        // kernels that learn the window's size from here
        } window;
    };
    int H, W, Cin, Cout, sh, sw, ph, pw, P, Ho, Wo;
    unsigned howo_mul, wo_mul;
    unsigned m_mul;           // division by tiles_m, or (few-pixel kernels) by kw
    unsigned extra;           // nsplit, or (few-pixel kernels) the division by Cin; activation-stationary kernel: see there
    unsigned bits;            // act, then the shifts that go with howo_mul, wo_mul, m_mul and extra, six bits each from bit 2 on
};
static_assert(sizeof(ConvArgs) == 112, "a cheap launch");

// small: the few-pixel kernels' reading of m_mul and extra.  window: the kernel learns the window's size from the arguments.
static inline ConvArgs conv_args(const ConvParams &p, bool small, bool window)
{
    ConvArgs a;
    a.x = p.x; a.a_vals = p.a_vals; a.bias = p.bias; a.y = p.y;
    a.tail = p.residual != nullptr ? static_cast<const void *>(p.residual) : p.scale;      // (never both)
    if (window) { a.window.K = p.K; a.window.kw = p.kw; }
    else a.ws_part = p.ws_part;
    a.H = p.H; a.W = p.W; a.Cin = p.Cin; a.Cout = p.Cout; a.sh = p.sh; a.sw = p.sw; a.ph = p.ph; a.pw = p.pw;
    a.P = p.P; a.Ho = p.Ho; a.Wo = p.Wo;
    a.howo_mul = p.howo_mul; a.wo_mul = p.wo_mul;
    a.m_mul = small ? p.kw_mul : p.tm_mul;
    a.extra = small ? p.cin_mul : (unsigned)p.nsplit;
    a.bits = (unsigned)p.act | p.howo_sh << 2 | p.wo_sh << 8 | (small ? p.kw_sh : p.tm_sh) << 14 | (small ? p.cin_sh : 0u) << 20;
    return a;
}

// Bytes of the ticket counters of a split reduction over so many tiles.  Every plan the library makes by itself has at most 128 tiles (half of
// 256 compute units): their counters take the same 512 bytes, so that plans of different sizes can follow each other in one workspace
// without one's partial sums lying where the other expects its counters at zero.
#ifdef __HIPCC__
__host__ __device__
#endif
static inline size_t ticket_bytes(long long tiles) { return (size_t)((tiles * 4 + 511) / 512 * 512); }

// floor(n / d) for 0 <= n < 2^31 as (n * mul) >> sh with s = ceil(log2 d), sh = 31 + s, mul = ceil(2^sh / d):
// mul * d - 2^sh < d <= 2^s, so the product overshoots n / d by less than 1 / d, never reaching the next integer.
static inline void fast_div_setup(unsigned d, unsigned *mul, unsigned *sh)
{
    unsigned s = 0;
    while ((1ull << s) < d) s++;
    *sh = 31 + s;
    *mul = (unsigned)(((1ull << (31 + s)) + d - 1) / d);
}

struct MlpParams {            // (a cheap launch, see ConvArgs; all channel counts are multiples of 32)
    const uint16_t *x;        // [P][Cin]
    const uint8_t *a1_vals, *a2_vals;
    const float *bias1, *bias2;
    const uint16_t *res2;     // [P][Cout2] or nullptr
    uint16_t *y2;             // [P][Cout2]
    int P, Cin, Cmid, Cout2, act1, act2;
    int blocks;               // workgroups of a resident launch
};

constexpr int kMlpKs1 = 4;        // first reduction: at most 128 input channels
constexpr int kMlpTiles = 2;      // 32x32 output tiles of the second layer per wave: at most 128 output channels x 64 pixels over 4 waves

// The resident kernel's LDS copy of the weights is in the order of use, two row tiles of the intermediate (32 channels each) after the other, so that all
// offsets inside a pair are constants: the first layer's tiles, the second layer's steps, their index words, the first layer's bias.
template <bool SPARSE, int TILES>
struct MlpPair {
    static constexpr int STEP = SPARSE ? 1024 : 2048, KP1 = (TILES + 1) / 2, W2 = 2 * TILES * STEP, I1 = 2 * W2, I2 = I1 + (SPARSE ? 2 * KP1 * 256 : 0),
                         BIAS = I2 + (SPARSE ? TILES * 256 : 0), BYTES = BIAS + 2 * 128;
    static constexpr size_t smem(int Cmid) { return (size_t)(Cmid / 64) * BYTES + TILES * 128; }      // (with the second layer's bias)
};
constexpr size_t kMlpResidentSmem = 160 * 1024;
constexpr int kMlpWideWaves = 16;         // wide kernel: at most 512 intermediate channels

// Can the kernel of this id (ss_debug_force_tile) run the inverted bottleneck?  40 all of them; 41 the wide one; 42 the resident one: built for 96 channels
// at both ends and sparse 128, if the weights fit the LDS (sparse 96 up to 640 intermediate channels, dense 96 up to 384, sparse 128 up to 512),
// and not for the sparse path with GELU, where both are bound by the vector ALU (96 channels 0.92 to 1.05 of mlp_kernel's time by itself but 0.99 to 1.04
// in a ConvNeXt block, 128 0.95 to 1.11 and 1.02 to 1.08), nor for 64 and 32 channels (with GELU 1.0 to 1.2).
static inline bool mlp_takes(const MlpParams &p, bool sparse, int id)
{
    if (id == 41) return p.Cmid <= 32 * kMlpWideWaves;
    if (id != 42) return true;
    if (p.Cin != p.Cout2 || (p.Cin != 96 && !(sparse && p.Cin == 128)) || (sparse && p.act1 == SS_ACT_GELU)) return false;
    return (p.Cin == 128 ? MlpPair<true, 4>::smem(p.Cmid) : (sparse ? MlpPair<true, 3>::smem(p.Cmid) : MlpPair<false, 3>::smem(p.Cmid))) <= kMlpResidentSmem;
}

// Which one pays:
//   * the wide one, a wave per 32 intermediate channels, while its workgroups of 32 pixels all run at once, from eight waves on.  bf16 with GELU, C -> 4 C ->
//     C, sparse / dense, mlp_kernel against it: 3136 pixels C = 64 5.3 / 5.4 against 4.35 / 4.5 us, 96 7.6 / 8.4 against 5.5 / 5.9, 128 10.3 /
//     11.4 against 6.65 / 7.5; 8192 pixels, the last that fit, C = 96 7.7 / 8.6 against 5.8 / 6.3; 10000 pixels, 313 workgroups of 12 waves, 7.8 / 8.75
//     against 9.5 / 10.9.  Four waves (C = 32) make no difference: 3.7 and 3.6.  Over 588 layers of 32 to 128 channels at either end and 256 to 512 between
//     them 0.82 of its time in the mean and with GELU always below 1; without, few channels leave it nothing to do at once: 32 and 32 1.03 to 1.11,
//     32 and 64 0.98 to 1.07, from 128 together on 0.63 to 1.03.
//   * the resident one from some pixel tiles per compute unit on.  A SIMD that gets a tile more than its neighbours keeps
//     the chip waiting for it, and the weights' way to LDS is some 3 us, so it takes a few tiles per SIMD.  Times against mlp_kernel's at 1.6, 2.4, 3.2, 4,
//     5.5, 7 and 12.25 tiles of 32 pixels per SIMD, bf16, C -> 4 C -> C:
//       ReLU   sparse  96   0.85 0.82 0.78 0.80 0.77 0.72 0.68      dense  96   0.79 0.82 0.73 0.72 0.73 0.69 0.62
//              sparse 128   0.94 0.96 0.88 0.85 0.86 0.79 0.76
//       GELU   dense   96   0.95 1.01 0.95 0.86 0.90 0.83 0.84     (in a ConvNeXt block on new inputs each time 0.95 to 0.90, 173 -> 163 us at 128 x 56 x 56)
//     With other intermediates, from 1.5 tiles per SIMD on: 96 channels and 128 between them 0.83 to 1.03, 256 0.62 to 0.90 (dense GELU 0.91 to 1.03), sparse
//     512 and 640 0.68 to 0.86.  128 channels live less from the pixels that they save and more on the weights' way: 128 between them 1.04 to 1.11, so never;
//     256 and 384 0.98 to 1.05 below 3 tiles per SIMD, 0.81 to 1.0 from there on.
static inline int choose_mlp(const MlpParams &p, bool sparse, int ncu)
{
    const long long tiles = ((long long)p.P + 31) / 32;
    if (tiles <= ncu && p.Cmid >= 256 && (p.act1 == SS_ACT_GELU || p.Cin + p.Cout2 >= 128) && mlp_takes(p, sparse, 41)) return 41;
    if (!mlp_takes(p, sparse, 42) || (p.Cin == 128 && p.Cmid < 256)) return 40;
    return tiles > (p.Cin == 128 && p.Cmid < 512 ? 12ll : 6ll) * ncu ? 42 : 40;
}

static inline long long n_blocks(const ConvParams &p, int bm, int bn)
{
    return (long long)((p.Cout + bm - 1) / bm) * (((long long)p.P + bn - 1) / bn);
}


// Tile id for a problem.  Measured on MI355X (tile sweep over the ResNet-50 / ConvNeXt-T layer shapes, 256 compute
// units).  pointwise: 1x1 staging; bigchunk: staging in chunks of 256+ reduction indices (3x3 tap transpose, long
// channels-last reductions).
static inline int choose_tile(const ConvParams &p, bool pointwise, bool bigchunk)
{
    if (p.Cout <= 64) {
        const bool deep = n_blocks(p, 64, 64) <= 1024 || (pointwise && p.K >= 256);
        return deep ? 1 : 0;
    }
    // Grids of at most one workgroup per compute unit: nothing else hides a wave's stalls, so separate producer
    // waves pay.  Larger grids do better with two four-wave workgroups per compute unit.
    const long long b128 = n_blocks(p, 128, 64), b256 = n_blocks(p, 256, 64);
    if (p.Cout > 128 && b256 > 128 && b256 <= 256) return 5;
    if (b128 <= 256) return 4;
    if (p.Cout >= 512 && p.K >= 512) return 3;
    if (bigchunk && p.Cout >= 256 && b256 >= 512) return 3;
    return 2;
}


// Tile id in the channels-last flattening with taps, from K = 512 on (p.K counts 2-byte units: pairs of 8-bit indices).  Ids 4 and 5
// then stage chunks of 256 units, a quarter of the barriers and four times the LDS: right for producer waves, which run
// few workgroups per compute unit anyway; the others stage 64.
// choose_tile except where it takes the four-wave 256x64 tile (large grids).  From a sweep over 2566 such layers with each tile forced
// (profiles/channels_last_large_grids.md; 256 to 1024 output channels, K 512 to 3456, five image sizes):
//   * dense 16-bit: 128x64 where it computes fewer rows (0.60 to 0.92 of the 256x64 tile's time, mean 0.76) and below K = 1792
//     (0.78 to 1.02, mean 0.92); with equal rows and K from there on 256x64 with producer waves (0.78 to 0.96, mean 0.87; 128x64
//     0.98);
//   * sparse 16-bit, half the matrix instructions per weight fetched, so that two 128-row tiles cost more than a 256-row one: by
//     the tiles of the fullest compute unit, two 128-row tiles counted as 9/8 of a 256-row tile.  That is 128x64 where
//     256 rows are mostly padding (288 to 384 channels: 0.72 to 0.98, mean 0.90) or leave units idle in the last round (256 channels on 64
//     28x28 images 0.91 to 1.02), 256x64 elsewhere (with equal rows 128x64 takes up to 1.46 of its time);
//   * dense 8-bit: 128x64 (int8 0.60 to 1.15, mean 0.84; FP8, whose general choice is producer waves, 0.58 to 1.31, mean 0.87: the
//     losses are at 784 workgroups, two per cent more than the chip holds at once).
// Over the sweep the choice is 1 % (dense 8-bit 1.6 %) above the best of the three in the mean, the four-wave 256x64 tile everywhere
// would be 4 to 21 %.  Sparse 8-bit layers, whose steps are the cheapest, start from the rule for short chunks (256x64 from 512 channels on) and have costs
// of their own behind it (choose_vec8_sparse).
static inline int choose_vec(const ConvParams &p, bool bytes, bool sparse, int ncu)
{
    const int id = choose_tile(p, false, true);
    if (id != 3) return id;
    if (bytes) return sparse ? choose_tile(p, false, false) : 2;
    const long long b128 = n_blocks(p, 128, 64), b256 = n_blocks(p, 256, 64);
    if (sparse) return 9 * ((b128 + ncu - 1) / ncu) < 16 * ((b256 + ncu - 1) / ncu) ? 2 : 3;
    return b128 == 2 * b256 && p.K >= 1792 ? 5 : 2;
}

// Tile id of a 3x3 layer in the paper's flattening (taps), or of a channels-last layer with taps and K >= 512, on a grid of more than one
// workgroup per compute unit, given the choice made so far.  Rows past the last output channel cost as much as any others, so
// there are tiles of 96, 160 and 224 rows too (136 channels in one tile of 160 instead of two of 128: 12.1 -> 10.8 us on six 45x61 images,
// 80 -> 136, sparse, with a residual).
// By the tiles of the fullest compute unit (halfway between that and the mean, since two or three workgroups share a unit) times the time
// of a tile, in hundredths of the 128-row one's, set by a sweep of 7000 drawn layers with each tile forced (profiles/tile_heights.md: medians by
// staging and operands 81 to 97 for 96 rows, 132 to 156 for 160, 164 to 183 for 224, 180 up for 256).  The taller ones have less to
// overlap with (two workgroups of five waves per unit, one of seven); dense 8-bit steps are bound by their registers.  Over the layers
// that come here the choice takes 0.90 of the time of the tiles of 64, 128 and 256 rows alone (1st to 99th percentile 0.57 to 1.11) and is 4 % above
// the best of all, half of which is noise.  In the paper's flattening the 128- and 256-row tiles are compared in the same way; the
// channels-last choice between those (choose_vec) stands.  Dense 256 rows: twice 128 and more, so never by this rule.
// Dense FP8 has costs of its own.  Its instruction wants eight consecutive registers per operand: tiles of 160 and 224 rows take as long as 256
// (1.95 to 2.24) and are not built; 96 rows gain channels-last (0.84) and not in the paper's flattening (0.99, spilling), where the tile
// with producer waves stands for 256 rows: the longer the reduction the better (2.12 at one chunk, 1.77, 1.56, 1.45 ... 1.28 at eight).  Over 2300
// layers 0.2 % and 2 % above the best of all, 0.92 and 0.98 of the time without a choice of heights; with int8's costs it was 1.03 and 1.00 of that (1.08 to 1.13
// in the paper's flattening at 129 to 224 channels).
static inline int choose_height(const ConvParams &p, int id, bool taps, bool bytes, bool sparse, int ncu, bool f8 = false)
{
    if (id != 2 && id != 3) return id;
    struct Tile {
        int id, rows, cost;           // (cost 0: not a choice)
    };
    const bool wide = bytes && !sparse;
    const Tile usual[] = {{2, 128, 100}, {6, 96, 92}, {7, 160, wide ? 170 : 145}, {8, 224, wide ? 180 : 162}, {3, 256, sparse ? 185 : 205}};
    const Tile dense_f8[] = {{2, 128, 100}, {6, 96, taps ? 0 : 88}, {7, 160, 0}, {8, 224, 0}, {3, 256, f8 && taps ? 125 + 90 * 9 / p.Ks : 0}};
    long long best = -1;
    int pick = id;
    for (const auto &t : f8 && !sparse ? dense_f8 : usual) {
        if (t.cost == 0 || (!taps && (t.id == 2 || t.id == 3) && t.id != id)) continue;
        const long long n = n_blocks(p, t.rows, 64), cost = (n + (n + ncu - 1) / ncu * ncu) * t.cost;
        if (best < 0 || cost < best) { best = cost; pick = t.id; }
    }
    return pick;
}

// Sparse 8-bit channels-last layers with taps and K >= 512, given the choice made so far: the tile of 128 or of 256 rows where it clearly beats that,
// by the tiles of the fullest compute unit (nearer to it than in choose_height) times the time of a tile.  Their weight fragments are half a
// 16-bit layer's, so a tall tile, which reads an activation fragment once for more rows, gains the more the longer the reduction: 256 rows
// take 1.75 of the 128-row tile's time at K = 640 (2-byte units), 1.63 at 1280, 1.57 at 2300; choose_vec never compares the two here, and choose_height takes K
// not into account.  Of 12264 layers on cold inputs with each tile forced (profiles/tile_heights.md) 1643 change their tile, 0.862 of its time in the mean,
// 99 % of them at most 1.00: 225 to 256 and 449 to 511 channels from 128 rows to 256, above those layers whose last round would be nearly empty.
// (In calls on new inputs each time: int8 160 -> 256 on 62 28x28 images 22.65 -> 19.2 us, 144 -> 452 on fifteen 40x40 21.6 -> 18.1, 256 -> 484 on twenty
// 35.0 -> 33.9.)  The line of 0.86 is below 1 because the grid's rounding is not known better: at 0.92 2886 layers change (0.897), but 8 % of them lose.
static inline int choose_vec8_sparse(const ConvParams &p, int id, int ncu)
{
    auto time = [&](int rows, int base, int start) {      // base + start / K: a tile's time in hundredths of the 128-row one's
        const long long n = n_blocks(p, rows, 64);
        return (3 * n + 7 * ((n + ncu - 1) / ncu * ncu)) * ((long long)base * p.K + start);
    };
    const long long t128 = time(128, 100, 0), t256 = time(256, 153, 11840);
    long long now;
    switch (id) {
        case 2: now = t128; break;
        case 3: now = t256; break;
        case 7: now = time(160, 125, 7680); break;
        case 8: now = time(224, 157, 11520); break;
        default: return id;
    }
    return (t128 < t256 ? t128 : t256) / 86 < now / 100 ? (t128 < t256 ? 2 : 3) : id;
}

// Tile id of a channels-last layer with taps and K < 512 (2-byte units), where it is not choose_tile's (8806 layers on cold inputs, profiles/tile_heights.md):
//   * sparse, 129 to 160 channels: one tile of 160 rows instead of two of 128 (0.89 of their time in the mean over 543 layers, 0.73 to 1.00, 16- and 8-bit
//     alike; dense 0.97, up to 1.21);
//   * 96 rows where they are no more tiles (65 to 96, 129 to 192, 257 to 288 channels).  A compute unit holds four workgroups of 128 rows or five of 96
//     (without a residual), so by workgroups per unit: up to two no gain (0.99 to 1.03), two to three 0.98 for dense int8 and 1.00 for the others, three to
//     four 0.92 dense (sparse 0.95), four to five, one round instead of two, 0.79 (0.95), five to six, two rounds on both sides, 0.98 to 1.01, above 0.89 to
//     0.92 (0.98, one in fifteen slower: not taken).  Not measured for dense FP8.
// In calls on new inputs, us: bf16 40 -> 136 on thirty 40x40 images 12.9 -> 9.65, int8 96 -> 148 on twenty 10.5 -> 9.0 (dense 11.4 -> 10.5), FP8 64 -> 132 on
// a hundred 28x28 16.9 -> 15.3, int8 dense 64 -> 92 13.75 -> 11.0,
// f16 dense 56 -> 90 on 42 40x40 19.2 -> 14.4 and 56 -> 180 27.6 -> 22.8, bf16 sparse 40 -> 92 11.45 -> 10.6.
// With a residual, whose fp32 tile changes the LDS of a workgroup (33 KB for 128 rows, 25 for 96, 42 for 160), the layers that move gain more: 292 16-bit ones
// with and without, strides of one and two: sparse 160 rows 0.83 of the time of 128 in the mean (0.68 to 0.98; without 0.88), sparse 96 rows 0.89 (0.95),
// dense 0.87 (0.89).
static inline int choose_vec_short(const ConvParams &p, bool bytes, bool sparse, bool f8, int ncu)
{
    const int id = choose_tile(p, false, false);
    if (id != 2) return id;
    if (sparse && p.Cout > 128 && p.Cout <= 160) return 7;
    if ((f8 && !sparse) || (p.Cout + 95) / 96 != (p.Cout + 127) / 128) return id;
    const long long n = n_blocks(p, 96, 64);
    const bool fits = n <= 5ll * ncu && n > (bytes && !sparse ? 2ll : 3ll) * ncu;
    return fits || (!sparse && n > 6ll * ncu) ? 6 : id;
}

// ---------------------------------------------------------------------------------------------
// Few output pixels: which of the one-latency kernels (ss_conv_small.h) takes a problem.  Here and not beside them because the
// workspace query and the entry points must know: a problem that they take never splits its reduction.
// ---------------------------------------------------------------------------------------------
// (RSCW: cin % 32 == 0, a reduction step lies in one tap; TAPSR: cin % 32 != 0, as MODE_TAPSR)
enum { SMALL_PW = 0, SMALL_RSC = 1, SMALL_TAPS = 2, SMALL_TAPSR = 3, SMALL_RSCW = 4 };
constexpr bool small_taps(int mode) { return mode == SMALL_TAPS || mode == SMALL_TAPSR; }

// Workgroups of a problem.
static inline long long small_blocks(const ConvParams &p, int px, int tm)
{
    return (long long)((p.Mt + tm - 1) / tm) * (((long long)p.P + px - 1) / px);
}

// How such a kernel would stage the problem, or -1 where none of them can.
static inline int small_staging(const ss_weight_desc *d, const ConvParams &p)
{
    if ((long long)p.P * p.Cout * 2 > 0x7FFFFFFF) return -1;      // (32-bit offsets; such outputs are far above these kernels' range)
    const bool square = (d->kh == 3 && d->kw == 3) || (d->kh == 2 && d->kw == 2);
    if (d->kh * d->kw == 1 && p.Cin % 8 == 0) return SMALL_PW;
    if (d->korder == SS_K_RSC && p.Cin % 32 == 0) return SMALL_RSCW;
    if (d->korder == SS_K_RSC && p.Cin % 8 == 0) return SMALL_RSC;
    if (d->korder == SS_K_CRS && square && p.Cin % 32 == 0) return SMALL_TAPS;
    if (d->korder == SS_K_CRS && square && p.Cin % 4 == 0 && p.Cin >= 8 && !is_byte_type(d->dtype)) return SMALL_TAPSR;
    return -1;
}

// Waves per workgroup: one per chunk of 32 channels (taps: the kernel's tap count, 0 = direct) or per four steps (direct), at most eight
// (sixteen with the 16-pixel tiles of the direct modes, whose fragments leave the registers for it).
static inline int small_waves(const ConvParams &p, int taps, bool tile16)
{
    const int shares = taps ? (p.Ks + taps - 1) / taps : (p.Ks + 3) / 4;
    return shares <= 2 ? 2 : (shares <= 4 ? 4 : (shares <= 8 || taps || !tile16 ? 8 : 16));
}

enum { SMALL_NONE = -1, SMALL_16 = 0, SMALL_32 = 1, SMALL_64X32 = 2 };      // 32 channels x 16 / x 32 pixels, 64 x 32

// Which variant pays, from a sweep of all of them and the tiled kernels over the ResNet-50 layers at batches 1 to 32, both
// flattenings, sparse and dense, 16- and 8-bit operands (profiles/small_grids.md):
//   * 16-pixel tiles while one per compute unit holds them all, and with two waves (short reductions) up to eight waves
//     per compute unit: 3x3 256 -> 256 on one 14x14 image 9.0 -> 4.4 us, 64 -> 64 on one 56x56 4.9 -> 3.7;
//   * 32-pixel tiles under the same conditions (four waves up to eight waves per unit, 2x2 kernels two workgroups):
//     the 256 -> 256 layer on four images 9.1 -> 5.4;
//   * 64 x 32 tiles for long reductions while one per unit holds them: 512 -> 512 on sixteen 7x7 images 19 -> 9.6 us.  Not for the
//     dense form of the tap modes (its fragments spill: 11.4 vs 9.8).  Direct loads from sixteen steps on (1x1 512 -> 128 on
//     four 28x28 images 5.0 -> 4.2 us, 3x3 channels-last 128 -> 512 on one 8.3 -> 6.6, int8 1x1 1024 -> 256 on eight 14x14
//     4.8 -> 4.1); below that the 32-pixel tiles are as good.
//   * direct loads, 32-pixel tiles up to two per unit while the reduction is short (1x1 128 -> 512 on one 28x28 image 4.0 -> 3.3,
//     64 -> 64 on two 56x56 3.5 -> 3.1, int8 3x3 64 -> 128 on four 28x28 4.8 -> 3.4; at 32 steps 6.7 against the tiled 6.4, and at
//     three per unit no gain).
static inline int small_variant(const ConvParams &p, int taps, bool sparse, int ncu)
{
    const long long b16 = small_blocks(p, 16, 1), b32 = small_blocks(p, 32, 1), b64 = small_blocks(p, 32, 2);
    const int nw = small_waves(p, taps, false);
    if (b16 <= ncu || (taps && nw == 2 && b16 * nw <= 8ll * ncu)) return SMALL_16;
    if (b32 <= ncu || (taps && nw == 4 && b32 * nw <= 8ll * ncu) || (taps == 4 && b32 <= 2ll * ncu)) return SMALL_32;
    if (b64 <= ncu && (taps ? nw == 8 && sparse : p.Ks >= 16)) return SMALL_64X32;
    if (!taps && p.Ks <= 20 && b32 <= 2ll * ncu) return SMALL_32;
    return SMALL_NONE;
}

// Shares of equal numbers of steps, added up in their order, in which a 1x1 layer's own call adds its reduction (1: one chain of products).
static inline int pw_shares(int P, int Ks, int Mt, bool sparse, int ncu)
{
    ConvParams q{};
    q.P = P; q.Ks = Ks; q.Mt = Mt;
    const int variant = small_variant(q, 0, sparse, ncu);
    return variant == SMALL_NONE ? 1 : small_waves(q, 0, variant == SMALL_16);
}

// Would the library by itself run this problem on one of them?
static inline bool takes_small(const ss_weight_desc *d, const ConvParams &p, bool sparse, int ncu)
{
    const int mode = small_staging(d, p);
    return mode >= 0 && small_variant(p, small_taps(mode) ? d->kh * d->kw : 0, sparse, ncu) != SMALL_NONE;
}

// ---------------------------------------------------------------------------------------------
// The fused pair and its third layer.
// ---------------------------------------------------------------------------------------------
constexpr int kFuseRow = 32 + 4;      // floats per pixel row of a wave's 32 x 32 result in LDS

// The tile must hold every output channel of the first convolution: 64, 128 or 256 rows; among the tiles of that
// height the grid size decides as in choose_tile.
static inline int choose_fused_tile(const ConvParams &p)
{
    if (p.Cout <= 64) return n_blocks(p, 64, 64) <= 1024 ? 1 : 0;
    if (p.Cout <= 128) return n_blocks(p, 128, 64) <= 256 ? 4 : 2;
    return n_blocks(p, 256, 64) <= 256 ? 5 : 3;
}

// Few pixels (pair_small_kernel, ss_conv_small.h).
constexpr int kPairWaves = 8;
struct PairShape {                    // LDS map of a workgroup, in bytes
    size_t stage, part, tile, third, total;  // [0, stage): staging, later the output slabs; then partial sums; then the 16-bit tile; the second layer's
};                                           // output where a third one follows; then the first layer's bias
#ifdef __HIPCC__
__host__ __device__
#endif
static inline PairShape pair_shape(int px, int nchunks, int cout1, int cout2)      // cout2: 0 without a third layer
{
    PairShape h;
    h.stage = (size_t)nchunks * px * 576;
    const size_t slabs = (size_t)kPairWaves * px * kFuseRow * 4;
    if (h.stage < slabs) h.stage = slabs;
    h.part = (size_t)kPairWaves * 4096;
    h.tile = (size_t)px * (cout1 + 8) * 2;
    h.third = cout2 > 0 ? (size_t)px * (cout2 + 8) * 2 : 0;
    h.total = h.stage + h.part + h.tile + h.third + (size_t)cout1 * 4;
    return h;
}

// Pixels per workgroup while one workgroup per compute unit holds them all, or 0.
static inline int pair_small_pixels(long long P, int ncu) { return (P + 15) / 16 <= ncu ? 16 : ((P + 31) / 32 <= ncu ? 32 : 0); }

// Does the kernel take these layers, px pixels at a time?  cout2, cout3: 0 without a third layer (with one: widths known at compile time, two waves at
// least to a row tile, weights of at most sixteen steps).
static inline bool pair_small_fits(const ss_weight_desc *d1, int px, int cout2, int cout3)
{
    if (d1->korder != SS_K_CRS || d1->kh != 3 || d1->kw != 3 || d1->cin % 32 != 0 || d1->cout % 32 != 0 || d1->cout > 32 * kPairWaves) return false;
    if (cout2 > 0 && ((d1->cout != 64 && d1->cout != 128) || cout2 > 512 || cout3 < 64 || cout3 > 128)) return false;
    return pair_shape(px, d1->cin / 32, d1->cout, cout2).total <= 160 * 1024;
}


// Split of a convolution's reduction over several workgroups per output tile (for grids that leave most compute
// units idle: few output pixels, long reductions -- small-batch inference and the last stages of a network).
struct SplitPlan {
    int tile, bm, bn, nsplit;        // tile id and shape; workgroups per output tile (1 = no split, nothing else is used)
    long long tiles;
    size_t ctr_bytes, part_bytes;    // workspace: ticket counters, then fp32 partial sums [tile][split][bm * bn]
};
// Decides tile and split for a 16-bit problem.  Only the two staging modes of the networks' own layers split (1x1
// kernels with more than two 32-wide steps; 3x3 kernels in the channel-slowest flattening with cin % 32 == 0).
// forced_tile / forced_split: test hooks (negative / zero: the library decides).  A split happens by itself when the
// grid would leave at least half of the compute units idle and the reduction is long enough to pay for the hand-over.
inline SplitPlan plan_split(const ss_weight_desc *d, long long P, int Ks, int ncu, int forced_tile, int forced_split)
{
    SplitPlan pl{};
    pl.nsplit = 1;
    if (is_byte_type(d->dtype)) return pl;
    if (forced_tile >= 10) return pl;              // the resident-grid, image and activation-stationary kernels do not split
    const bool pw = d->kh * d->kw == 1 && d->cin % 8 == 0 && Ks > 2;
    const bool taps = d->korder == SS_K_CRS && d->kh == 3 && d->kw == 3 && d->cin % 32 == 0;
    if (!pw && !taps) return pl;
    const int ksteps = taps ? 9 : 4;
    ConvParams q{};
    q.Cout = d->cout; q.P = (int)P; q.K = d->cin * d->kh * d->kw;
    pl.tile = (forced_tile >= 0 && forced_tile <= 5) ? forced_tile : choose_tile(q, pw, taps);
    pl.bm = pl.tile <= 1 ? 64 : ((pl.tile == 2 || pl.tile == 4) ? 128 : 256);
    pl.bn = 64;
    pl.tiles = n_blocks(q, pl.bm, pl.bn);
    const int nchunks = (Ks + ksteps - 1) / ksteps;
    int n = 1;
    if (forced_split > 0) n = forced_split;
    else if (forced_tile < 0 && pl.tiles * 2 <= ncu) {
        // Measured on MI355X: handing the partial sums over costs about as much as four 3x3 chunks (sixteen of the
        // shorter 1x1 chunks), so a share keeps at least that many.  (512 -> 512 3x3 at 7x7: batch 1, 4 tiles, 14.5 us
        // whole, 9.6 us in four shares; batch 8, 28 tiles, 14.8 -> 11.7 us; reductions of 2304 and the 1x1 layers up
        // to 2048 channels gained nothing and stay whole.)
        const int per_share = taps ? 4 : 16;
        n = (int)(ncu / pl.tiles);
        if (n > nchunks / per_share) n = nchunks / per_share;
        if (n > 8) n = 8;
        if (nchunks < 3 * per_share) n = 1;
    }
    if (n > nchunks) n = nchunks;
    if (n < 1) n = 1;
    pl.nsplit = n;
    pl.ctr_bytes = ticket_bytes(pl.tiles);
    pl.part_bytes = (size_t)pl.tiles * n * pl.bm * pl.bn * 4;
    return pl;
}

// Test hook (ss_debug.h): the tile id forced by ss_debug_force_tile, or -1 when the library chooses.
int forced_tile();
// Test hook (ss_debug.h): upper bound on the workgroups of the resident-grid kernels, or 0 for none.
int block_limit();
// Test hook (ss_debug.h): workgroups per output tile forced by ss_debug_force_split, or 0 when the library decides.
int forced_split();

// One function per operand type and operand form, each defined in its own translation unit.  conv_dispatch_* picks
// the staging mode and tile for the problem and launches; fused_dispatch_* does so for a k x k convolution followed by
// a 1x1 one; mlp_dispatch_* launches the 1x1 -> 1x1 kernel.  All return an SS_* status.
#define SS_DECLARE_CONV(NAME) \
    int conv_dispatch_##NAME(const ss_weight_desc *desc, const ConvParams &p, hipStream_t s);
#define SS_DECLARE_FUSED(NAME) \
    int fused_dispatch_##NAME(const ss_weight_desc *d1, const ChainParams &p, hipStream_t s); \
    int mlp_dispatch_##NAME(const MlpParams &p, hipStream_t s);
SS_DECLARE_CONV(f16_sparse) SS_DECLARE_CONV(f16_dense) SS_DECLARE_CONV(bf16_sparse) SS_DECLARE_CONV(bf16_dense)
SS_DECLARE_CONV(i8_sparse) SS_DECLARE_CONV(i8_dense) SS_DECLARE_CONV(f8_sparse) SS_DECLARE_CONV(f8_dense)
// Can the image kernel take this problem?  Dense 16-bit 7x7 kernel with stride 2 on three or four channels, 16-byte
// output runs, no residual, output below 2 GiB (32-bit store offsets, out-of-range mark above every real one).
static inline bool image_eligible(const ss_weight_desc *desc, const ConvParams &p)
{
    return !is_byte_type(desc->dtype) && desc->kh == 7 && desc->kw == 7 && (desc->cin == 3 || desc->cin == 4) && p.sh == 2 &&
           p.sw == 2 && desc->cout % 8 == 0 && p.residual == nullptr && p.nsplit <= 1 &&
           (long long)p.P * p.Cout * 2 < (1ll << 31) - (1ll << 27);
}

// The first layer of an image network with the max pooling behind it (dense 16-bit operands), the pooled output at p.y2.
int pooled_dispatch_f16_dense(const ss_weight_desc *desc, const ConvParams &p, int pool_h, int pool_w, hipStream_t s);
int pooled_dispatch_bf16_dense(const ss_weight_desc *desc, const ConvParams &p, int pool_h, int pool_w, hipStream_t s);
SS_DECLARE_FUSED(f16_sparse) SS_DECLARE_FUSED(f16_dense) SS_DECLARE_FUSED(bf16_sparse) SS_DECLARE_FUSED(bf16_dense)

}  // namespace ss

#endif
