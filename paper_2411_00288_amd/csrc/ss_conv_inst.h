// Instantiates the convolution kernels for one operand type and one operand form (2:4-sparse or dense), named by the
// including file through SS_INST_NAME / SS_INST_DT / SS_INST_SPARSE / SS_INST_FUSED.
#include "ss_conv_kernel.h"
#include "ss_conv_stream.h"
#include "ss_conv_image.h"
#include "ss_conv_rows.h"
#include "ss_conv_small.h"

#define SS_CAT2(a, b) a##b
#define SS_CAT(a, b) SS_CAT2(a, b)

namespace ss {

int SS_CAT(conv_dispatch_, SS_INST_NAME)(const ss_weight_desc *desc, const ConvParams &p, hipStream_t s)
{
    // Few output pixels: the one-latency kernels (tile ids 20 to 22 when forced; a forced split means the tiled kernels)
    if (forced_tile() < 0 ? forced_split() == 0 : forced_tile() >= 20 && forced_tile() <= 22) {
        const int st = small_mode<SS_INST_DT, SS_INST_SPARSE>(desc, p, forced_tile() < 0 ? -1 : forced_tile() - 20, s);
        if (st != SS_ERR_INVALID_ARG) return st;
    }
    if constexpr (!is_byte_type(SS_INST_DT) || SS_INST_SPARSE) {
        if (p.nsplit <= 1 && stream_eligible(desc, p)) {
            int ncu = compute_units();
            if (ncu <= 0) return SS_ERR_HIP;
            if (block_limit() > 0 && block_limit() < ncu) ncu = block_limit();
            const int forced = forced_tile();
            // Two pixel-tile widths: 128 pixels make the cheapest step, 64 waste less of the last round.  A workgroup takes
            // its tiles one after the other, so the time goes with the rounds of the fullest compute unit; a round of the
            // narrow tile measured 0.59 of a wide one (256 -> 256 on N 14x14 images, f16: N = 125, rounds 1 / 3, 20.4 / 24.9
            // us; 200, 2 / 3, 37.2 / 35.8; 500, 3 / 6, 60.9 / 69.7).
            // Against the one-tile-per-workgroup kernels: faster as soon as the narrow grid fills more than half of the
            // compute units (256 -> 256, N = 50, 154 tiles: 12.6 against 13.0 us, fp8 N = 64: 9.4 / 9.8; N = 40, 123 tiles:
            // 12.3 / 10.3), provided the 256-row tiles are not mostly padding.  3x3: above 176 channels per 256-row tile with 16-bit
            // operands (5 row tiles of 32: the one-tile kernels' 160-row tile takes 0.96 of this one's time, 6 to 8: 1.01 to 1.09; 9 to 11 in two: 0.91
            // to 0.94, 12: 0.99), above 224 with 8-bit ones, whose steps are half as long (their 224-row tile 0.92, eight row tiles: 0.96 to
            // 1.05).  2x2: above half.
            const long long rows = (p.Cout + 255) / 256, wide = ((long long)p.P + 127) / 128, narrow = ((long long)p.P + 63) / 64;
            const long long slots = ncu > rows ? ncu / rows : 1;          // pixel tiles of one round, as the launch deals them out
            const long long rounds_w = (wide + slots - 1) / slots, rounds_n = (narrow + slots - 1) / slots;
            const bool filled = desc->kh == 2 ? 2ll * p.Cout > 256 * rows : (is_byte_type(SS_INST_DT) ? (long long)p.Cout > 224 * rows : (long long)p.Cout > 176 * rows);
            const bool pays = filled && 2 * rows * narrow > ncu;
            if (desc->kh == 2) {
                // The same line for 2x2 kernels of 16-bit operands with at least two chunks (96 -> 192 on 128 images of 56x56: 30-35
                // -> 25.4 us, on 32: 9.8 -> 7.7; 192 -> 384 on 64 of 28x28 12.6 -> 10.4; one chunk, 32 -> 200: 5.6 against 6.7 stays).
                // Sparse, a narrow round is worth 0.56 of a wide one.  8-bit operands gain nothing (23.4 / 23.2, 24.1 / 23.5): not built.
                if constexpr (!is_byte_type(SS_INST_DT)) {
                    const bool wide_pays = 100 * rounds_w <= (SS_INST_SPARSE ? 56 : 59) * rounds_n;
                    if (forced == 10 || (forced < 0 && pays && p.Ks > 4 && wide_pays))
                        return launch_stream<SS_INST_DT, SS_INST_SPARSE, 2, 4, 2>(p, ncu, s);
                    if (forced == 11 || (forced < 0 && pays && p.Ks > 4)) return launch_stream<SS_INST_DT, SS_INST_SPARSE, 2, 2, 2>(p, ncu, s);
                }
            } else {
                if (forced == 10 || (forced < 0 && pays && 100 * rounds_w <= 59 * rounds_n))
                    return launch_stream<SS_INST_DT, SS_INST_SPARSE, 2, 4, 3>(p, ncu, s);
                if (forced == 11 || (forced < 0 && pays)) return launch_stream<SS_INST_DT, SS_INST_SPARSE, 2, 2, 3>(p, ncu, s);
            }
        }
    }
    if constexpr (!is_byte_type(SS_INST_DT)) {
        // 1x1 layers with short reductions and many output channels: activations stationary (tile id 13 when forced)
        const int forced = forced_tile();
        // Measured on the ResNet-50 / ConvNeXt-T layers: it pays for the channel-expanding layers (64 -> 256 ... 512 -> 2048
        // and the 512 -> 1024 projection: 5-13 % faster; 96 -> 384 with GELU: 117 -> 84 us) and loses on the reducing
        // ones, whose few output channels leave nothing to walk over.
        // With a residual tail the gain is smaller (the residual runs are fetched by the same waves that multiply), and
        // at 512 channels, where LDS leaves room for one workgroup per compute unit, it turns into a loss.
        // With few pixel tiles (small batches of the late stages) the long reductions do better in the tiled kernels
        // (7x7 images, 512 -> 2048: 4.4 vs 5.7 us at batch 1, 4.7 vs 6.0 us at batch 8).
        const bool pays = p.Cout >= 2 * desc->cin && p.Cout >= 256 && !(desc->cin >= 512 && p.residual != nullptr) &&
                          (desc->cin <= 128 || (long long)p.P >= 48 * 64);
        if ((forced == 13 || (forced < 0 && pays)) && rows_eligible(desc, p)) {
            int ncu = compute_units();
            if (ncu <= 0) return SS_ERR_HIP;
            if (block_limit() > 0 && block_limit() < ncu) ncu = block_limit();
            return launch_rows<SS_INST_DT, SS_INST_SPARSE>(desc, p, ncu, s);
        }
    }
    if constexpr (!is_byte_type(SS_INST_DT) && !SS_INST_SPARSE) {
        // the dense first layer of an image network (tile id 12 when forced)
        const int forced = forced_tile();
        if ((forced < 0 || forced == 12) && image_eligible(desc, p)) {
            int ncu = compute_units();
            if (ncu <= 0) return SS_ERR_HIP;
            if (block_limit() > 0 && block_limit() < ncu) ncu = block_limit();
            return launch_image<SS_INST_DT>(desc, p, ncu, s);
        }
    }
    return pick_mode<SS_INST_DT, SS_INST_SPARSE>(desc, p, s);
}

#if SS_INST_FUSED
#if !SS_INST_SPARSE
int SS_CAT(pooled_dispatch_, SS_INST_NAME)(const ss_weight_desc *desc, const ConvParams &p, int pool_h, int pool_w, hipStream_t s)
{
    int ncu = compute_units();
    if (ncu <= 0) return SS_ERR_HIP;
    if (block_limit() > 0 && block_limit() < ncu) ncu = block_limit();
    return image_eligible(desc, p) ? launch_image<SS_INST_DT, true>(desc, p, ncu, s, pool_h, pool_w) : (int)SS_ERR_UNSUPPORTED;
}
#endif

int SS_CAT(fused_dispatch_, SS_INST_NAME)(const ss_weight_desc *d1, const ChainParams &p, hipStream_t s)
{
    if (forced_tile() < 0 || forced_tile() == 20 || forced_tile() == 21) {       // few output pixels
        const int st = pair_small<SS_INST_DT, SS_INST_SPARSE>(d1, p, forced_tile() < 0 ? 0 : (forced_tile() == 20 ? 16 : 32), s);
        if (st != SS_ERR_INVALID_ARG) return st;
    }
    return fused_mode<SS_INST_DT, SS_INST_SPARSE>(d1, p, s);
}

int SS_CAT(mlp_dispatch_, SS_INST_NAME)(const MlpParams &p, hipStream_t s)
{
    return launch_mlp<SS_INST_DT, SS_INST_SPARSE>(p, s);
}
#endif

}  // namespace ss
