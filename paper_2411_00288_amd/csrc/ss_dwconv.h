// Which kernel a depthwise convolution takes (ss_dwconv.hip), host code only.
#ifndef SS_DWCONV_H_
#define SS_DWCONV_H_
#include <stdint.h>

namespace ss {

// The kernels by their ids of ss_debug_force_tile: vector ALU, matrix unit, and few outputs with 1 x 2, 1 x 4, 2 x 4 and 4 x 4 outputs per thread.
enum { DW_VECTOR = 60, DW_MATRIX = 61, DW_FEW_1X2 = 62, DW_FEW_1X4 = 63, DW_FEW_2X4 = 64, DW_FEW_4X4 = 65 };

constexpr int kDwFewTaps = 8192;          // kernel for few outputs: K K C at most, 32 KiB of LDS

struct DwShape {
    int N, H, W, C, kh, kw, ph, Ho, Wo;
};

// Can this kernel run the layer?
static inline bool dw_fits(const DwShape &s, int id)
{
    if (id == DW_VECTOR) return true;
    if (s.kh != s.kw) return false;
    // Offsets outside the image start at 2 GiB and go on by rows: they must not come round to the image again.  The matrix kernel's go on from the first
    // padding row to the image's last, those of the kernel for few outputs over one thread's rows.
    if (id == DW_MATRIX) return s.kw > 3 && ((long long)s.H + s.ph) * s.W * s.C * 2 < (1ll << 31) && (long long)s.N * s.Ho * s.Wo * s.C * 2 < (1ll << 31);
    if (s.kw * s.kw * s.C > kDwFewTaps || (long long)(s.kw + 3) * s.W * s.C * 2 >= (1ll << 31)) return false;
    if ((id == DW_FEW_1X2 && s.kw != 7) || (id == DW_FEW_2X4 && s.kw == 5) || (id == DW_FEW_4X4 && s.kw != 3)) return false;
    const int rows = id == DW_FEW_4X4 ? 4 : (id == DW_FEW_2X4 ? 2 : 1), cols = id == DW_FEW_1X2 ? 2 : 4;
    return (long long)s.N * ((s.Ho + rows - 1) / rows) * ((s.Wo + cols - 1) / cols) * (s.C / 2) <= 0x7FFFFF00ll;      // (its threads have 31-bit numbers)
}

// Few outputs: the kernel for them, 3x3 always.  Against the vector one it wins (see there), except on images of one row, of whose inputs it loads
// the missing rows as well (3x3, from 2.5 M outputs on 1.1 to 2.2 of the vector kernel's time, below 0.7 to 0.9; 5x5 from 1.2 M on 1.1 to 1.45), and 5x5 on two
// rows (from 2.5 M on 1.0 to 1.2).  Against the matrix one, us: 5x5 16 x 56 x 56 x 96
// (4.8 M outputs) 10.0 / 10.3, 64 x 28 x 28 x 128 (6.4 M) 11.9 / 11.2; with more than 128 channels, whose taps each workgroup fetches whole, the line is the
// vector kernel's, 11 x 47 x 63 x 152 (4.95 M) 13.7 / 10.8; 7x7 8 x 56 x 56 x 96 (2.4 M) 9.35 / 10.6, 12 x 56 x 56 x 96 (3.6 M) 11.0 / 10.95, 16 (4.8 M)
// 13.5 / 11.6.  Rows per thread: 3x3 at 1.9 M outputs 4.2 / 4.3 / 4.7 for one, two and four, 4.8 M 7.5 / 6.3 / 6.6, 9.6 M 14 / 11.1 / 10.2 (four are 1.2 of
// two where there are only two rows); 7x7 at 1.4 M 6.6 / 7.1 for one and two, 1.9 M 8.0 / 7.6.  7x7 in pairs of columns while that is one workgroup per
// compute unit: 14 x 14 x 14 x 96 4.4 -> 3.9.
// The matrix kernel costs about the same for every filter width and has a longer set-up.  Measured against the vector one, where the taps or
// the rows do not fit the kernel for few outputs: 7x7 faster or equal from 1 x 7 x 7 x 96 up, 5x5 from about 4 M outputs.
static inline int choose_dw(const DwShape &s, int ncu)
{
    const long long outputs = (long long)s.N * s.Ho * s.Wo * s.C;
    int few = -1;
    if (s.kw == 3) {
        if (s.H > 1 || outputs < 2500000) few = outputs < 2500000 ? DW_FEW_1X4 : (outputs < 8000000 || s.H == 2 ? DW_FEW_2X4 : DW_FEW_4X4);
    } else if (s.kw == 5) {
        if (outputs < (s.H == 1 ? 1200000 : (s.H == 2 ? 2500000 : (s.C > 128 ? 1 << 22 : 5000000)))) few = DW_FEW_1X4;
    } else if (outputs < 3200000) {
        const bool narrow = (long long)s.N * s.Ho * ((s.Wo + 1) / 2) * (s.C / 2) <= 256ll * ncu;
        few = narrow ? DW_FEW_1X2 : (outputs >= 1700000 ? DW_FEW_2X4 : DW_FEW_1X4);
    }
    if (few >= 0 && dw_fits(s, few)) return few;
    return (s.kw == 7 || (s.kw == 5 && outputs >= 1 << 22)) && dw_fits(s, DW_MATRIX) ? DW_MATRIX : DW_VECTOR;
}

}  // namespace ss

#endif
