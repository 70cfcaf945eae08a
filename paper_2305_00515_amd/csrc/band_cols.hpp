// Which bytes of a row the banded uint8 kernels load, and which byte stands
// where in a lane's window.  Plain integer code, shared by the kernels and by
// a host-side check that enumerates every width, column and border rule.
//
// A lane's window is a run of 4-byte words of one image row.  Word `x`
// (columns x .. x + 3, any of them possibly outside the row) is loaded as
// the four bytes at window_load(x, W), which always lie inside the row of
// W >= 4 bytes, and its bytes are put in place by one byte permute with
// window_sel(x, ...): the permute also does the border rule, because the
// columns that REPLICATE and REFLECT101 read for the two columns beyond an
// edge lie in the same four bytes.  Bytes further outside meet only zero
// weights or unwanted outputs and hold some byte of the row.
#pragma once

#if defined(__HIPCC__)
#define S4X5_BAND_HD __host__ __device__
#else
#define S4X5_BAND_HD
#endif

namespace s4x5 {

S4X5_BAND_HD inline int band_clamp(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// Border rules as the kernels take them (VALID reads like REPLICATE, at
// positions that lie inside).
constexpr int kBandRep = 0, kBandZero = 1, kBandRefl = 2;

// Index that position i of an axis of n >= 1 pixels reads, for i at most two
// outside the axis (REFLECT101 bounces twice on an axis of two pixels);
// always in [0, n - 1], also for positions further out and under ZERO, whose
// callers mask the value.
S4X5_BAND_HD inline int band_index(int i, int n, int bm)
{
    if (bm == kBandRefl) {
        i = i < 0 ? -i : i;
        const int m = 2 * (n - 1) - i;
        i = m < i ? m : i;
        i = i < 0 ? -i : i;
    }
    return band_clamp(i, 0, n - 1);
}

S4X5_BAND_HD inline int window_load(int x, int W) { return band_clamp(x, 0, W > 4 ? W - 4 : 0); }

// Byte selector (one byte per window byte: 0..3 picks a loaded byte, 0x0c
// gives zero) of the window word at column x.
S4X5_BAND_HD inline unsigned window_sel(int x, int W, int bm)
{
    const int base = window_load(x, W);
    unsigned sel = 0;
    for (int t = 0; t < 4; ++t) {
        const int c = x + t;
        const int s = band_clamp(band_index(c, W, bm) - base, 0, 3);
        sel |= (bm == kBandZero && (c < 0 || c >= W) ? 0x0cu : (unsigned)s) << (8 * t);
    }
    return sel;
}

}  // namespace s4x5
