// The uint8 operators as banded matrix products on the int8 matrix cores,
// streamed from memory: no LDS, no barrier, any alignment of rows and bases.
//
// One v_mfma_i32_16x16x64_i8 multiplies a 16 x 64 weight block A by a 64 x 16
// image block B.  The kernels lay it out so that the lane that loads a piece
// of the image is the lane that stores the piece of the result at the same
// place (n = lane % 16, g = lane / 16):
//   B[k][n]: n = one of 16 tiles; k = (g, byte) is held by lane (g, n): four
//            rows of a "quad" of input rows, one per lane group g, as two
//            8-byte windows: one of quad q, one of quad q + 1 (the five rows
//            of any of four consecutive output rows lie in two quads);
//   A[m][k]: m = (output row j of four, response f of four): response f's
//            weight at row offset (g or g + 4) - j, column offset byte - s,
//            for the output column whose taps start at byte s of the window;
//            zero off the band;
//   D[m][n]: lane (g, n) receives m = 4 g .. 4 g + 3: the four responses of
//            output row g, column c of tile n.
// So a step of a wave covers 4 rows x (4 NB) columns of 16 tiles: each lane
// loads one window of 4 NB + 8 bytes of a row (NB words and one on each
// side), and after 4 NB products holds all responses of 4 NB consecutive
// pixels of one row.  The first two columns of a word take the windows of
// that word and the one before, the last two of that word and the next.  An
// image quad enters once and serves two steps (its operand registers keep
// their place, and the weight operands come in two orders instead).
//
// The tiles of a wave are 16 consecutive ones of the image's tile grid, row
// band by row band; each lane addresses its own, so narrow images and the
// last columns waste nothing but the last wave.  A tile whose columns would
// pass the right edge is moved left until it ends at it: the columns it
// shares with its neighbour get the same bytes twice.
//
// uint8 pixels enter as int8 through x ^ 0x80 = x - 128: every filter here
// is antisymmetric under a half turn, so its weights sum to zero and the
// shift leaves the response unchanged.  Responses are exact in int32.
//
// What bounds it: memory.  A four-directional magnitude takes 9.3 vector
// instructions and one product a pixel (8192^2: 10.7 M wave instructions,
// 1.05 M of them products; 18 us of issue), and HBM moves 1.03 times the
// input and 1.00 times the output.  8192^2 takes 30.0 us from HBM (buffers in
// turn, 4.5 TB/s) and 25.0 us on one pair of buffers, which the Infinity Cache
// holds in part and where torch's copy of the same bytes takes 27.0 us; the
// packed int16 sweep that ran here before took 20.4 instructions a pixel and
// 45.1 us.  What counted, on one pair of buffers:
//   - 16-byte stores past the L2: 31.7 -> 25.8 us, and rows of the output
//     that are not aligned to lines cost 2 us instead of 5;
//   - windows loaded at multiples of 4 bytes: at odd addresses (kShift) a
//     launch took 38 us before, 33 us with it (26.8 us with the stores above);
//   - neighbouring workgroups on one XCD: 35.7 -> 31.7 us;
//   - taking the words beside a tile from the neighbour lane's registers
//     instead of loading them gained nothing.
#pragma once

#include "band_cols.hpp"
#include "internal.hpp"

#include <type_traits>

namespace s4x5 {

// `v` with lane `lane` replaced by the scalar `s`: the compiler's intrinsic,
// which keeps the two wait states between a vector instruction that writes `s`
// (the reload of a spilled argument) and this one; asm would not.
__device__ unsigned int write_lane(unsigned int s, unsigned int lane, unsigned int v) __asm("llvm.amdgcn.writelane.i32");

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef unsigned int u32;
typedef unsigned long long u64;
typedef u32 bv4 __attribute__((ext_vector_type(4)));
typedef u32 bv3 __attribute__((ext_vector_type(3)));
typedef u32 bv2 __attribute__((ext_vector_type(2)));
// global memory at any byte address (the runtime runs the GPU in unaligned
// access mode)
#define BAND_G __attribute__((address_space(1)))
typedef bv4 bv4_u __attribute__((aligned(1)));
typedef bv2 bv2_u __attribute__((aligned(1)));
typedef bv4 bv4_a __attribute__((aligned(4)));
typedef bv3 bv3_a __attribute__((aligned(4)));
typedef bv2 bv2_a __attribute__((aligned(4)));
typedef u32 u32_u1 __attribute__((aligned(1)));
typedef const BAND_G uint8_t *gsrc;
typedef BAND_G uint8_t *gdst;

constexpr int kBandWaves = kGroupWaves;
constexpr int kBandResident = 16; // waves a CU holds: 4 on each SIMD, at up to 128 VGPRs

// Weights of an operator: bytes 0..4 of row[5 f + dy] are the int8 weights of
// row dy of response f.
struct BandTaps {
    uint64_t row[20];
};
template <class K>
constexpr BandTaps band_taps(const K &k, int responses)
{
    BandTaps t{};
    for (int f = 0; f < responses; ++f)
        for (int dy = 0; dy < 5; ++dy)
            for (int dx = 0; dx < 5; ++dx) t.row[5 * f + dy] |= (uint64_t)(uint8_t)(int8_t)k[f][dy][dx] << (8 * dx);
    return t;
}

// Eq. (sobel5_1) in plane order: 0, 45, 90, 135 degrees.
constexpr int kSobel5[4][5][5] = {
    {{-1, -2, 0, 2, 1}, {-4, -8, 0, 8, 4}, {-6, -12, 0, 12, 6}, {-4, -8, 0, 8, 4}, {-1, -2, 0, 2, 1}},
    {{-6, -4, -1, -2, 0}, {-4, -12, -8, 0, 2}, {-1, -8, 0, 8, 1}, {-2, 0, 8, 12, 4}, {0, 2, 1, 4, 6}},
    {{-1, -4, -6, -4, -1}, {-2, -8, -12, -8, -2}, {0, 0, 0, 0, 0}, {2, 8, 12, 8, 2}, {1, 4, 6, 4, 1}},
    {{0, -2, -1, -4, -6}, {2, 0, -8, -12, -4}, {1, 8, 0, -8, -1}, {4, 12, 8, 0, -2}, {6, 4, 1, 2, 0}},
};
// Eq. (sobel3_1), 0 and 90 degrees, in the middle of a 5x5 window.
constexpr int kSobel3[2][5][5] = {
    {{0, 0, 0, 0, 0}, {0, -1, 0, 1, 0}, {0, -2, 0, 2, 0}, {0, -1, 0, 1, 0}, {0, 0, 0, 0, 0}},
    {{0, 0, 0, 0, 0}, {0, -1, -2, -1, 0}, {0, 0, 0, 0, 0}, {0, 1, 2, 1, 0}, {0, 0, 0, 0, 0}},
};
struct Pair5 {   // the 0 and 90 degree filters of Eq. (sobel5_1)
    constexpr const int (&operator[](int f) const)[5][5] { return kSobel5[2 * f]; }
};
constexpr BandTaps kTaps4x5 = band_taps(kSobel5, 4), kTaps2x5 = band_taps(Pair5{}, 2), kTaps2x3 = band_taps(kSobel3, 2);

// Operand word of the lane's weights: bytes 0..4 of the result are the five
// weights of row dy of response f (zero outside the filter).  The twenty
// rows come as kernel arguments; lane i takes row i, and each lane then
// fetches its row from there, which costs no memory access.
__device__ __forceinline__ u64 band_tap(u32 lo, u32 hi, int f, int dy)
{
    const int at = 4 * (5 * f + band_clamp(dy, 0, 4));
    const u32 a = (u32)__builtin_amdgcn_ds_bpermute(at, (int)lo);
    const u32 b = (u32)__builtin_amdgcn_ds_bpermute(at, (int)hi);
    return (dy >= 0 && dy <= 4) ? ((u64)b << 32 | a) : 0ull;
}

// Weight operands: NR responses a pixel (4, or 2 for the two-directional
// operators, whose products serve two columns each), in both quad orders.
template <int NR>
struct BandA {
    v4i w[2][NR];
};

template <int NR>
__device__ __forceinline__ void band_weights(const BandTaps &T, BandA<NR> &A)
{
    const int lane = threadIdx.x & 63, g = lane >> 4, j = (lane >> 2) & 3, r = lane & 3;
    const int f = r % NR, cc = r / NR;
    u32 lo = 0, hi = 0;
#pragma unroll
    for (int i = 0; i < 5 * NR; ++i) {
        lo = write_lane((u32)T.row[i], i, lo);
        hi = write_lane((u32)(T.row[i] >> 32), i, hi);
    }
    const u64 near = band_tap(lo, hi, f, g - j), far = band_tap(lo, hi, f, g + 4 - j);
#pragma unroll
    for (int p = 0; p < NR; ++p) {
        const int sh = 8 * ((p * (4 / NR) + cc) ^ 2);   // columns 0..3 of a word start at bytes 2, 3, 0, 1
        const u64 a = near << sh, b = far << sh;
        A.w[0][p] = v4i{(int)(u32)a, (int)(u32)(a >> 32), (int)(u32)b, (int)(u32)(b >> 32)};
        A.w[1][p] = v4i{(int)(u32)b, (int)(u32)(b >> 32), (int)(u32)a, (int)(u32)(a >> 32)};
    }
}

// a * a + acc on the 24-bit multiplier (|a| < 2^23), one instruction.  `a` may
// come from a matrix product only if a compiled instruction has read that
// product before: the wait for it stands there, and none before asm.
__device__ __forceinline__ int sq24(int a, int acc)
{
    int r;
    asm("v_mad_i32_i24 %0, %1, %1, %2" : "=v"(r) : "v"(a), "v"(acc));
    return r;
}

// One lane's tile: its first output column and row, and the number of steps
// of four rows (the same in all lanes of a wave).
struct BandTile {
    int xo, yo, steps;
};

// How a wave reads its windows.
//   kInside:  every byte and row of every lane lies in the image, and windows
//             start at multiples of 4 bytes;
//   kShift:   the same at other addresses: the aligned words around a window
//             are loaded and shifted (a load of several words at an address
//             that is no multiple of 4 takes about twice as long);
//   kCols:    every row lies in the image; the words beside the lane's own
//             columns are loaded inside the row and permuted;
//   kEdge:    the same, and rows are mapped;
//   kNarrow:  rows narrower than a tile: every word is loaded inside the row
//             and permuted.
constexpr int kInside = 0, kShift = 1, kCols = 2, kEdge = 3, kNarrow = 4;

// Windows of the quads of one lane's tile.  load() issues the loads of the
// next quad into `d`, words(d) puts the oldest loaded quad's words in place.
template <int NB, int MODE>
struct BandSource {
    static constexpr bool kWhole = MODE != kEdge && MODE != kNarrow;   // every row of every lane lies in the image
    static constexpr bool kBeside = MODE == kCols || MODE == kEdge;
    static_assert(NB == 1 || NB == 2 || NB == 4, "words per lane");
    static constexpr int kWords = NB + 2;
    static constexpr int kRaw = MODE == kShift ? NB + 3 : NB + 2;
    static constexpr int kMoved = MODE == kNarrow ? kWords : 2;   // words that are permuted

    gsrc p;              // kInside, kShift: the lane's window, kNarrow: the row's start, else its own
                         // columns; in its row of the next quad (kEdge, kNarrow: in row 0)
    int64_t pitch;
    int quads;           // quads not loaded yet; the last one is loaded again when none is left
    int y, yf;           // the lane's row of the next quad to load / to put in place
    int H, W, bm;
    int col[kMoved];     // kNarrow: columns of the words; else offsets of the words beside
    u32 sel[kMoved];
    u32 shift;           // kShift: bytes before the window in its first word
    int last;            // kShift: offset of the word that holds the window's last byte

    __device__ __forceinline__ void init(const U8Job &J, const BandTile &t, int off, int border_mode)
    {
        const int g = (threadIdx.x >> 4) & 3;
        const int x = t.xo + off - 4;
        y = yf = t.yo + off - 2 + g;
        H = J.H;
        W = J.W;
        bm = border_mode;
        pitch = J.src_pitch;
        quads = t.steps + 1;
        p = (gsrc)J.src + (MODE == kNarrow ? 0 : kBeside ? x + 4 : x);
        if (kWhole) p += (int64_t)y * pitch;
        if constexpr (MODE == kShift) {
            // four rows below, the shift is the same
            shift = (u32)(uintptr_t)p & 3;
            p -= shift;
            last = shift ? 4 * kWords : 4 * kWords - 4;
        } else if constexpr (kBeside) {
            col[0] = window_load(x, W) - (x + 4);
            sel[0] = window_sel(x, W, bm);
            col[1] = window_load(x + 4 + 4 * NB, W) - (x + 4);
            sel[1] = window_sel(x + 4 + 4 * NB, W, bm);
        } else if constexpr (MODE == kNarrow) {
#pragma unroll
            for (int b = 0; b < kWords; ++b) {
                col[b] = window_load(x + 4 * b, W);
                sel[b] = window_sel(x + 4 * b, W, bm);
            }
        }
    }

    __device__ __forceinline__ void load(u32 (&d)[kRaw])
    {
        gsrc r = p;
        if (!kWhole) r += (int64_t)band_index(y, H, bm) * pitch;
        if constexpr (kBeside) {
            if constexpr (NB == 4) {
                const bv4 v = *reinterpret_cast<const BAND_G bv4_u *>(r);
                d[1] = v.x, d[2] = v.y, d[3] = v.z, d[4] = v.w;
            } else if constexpr (NB == 2) {
                const bv2 v = *reinterpret_cast<const BAND_G bv2_u *>(r);
                d[1] = v.x, d[2] = v.y;
            } else {
                d[1] = *reinterpret_cast<const BAND_G u32_u1 *>(r);
            }
            d[0] = *reinterpret_cast<const BAND_G u32_u1 *>(r + col[0]);
            d[NB + 1] = *reinterpret_cast<const BAND_G u32_u1 *>(r + col[1]);
        } else if constexpr (MODE == kInside || MODE == kShift) {
            if constexpr (NB >= 2) {
                const bv4 v = *reinterpret_cast<const BAND_G bv4_a *>(r);
                d[0] = v.x, d[1] = v.y, d[2] = v.z, d[3] = v.w;
            } else {
                const bv3 v = *reinterpret_cast<const BAND_G bv3_a *>(r);
                d[0] = v.x, d[1] = v.y, d[2] = v.z;
            }
            if constexpr (NB == 4) {
                const bv2 w = *reinterpret_cast<const BAND_G bv2_a *>(r + 16);
                d[4] = w.x, d[5] = w.y;
            }
            if constexpr (MODE == kShift) d[kRaw - 1] = *reinterpret_cast<const BAND_G u32 *>(r + last);
        } else if (W >= 4) {
#pragma unroll
            for (int b = 0; b < kWords; ++b) d[b] = *reinterpret_cast<const BAND_G u32_u1 *>(r + col[b]);
        } else {
            u32 v = 0;
#pragma unroll
            for (int t = 0; t < 3; ++t) v |= (u32)r[band_clamp(t, 0, W - 1)] << (8 * t);
#pragma unroll
            for (int b = 0; b < kWords; ++b) d[b] = v;
        }
        const bool more = --quads > 0;
        if (kWhole)
            p += more ? 4 * pitch : 0;
        else
            y += more ? 4 : 0;
    }

    // the window as int8
    __device__ __forceinline__ void words(const u32 (&d)[kRaw], u32 (&e)[kWords])
    {
#pragma unroll
        for (int b = 0; b < kWords; ++b)
            {
            if constexpr (MODE == kShift)
                e[b] = __builtin_amdgcn_alignbyte(d[b + 1], d[b], shift);
            else
                e[b] = d[b];
        }
        if constexpr (kBeside || MODE == kNarrow) {
            if constexpr (kBeside) {
                e[0] = __builtin_amdgcn_perm(0u, d[0], sel[0]);
                e[NB + 1] = __builtin_amdgcn_perm(0u, d[NB + 1], sel[1]);
            } else {
#pragma unroll
                for (int b = 0; b < kWords; ++b) e[b] = __builtin_amdgcn_perm(0u, d[b], sel[b]);
            }
            if (!kWhole) {
                const u32 keep = bm == kBandZero && (yf < 0 || yf >= H) ? 0u : ~0u;
#pragma unroll
                for (int b = 0; b < kWords; ++b) e[b] &= keep;
                yf += 4;
            }
        }
#pragma unroll
        for (int b = 0; b < kWords; ++b) e[b] ^= 0x80808080u;
    }
};

// The magnitude byte of the sum of squares S: the float conversion is exact
// below 2^24 and anything above saturates, the root is within 1 ulp, and no
// integer S comes nearer than 4.9e-4 to a half-way point.  Inserted as byte
// `at` of `w` by the same instruction that rounds and saturates.
__device__ __forceinline__ u32 mag_byte(int S, int at, u32 w)
{
    return __builtin_amdgcn_cvt_pk_u8_f32(__builtin_amdgcn_sqrtf((float)S), at, w);
}

// CLAMP, for run-time weights of large sums: a response beyond 256 saturates
// the magnitude alone, and clamped responses keep the sum below 2^31.
template <int NR, bool CLAMP>
__device__ __forceinline__ int sum_squares(const int (&G)[NR])
{
    int S = 0;
#pragma unroll
    for (int f = 0; f < NR; ++f) {
        const int v = CLAMP ? band_clamp(G[f], -256, 256) : G[f];
        S = f == 0 ? __mul24(v, v) : sq24(v, S);   // the compiled product comes first (see sq24)
    }
    return S;
}

// 4 N bytes at any address, stored as OutputStores says (a constant: the
// compiler makes one ordinary store of a choice).  The 4 or 8 bytes of a
// magnitude beside planes are left to the L2, where they meet their neighbours,
// unless everything goes past both caches.
template <int TO, int N>
__device__ __forceinline__ void store_words(gdst p, const u32 (&w)[N])
{
    if constexpr (N % 4 == 0) {
#pragma unroll
        for (int i = 0; i < N; i += 4) {
            const bv4 v{w[i], w[i + 1], w[i + 2], w[i + 3]};
            if constexpr (TO == OutputStores::kToMemory)
                __builtin_nontemporal_store(v, reinterpret_cast<BAND_G bv4_u *>(p + 4 * i));
            else if constexpr (TO == OutputStores::kToCache)
                __builtin_amdgcn_global_store_b128(reinterpret_cast<BAND_G bv4 *>(p + 4 * i), v, "agent");
            else
                *reinterpret_cast<BAND_G bv4_u *>(p + 4 * i) = v;
        }
    } else if constexpr (N == 2) {
        const bv2 v{w[0], w[1]};
        if constexpr (TO == OutputStores::kToMemory)
            __builtin_nontemporal_store(v, reinterpret_cast<BAND_G bv2_u *>(p));
        else
            *reinterpret_cast<BAND_G bv2_u *>(p) = v;
    } else {
        static_assert(N == 1, "words");
        if constexpr (TO == OutputStores::kToMemory)
            __builtin_nontemporal_store(w[0], reinterpret_cast<BAND_G u32_u1 *>(p));
        else
            *reinterpret_cast<BAND_G u32_u1 *>(p) = w[0];
    }
}

// The same of a tile that is wider than the image: the first `left` of its
// elements of ES bytes.
template <int ES, int N>
__device__ __forceinline__ void store_left(gdst p, const u32 (&w)[N], int left)
{
#pragma unroll
    for (int c = 0; c < 4 * N / ES; ++c)
        if (c < left) {
            if constexpr (ES == 1)
                p[c] = (uint8_t)(w[c / 4] >> (8 * (c % 4)));
            else if constexpr (ES == 2)
                *reinterpret_cast<BAND_G uint16_t *>(p + 2 * c) = (uint16_t)(w[c / 2] >> (16 * (c % 2)));
            else
                *reinterpret_cast<BAND_G u32 *>(p + 4 * c) = w[c];
        }
}

// One lane's share of a wave: all steps of its tile.  DIR: the job may also
// ask for the responses themselves (directional planes) and do without the
// magnitude; the planes are int16 (kPlanes16), int32 (kPlanes32) or what the
// job says, none included (kPlanesAny).
constexpr int kPlanes16 = 1, kPlanes32 = 2, kPlanesAny = 3;

template <int NB, int NR, int MODE, bool CLAMP, int DIR, int TO>
__device__ __forceinline__ void band_sweep(const U8Job &J, const BandTile &t, int off, int bm, const BandTaps &T)
{
    constexpr int NC = 4 * NB;
    constexpr bool AHEAD = MODE != kNarrow;                    // two quads in flight; narrow images are small
    using Source = BandSource<NB, MODE>;
    Source src;
    src.init(J, t, off, bm);
    u32 raw[2][Source::kRaw];
    v4i B[NB + 1];   // windows (word b, word b + 1), of the quad in even and the one in odd place
    auto place = [&](const u32 (&d)[Source::kRaw], auto half) __attribute__((always_inline)) {
        constexpr int h = decltype(half)::value;
        u32 e[Source::kWords];
        src.words(d, e);
#pragma unroll
        for (int b = 0; b <= NB; ++b) B[b][2 * h] = (int)e[b], B[b][2 * h + 1] = (int)e[b + 1];
    };
    BandA<NR> A;
    if constexpr (AHEAD) {
        src.load(raw[0]);
        src.load(raw[1]);
        band_weights<NR>(T, A);   // while the first rows travel
        place(raw[0], std::integral_constant<int, 0>{});
        src.load(raw[0]);
    } else {
        band_weights<NR>(T, A);
        src.load(raw[0]);
        place(raw[0], std::integral_constant<int, 0>{});
    }

    const int g = (threadIdx.x >> 4) & 3;
    int yo = t.yo + g;
    gdst mag = (gdst)J.mag + (int64_t)yo * J.mag_pitch + t.xo;
    int64_t plane = DIR ? (int64_t)yo * J.dir_pitch + (int64_t)t.xo * (2 * J.dir_type) : 0;
    const int left = J.Wo - t.xo;
    auto step = [&](auto par) __attribute__((always_inline)) {
        constexpr int P = decltype(par)::value;
        u32(&d)[Source::kRaw] = raw[AHEAD ? P ^ 1 : 0];
        if constexpr (!AHEAD) src.load(d);
        place(d, std::integral_constant<int, P ^ 1>{});
        if constexpr (AHEAD) src.load(d);
        // the products of a block are issued ahead of the squares of the one before
        v4i D[2][NR];
        auto products = [&](int b) __attribute__((always_inline)) {
#pragma unroll
            for (int p = 0; p < NR; ++p)
                D[b & 1][p] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A.w[P][p], B[b + (p >= NR / 2)], v4i{0, 0, 0, 0}, 0, 0, 0);
        };
        u32 m[NB];
        u32 s16[NR][2 * NB], s32[NR][4 * NB];
        products(0);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (b + 1 < NB) products(b + 1);
            int G[4][NR];
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int f = 0; f < NR; ++f) G[c][f] = D[b & 1][c * NR / 4][(c * NR + f) & 3];
            m[b] = 0;
            if (!DIR || J.mag) {
#pragma unroll
                for (int c = 0; c < 4; ++c) m[b] = mag_byte(sum_squares<NR, CLAMP>(G[c]), c, m[b]);
            }
            if constexpr (DIR) {
#pragma unroll
                for (int f = 0; f < NR; ++f) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) s32[f][4 * b + c] = (u32)G[c][f];
                    s16[f][2 * b] = __builtin_amdgcn_perm((u32)G[1][f], (u32)G[0][f], 0x05040100u);
                    s16[f][2 * b + 1] = __builtin_amdgcn_perm((u32)G[3][f], (u32)G[2][f], 0x05040100u);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (Source::kWhole || yo < J.Ho) {
            const bool full = MODE != kNarrow || left >= NC;
            if (!DIR || J.mag) {
                if (full)
                    store_words<TO>(mag, m);
                else
                    store_left<1>(mag, m, left);
            }
            if constexpr (DIR) {
                // the two-directional operators fill planes 0 and 2
#pragma unroll
                for (int f = 0; f < NR; ++f) {
                    gdst p = (gdst)J.dir[f * 4 / NR] + plane;
                    if ((DIR & kPlanes16) && (DIR != kPlanesAny || J.dir_type == 1)) {
                        if (full)
                            store_words<TO>(p, s16[f]);
                        else
                            store_left<2>(p, s16[f], left);
                    } else if ((DIR & kPlanes32) && (DIR != kPlanesAny || J.dir_type == 2)) {
                        if (full)
                            store_words<TO>(p, s32[f]);
                        else
                            store_left<4>(p, s32[f], left);
                    }
                }
            }
        }
        if (DIR) plane += 4 * J.dir_pitch;
        yo += 4;
        mag += 4 * J.mag_pitch;
    };
    // the first two steps stand before the loop: the loop then starts with the
    // loads and stores in flight that it also ends with, and its waits leave
    // them all out
    int k = t.steps;
    if (AHEAD && k >= 2) {
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
        for (k -= 2; k >= 2; k -= 2) {
            step(std::integral_constant<int, 0>{});
            step(std::integral_constant<int, 1>{});
        }
    }
    if constexpr (!AHEAD) {
        for (; k >= 2; k -= 2) {
            step(std::integral_constant<int, 0>{});
            step(std::integral_constant<int, 1>{});
        }
    }
    if (k > 0) step(std::integral_constant<int, 0>{});
}

// Tile `id` of an image's tile grid: J.nt tile columns of 4 NB pixels, bands
// of bq steps.
template <int NB>
__device__ __forceinline__ BandTile band_tile(const U8Job &J, u32 id, int bq)
{
    BandTile t;
    u32 band = __umulhi(id, J.inv_nt), tx = id - band * J.nt;   // at most one short
    if (tx >= J.nt) ++band, tx -= J.nt;
    // a tile beyond the last one that fits ends at the edge (nt may be rounded up)
    t.xo = min((int)(tx * 4 * NB), max(J.Wo - 4 * NB, 0));
    t.yo = 4 * bq * (int)band;
    // tiles of the last band are shorter; a wave that starts above it runs
    // whole bands and its rows past the image are not stored
    t.steps = __builtin_amdgcn_readfirstlane(min(bq, (J.Ho + 3 - t.yo) / 4));
    return t;
}

template <int NB, int NR, bool CLAMP, int DIR, int TO>
__device__ __forceinline__ void band_run(const U8Job &J, const BandTile &t, int off, int bm, const BandTaps &T)
{
    const int x = t.xo + off - 4, y = t.yo + off - 2;
    auto all = [](bool v) { return __builtin_amdgcn_ballot_w64(v) == ~0ull; };
    const bool rows_in = all(y >= 0 && y + 4 * (t.steps + 1) <= J.H && t.yo + 4 * t.steps <= J.Ho);
    const bool cols_in = all(x >= 0 && x + 4 * NB + 8 <= J.W && J.Wo >= 4 * NB);
    const bool word = all((((u32)(uintptr_t)J.src + (u32)x) & 3) == 0) && (J.src_pitch & 3) == 0;
    if (rows_in && cols_in && word)
        band_sweep<NB, NR, kInside, CLAMP, DIR, TO>(J, t, off, bm, T);
    else if (rows_in && cols_in)
        band_sweep<NB, NR, kShift, CLAMP, DIR, TO>(J, t, off, bm, T);
    else if (rows_in && J.Wo >= 4 * NB)
        band_sweep<NB, NR, kCols, CLAMP, DIR, TO>(J, t, off, bm, T);
    else if (J.Wo >= 4 * NB)
        band_sweep<NB, NR, kEdge, CLAMP, DIR, TO>(J, t, off, bm, T);
    else
        band_sweep<NB, NR, kNarrow, CLAMP, DIR, TO>(J, t, off, bm, T);
}

struct BandGrid {
    u32 tiles;       // tiles of the image
    int bq;          // steps of a band
    int off, bm;     // output (0, 0) is centred at input (off, off); border rule
};

// Workgroup b runs on XCD b mod 8: each XCD takes one of eight contiguous
// stretches of the grid, so the lines that neighbours share meet in one L2.
__device__ __forceinline__ u32 band_workgroup(u32 b, u32 groups)
{
    const u32 per = groups / 8;
    return b < 8 * per ? (b & 7) * per + b / 8 : b;
}

template <int NB, int NR, bool CLAMP, int DIR, int TO>
__global__ __launch_bounds__(64 * kBandWaves) __attribute__((amdgpu_waves_per_eu(DIR ? 3 : 4, 4))) void k_band_single(
    const U8Job J, const BandTaps T, const BandGrid gr)
{
    const u32 wave = band_workgroup(blockIdx.x, gridDim.x) * kBandWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const u32 id = min(16 * wave + (threadIdx.x & 15), gr.tiles - 1);
    const BandTile t = band_tile<NB>(J, id, gr.bq);
    if (16 * wave >= gr.tiles) return;
    band_run<NB, NR, CLAMP, DIR, TO>(J, t, gr.off, gr.bm, T);
}

// Batch of images: wave-tile t of the host-built table is {image, first tile,
// steps of a band, tiles of the image}.  With queue == nullptr the grid holds
// one wave for each (static form).  Otherwise a persistent grid draws them
// from queue[0] until none are left; each wave then counts itself out in
// queue[1], and the last one resets both words for the next launch.  claims
// (debug launches only, else nullptr): one counter per wave-tile, plus one
// for every time a wave takes it, so a launch that leaves any counter other
// than 1 has skipped or repeated one.
template <int NB, int DIR, int TO>
__global__ __launch_bounds__(64 * kBandWaves) __attribute__((amdgpu_waves_per_eu(DIR ? 3 : 4, 4))) void k_band_batched(
    const U8Job *__restrict__ jobs, const int4 *__restrict__ table, int32_t total, uint32_t *queue, uint32_t *claims,
    const BandTaps T, int off, int bm)
{
    for (;;) {
        int t;
        if (queue == nullptr) {
            t = (int)band_workgroup(blockIdx.x, gridDim.x) * kBandWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        } else {
            u32 tv = 0;
            if ((threadIdx.x & 63) == 0) tv = atomicAdd(&queue[0], 1u);
            t = __builtin_amdgcn_readfirstlane((int)tv);
        }
        if (t >= total) break;
        const int4 e = table[t];
        const U8Job J = jobs[e.x];
        if (claims != nullptr && (threadIdx.x & 63) == 0) atomicAdd(&claims[t], 1u);
        const BandTile tile = band_tile<NB>(J, min((u32)e.y + (threadIdx.x & 15), (u32)e.w - 1), e.z);
        band_run<NB, 4, false, DIR, TO>(J, tile, off, bm, T);
        if (queue == nullptr) break;
    }
    if (queue == nullptr) return;
    const int lane = threadIdx.x & 63;
    if (lane == 0) {
        __threadfence();
        const u32 nwaves = gridDim.x * kBandWaves;
        if (atomicAdd(&queue[1], 1u) == nwaves - 1) {
            queue[0] = 0;
            queue[1] = 0;
            __threadfence();
        }
    }
}

// A small batch of magnitudes in the kernel's arguments: no table to upload, to
// keep or to wait for.  Wave w of the grid belongs to the last image whose
// first wave is not beyond it.
struct BandImage {
    const uint8_t *src;
    uint8_t *mag;
    int64_t src_pitch, mag_pitch;
    int32_t W, H;
    u32 nt, inv_nt, tiles;
};
struct BandImages {
    BandImage img[kBatchArgs];
    u32 first[64];      // first wave of each image, ~0 beyond the last one
};

// (256 bytes of the 4 KB of arguments belong to the runtime)
static_assert(kBatchArgs < 64 && sizeof(BandImages) + sizeof(BandTaps) + 4 * sizeof(u32) + 256 <= 4096,
              "one lane an image, and a kernel's arguments");

template <int TO>
__global__ __launch_bounds__(64 * kBandWaves) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_band_args(
    const BandImages B, const BandTaps T, u32 waves, int bq, int off, int bm)
{
    const u32 w = band_workgroup(blockIdx.x, gridDim.x) * kBandWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const u64 at = __builtin_amdgcn_ballot_w64(B.first[threadIdx.x & 63] <= w);
    const int i = __builtin_popcountll(at) - 1;   // first[0] is 0
    const BandImage &I = B.img[i];
    U8Job J{};
    J.src = I.src;
    J.mag = I.mag;
    J.src_pitch = I.src_pitch;
    J.mag_pitch = I.mag_pitch;
    J.W = I.W;
    J.H = I.H;
    J.Wo = I.W - 2 * off;
    J.Ho = I.H - 2 * off;
    J.nt = I.nt;
    J.inv_nt = I.inv_nt;
    const BandTile t = band_tile<4>(J, min(16 * (w - B.first[i]) + (threadIdx.x & 15), I.tiles - 1), bq);
    if (w >= waves) return;
    band_run<4, 4, false, 0, TO>(J, t, off, bm, T);
}

}  // namespace
}  // namespace s4x5
