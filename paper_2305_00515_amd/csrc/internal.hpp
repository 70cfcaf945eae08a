// Internal declarations shared by the C-ABI layer (sobel4x5_api.cpp) and the
// HIP kernel translation units.  Not part of the public interface.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "launch_rules.hpp"

namespace s4x5 {

// One uint8 image as the kernels see it.  Output pixel (yo, xo) is the
// operator centred on input pixel (yo + off, xo + off): off = 0 for the
// replicate border, the operator's radius (2, or 1 for the 3x3 pair) for the
// valid border.
struct U8Job {
    const uint8_t *src;
    uint8_t *mag;          // may be null
    void *dir[4];          // used iff dir_type != 0
    int64_t src_pitch;
    int64_t mag_pitch;
    int64_t dir_pitch;
    int32_t W, H;          // input size
    int32_t Wo, Ho;        // output size
    int32_t dir_type;      // 0 none, 1 int16, 2 int32
    uint32_t nt;           // tile columns (u8_tile)
    uint32_t inv_nt;       // floor(2^32 / nt), at most 2^32 - 1
};

// Shape of a launch.
struct U8Shape {
    int ppl;        // batched: pixels per lane (OutputStores::ppl)
    int th;         // batched: rows of a wave's tiles, a multiple of 4
    int waves = 0;  // single image: waves to launch (0 = by size); batched: kStaticGrid or a persistent grid
};

// Fills the tile columns of `j` for tiles of s.ppl pixels (tile_columns).
void u8_tile(U8Job &j, const U8Shape &s);

// How a launch's outputs are stored: through the L2, past it into the Infinity
// Cache (agent scope), or past both (nontemporal).  Measured on single images,
// and with a torch kernel that reads the outputs next:
// - Rows of whole 64-byte pieces: past the L2 (4096^2 int16 planes 24.6 us past
//   both, 40.5 through it).  Up to 32 MiB, an eighth of the Infinity Cache, the
//   outputs stay there for their reader (over many inputs, each converted to
//   float next: 2160x3840 22.4 us an image, 29.0 past both; 4096^2 37.7 and
//   50.0; 1080x1920 with int16 planes 37.3 and 39.8), which costs the call
//   nothing where its output memory is used again (2160x3840 6.49 and 6.66;
//   4096^2 9.98 and 10.2).  Larger ones are faster alone past both (a few
//   images in turn: 8192^2 24.8 and 28.2 us, 4096^2 with int16 planes 25.0 and
//   40.4), and a reader pays for it (8192^2 converted to float 193 and 159).
// - Other rows, whose ends share lines with a neighbouring wave: planes
//   through the L2 (4096 x 4104 int16 39.7 us, past both 51.0), magnitudes past
//   it up to 128 MiB, half of what the Infinity Cache holds to put the pieces
//   together (8193 x 8192 29.3 us, through the L2 35.6; 11001 x 11000 49.6 and
//   59.0; 12001 x 12000 74.5 and 70.9; 15001 x 15000 121 and 104).
struct OutputStores {
    enum Kind { kThroughL2 = 0, kToCache = 1, kToMemory = 2 };
    bool planes = false, whole = true, s32 = true;
    int64_t pixels = 0, bytes = 0;
    void add(const U8Job &j)
    {
        uint64_t low = 0;
        if (j.mag) low |= reinterpret_cast<uintptr_t>(j.mag) | (uint64_t)j.mag_pitch;
        if (j.dir_type) {
            planes = true;
            s32 = s32 && j.dir_type == 2;
            low |= (uint64_t)j.dir_pitch;
            for (const void *d : j.dir) low |= reinterpret_cast<uintptr_t>(d);
        }
        whole = whole && (low & 63) == 0;
        int64_t each = j.mag != nullptr;
        for (const void *d : j.dir) each += j.dir_type && d ? 2 * j.dir_type : 0;
        pixels += (int64_t)j.Wo * j.Ho;
        bytes += (int64_t)j.Wo * j.Ho * each;
    }
    // Pixels of a batch's lane: 16 bytes of a magnitude row or of a plane's, so
    // that a wave's store covers whole pieces of lines (12 images of 1024^2 with
    // int32 planes 40.6 us, with two stores a lane and plane 90.8; 4 of 2048^2
    // 54.0 and 118.9).  int32 planes beside int16 ones take the int16 form.
    int ppl() const { return !planes ? 16 : s32 ? 4 : 8; }
    bool large() const { return pixels > ((int64_t)128 << 20); }
    Kind kind() const
    {
        if (!whole && (planes || large())) return kThroughL2;
        return bytes <= (int64_t)32 << 20 ? kToCache : kToMemory;
    }
};

// Single image: one launch of the banded matrix-core kernels (u8_band.hpp),
// magnitude and/or planes.  `border` is the public SOBEL4X5_BORDER_* code
// (replicate 0, valid 1, zero 2, reflect-101 3).
hipError_t launch_u8_single(const U8Job &j, int border, const U8Shape &s, hipStream_t stream);

// Four run-time kernels (HOST array of 4*25 int32, the layout of
// sobel4x5_u8_weighted, already validated) on the banded kernels, when every
// weight fits int8 (mfma_weights_fit).
bool mfma_weights_fit(const int32_t *weights);
hipError_t launch_u8_mfma_weighted(const U8Job &j, int border, const int32_t *weights, int waves, hipStream_t stream);

// The same for the two-directional operators: op 1 = the 0 / 90 deg filters of
// the 5x5 operator, op 2 = the 3x3 pair (VALID: output (0, 0) is centred at
// input (1, 1)).  The job's Wo, Ho are those of the operator's own border rule.
hipError_t launch_u8_2dir(const U8Job &j, int op, int border, const U8Shape &s, hipStream_t stream);

// Batched launch.  `jobs` (device) holds the images; `tiles` (device, `total`
// entries) lists every wave-tile of the batch (batched_tiles); `queue`
// (device, 2 words, zero before the first launch) is the work counter and
// the exit counter of a persistent grid, reset by the last wave to finish,
// or null for one wave per wave-tile.  `border`: the public code; `dir`: some
// job asks for directional planes, which s.ppl = 4 or 8 can write.  `claims` (device, `total` counters, or
// null): each wave-tile's counter gains one for every wave that takes it.
// `kind`: how outputs are stored (OutputStores).
// tiles == nullptr: `jobs` is a HOST array of `total` <= kBatchArgs images,
// magnitudes only, tiled for bands of s.th rows; they go into the kernel's
// arguments (`queue`, `grid` and `claims` are not looked at).  48 images take
// 2.9 KB of the 4 KB of a kernel's arguments; 60 would be the most.
constexpr int32_t kBatchArgs = 48;
hipError_t launch_u8_batched(const U8Job *jobs, const int4 *tiles, int32_t total, uint32_t *queue, int border,
                             int kind, bool dir, const U8Shape &s, int grid, hipStream_t stream,
                             uint32_t *claims = nullptr);

// Wave-tiles of image `img` (tiled by u8_tile): 16 consecutive tiles of its
// tile grid each, in bands of `th` rows, as {image, first tile, steps of four
// rows, tiles of the image}.
template <class Push>
void batched_tiles_each(const U8Job &j, int32_t img, int th, Push &&push)
{
    const int64_t tiles = batched_image_tiles(j, th);
    for (int64_t t = 0; t < tiles; t += 16) push(make_int4(img, (int)t, th / 4, (int)tiles));
}

// Allocation-free batched call (sobel4x5_batched_noalloc): the queue
// words, the job table and the tile table of one batch live in a fixed
// device buffer of kNoallocBytes per device, laid out as below.  The limits
// are the public SOBEL4X5_NOALLOC_MAX_* (launch_rules.hpp).
constexpr size_t kNoallocJobsOff = 256;   // bytes [0, 8): queue[0], queue[1]
constexpr size_t kNoallocTilesOff = (kNoallocJobsOff + sizeof(U8Job) * kNoallocMaxImages + 255) / 256 * 256;
constexpr size_t kNoallocBytes = kNoallocTilesOff + sizeof(int4) * kNoallocTable;

// Device address of this device's buffer (looked up once per device, with
// that device current).
hipError_t noalloc_scratch(void **out);

// Number of workgroups of the persistent kernel that fit on the device at
// once for shape `s` (occupancy x CUs), or 0 on error.
int u8_persistent_grid(const U8Shape &s, int kind, bool dir);

// uint8 operator with run-time weights (four integer kernels that are
// antisymmetric under a half turn), as coefficients of the 12 upper-half
// pair differences: coef[plane][t] = k_plane[i_t][j_t] with taps (0,0..4),
// (1,0..4), (2,0), (2,1).
struct WJob {
    const uint8_t *src;
    uint8_t *mag;          // may be null
    void *dir[4];          // used iff dir_type != 0
    int64_t src_pitch, mag_pitch, dir_pitch;
    int32_t W, H, Wo, Ho;
    int32_t off;           // 0 replicate / zero / reflect-101, 2 valid
    int32_t bmode;         // pixels outside the image: 0 nearest, 1 zero, 2 reflect-101
    int32_t dir_type;      // 0 none, 1 int16, 2 int32
    int32_t coef[4][12];
};
hipError_t launch_u8_weighted(const WJob &j, hipStream_t stream);

hipError_t launch_copy16(const void *src, void *dst, int64_t n16, hipStream_t stream);

// Fingerprint of one plane of `rows` rows of `row_bytes` bytes (device):
// fingerprint_blocks(rows) workgroup sums written to `partials` (device).
int64_t fingerprint_blocks(int64_t rows);
hipError_t launch_fingerprint(const void *base, int64_t pitch, int64_t row_bytes, int64_t rows, uint64_t *partials,
                              hipStream_t stream);
// method 0: the square-root rounding of the kernels; 1: an integer root
hipError_t launch_round_mag(const int32_t *S, uint8_t *out, int64_t n, int method, hipStream_t stream);
// The four-directional kernel's rounding of n int16 quadruples (E1, E2, Hp, Hm)
hipError_t launch_round_quad(const int16_t *q, uint8_t *out, int64_t n, hipStream_t stream);

// fp32 path (pointers and strides as in the public header).
struct F32Args {
    const float *src;
    int64_t src_pitch, src_bstride;       // bytes
    float *out;
    int64_t out_pitch, out_bstride;       // bytes
    const float *grad;                    // bwd only
    int64_t g_pitch, g_bstride;           // bytes
    int32_t B, W, H, Wo, Ho;
    int32_t off;                          // 0 replicate / zero / reflect-101, 2 valid
    int32_t bmode;                        // 0 clamp (replicate, valid), 1 zero, 2 reflect-101
};

hipError_t launch_f32_fwd(const F32Args &a, hipStream_t stream);
hipError_t launch_f32_bwd(const F32Args &a, hipStream_t stream);

}  // namespace s4x5
