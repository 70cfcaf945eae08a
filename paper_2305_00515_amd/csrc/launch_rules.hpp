// Sizes of launches: how the row ranges, bands and tables of a call are cut.
// Plain integer code, shared by the launches and by a host-side check that
// enumerates sizes up to the largest that the entry points take.
#pragma once

#include <algorithm>
#include <cstdint>

namespace s4x5 {

// Every workgroup has four waves.  A launch has fewer than 2^32 work-items, in
// workgroups and in waves:
constexpr int kGroupWaves = 4;
constexpr int64_t kLaunchGroups = 0xffffffffll / (64 * kGroupWaves);
constexpr int64_t kLaunchWaves = kGroupWaves * kLaunchGroups;

// fp32: row ranges per strip, for a kernel of which `slots` waves are resident
// at once: as many as fill one round of them (rounding up would leave a few
// waves to run as a second, nearly empty round), of at least 4 rows, though a
// range costs 4 (forward) or 8 (adjoint) warm-up rows: small batches are bound
// by the serial steps of a wave (forward + adjoint of 1 x 256^2: 10.5 us at 4
// rows, 31.5 at 32; 8 x 512^2 23.7 and 33.7).  `most` rows at most: the forward
// of a large batch, which is bound by memory, runs several rounds that follow
// each other through the image (32 x 1024^2: 59.5 us at 16 rows, 67.0 in one
// round of 36); the adjoint, bound by its arithmetic, does not (one round of 73
// rows 105 us, 32 rows 107, 16 rows 113).  Never more waves than a launch holds.
inline int f32_ranges(int64_t slots, int64_t strips, int rows, int most)
{
    int64_t n = std::max<int64_t>(slots / strips, rows / most);
    n = std::min<int64_t>(n, std::min<int64_t>(rows / 4, kLaunchWaves / strips));
    return (int)std::max<int64_t>(1, n);
}

// Single uint8 image: steps (of four rows) of a wave's bands, for nt tile
// columns, nq quads of rows and `slots` resident waves of 16 tiles.
// (Times of calls back to back on one set of buffers.)
// - The fewest steps with which all waves are resident at once, as a wave that
//   waits for a slot starts with a trip to memory (4096^2 at 4 steps 8.1 us, at
//   2 9.1, at 1 11.2; 3840x2160 at 2 steps 5.9 us, at 1 7.2).  Above one step
//   an even number (the steps come in pairs: 4001x2999 7.0 us at 4 steps, 7.2
//   at 3).  At most 8 steps: larger images run several rounds, which hide each
//   other's first loads and end more evenly (4096^2 9.6 us at 16 steps and 29.7
//   at 64; 8192^2 25.0 at 8, 24.7 at 16 and 30.7 at 64).
// - With planes one step: the stores bound it, and many short waves store in
//   the order of memory (the four planes of 4096^2, int16, 23.1 us at 1 step,
//   23.6 at 2, 26.1 at 8; int32 46.6, 47.8, 49.7).
// More only where a launch would not hold the waves.
inline int band_steps(int64_t nt, int64_t nq, int64_t slots, bool planes)
{
    const int64_t bands = std::max<int64_t>(1, slots * 16 / nt);
    int64_t bq = planes ? 1 : (nq + bands - 1) / bands;
    if (bq > 1) bq = std::min<int64_t>((bq + 1) / 2 * 2, 8);
    while (nt * ((nq + bq - 1) / bq) > 16 * kLaunchWaves) bq *= 2;
    return (int)bq;
}

// Tile columns of an image of Wo columns, for tiles of ppl pixels.  Rows of
// tiles start at multiples of 8 tiles (128 bytes of magnitudes) where that adds
// at most a sixteenth of the tiles, so that a wave's bytes of a row are whole
// lines.
inline uint32_t tile_columns(int32_t Wo, int ppl)
{
    const int64_t nt = ((int64_t)Wo + ppl - 1) / ppl, whole = (nt + 7) / 8 * 8;
    return (uint32_t)((whole - nt) * 16 <= nt ? whole : nt);
}

// Batches: tiles of an image of j.nt tile columns and j.Ho rows in bands of th
// rows, and the wave-tiles (16 tiles) that hold them.
template <class Job>
int64_t batched_image_tiles(const Job &j, int th)
{
    return (int64_t)j.nt * (((int64_t)j.Ho + th - 1) / th);
}
template <class Job>
int64_t batched_count(const Job &j, int th)
{
    return (batched_image_tiles(j, th) + 15) / 16;
}

// The height of a batch's bands: `th`, doubled until the batch has at most
// `limit` wave-tiles and every image's tiles are numbered in 31 bits; 0 if that
// is not so even with one band an image.
template <class Job>
int batched_fit(const Job *jobs, int32_t count, int th, int64_t limit, int64_t *total)
{
    for (;; th *= 2) {
        int64_t most = 0;
        int32_t rows = 0;
        *total = 0;
        for (int32_t i = 0; i < count; ++i) {
            *total += batched_count(jobs[i], th);
            most = std::max(most, batched_image_tiles(jobs[i], th));
            rows = std::max(rows, jobs[i].Ho);
        }
        if (*total <= limit && most <= INT32_MAX) return th;
        if (th >= rows) return 0;
    }
}

// The unit in which the allocation-free call's public limit is counted: per
// image, strips of 512 columns in chunks of `tallx` * 32 rows, the last
// 1 / `shortq` of the rows in chunks of 32; the 128-column tiles that no whole
// strip holds in chunks of 128 rows.
struct BatchSplit {
    int tallx;
    int shortq;
};
inline int64_t budget_tiles(int32_t Wo, int32_t Ho, const BatchSplit &sp = BatchSplit{2, 4})
{
    const int64_t ntx = ((int64_t)Wo + 127) / 128, strips = ntx / 4, tall = 32 * sp.tallx;
    const int64_t rows = (Ho - Ho / sp.shortq) / tall * tall;
    return strips * (rows / tall + (Ho - rows + 31) / 32) + (ntx - 4 * strips) * (((int64_t)Ho + 127) / 128);
}

// Limits of the allocation-free batched call: images, tiles in that unit, and
// entries of the tile table (a wave-tile is half as wide as the budget's strip,
// and rows of tiles are rounded up by at most a sixteenth: a batch within the
// budget fits with one band an image at the latest).
constexpr int32_t kNoallocMaxImages = 1024;
constexpr int32_t kNoallocMaxTiles = 65536;
constexpr int32_t kNoallocTable = 2 * kNoallocMaxTiles + kNoallocMaxTiles / 4 + kNoallocMaxImages;

}  // namespace s4x5
