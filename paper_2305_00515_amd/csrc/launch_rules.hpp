// Sizes of launches: how the row ranges, bands and tables of a call are cut.
// Plain integer code, shared by the launches and by a host-side check that
// enumerates sizes up to the largest that the entry points take.
#pragma once

#include <algorithm>
#include <cstdint>

namespace s4x5 {

// A launch has fewer than 2^32 work-items: workgroups of four waves, and waves.
constexpr int64_t kLaunchGroups = 0xffffffffll / 256;
constexpr int64_t kLaunchWaves = 4 * kLaunchGroups;

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
// - The fewest steps with which all waves are resident at once, as a wave that
//   waits for a slot starts with a trip to memory (4096^2 at 4 steps 10.7 us,
//   at 2 12.1; 3840x2160 at 2 steps 6.9 us, at 1 8.5).  Above one step an
//   even number (the steps come in pairs: 4001x2999 9.1 us at 4 steps, 10.0
//   at 3).  At most 8 steps: larger images run several rounds, which hide
//   each other's first loads and end more evenly (16384^2: 103.6 us at 8
//   steps, 114.8 at 64; 8192^2: 25.8 at 8 and 25.7 at 16).
// - With planes one step: the stores bound it, and many short waves store in
//   the order of memory (4096^2 with int16 planes 24.6 us at 1 step, 27.8 at
//   2, 31.5 at 8; int32 52.5, 53.3, 55.0).
// More only where a launch would not hold the waves.
inline int band_steps(int64_t nt, int64_t nq, int64_t slots, bool planes)
{
    const int64_t bands = std::max<int64_t>(1, slots * 16 / nt);
    int64_t bq = planes ? 1 : (nq + bands - 1) / bands;
    if (bq > 1) bq = std::min<int64_t>((bq + 1) / 2 * 2, 8);
    while (nt * ((nq + bq - 1) / bq) > 16 * kLaunchWaves) bq *= 2;
    return (int)bq;
}

}  // namespace s4x5
