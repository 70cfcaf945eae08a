// Launches of the banded matrix-core kernels (u8_band.hpp).

#include "u8_band.hpp"

#include <algorithm>
#include <atomic>

namespace s4x5 {
namespace {

// Waves the current device holds at once (256 CUs if unknown).
int64_t band_slots()
{
    static std::atomic<int> cus[64];
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256 * kBandResident;
    n = cus[dev].load(std::memory_order_relaxed);
    if (n <= 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cus[dev].store(n, std::memory_order_relaxed);
    }
    return (int64_t)n * kBandResident;
}

// The tile grid of one image.
// - Rows of tiles start at multiples of 8 tiles (128 bytes of magnitudes)
//   where that adds at most a sixteenth of the tiles, so that a wave's 256
//   bytes of a row are whole lines.
// - Bands: the fewest steps with which all waves are resident at once, as a
//   wave that waits for a slot starts with a trip to memory (4096^2 at 4
//   steps 10.7 us, at 2 12.1; 3840x2160 at 2 steps 6.9 us, at 1 8.5).  Above
//   one step an even number (the steps come in pairs: 4001x2999 9.1 us at 4
//   steps, 10.0 at 3).  At most 8 steps: larger images run several rounds,
//   which hide each other's first loads and end more evenly (16384^2: 103.6
//   us at 8 steps, 114.8 at 64; 8192^2: 25.8 at 8 and 25.7 at 16).
// - With planes one step: the stores bound it, and many short waves store in
//   the order of memory (4096^2 with int16 planes 24.6 us at 1 step, 27.8 at
//   2, 31.5 at 8; int32 52.5, 53.3, 55.0).
template <int NB>
BandGrid band_grid(const U8Job &j, int off, int border, int64_t slots, bool planes)
{
    int64_t nt = (j.Wo + 4 * NB - 1) / (4 * NB);
    const int64_t nq = (j.Ho + 3) / 4, whole = (nt + 7) / 8 * 8;
    if ((whole - nt) * 16 <= nt) nt = whole;
    const int64_t bands = std::max<int64_t>(1, slots * 16 / nt);
    int64_t bq = (nq + bands - 1) / bands;
    if (planes)
        bq = 1;
    else if (bq > 1)
        bq = std::min<int64_t>((bq + 1) / 2 * 2, 8);
    while (nt * ((nq + bq - 1) / bq) > INT32_MAX) bq *= 2;   // tiles are numbered in 32 bits
    BandGrid g;
    g.nt = (u32)nt;
    g.inv_nt = (u32)std::min<uint64_t>((1ull << 32) / (uint64_t)nt, 0xffffffffull);
    g.tiles = (u32)(nt * ((nq + bq - 1) / bq));
    g.bq = (int)bq;
    g.off = off;
    g.bm = border == 2 ? kBandZero : border == 3 ? kBandRefl : kBandRep;
    return g;
}

template <int NB, int NR, bool CLAMP, int DIR>
hipError_t launch_band(const U8Job &j, const BandTaps &taps, int off, int border, int waves, hipStream_t st)
{
    if (j.Wo <= 0 || j.Ho <= 0) return hipSuccess;
    const BandGrid g = band_grid<NB>(j, off, border, waves > 0 ? waves : band_slots(), DIR != 0);
    const u32 groups = (g.tiles + 16 * kBandWaves - 1) / (16 * kBandWaves);
    void *args[] = {const_cast<U8Job *>(&j), const_cast<BandTaps *>(&taps), const_cast<BandGrid *>(&g)};
    return hipLaunchKernel(reinterpret_cast<const void *>(&k_band_single<NB, NR, CLAMP, DIR>), dim3(groups),
                           dim3(64 * kBandWaves), args, 0, st);
}

}  // namespace

hipError_t launch_u8_single(const U8Job &j, int border, const U8Shape &s, hipStream_t st)
{
    const int off = border == 1 ? 2 : 0;
    if (!j.dir_type) return launch_band<4, 4, false, 0>(j, kTaps4x5, off, border, s.waves, st);
    // planes: 16 bytes of a plane a lane, so that a wave's stores are whole
    // lines (int32 planes of 4096^2: 52.5 us, with two stores a lane 113)
    if (j.dir_type == 1) return launch_band<2, 4, false, kPlanes16>(j, kTaps4x5, off, border, s.waves, st);
    return launch_band<1, 4, false, kPlanes32>(j, kTaps4x5, off, border, s.waves, st);
}

hipError_t launch_u8_2dir(const U8Job &j, int op, int border, const U8Shape &s, hipStream_t st)
{
    const bool small = op == 2;
    const int off = border != 1 ? 0 : small ? 1 : 2;
    const BandTaps &taps = small ? kTaps2x3 : kTaps2x5;
    if (!j.dir_type) return launch_band<4, 2, false, 0>(j, taps, off, border, s.waves, st);
    if (j.dir_type == 1) return launch_band<2, 2, false, kPlanes16>(j, taps, off, border, s.waves, st);
    return launch_band<1, 2, false, kPlanes32>(j, taps, off, border, s.waves, st);
}

bool mfma_weights_fit(const int32_t *weights)
{
    for (int i = 0; i < 100; ++i)
        if (weights[i] < -128 || weights[i] > 127) return false;
    return true;
}

hipError_t launch_u8_mfma_weighted(const U8Job &j, int border, const int32_t *weights, int waves, hipStream_t st)
{
    struct Kernels {
        const int32_t *w;
        struct Kernel {
            const int32_t *k;
            const int32_t *operator[](int dy) const { return k + 5 * dy; }
        };
        Kernel operator[](int f) const { return {w + 25 * f}; }
    };
    const BandTaps taps = band_taps(Kernels{weights}, 4);
    // |G| is at most 255 times half the sum of |weights|; without the clamp,
    // four squares must stay below 2^31
    int64_t most = 0;
    for (int f = 0; f < 4; ++f) {
        int64_t sum = 0;
        for (int t = 0; t < 25; ++t) sum += weights[25 * f + t] < 0 ? -(int64_t)weights[25 * f + t] : weights[25 * f + t];
        most = std::max(most, sum);
    }
    const bool clamp = most > 181;
    const int off = border == 1 ? 2 : 0;
    if (j.dir_type == 1) return launch_band<2, 4, false, kPlanes16>(j, taps, off, border, waves, st);   // sums <= 128
    if (j.dir_type == 2)
        return clamp ? launch_band<1, 4, true, kPlanes32>(j, taps, off, border, waves, st)
                     : launch_band<1, 4, false, kPlanes32>(j, taps, off, border, waves, st);
    return clamp ? launch_band<4, 4, true, 0>(j, taps, off, border, waves, st)
                 : launch_band<4, 4, false, 0>(j, taps, off, border, waves, st);
}

}  // namespace s4x5
