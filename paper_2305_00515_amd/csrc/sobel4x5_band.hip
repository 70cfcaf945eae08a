// Launches of the banded matrix-core kernels (u8_band.hpp).

#include "u8_band.hpp"

#include <algorithm>
#include <atomic>
#include <mutex>

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

template <int NB, int DIR>
const void *batched_fn(int kind)
{
    return kind == OutputStores::kToCache    ? reinterpret_cast<const void *>(&k_band_batched<NB, DIR, 1>)
           : kind == OutputStores::kToMemory ? reinterpret_cast<const void *>(&k_band_batched<NB, DIR, 2>)
                                             : reinterpret_cast<const void *>(&k_band_batched<NB, DIR, 0>);
}
const void *batched_fn(const U8Shape &s, int kind, bool dir)
{
    return !dir ? batched_fn<4, 0>(kind) : s.ppl == 4 ? batched_fn<1, kPlanesAny>(kind) : batched_fn<2, kPlanesAny>(kind);
}

int border_mode(int border) { return border == 2 ? kBandZero : border == 3 ? kBandRefl : kBandRep; }

template <int NB, int NR, bool CLAMP, int DIR, int TO>
hipError_t launch_band(const U8Job &j, const BandTaps &taps, int off, int border, int waves, hipStream_t st)
{
    if (j.Wo <= 0 || j.Ho <= 0) return hipSuccess;
    U8Job job = j;
    u8_tile(job, U8Shape{4 * NB, 0});
    const int64_t nq = ((int64_t)j.Ho + 3) / 4;
    const int bq = band_steps(job.nt, nq, waves > 0 ? waves : band_slots(), DIR != 0);
    const BandGrid g{(u32)(job.nt * ((nq + bq - 1) / bq)), bq, off, border_mode(border)};
    const u32 groups = (g.tiles + 16 * kBandWaves - 1) / (16 * kBandWaves);
    void *args[] = {&job, const_cast<BandTaps *>(&taps), const_cast<BandGrid *>(&g)};
    return hipLaunchKernel(reinterpret_cast<const void *>(&k_band_single<NB, NR, CLAMP, DIR, TO>), dim3(groups),
                           dim3(64 * kBandWaves), args, 0, st);
}

template <int NB, int NR, bool CLAMP, int DIR>
hipError_t launch_any(const U8Job &j, const BandTaps &taps, int off, int border, int waves, hipStream_t st)
{
    OutputStores o;
    o.add(j);
    switch (o.kind()) {
    case OutputStores::kToCache: return launch_band<NB, NR, CLAMP, DIR, 1>(j, taps, off, border, waves, st);
    case OutputStores::kToMemory: return launch_band<NB, NR, CLAMP, DIR, 2>(j, taps, off, border, waves, st);
    default: return launch_band<NB, NR, CLAMP, DIR, 0>(j, taps, off, border, waves, st);
    }
}

}  // namespace

void u8_tile(U8Job &j, const U8Shape &s)
{
    j.nt = tile_columns(j.Wo, s.ppl);
    j.inv_nt = (u32)std::min<uint64_t>((1ull << 32) / std::max<u32>(1, j.nt), 0xffffffffull);
}

hipError_t launch_u8_single(const U8Job &j, int border, const U8Shape &s, hipStream_t st)
{
    const int off = border == 1 ? 2 : 0;
    if (!j.dir_type) return launch_any<4, 4, false, 0>(j, kTaps4x5, off, border, s.waves, st);
    // planes: 16 bytes of a plane a lane, so that a wave's stores are whole
    // lines (int32 planes of 4096^2: 52.5 us, with two stores a lane 113)
    if (j.dir_type == 1) return launch_any<2, 4, false, kPlanes16>(j, kTaps4x5, off, border, s.waves, st);
    return launch_any<1, 4, false, kPlanes32>(j, kTaps4x5, off, border, s.waves, st);
}

hipError_t launch_u8_2dir(const U8Job &j, int op, int border, const U8Shape &s, hipStream_t st)
{
    const bool small = op == 2;
    const int off = border != 1 ? 0 : small ? 1 : 2;
    const BandTaps &taps = small ? kTaps2x3 : kTaps2x5;
    if (!j.dir_type) return launch_any<4, 2, false, 0>(j, taps, off, border, s.waves, st);
    if (j.dir_type == 1) return launch_any<2, 2, false, kPlanes16>(j, taps, off, border, s.waves, st);
    return launch_any<1, 2, false, kPlanes32>(j, taps, off, border, s.waves, st);
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
    if (j.dir_type == 1) return launch_any<2, 4, false, kPlanes16>(j, taps, off, border, waves, st);   // sums <= 128
    if (j.dir_type == 2)
        return clamp ? launch_any<1, 4, true, kPlanes32>(j, taps, off, border, waves, st)
                     : launch_any<1, 4, false, kPlanes32>(j, taps, off, border, waves, st);
    return clamp ? launch_any<4, 4, true, 0>(j, taps, off, border, waves, st)
                 : launch_any<4, 4, false, 0>(j, taps, off, border, waves, st);
}

hipError_t launch_u8_batched(const U8Job *jobs, const int4 *tiles, int32_t total, uint32_t *queue, int border, int kind,
                             bool dir, const U8Shape &s, int grid, hipStream_t st, uint32_t *claims)
{
    int off = border == 1 ? 2 : 0, bm = border_mode(border);
    if (!tiles) {
        BandImages b;
        int64_t waves = 0;
        for (int32_t i = 0; i < 64; ++i) {
            b.first[i] = i < total ? (u32)waves : 0xffffffffu;
            if (i >= total) continue;
            const U8Job &j = jobs[i];
            b.img[i] = BandImage{j.src, j.mag, j.src_pitch, j.mag_pitch, j.W, j.H, j.nt, j.inv_nt,
                                 (u32)batched_image_tiles(j, s.th)};
            waves += batched_count(j, s.th);
        }
        u32 w = (u32)waves;
        int bq = s.th / 4;
        void *args[] = {(void *)&b, const_cast<BandTaps *>(&kTaps4x5), (void *)&w, (void *)&bq, (void *)&off, (void *)&bm};
        const void *fn = kind == OutputStores::kToCache    ? reinterpret_cast<const void *>(&k_band_args<1>)
                         : kind == OutputStores::kToMemory ? reinterpret_cast<const void *>(&k_band_args<2>)
                                                           : reinterpret_cast<const void *>(&k_band_args<0>);
        return hipLaunchKernel(fn, dim3((w + kBandWaves - 1) / kBandWaves), dim3(64 * kBandWaves), args, 0, st);
    }
    void *args[] = {(void *)&jobs, (void *)&tiles, (void *)&total, (void *)&queue, (void *)&claims,
                    const_cast<BandTaps *>(&kTaps4x5), (void *)&off, (void *)&bm};
    return hipLaunchKernel(batched_fn(s, kind, dir), dim3(grid), dim3(64 * kBandWaves), args, 0, st);
}

int u8_persistent_grid(const U8Shape &s, int kind, bool dir)
{
    int dev = 0, ncu = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, batched_fn(s, kind, dir), 64 * kBandWaves, 0) != hipSuccess)
        return 0;
    if (per_cu < 1) per_cu = 1;
    return ncu * per_cu;
}

// The fixed buffer of the allocation-free batched call.  In host code this
// name is only a handle for hipGetSymbolAddress; kernels get the device
// address that call returns.
static __device__ __align__(256) unsigned char scratch[kNoallocBytes];

hipError_t noalloc_scratch(void **out)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        if ((e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch))) != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[dev] = p;
    }
    *out = addr[dev];
    return hipSuccess;
}

}  // namespace s4x5
