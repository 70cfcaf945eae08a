// Host-only check of what the C-ABI layer does while its stream is captured
// into a graph.  Linked with sobel4x5_api.cpp in place of the kernels and of
// the HIP runtime: "device" memory is host memory, and a launch is recorded.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../../include/sobel4x5.h"
#include "../../paper_2305_00515_amd/csrc/internal.hpp"

namespace {

bool capturing = false;
struct Launch {
    bool in_arguments;            // the images travel in the kernel's arguments
    int kind;                     // how outputs are stored
    std::vector<const uint8_t *> srcs;
};
std::vector<Launch> launches;
int copies = 0, allocations = 0, bad = 0;

#define CHECK(x) \
    do { \
        if (!(x)) { \
            std::printf("line %d: %s (%s)\n", __LINE__, #x, sobel4x5_last_error()); \
            bad = 1; \
        } \
    } while (0)

}  // namespace

namespace s4x5 {

void u8_tile(U8Job &j, const U8Shape &s)
{
    j.nt = (uint32_t)((j.Wo + s.ppl - 1) / s.ppl);
    j.inv_nt = 0;
}
hipError_t launch_u8_batched(const U8Job *jobs, const int4 *tiles, int32_t total, uint32_t *, int, int kind, bool,
                             const U8Shape &, int, hipStream_t, uint32_t *)
{
    Launch l{tiles == nullptr, kind, {}};
    for (int32_t i = 0; i < total; ++i) l.srcs.push_back(jobs[tiles ? tiles[i].x : i].src);
    launches.push_back(l);
    return hipSuccess;
}
hipError_t noalloc_scratch(void **p)
{
    static unsigned char buf[kNoallocBytes];
    *p = buf;
    return hipSuccess;
}
hipError_t launch_u8_single(const U8Job &, int, const U8Shape &, hipStream_t) { return hipErrorNoDevice; }
bool mfma_weights_fit(const int32_t *) { return false; }
hipError_t launch_u8_mfma_weighted(const U8Job &, int, const int32_t *, int, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_u8_2dir(const U8Job &, int, int, const U8Shape &, hipStream_t) { return hipErrorNoDevice; }
int u8_persistent_grid(const U8Shape &, int, bool) { return 0; }
hipError_t launch_u8_weighted(const WJob &, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_copy16(const void *, void *, int64_t, hipStream_t) { return hipErrorNoDevice; }
int64_t fingerprint_blocks(int64_t rows) { return rows; }
hipError_t launch_fingerprint(const void *, int64_t, int64_t, int64_t, uint64_t *, hipStream_t)
{
    return hipErrorNoDevice;
}
hipError_t launch_round_mag(const int32_t *, uint8_t *, int64_t, int, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_round_quad(const int16_t *, uint8_t *, int64_t, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_f32_fwd(const F32Args &, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_f32_bwd(const F32Args &, hipStream_t) { return hipErrorNoDevice; }

}  // namespace s4x5

// The runtime calls that the batched entry points make (the linker takes these
// before the runtime's own).
extern "C" {
hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n)
{
    ++allocations;
    return (*p = std::malloc(n)) ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p)
{
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind)
{
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    ++copies;
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s)
{
    *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
}

int main()
{
    const int n = 130, side = 8;
    std::vector<uint8_t> src(n * side * side), mag(n * side * side);
    std::vector<int16_t> planes(4 * n * side * side);
    std::vector<sobel4x5_image> imgs(n);
    std::vector<sobel4x5_outputs> outs(n);
    for (int i = 0; i < n; ++i) {
        imgs[i] = {&src[i * side * side], &mag[i * side * side], side, side, side, side};
        outs[i] = {};
        outs[i].dir_type = SOBEL4X5_DIR_S16;
        outs[i].dir_pitch = 2 * side;
        for (int k = 0; k < 4; ++k) outs[i].dir[k] = &planes[(4 * i + k) * side * side];
    }
    int stream_stands_here = 0;
    void *st = &stream_stands_here;

    // Batches that a cached plan serves: the cache may drop the plan while a
    // graph still holds its launch, so a captured call is refused, whether the
    // plan is there already or not, and takes nothing.
    for (int warm = 0; warm < 2; ++warm) {
        capturing = true;
        launches.clear();
        allocations = 0;
        CHECK(sobel4x5_batched(imgs.data(), 49, 0, st) == SOBEL4X5_EUNSUPPORTED);
        CHECK(sobel4x5_batched_ex(imgs.data(), outs.data(), 3, 0, st) == SOBEL4X5_EUNSUPPORTED);
        CHECK(launches.empty() && allocations == 0);
        CHECK(sobel4x5_batched(imgs.data(), 48, 0, st) == SOBEL4X5_OK);
        CHECK(launches.size() == 1 && launches[0].in_arguments && allocations == 0);
        capturing = false;
        CHECK(sobel4x5_batched(imgs.data(), 49, 0, st) == SOBEL4X5_OK);
        CHECK(sobel4x5_batched_ex(imgs.data(), outs.data(), 3, 0, st) == SOBEL4X5_OK);
        CHECK(launches.size() == 3 && !launches[1].in_arguments && !launches[2].in_arguments);
        allocations = 0;
    }

    // The allocation-free call: a graph must hold all that its launches read, so
    // that another batch in between changes nothing for a replay.
    for (int32_t count : {1, 48, 49, 130}) {
        capturing = true;
        launches.clear();
        copies = 0;
        CHECK(sobel4x5_batched_noalloc(imgs.data(), count, 0, st) == SOBEL4X5_OK);
        std::vector<const uint8_t *> seen;
        for (const Launch &l : launches) {
            CHECK(l.in_arguments && (int)l.srcs.size() <= s4x5::kBatchArgs);
            seen.insert(seen.end(), l.srcs.begin(), l.srcs.end());
        }
        CHECK(copies == 0 && allocations == 0);
        CHECK((int)seen.size() == count);
        for (int i = 0; i < (int)seen.size() && i < count; ++i) CHECK(seen[i] == imgs[i].src);
        capturing = false;
        launches.clear();
        CHECK(sobel4x5_batched_noalloc(imgs.data(), count, 0, st) == SOBEL4X5_OK);
        CHECK(launches.size() == 1 && !launches[0].in_arguments && allocations == 0);
    }

    // Outputs stay in the Infinity Cache up to 32 MiB.
    {
        std::vector<uint8_t> in((size_t)4096 * 8193), out((size_t)4096 * 8193 + 64);
        uint8_t *line = out.data() + (64 - (uintptr_t)out.data() % 64) % 64;
        for (int rows : {8192, 8193}) {
            const sobel4x5_image one = {in.data(), line, 4096, rows, 4096, 4096};
            launches.clear();
            CHECK(sobel4x5_batched(&one, 1, 0, st) == SOBEL4X5_OK && launches.size() == 1);
            CHECK(launches[0].kind == (rows == 8192 ? s4x5::OutputStores::kToCache : s4x5::OutputStores::kToMemory));
        }
    }

    if (bad) return 1;
    std::puts("capture checks ok");
    return 0;
}
