// C-ABI layer of the four-directional 5x5 Sobel library: argument checks,
// tile-shape choice, launches, batched plans (hipGraph), autotuning.
#include "../../include/sobel4x5.h"

#include <algorithm>
#include <atomic>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <unordered_map>
#include <vector>

#include <sys/stat.h>

#include "internal.hpp"

using namespace s4x5;

namespace {

thread_local std::string g_last_error;

int fail(int code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    std::vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return code;
}

int ok()
{
    return SOBEL4X5_OK;
}

int hip_fail(hipError_t e, const char *what)
{
    return fail(SOBEL4X5_EHIP, "%s: %s", what, hipGetErrorString(e));
}

// Test hook (sobel4x5_debug_inject_failure): while armed with n > 0, the
// n-th HIP call that passes through guard() reports hipErrorUnknown in place
// of its own result, which exercises the error paths without a real runtime
// failure.  The call itself still ran (an enqueued copy is still queued).
std::atomic<int> g_inject{0};

hipError_t guard(hipError_t e)
{
    int n = g_inject.load(std::memory_order_relaxed);
    while (n > 0) {
        if (g_inject.compare_exchange_weak(n, n - 1, std::memory_order_relaxed)) return n == 1 ? hipErrorUnknown : e;
    }
    return e;
}

constexpr int64_t kMaxDim = 1 << 30;

// Output size of an operator of radius r (2 for the 5x5 filters, 1 for 3x3).
int out_dims_r(int32_t W, int32_t H, int32_t border, int r, int32_t *Wo, int32_t *Ho)
{
    if (border != SOBEL4X5_BORDER_REPLICATE && border != SOBEL4X5_BORDER_VALID && border != SOBEL4X5_BORDER_ZERO &&
        border != SOBEL4X5_BORDER_REFLECT101)
        return fail(SOBEL4X5_EINVAL, "border must be REPLICATE (0), VALID (1), ZERO (2) or REFLECT101 (3), got %d",
                    border);
    if (W < 1 || H < 1) return fail(SOBEL4X5_EINVAL, "width and height must be >= 1 (got %d x %d)", W, H);
    if (W > kMaxDim || H > kMaxDim) return fail(SOBEL4X5_EINVAL, "image too large");
    if (border == SOBEL4X5_BORDER_VALID) {
        if (W < 2 * r + 1 || H < 2 * r + 1)
            return fail(SOBEL4X5_EINVAL, "VALID border needs width and height >= %d (got %d x %d)", 2 * r + 1, W, H);
        *Wo = W - 2 * r;
        *Ho = H - 2 * r;
    } else {
        *Wo = W;
        *Ho = H;
    }
    return ok();
}

int out_dims(int32_t W, int32_t H, int32_t border, int32_t *Wo, int32_t *Ho)
{
    return out_dims_r(W, H, border, 2, Wo, Ho);
}

struct Range {
    uintptr_t lo, hi;   // [lo, hi)
};

Range span(const void *p, int64_t rows, int64_t pitch, int64_t row_bytes)
{
    const uintptr_t a = reinterpret_cast<uintptr_t>(p);
    return {a, a + (uintptr_t)((rows - 1) * pitch + row_bytes)};
}

bool overlap(Range a, Range b) { return a.lo < b.hi && b.lo < a.hi; }

int check_pitch(const char *name, int64_t pitch, int64_t row_bytes, int64_t rows)
{
    if (pitch < row_bytes)
        return fail(SOBEL4X5_EINVAL, "%s pitch %lld is smaller than a row (%lld bytes)", name,
                    (long long)pitch, (long long)row_bytes);
    if (rows > 0 && pitch > (INT64_MAX / 2) / rows) return fail(SOBEL4X5_EINVAL, "%s pitch overflows", name);
    return ok();
}

// Arguments of one uint8 image for operator `op` (SOBEL4X5_OP_*): the
// two-directional operators write directional planes 0 and 2 only.
int validate_u8(const uint8_t *src, int32_t W, int32_t H, int64_t pitch, int32_t border,
                const sobel4x5_outputs *out, int32_t *pWo, int32_t *pHo, int32_t op = SOBEL4X5_OP_4DIR_5X5)
{
    int32_t Wo, Ho;
    if (op != SOBEL4X5_OP_4DIR_5X5 && op != SOBEL4X5_OP_2DIR_5X5 && op != SOBEL4X5_OP_2DIR_3X3)
        return fail(SOBEL4X5_EINVAL, "op must be 0, 1 or 2, got %d", op);
    if (int rc = out_dims_r(W, H, border, op == SOBEL4X5_OP_2DIR_3X3 ? 1 : 2, &Wo, &Ho)) return rc;
    if (!src) return fail(SOBEL4X5_EINVAL, "src is NULL");
    if (!out) return fail(SOBEL4X5_EINVAL, "out is NULL");
    if (int rc = check_pitch("src", pitch, W, H)) return rc;
    if (out->dir_type != SOBEL4X5_DIR_NONE && out->dir_type != SOBEL4X5_DIR_S16 &&
        out->dir_type != SOBEL4X5_DIR_S32)
        return fail(SOBEL4X5_EINVAL, "dir_type must be 0, 1 or 2, got %d", out->dir_type);
    if (!out->mag && out->dir_type == SOBEL4X5_DIR_NONE)
        return fail(SOBEL4X5_EINVAL, "no output requested (mag is NULL and dir_type is NONE)");
    const Range rs = span(src, H, pitch, W);
    std::vector<Range> outs;
    if (out->mag) {
        if (int rc = check_pitch("mag", out->mag_pitch, Wo, Ho)) return rc;
        outs.push_back(span(out->mag, Ho, out->mag_pitch, Wo));
    }
    if (out->dir_type != SOBEL4X5_DIR_NONE) {
        const int64_t es = out->dir_type == SOBEL4X5_DIR_S16 ? 2 : 4;
        if (int rc = check_pitch("dir", out->dir_pitch, (int64_t)Wo * es, Ho)) return rc;
        if (out->dir_pitch % es) return fail(SOBEL4X5_EINVAL, "dir pitch must be a multiple of the element size");
        for (int k = 0; k < 4; ++k) {
            if (op != SOBEL4X5_OP_4DIR_5X5 && (k & 1)) continue;
            if (!out->dir[k]) return fail(SOBEL4X5_EINVAL, "dir[%d] is NULL", k);
            if (reinterpret_cast<uintptr_t>(out->dir[k]) % es)
                return fail(SOBEL4X5_EINVAL, "dir[%d] is not aligned to its element size", k);
            outs.push_back(span(out->dir[k], Ho, out->dir_pitch, (int64_t)Wo * es));
        }
    }
    for (size_t i = 0; i < outs.size(); ++i) {
        if (overlap(outs[i], rs)) return fail(SOBEL4X5_EINVAL, "an output overlaps src");
        for (size_t k = i + 1; k < outs.size(); ++k)
            if (overlap(outs[i], outs[k])) return fail(SOBEL4X5_EINVAL, "two outputs overlap");
    }
    *pWo = Wo;
    *pHo = Ho;
    return ok();
}

U8Job make_job(const uint8_t *src, int32_t W, int32_t H, int64_t pitch, int32_t Wo, int32_t Ho,
               uint8_t *mag, int64_t mag_pitch, const void *const dir[4], int64_t dir_pitch, int32_t dir_type)
{
    U8Job j;
    std::memset(&j, 0, sizeof j);
    j.src = src;
    j.mag = mag;
    for (int k = 0; k < 4; ++k) j.dir[k] = dir ? const_cast<void *>(dir[k]) : nullptr;
    j.src_pitch = pitch;
    j.mag_pitch = mag_pitch;
    j.dir_pitch = dir_pitch;
    j.W = W;
    j.H = H;
    j.Wo = Wo;
    j.Ho = Ho;
    j.dir_type = dir_type;
    return j;
}

int env_int(const char *name, int dflt)
{
    const char *v = std::getenv(name);
    if (!v || !*v) return dflt;
    char *end = nullptr;
    const long x = std::strtol(v, &end, 10);
    return (end && *end == 0 && x >= 0 && x < (1 << 30)) ? (int)x : dflt;
}

// U8Shape::waves of a batched plan that launches one wave per tile (static
// form, no work queue) instead of a persistent grid.
constexpr int kStaticGrid = 1 << 30;

// Shape of a single-image launch: by size, unless SOBEL4X5_U8_WAVES (waves to
// launch) overrides it for tuning runs.
U8Shape single_shape()
{
    U8Shape s{};
    s.waves = env_int("SOBEL4X5_U8_WAVES", 0);
    return s;
}

// Border rule of the fp32 kernels: 0 reads the nearest pixel (REPLICATE,
// and VALID, whose taps stay inside), 1 ZERO, 2 REFLECT101.
int f32_bmode(int32_t border)
{
    return border == SOBEL4X5_BORDER_ZERO ? 1 : border == SOBEL4X5_BORDER_REFLECT101 ? 2 : 0;
}

// A batch of `batch` fp32 images of rows x cols, image b at p + b*bstride.
int check_f32_buf(const char *name, const float *p, int32_t batch, int32_t cols, int32_t rows, int64_t pitch,
                  int64_t bstride, Range *r)
{
    if (!p) return fail(SOBEL4X5_EINVAL, "%s is NULL", name);
    if ((reinterpret_cast<uintptr_t>(p) & 3u) || (pitch & 3) || (bstride & 3))
        return fail(SOBEL4X5_EINVAL, "%s: pointer, pitch and batch stride must be multiples of 4 bytes", name);
    if (int rc = check_pitch(name, pitch, (int64_t)cols * 4, rows)) return rc;
    const int64_t img = (int64_t)(rows - 1) * pitch + (int64_t)cols * 4;
    if (batch > 1 && bstride < img) return fail(SOBEL4X5_EINVAL, "%s batch stride is smaller than an image", name);
    if (batch > 1 && bstride > (INT64_MAX / 2) / batch) return fail(SOBEL4X5_EINVAL, "%s batch stride overflows", name);
    const uintptr_t a = reinterpret_cast<uintptr_t>(p);
    *r = {a, a + (uintptr_t)((batch > 0 ? batch - 1 : 0) * bstride + img)};
    return ok();
}

// Outputs of batch image i: outs[i] when given, else the image's own mag.
sobel4x5_outputs batch_outputs(const sobel4x5_image *imgs, const sobel4x5_outputs *outs, int32_t i)
{
    if (outs) return outs[i];
    sobel4x5_outputs o;
    std::memset(&o, 0, sizeof o);
    o.mag = imgs[i].mag;
    o.mag_pitch = imgs[i].mag_pitch;
    return o;
}

// Memory ranges every output of one image writes.
void output_ranges(const sobel4x5_outputs &o, int32_t Wo, int32_t Ho, std::vector<Range> &v)
{
    if (o.mag) v.push_back(span(o.mag, Ho, o.mag_pitch, Wo));
    if (o.dir_type != SOBEL4X5_DIR_NONE) {
        const int64_t es = o.dir_type == SOBEL4X5_DIR_S16 ? 2 : 4;
        for (int k = 0; k < 4; ++k) v.push_back(span(o.dir[k], Ho, o.dir_pitch, (int64_t)Wo * es));
    }
}

int validate_batch(const sobel4x5_image *imgs, const sobel4x5_outputs *outs_in, int32_t count, int32_t border)
{
    if (!imgs) return fail(SOBEL4X5_EINVAL, "imgs is NULL");
    if (count < 1) return fail(SOBEL4X5_EINVAL, "count must be >= 1 (got %d)", count);
    std::vector<Range> outs;
    for (int32_t i = 0; i < count; ++i) {
        const sobel4x5_image &m = imgs[i];
        const sobel4x5_outputs o = batch_outputs(imgs, outs_in, i);
        if (!outs_in && !m.mag) return fail(SOBEL4X5_EINVAL, "image %d: mag is NULL", i);
        int32_t Wo, Ho;
        if (validate_u8(m.src, m.width, m.height, m.src_pitch, border, &o, &Wo, &Ho))
            return fail(SOBEL4X5_EINVAL, "image %d: %s", i, g_last_error.c_str());
        output_ranges(o, Wo, Ho, outs);
    }
    // outputs of different images must not overlap each other (sorted sweep)
    std::sort(outs.begin(), outs.end(), [](const Range &a, const Range &b) { return a.lo < b.lo; });
    for (size_t i = 1; i < outs.size(); ++i)
        if (outs[i].lo < outs[i - 1].hi) return fail(SOBEL4X5_EINVAL, "outputs of two images overlap");
    // no output may overlap any input
    std::vector<Range> ins(count);
    for (int32_t i = 0; i < count; ++i) ins[i] = span(imgs[i].src, imgs[i].height, imgs[i].src_pitch, imgs[i].width);
    std::sort(ins.begin(), ins.end(), [](const Range &a, const Range &b) { return a.lo < b.lo; });
    for (const Range &o : outs) {
        auto it = std::upper_bound(ins.begin(), ins.end(), o.hi,
                                   [](uintptr_t v, const Range &r) { return v <= r.lo; });
        for (auto k = ins.begin(); k != it; ++k)
            if (overlap(*k, o)) return fail(SOBEL4X5_EINVAL, "an output overlaps an input");
    }
    return ok();
}

// ------------------------------------------------------------------ plans

constexpr uint32_t kPlanMagic = 0x534f4234u;   // "SOB4"

}  // namespace

struct sobel4x5_plan_s {
    uint32_t magic = kPlanMagic;
    int device = 0;
    int32_t count = 0;
    int32_t border = 0;
    U8Shape shape{};
    int grid = 0;
    bool use_graph = true;
    std::vector<sobel4x5_image> imgs;
    std::vector<sobel4x5_outputs> outs;   // per image: mag and/or directional planes
    bool dir = false;                     // some image asks for directional planes
    OutputStores stores;
    unsigned char *d_base = nullptr;   // the tables' device memory
    U8Job *d_jobs = nullptr;
    int4 *d_tiles = nullptr;      // wave-tiles, one per queue ticket (batched_tiles_each)
    int32_t total = 0;            // wave-tiles of the batch
    uint32_t *d_queue = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
};

namespace {

void plan_free_device(sobel4x5_plan_s *p)
{
    if (p->exec) hipGraphExecDestroy(p->exec);
    if (p->graph) hipGraphDestroy(p->graph);
    if (p->d_base) hipFree(p->d_base);
    p->exec = nullptr;
    p->graph = nullptr;
    p->d_base = nullptr;
}

U8Job plan_job(const sobel4x5_plan_s *p, int32_t i)
{
    const sobel4x5_image &m = p->imgs[i];
    const sobel4x5_outputs &o = p->outs[i];
    int32_t Wo, Ho;
    out_dims(m.width, m.height, p->border, &Wo, &Ho);
    return make_job(m.src, m.width, m.height, m.src_pitch, Wo, Ho, o.mag, o.mag_pitch, o.dir_type ? o.dir : nullptr,
                    o.dir_pitch, o.dir_type);
}

// Build device tables for `shape` (no graph): the queue words, the jobs and
// the wave-tiles in one allocation, uploaded by one copy.
int plan_setup(sobel4x5_plan_s *p, const U8Shape &shape)
{
    plan_free_device(p);
    p->shape = shape;
    std::vector<U8Job> jobs(p->count);
    for (int32_t i = 0; i < p->count; ++i) {
        jobs[i] = plan_job(p, i);
        u8_tile(jobs[i], shape);
    }
    int64_t total = 0;
    p->shape.th = batched_fit(jobs.data(), p->count, shape.th, shape.waves == kStaticGrid ? kLaunchWaves : INT32_MAX,
                              &total);
    if (!p->shape.th) return fail(SOBEL4X5_EINVAL, "batch too large for one plan");
    p->total = (int32_t)total;
    const size_t tiles_off = kNoallocJobsOff + (sizeof(U8Job) * p->count + 255) / 256 * 256;
    std::vector<unsigned char> host(tiles_off + sizeof(int4) * (size_t)total);
    std::memcpy(host.data() + kNoallocJobsOff, jobs.data(), sizeof(U8Job) * p->count);
    int4 *t = reinterpret_cast<int4 *>(host.data() + tiles_off);
    for (int32_t i = 0; i < p->count; ++i) batched_tiles_each(jobs[i], i, p->shape.th, [&](int4 e) { *t++ = e; });
    hipError_t e;
    if ((e = hipMalloc(&p->d_base, host.size())) != hipSuccess) {
        p->d_base = nullptr;
        return fail(SOBEL4X5_ENOMEM, "hipMalloc for plan tables: %s", hipGetErrorString(e));
    }
    if ((e = hipMemcpy(p->d_base, host.data(), host.size(), hipMemcpyHostToDevice)) != hipSuccess) {
        plan_free_device(p);
        return hip_fail(e, "uploading plan tables");
    }
    p->d_queue = reinterpret_cast<uint32_t *>(p->d_base);
    p->d_jobs = reinterpret_cast<U8Job *>(p->d_base + kNoallocJobsOff);
    p->d_tiles = reinterpret_cast<int4 *>(p->d_base + tiles_off);
    const int need = (int)(((int64_t)p->total + 3) / 4);   // never more workgroups than work (4 waves each)
    if (shape.waves == kStaticGrid) {       // one wave per wave-tile, no queue
        p->grid = std::max(1, need);
        return ok();
    }
    p->grid = u8_persistent_grid(shape, p->stores.kind(), p->dir);
    if (p->grid <= 0) {
        plan_free_device(p);
        return fail(SOBEL4X5_EHIP, "could not query occupancy");
    }
    p->grid = std::max(1, std::min(p->grid, need));
    return ok();
}

hipError_t plan_kernel(sobel4x5_plan_s *p, hipStream_t st, uint32_t *claims)
{
    uint32_t *queue = p->shape.waves == kStaticGrid ? nullptr : p->d_queue;
    return launch_u8_batched(p->d_jobs, p->d_tiles, p->total, queue, p->border, p->stores.kind(), p->dir, p->shape,
                             p->grid, st, claims);
}

int plan_direct_launch(sobel4x5_plan_s *p, hipStream_t st, uint32_t *claims = nullptr)
{
    hipError_t e = plan_kernel(p, st, claims);
    return e == hipSuccess ? ok() : hip_fail(e, "batched launch");
}

int plan_capture(sobel4x5_plan_s *p)
{
    hipStream_t st;
    hipError_t e = hipStreamCreateWithFlags(&st, hipStreamNonBlocking);
    if (e != hipSuccess) return hip_fail(e, "hipStreamCreate");
    int rc = ok();
    if ((e = hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal)) != hipSuccess) {
        rc = hip_fail(e, "hipStreamBeginCapture");
    } else {
        const int lrc = plan_direct_launch(p, st);
        hipGraph_t g = nullptr;
        e = hipStreamEndCapture(st, &g);
        if (lrc != SOBEL4X5_OK) {
            rc = lrc;
            if (g) hipGraphDestroy(g);
        } else if (e != hipSuccess) {
            rc = hip_fail(e, "hipStreamEndCapture");
        } else {
            p->graph = g;
            if ((e = hipGraphInstantiate(&p->exec, g, nullptr, nullptr, 0)) != hipSuccess)
                rc = hip_fail(e, "hipGraphInstantiate");
        }
    }
    hipStreamDestroy(st);
    return rc;
}

// Every output plane of image i: (device pointer, pitch, row bytes, rows).
struct Plane {
    void *p;
    int64_t pitch, row_bytes, rows;
};

std::vector<Plane> image_planes(const sobel4x5_plan_s *p, int32_t i)
{
    const sobel4x5_image &m = p->imgs[i];
    const sobel4x5_outputs &o = p->outs[i];
    int32_t Wo, Ho;
    out_dims(m.width, m.height, p->border, &Wo, &Ho);
    std::vector<Plane> v;
    if (o.mag) v.push_back({o.mag, o.mag_pitch, Wo, Ho});
    if (o.dir_type != SOBEL4X5_DIR_NONE) {
        const int64_t es = o.dir_type == SOBEL4X5_DIR_S16 ? 2 : 4;
        for (int k = 0; k < 4; ++k) v.push_back({o.dir[k], o.dir_pitch, Wo * es, Ho});
    }
    return v;
}

// 64-bit fingerprint of every output plane, used by the autotuner to check
// that a candidate shape reproduces the reference bytes: a device kernel sums
// a mix of (row, column, byte) per 16-row block, and the host folds the block
// sums of each plane in order.
int batch_fingerprint(const sobel4x5_plan_s *p, std::vector<uint64_t> &out)
{
    out.clear();
    int64_t most = 1;
    for (int32_t i = 0; i < p->count; ++i)
        for (const Plane &pl : image_planes(p, i)) most = std::max(most, fingerprint_blocks(pl.rows));
    uint64_t *d_part = nullptr;
    hipError_t e = hipMalloc(&d_part, sizeof(uint64_t) * most);
    if (e != hipSuccess) return fail(SOBEL4X5_ENOMEM, "hipMalloc for the autotuner's check: %s", hipGetErrorString(e));
    std::vector<uint64_t> part;
    int rc = ok();
    for (int32_t i = 0; i < p->count && rc == SOBEL4X5_OK; ++i)
        for (const Plane &pl : image_planes(p, i)) {
            const int64_t nb = fingerprint_blocks(pl.rows);
            part.assign(nb, 0);
            if ((e = launch_fingerprint(pl.p, pl.pitch, pl.row_bytes, pl.rows, d_part, nullptr)) != hipSuccess ||
                (e = hipMemcpy(part.data(), d_part, sizeof(uint64_t) * nb, hipMemcpyDeviceToHost)) != hipSuccess) {
                rc = hip_fail(e, "reading outputs for verification");
                break;
            }
            uint64_t h = 1469598103934665603ull;
            for (uint64_t v : part) h = (h ^ v) * 1099511628211ull;
            out.push_back(h);
        }
    hipFree(d_part);
    return rc;
}

double time_plan(sobel4x5_plan_s *p, int reps)
{
    hipEvent_t a, b;
    if (hipEventCreate(&a) != hipSuccess) return -1;
    if (hipEventCreate(&b) != hipSuccess) {
        hipEventDestroy(a);
        return -1;
    }
    // the best of `reps` rounds of four back-to-back launches (per launch):
    // candidates a few percent apart need more than single launches
    constexpr int kPerRound = 4;
    double best = 1e30;
    for (int r = 0; r < reps && best >= 0; ++r) {
        hipEventRecord(a, nullptr);
        for (int k = 0; k < kPerRound; ++k)
            if (plan_direct_launch(p, nullptr) != SOBEL4X5_OK) {
                best = -1;
                break;
            }
        hipEventRecord(b, nullptr);
        hipEventSynchronize(b);
        float ms = 0;
        hipEventElapsedTime(&ms, a, b);
        if (best >= 0) best = std::min(best, (double)ms / kPerRound);
    }
    hipEventDestroy(a);
    hipEventDestroy(b);
    return best;
}

std::string tune_cache_path()
{
    if (const char *e = std::getenv("SOBEL4X5_TUNE_CACHE")) return e;
    const char *home = std::getenv("HOME");
    return std::string(home ? home : "/tmp") + "/.cache/sobel4x5_tune.txt";
}

// Hash of the kernel sources the library was built from (set by the build):
// a tuned shape is only as good as the code it was timed and checked with.
#ifndef SOBEL4X5_KERNEL_HASH
#define SOBEL4X5_KERNEL_HASH 0ull
#endif

std::string tune_key(const sobel4x5_plan_s *p)
{
    hipDeviceProp_t prop;
    std::memset(&prop, 0, sizeof prop);
    hipGetDeviceProperties(&prop, p->device);
    // the key describes the workload shape, not the pointers: sizes, outputs
    // asked for, and what selects the kernel and the default shape
    uint64_t h = 1469598103934665603ull;
    auto mix = [&](uint64_t v) { h = (h ^ v) * 1099511628211ull; };
    int64_t px = 0;
    for (const auto &m : p->imgs) {
        mix((uint64_t)m.width);
        mix((uint64_t)m.height);
        px += (int64_t)m.width * m.height;
    }
    for (const auto &o : p->outs) mix(((uint64_t)(uint32_t)o.dir_type << 1) | (o.mag != nullptr));
    char buf[256];
    std::snprintf(buf, sizeof buf, "v%d|k%016llx|%s|b%d|d%d|s%d%d|n%d|px%lld|h%016llx", SOBEL4X5_VERSION,
                  (unsigned long long)(SOBEL4X5_KERNEL_HASH), prop.gcnArchName, p->border, (int)p->dir,
                  (int)p->stores.kind(), (int)p->stores.whole, p->count, (long long)px, (unsigned long long)h);
    std::string key = buf;
    for (char &c : key)
        if (c == ' ' || c == '\n') c = '_';
    return key;
}

bool tune_lookup(const std::string &key, U8Shape &s)
{
    FILE *f = std::fopen(tune_cache_path().c_str(), "r");
    if (!f) return false;
    // one entry a line: key ppl th wpg [static]; a line without the static
    // field is a persistent grid
    char line[1024], k[512];
    bool found = false;
    while (std::fgets(line, sizeof line, f)) {
        int ppl = 0, th = 0, wpg = 0, st = 0;
        const int n = std::sscanf(line, "%511s %d %d %d %d", k, &ppl, &th, &wpg, &st);
        if (n >= 4 && key == k && ppl == s.ppl && th >= 4 && th <= 256 && th % 4 == 0 && wpg == kGroupWaves &&
            (st == 0 || st == 1)) {
            s = U8Shape{ppl, th};
            if (n >= 5 && st == 1) s.waves = kStaticGrid;
            found = true;   // last entry wins
        }
    }
    std::fclose(f);
    return found;
}

void tune_store(const std::string &key, const U8Shape &s)
{
    const std::string path = tune_cache_path();
    const size_t slash = path.rfind('/');
    if (slash != std::string::npos && slash > 0) mkdir(path.substr(0, slash).c_str(), 0755);   // best effort
    FILE *f = std::fopen(path.c_str(), "a");
    if (!f) return;
    std::fprintf(f, "%s %d %d %d %d\n", key.c_str(), s.ppl, s.th, kGroupWaves, s.waves == kStaticGrid ? 1 : 0);
    std::fclose(f);
}

// Shape of a batch without autotuning: the static grid (a persistent grid
// loads ticket, table entry and job in series before each wave-tile's first
// row), and bands of
// - 16 rows for magnitudes, 32 in a large batch (256 images of 128..4096, 1182
//   Mpx: 527 us at 32 rows, 560 at 16; 64 of 2048^2: 117 and 126; but 12 of
//   2101^2: 36.2 and 34.6, 40 of 64..1080: 18.1 and 16.6);
// - 4 rows with directional planes, which are bound by their stores, or 8
//   where rows share lines (32 images of 128..4096 with int16 planes: 312 us
//   at 8 rows, 361 at 4 and at 16; int32: 4 of 2048^2 54.0 us at 4 rows, 57.5
//   at 8; 6 of 2999x3001 260 and 196).
// SOBEL4X5_BATCH_TH (4..256) and SOBEL4X5_BATCH_STATIC (0 or 1) override it.
U8Shape batch_default_shape(const OutputStores &o)
{
    U8Shape s{o.ppl(), o.planes ? (o.whole ? 4 : 8) : o.large() ? 32 : 16};
    s.waves = kStaticGrid;
    const int th = env_int("SOBEL4X5_BATCH_TH", 0);
    if (th >= 4 && th <= 256) s.th = th / 4 * 4;
    if (env_int("SOBEL4X5_BATCH_STATIC", -1) == 0) s.waves = 0;
    return s;
}

// Clear every output plane, so that a candidate that skips pixels cannot
// reproduce the reference bytes.
void clear_outputs(const sobel4x5_plan_s *p)
{
    for (int32_t i = 0; i < p->count; ++i)
        for (const Plane &pl : image_planes(p, i)) hipMemset2D(pl.p, pl.pitch, 0xA5, pl.row_bytes, pl.rows);
}

// Run shape c once on cleared outputs; true when its bytes equal `want`.
bool candidate_matches(sobel4x5_plan_s *p, const U8Shape &c, const std::vector<uint64_t> &want, int *rc)
{
    *rc = SOBEL4X5_OK;
    if (plan_setup(p, c) != SOBEL4X5_OK) return false;
    clear_outputs(p);
    if (plan_direct_launch(p, nullptr) != SOBEL4X5_OK) return false;
    if (hipDeviceSynchronize() != hipSuccess) {
        *rc = fail(SOBEL4X5_EHIP, "autotune candidate run failed");
        return false;
    }
    std::vector<uint64_t> got;
    return batch_fingerprint(p, got) == SOBEL4X5_OK && got == want;   // never trust a mismatch
}

int plan_autotune(sobel4x5_plan_s *p)
{
    const std::string key = tune_key(p);

    // reference bytes with the default shape
    const U8Shape ref = batch_default_shape(p->stores);
    if (int rc = plan_setup(p, ref)) return rc;
    if (int rc = plan_direct_launch(p, nullptr)) return rc;
    if (hipError_t e = hipDeviceSynchronize(); e != hipSuccess) return hip_fail(e, "autotune reference run");
    std::vector<uint64_t> want;
    if (int rc = batch_fingerprint(p, want)) return rc;

    // a cached shape is used only after it has reproduced the reference
    // bytes once on these images
    U8Shape cached = ref;
    if (tune_lookup(key, cached)) {
        int rc;
        if (candidate_matches(p, cached, want, &rc)) return ok();
        if (rc != SOBEL4X5_OK) return rc;
        if (int rc2 = plan_setup(p, ref)) return rc2;
    }

    U8Shape best = ref;
    double best_ms = time_plan(p, 10);
    const int ths[] = {8, 16, 32, 64, 128};
    for (int grid_form = 0; grid_form < 2; ++grid_form)   // persistent, static
        for (int th : ths) {
            U8Shape c{ref.ppl, th};
            if (grid_form == 1) c.waves = kStaticGrid;
            if (c.th == ref.th && c.waves == ref.waves) continue;
            int rc;
            if (!candidate_matches(p, c, want, &rc)) {
                if (rc != SOBEL4X5_OK) return rc;
                continue;
            }
            const double ms = time_plan(p, 10);
            if (ms > 0 && ms < best_ms) {
                best_ms = ms;
                best = c;
            }
        }
    tune_store(key, best);
    return plan_setup(p, best);
}

// --------------------------------------------------------- one-shot cache

struct CachedPlan {
    std::string key;
    sobel4x5_plan plan;
    hipStream_t stream;   // the only stream this plan is launched on
};

struct PlanCache {
    std::mutex mu;
    std::vector<CachedPlan> lru;   // most recent last
};

PlanCache &plan_cache()
{
    static PlanCache *c = new PlanCache();   // intentionally leaked: plans live to process end
    return *c;
}

// Whether `st` is being captured into a graph (the null stream cannot be; what
// is wrong with a stream that cannot be asked, the launch on it will say).
bool is_captured(hipStream_t st)
{
    hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
    if (st && hipStreamIsCapturing(st, &s) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return s != hipStreamCaptureStatusNone;
}

// Key of a one-shot batched call, from the descriptor fields one by one (not
// the structs' raw bytes, whose padding a C caller may leave uninitialised),
// the border, the device and the stream.  A plan's work queue admits one
// launch at a time, so every stream gets plans of its own; launches of one
// plan on one stream run in order.
std::string batch_key(const sobel4x5_image *imgs, const sobel4x5_outputs *outs, int32_t count, int32_t border,
                      int device, hipStream_t stream)
{
    std::string k;
    auto put = [&](uint64_t v) { k.append(reinterpret_cast<const char *>(&v), sizeof v); };
    put((uint64_t)(uint32_t)count);
    put((uint64_t)(uint32_t)border);
    put((uint64_t)(uint32_t)device);
    put((uint64_t)reinterpret_cast<uintptr_t>(stream));
    put(outs ? 1u : 0u);
    for (int32_t i = 0; i < count; ++i) {
        const sobel4x5_image &m = imgs[i];
        put((uint64_t)reinterpret_cast<uintptr_t>(m.src));
        put(((uint64_t)(uint32_t)m.width << 32) | (uint32_t)m.height);
        put((uint64_t)m.src_pitch);
        if (outs) {
            const sobel4x5_outputs &o = outs[i];
            put((uint64_t)reinterpret_cast<uintptr_t>(o.mag));
            put((uint64_t)o.mag_pitch);
            put((uint64_t)(uint32_t)o.dir_type);
            if (o.dir_type != SOBEL4X5_DIR_NONE) {
                for (int d = 0; d < 4; ++d) put((uint64_t)reinterpret_cast<uintptr_t>(o.dir[d]));
                put((uint64_t)o.dir_pitch);
            }
        } else {
            put((uint64_t)reinterpret_cast<uintptr_t>(m.mag));
            put((uint64_t)m.mag_pitch);
        }
    }
    return k;
}


// ------------------------------------------------------- host pipeline

// One in-flight image of a pipeline: device buffers (sized for the largest
// image), pinned staging buffers for callers whose host memory is pageable,
// and a stream of its own (default priority).
struct PipeSlot {
    hipStream_t st = nullptr;
    uint8_t *d_src = nullptr, *d_mag = nullptr;
    uint8_t *h_src = nullptr, *h_mag = nullptr;   // pinned staging
    int64_t pitch = 0;                            // device and staging row pitch
    int pending = -1;                             // image whose magnitudes are in flight
    bool staged_out = false;                      // D2H went to h_mag (copy on finish)
};

// true when p points to pinned (page-locked) host memory
bool is_pinned(const void *p)
{
    hipPointerAttribute_t a;
    if (hipPointerGetAttributes(&a, p) != hipSuccess) {
        (void)hipGetLastError();   // pageable memory is not an error here
        return false;
    }
    return a.type == hipMemoryTypeHost;
}

}  // namespace

struct sobel4x5_pipe_s {
    int32_t max_w = 0, max_h = 0;
    std::vector<PipeSlot> slots;
};

namespace {

void pipe_free(sobel4x5_pipe_s *p)
{
    for (auto &s : p->slots) {
        if (s.st) hipStreamSynchronize(s.st);
        if (s.d_src) hipFree(s.d_src);
        if (s.d_mag) hipFree(s.d_mag);
        if (s.h_src) hipHostFree(s.h_src);
        if (s.h_mag) hipHostFree(s.h_mag);
        if (s.st) hipStreamDestroy(s.st);
        s = PipeSlot{};
    }
}

// Rows that lie back to back are copied as rows of whole words: one, two or
// four of them at a time.
int rows_per_word_row(int64_t w) { return w % 4 == 0 ? 1 : w % 2 == 0 ? 2 : 4; }

// Rows in page-locked memory are copied from where they lie if their pitch is
// of whole words or they lie back to back.  (A pitched copy of whole words is
// one fast transfer; of any other pitch it goes row by row.  4 images of 896
// rows out: 154 us a run for 733 bytes at a pitch of 736, 23.6 ms at 733 or
// 734, 265 through the staging buffer.  A plain copy is slower than a pitched
// one: 239 against 154 for 736 bytes back to back.)  Rows left over take a
// second transfer, which a small image does not win back (3 of 301x301: 89 us
// against 69 staged; 4 of 401x701: 137 against 150).
bool pipe_direct(const void *p, int64_t pitch, int32_t w, int32_t h)
{
    if (pitch % 4 != 0 && (pitch != w || (h % rows_per_word_row(w) != 0 && (int64_t)w * h < 256 << 10))) return false;
    return is_pinned(p);
}

// The device's pitch for such rows: its own, or back to back as they are.
int64_t pipe_pitch(const PipeSlot &s, int64_t pitch, int32_t w) { return pitch % 4 ? w : s.pitch; }

hipError_t pipe_copy(uint8_t *dst, int64_t dpitch, const uint8_t *src, int64_t spitch, int32_t w, int32_t h,
                     hipMemcpyKind kind, hipStream_t st)
{
    if (spitch % 4 == 0 && dpitch % 4 == 0) return hipMemcpy2DAsync(dst, dpitch, src, spitch, w, h, kind, st);
    const int k = rows_per_word_row(w);
    const size_t row = k * (size_t)w, rows = h / k, rest = (h % k) * (size_t)w;
    hipError_t e = hipSuccess;
    if (rows) e = hipMemcpy2DAsync(dst, row, src, row, row, rows, kind, st);
    if (rest && e == hipSuccess)
        e = hipMemcpy2DAsync(dst + row * rows, row, src + row * rows, row, rest, 1, kind, st);
    return e;
}

// Copy the magnitudes of the slot's finished image out of pinned staging.
void pipe_finish(PipeSlot &s, const sobel4x5_image *imgs, int32_t border)
{
    if (s.pending < 0) return;
    if (s.staged_out) {
        const sobel4x5_image &m = imgs[s.pending];
        int32_t Wo, Ho;
        out_dims(m.width, m.height, border, &Wo, &Ho);
        for (int32_t r = 0; r < Ho; ++r) std::memcpy(m.mag + r * m.mag_pitch, s.h_mag + r * s.pitch, (size_t)Wo);
    }
    s.pending = -1;
    s.staged_out = false;
}

}  // namespace

extern "C" {

const char *sobel4x5_status_string(int status)
{
    switch (status) {
    case SOBEL4X5_OK: return "ok";
    case SOBEL4X5_EINVAL: return "invalid argument";
    case SOBEL4X5_EUNSUPPORTED: return "unsupported request";
    case SOBEL4X5_EHIP: return "HIP runtime error";
    case SOBEL4X5_ENOMEM: return "out of memory";
    default: return "unknown status";
    }
}

const char *sobel4x5_last_error(void) { return g_last_error.c_str(); }

int sobel4x5_version(void) { return SOBEL4X5_VERSION; }

int sobel4x5_validate_u8(const uint8_t *src, int32_t width, int32_t height, int64_t src_pitch, int32_t border,
                         const sobel4x5_outputs *out)
{
    int32_t Wo, Ho;
    return validate_u8(src, width, height, src_pitch, border, out, &Wo, &Ho);
}

int sobel4x5_u8(const uint8_t *src, int32_t width, int32_t height, int64_t src_pitch, int32_t border,
                const sobel4x5_outputs *out, void *stream)
{
    int32_t Wo, Ho;
    if (int rc = validate_u8(src, width, height, src_pitch, border, out, &Wo, &Ho)) return rc;
    U8Job j = make_job(src, width, height, src_pitch, Wo, Ho, out->mag, out->mag_pitch,
                       out->dir_type ? out->dir : nullptr, out->dir_pitch, out->dir_type);
    hipError_t e = guard(launch_u8_single(j, border, single_shape(), static_cast<hipStream_t>(stream)));
    return e == hipSuccess ? ok() : hip_fail(e, "sobel4x5_u8 launch");
}

int sobel4x5_validate_u8_op(const uint8_t *src, int32_t width, int32_t height, int64_t src_pitch, int32_t op,
                            int32_t border, const sobel4x5_outputs *out)
{
    int32_t Wo, Ho;
    return validate_u8(src, width, height, src_pitch, border, out, &Wo, &Ho, op);
}

int sobel4x5_u8_op(const uint8_t *src, int32_t width, int32_t height, int64_t src_pitch, int32_t op,
                   int32_t border, const sobel4x5_outputs *out, void *stream)
{
    int32_t Wo, Ho;
    if (int rc = validate_u8(src, width, height, src_pitch, border, out, &Wo, &Ho, op)) return rc;
    if (op == SOBEL4X5_OP_4DIR_5X5) return sobel4x5_u8(src, width, height, src_pitch, border, out, stream);
    void *dirs[4] = {nullptr, nullptr, nullptr, nullptr};
    if (out->dir_type) {
        dirs[0] = out->dir[0];
        dirs[2] = out->dir[2];
    }
    U8Job j = make_job(src, width, height, src_pitch, Wo, Ho, out->mag, out->mag_pitch,
                       out->dir_type ? dirs : nullptr, out->dir_pitch, out->dir_type);
    hipError_t e = launch_u8_2dir(j, op, border, single_shape(), static_cast<hipStream_t>(stream));
    return e == hipSuccess ? ok() : hip_fail(e, "sobel4x5_u8_op launch");
}

int sobel4x5_validate_batch(const sobel4x5_image *imgs, int32_t count, int32_t border)
{
    return validate_batch(imgs, nullptr, count, border);
}

int sobel4x5_validate_batch_ex(const sobel4x5_image *imgs, const sobel4x5_outputs *outs, int32_t count,
                               int32_t border)
{
    return validate_batch(imgs, outs, count, border);
}

int sobel4x5_plan_create_ex(const sobel4x5_image *imgs, const sobel4x5_outputs *outs, int32_t count, int32_t border,
                            uint32_t flags, sobel4x5_plan *out)
{
    if (!out) return fail(SOBEL4X5_EINVAL, "out is NULL");
    *out = nullptr;
    if (int rc = validate_batch(imgs, outs, count, border)) return rc;
    if (flags & ~(SOBEL4X5_PLAN_AUTOTUNE | SOBEL4X5_PLAN_NO_GRAPH))
        return fail(SOBEL4X5_EINVAL, "unknown plan flags 0x%x", flags);
    auto *p = new (std::nothrow) sobel4x5_plan_s();
    if (!p) return fail(SOBEL4X5_ENOMEM, "plan allocation");
    p->count = count;
    p->border = border;
    p->use_graph = !(flags & SOBEL4X5_PLAN_NO_GRAPH);
    p->imgs.assign(imgs, imgs + count);
    p->outs.resize(count);
    for (int32_t i = 0; i < count; ++i) {
        p->outs[i] = batch_outputs(imgs, outs, i);
        p->dir = p->dir || p->outs[i].dir_type != SOBEL4X5_DIR_NONE;
        p->stores.add(plan_job(p, i));
    }
    hipGetDevice(&p->device);
    int rc = (flags & SOBEL4X5_PLAN_AUTOTUNE) ? plan_autotune(p) : plan_setup(p, batch_default_shape(p->stores));
    // A static grid is one kernel without state, and the plan launches it as
    // such: 16 images of 64..640 cost the caller 5.5 us a launch, 18.6 when
    // waited for, where a captured graph of it cost 13.2 and 35.9, and 140 us
    // more to build.  A plan with a work queue keeps the graph: its launches
    // share the queue words.
    p->use_graph = p->use_graph && p->shape.waves != kStaticGrid;
    if (rc == SOBEL4X5_OK && p->use_graph) rc = plan_capture(p);
    if (rc != SOBEL4X5_OK) {
        plan_free_device(p);
        p->magic = 0;
        delete p;
        return rc;
    }
    *out = p;
    return ok();
}

int sobel4x5_plan_create(const sobel4x5_image *imgs, int32_t count, int32_t border, uint32_t flags,
                         sobel4x5_plan *out)
{
    return sobel4x5_plan_create_ex(imgs, nullptr, count, border, flags, out);
}

int sobel4x5_plan_launch(sobel4x5_plan plan, void *stream)
{
    if (!plan || plan->magic != kPlanMagic) return fail(SOBEL4X5_EINVAL, "invalid plan handle");
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (plan->use_graph) {
        hipError_t e = guard(hipGraphLaunch(plan->exec, st));
        return e == hipSuccess ? ok() : hip_fail(e, "hipGraphLaunch");
    }
    // The stream may belong to the plan's device while another is current.
    int dev = plan->device;
    hipGetDevice(&dev);
    const bool other = st && dev != plan->device;
    if (other) hipSetDevice(plan->device);
    hipError_t e = guard(plan_kernel(plan, st, nullptr));
    if (other) hipSetDevice(dev);
    return e == hipSuccess ? ok() : hip_fail(e, "batched launch");
}

int sobel4x5_debug_plan_claims(sobel4x5_plan plan, uint32_t *claims, int64_t capacity, int64_t *ntiles, void *stream)
{
    if (!plan || plan->magic != kPlanMagic) return fail(SOBEL4X5_EINVAL, "invalid plan handle");
    if (!ntiles) return fail(SOBEL4X5_EINVAL, "ntiles is NULL");
    *ntiles = plan->total;
    if (!claims) return ok();
    if (capacity < plan->total)
        return fail(SOBEL4X5_EINVAL, "claims holds %lld counters, the plan has %d tiles", (long long)capacity,
                    plan->total);
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipError_t e = guard(hipMemsetAsync(claims, 0, sizeof(uint32_t) * (size_t)std::max<int32_t>(plan->total, 1), st));
    if (e != hipSuccess) return hip_fail(e, "clearing the claim counters");
    return plan_direct_launch(plan, st, claims);
}

int sobel4x5_plan_info(sobel4x5_plan plan, int32_t *px_per_lane, int32_t *rows_per_tile, int32_t *waves_per_group,
                       int32_t *grid)
{
    if (!plan || plan->magic != kPlanMagic) return fail(SOBEL4X5_EINVAL, "invalid plan handle");
    if (px_per_lane) *px_per_lane = plan->shape.ppl;
    if (rows_per_tile) *rows_per_tile = plan->shape.th;
    if (waves_per_group) *waves_per_group = kGroupWaves;
    if (grid) *grid = plan->grid;
    return ok();
}

int sobel4x5_plan_destroy(sobel4x5_plan plan)
{
    if (!plan || plan->magic != kPlanMagic) return fail(SOBEL4X5_EINVAL, "invalid plan handle");
    plan_free_device(plan);
    plan->magic = 0;
    delete plan;
    return ok();
}

int sobel4x5_batched_ex(const sobel4x5_image *imgs, const sobel4x5_outputs *outs, int32_t count, int32_t border,
                        void *stream)
{
    if (int rc = validate_batch(imgs, outs, count, border)) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // A few images' magnitudes: the images go into the kernel's arguments, and
    // the call keeps nothing.  (16 images of 64..640: 5 us a launch, where a
    // plan's look-up and launch take 9 and a new plan 100.)
    if (!outs && count <= kBatchArgs) {
        U8Job jobs[kBatchArgs];
        OutputStores stores;
        for (int32_t i = 0; i < count; ++i) {
            const sobel4x5_image &m = imgs[i];
            int32_t Wo, Ho;
            out_dims(m.width, m.height, border, &Wo, &Ho);
            jobs[i] = make_job(m.src, m.width, m.height, m.src_pitch, Wo, Ho, m.mag, m.mag_pitch, nullptr, 0, 0);
            stores.add(jobs[i]);
        }
        U8Shape shape = batch_default_shape(stores);
        for (int32_t i = 0; i < count; ++i) u8_tile(jobs[i], shape);
        int64_t total = 0;
        shape.th = batched_fit(jobs, count, shape.th, kLaunchWaves, &total);
        if (shape.waves == kStaticGrid && shape.th) {
            hipError_t e = guard(launch_u8_batched(jobs, nullptr, count, nullptr, border, stores.kind(), false, shape,
                                                   0, st));
            return e == hipSuccess ? ok() : hip_fail(e, "batched launch");
        }
    }
    // A graph would replay the launch with the cached plan's tables, which the
    // cache frees at its own time: only a plan that the caller holds may be
    // captured.
    if (is_captured(st))
        return fail(SOBEL4X5_EUNSUPPORTED, "a stream capture takes batches of up to %d magnitudes; others need a plan "
                    "(sobel4x5_plan_create) that outlives the graph", kBatchArgs);
    int dev = 0;
    hipGetDevice(&dev);
    const std::string key = batch_key(imgs, outs, count, border, dev, st);
    // Lookups, launches and evictions all hold the cache lock, so a plan is
    // never destroyed between another thread's lookup and its launch.
    PlanCache &c = plan_cache();
    {
        std::lock_guard<std::mutex> lk(c.mu);
        for (size_t i = 0; i < c.lru.size(); ++i)
            if (c.lru[i].key == key) {
                CachedPlan e = c.lru[i];
                c.lru.erase(c.lru.begin() + i);
                c.lru.push_back(e);
                return sobel4x5_plan_launch(e.plan, stream);
            }
    }
    sobel4x5_plan plan = nullptr;
    if (int rc = sobel4x5_plan_create_ex(imgs, outs, count, border, 0, &plan)) return rc;
    std::lock_guard<std::mutex> lk(c.mu);
    c.lru.push_back(CachedPlan{key, plan, st});
    if (c.lru.size() > 8) {
        const CachedPlan evicted = c.lru.front();
        c.lru.erase(c.lru.begin());
        (void)hipStreamSynchronize(evicted.stream);   // it may still be running there
        sobel4x5_plan_destroy(evicted.plan);
    }
    return sobel4x5_plan_launch(plan, stream);
}

int sobel4x5_batched(const sobel4x5_image *imgs, int32_t count, int32_t border, void *stream)
{
    return sobel4x5_batched_ex(imgs, nullptr, count, border, stream);
}

static_assert(SOBEL4X5_NOALLOC_MAX_IMAGES == kNoallocMaxImages && SOBEL4X5_NOALLOC_MAX_TILES == kNoallocMaxTiles,
              "public limits of the allocation-free batched call");

int sobel4x5_batched_noalloc(const sobel4x5_image *imgs, int32_t count, int32_t border, void *stream)
{
    if (int rc = validate_batch(imgs, nullptr, count, border)) return rc;
    if (count > kNoallocMaxImages)
        return fail(SOBEL4X5_EINVAL, "%d images: the allocation-free call takes at most %d", count,
                    kNoallocMaxImages);
    // Tables built on the host in fixed static buffers (no allocation, host
    // or device), then copied into the fixed device buffer on `stream`.  The
    // lock covers the building and both copies: a copy from pageable memory
    // has read its source when hipMemcpyAsync returns (outside a capture).
    static std::mutex mu;
    static unsigned char stage[kNoallocBytes];     // queue words, jobs, tiles: the device layout
    std::lock_guard<std::mutex> lk(mu);
    std::memset(stage, 0, kNoallocJobsOff);   // queue words start at zero
    U8Job *jobs = reinterpret_cast<U8Job *>(stage + kNoallocJobsOff);
    int64_t budget = 0;
    OutputStores stores;
    for (int32_t i = 0; i < count; ++i) {
        const sobel4x5_image &m = imgs[i];
        int32_t Wo, Ho;
        out_dims(m.width, m.height, border, &Wo, &Ho);
        jobs[i] = make_job(m.src, m.width, m.height, m.src_pitch, Wo, Ho, m.mag, m.mag_pitch, nullptr, 0, 0);
        stores.add(jobs[i]);
        budget += budget_tiles(Wo, Ho);
    }
    U8Shape shape = batch_default_shape(stores);
    for (int32_t i = 0; i < count; ++i) u8_tile(jobs[i], shape);
    if (budget > kNoallocMaxTiles)
        return fail(SOBEL4X5_EINVAL, "the batch needs more than %d wave-tiles, the allocation-free call's limit",
                    kNoallocMaxTiles);
    hipStream_t st = static_cast<hipStream_t>(stream);
    // Under capture the copies below would read `stage` again at every replay,
    // and the device buffer would hold whatever call came last: the images go
    // into kernel arguments instead, which the graph keeps.
    hipError_t e = hipSuccess;
    const bool captured = is_captured(st);
    for (int32_t i = 0; captured && i < count; i += kBatchArgs) {
        e = guard(launch_u8_batched(jobs + i, nullptr, std::min(kBatchArgs, count - i), nullptr, border,
                                    stores.kind(), false, shape, 0, st));
        if (e != hipSuccess) return hip_fail(e, "batched launch");
    }
    if (captured) return ok();
    // bands high enough for the table
    int64_t total = 0;
    shape.th = batched_fit(jobs, count, shape.th, kNoallocTable, &total);
    if (!shape.th) return fail(SOBEL4X5_EINVAL, "the batch does not fit the allocation-free call's table");
    int4 *t = reinterpret_cast<int4 *>(stage + kNoallocTilesOff);
    for (int32_t i = 0; i < count; ++i) batched_tiles_each(jobs[i], i, shape.th, [&](int4 e) { *t++ = e; });
    void *scr = nullptr;
    if ((e = guard(noalloc_scratch(&scr))) != hipSuccess) return hip_fail(e, "looking up the fixed device buffer");
    unsigned char *base = static_cast<unsigned char *>(scr);
    // queue words and the count jobs, then the total tiles
    if ((e = guard(hipMemcpyAsync(base, stage, kNoallocJobsOff + sizeof(U8Job) * count, hipMemcpyHostToDevice,
                                  st))) != hipSuccess ||
        (e = guard(hipMemcpyAsync(base + kNoallocTilesOff, stage + kNoallocTilesOff, sizeof(int4) * total,
                                  hipMemcpyHostToDevice, st))) != hipSuccess)
        return hip_fail(e, "copying the batch tables");
    // the default shape's grid form: one wave per tile, or a persistent grid
    // on the queue words
    const int need = (int)((total + 3) / 4);
    int grid = std::max(1, need);
    uint32_t *queue = nullptr;
    if (shape.waves != kStaticGrid) {
        grid = u8_persistent_grid(shape, stores.kind(), false);
        if (grid <= 0) return fail(SOBEL4X5_EHIP, "could not query occupancy");
        grid = std::max(1, std::min(grid, need));
        queue = reinterpret_cast<uint32_t *>(base);
    }
    e = guard(launch_u8_batched(reinterpret_cast<const U8Job *>(base + kNoallocJobsOff),
                                reinterpret_cast<const int4 *>(base + kNoallocTilesOff), (int32_t)total, queue,
                                border, stores.kind(), false, shape, grid, st));
    return e == hipSuccess ? ok() : hip_fail(e, "batched launch");
}

int sobel4x5_validate_f32(const float *src, int32_t batch, int32_t width, int32_t height, int64_t src_pitch,
                          int64_t src_bstride, int32_t border, const float *out, int64_t out_pitch,
                          int64_t out_bstride)
{
    int32_t Wo, Ho;
    if (int rc = out_dims(width, height, border, &Wo, &Ho)) return rc;
    if (batch < 0) return fail(SOBEL4X5_EINVAL, "batch must be >= 0");
    Range rs, ro;
    if (int rc = check_f32_buf("src", src, batch, width, height, src_pitch, src_bstride, &rs)) return rc;
    if (int rc = check_f32_buf("output", out, batch, Wo, Ho, out_pitch, out_bstride, &ro)) return rc;
    if (batch > 0 && overlap(rs, ro)) return fail(SOBEL4X5_EINVAL, "output overlaps src");
    return ok();
}

int sobel4x5_f32_fwd(const float *src, int32_t batch, int32_t width, int32_t height, int64_t src_pitch,
                     int64_t src_bstride, int32_t border, float *mag, int64_t mag_pitch, int64_t mag_bstride,
                     void *stream)
{
    if (int rc = sobel4x5_validate_f32(src, batch, width, height, src_pitch, src_bstride, border, mag, mag_pitch,
                                       mag_bstride))
        return rc;
    F32Args a{};
    a.src = src;
    a.src_pitch = src_pitch;
    a.src_bstride = src_bstride;
    a.out = mag;
    a.out_pitch = mag_pitch;
    a.out_bstride = mag_bstride;
    a.B = batch;
    a.W = width;
    a.H = height;
    out_dims(width, height, border, &a.Wo, &a.Ho);
    a.off = border == SOBEL4X5_BORDER_VALID ? 2 : 0;
    a.bmode = f32_bmode(border);
    hipError_t e = launch_f32_fwd(a, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? ok() : hip_fail(e, "sobel4x5_f32_fwd launch");
}

int sobel4x5_f32_bwd(const float *src, int64_t src_pitch, int64_t src_bstride, const float *grad_mag,
                     int64_t g_pitch, int64_t g_bstride, int32_t batch, int32_t width, int32_t height,
                     int32_t border, float *grad_src, int64_t gs_pitch, int64_t gs_bstride, void *stream)
{
    int32_t Wo, Ho;
    if (int rc = out_dims(width, height, border, &Wo, &Ho)) return rc;
    if (batch < 0) return fail(SOBEL4X5_EINVAL, "batch must be >= 0");
    Range rs, rg, rd;
    if (int rc = check_f32_buf("src", src, batch, width, height, src_pitch, src_bstride, &rs)) return rc;
    if (int rc = check_f32_buf("grad_mag", grad_mag, batch, Wo, Ho, g_pitch, g_bstride, &rg)) return rc;
    if (int rc = check_f32_buf("grad_src", grad_src, batch, width, height, gs_pitch, gs_bstride, &rd)) return rc;
    if (batch > 0 && (overlap(rd, rs) || overlap(rd, rg)))
        return fail(SOBEL4X5_EINVAL, "grad_src overlaps src or grad_mag");
    F32Args a{};
    a.src = src;
    a.src_pitch = src_pitch;
    a.src_bstride = src_bstride;
    a.grad = grad_mag;
    a.g_pitch = g_pitch;
    a.g_bstride = g_bstride;
    a.out = grad_src;
    a.out_pitch = gs_pitch;
    a.out_bstride = gs_bstride;
    a.B = batch;
    a.W = width;
    a.H = height;
    a.Wo = Wo;
    a.Ho = Ho;
    a.off = border == SOBEL4X5_BORDER_VALID ? 2 : 0;
    a.bmode = f32_bmode(border);
    hipError_t e = launch_f32_bwd(a, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? ok() : hip_fail(e, "sobel4x5_f32_bwd launch");
}

int sobel4x5_validate_weights(const int32_t *w, int32_t dir_type)
{
    if (!w) return fail(SOBEL4X5_EINVAL, "weights is NULL");
    const int64_t limit = dir_type == SOBEL4X5_DIR_S16 ? 128 : 32768;
    for (int k = 0; k < 4; ++k) {
        const int32_t *K = w + 25 * k;
        int64_t sum = 0;
        for (int i = 0; i < 5; ++i)
            for (int j = 0; j < 5; ++j) {
                if ((int64_t)K[5 * i + j] != -(int64_t)K[5 * (4 - i) + (4 - j)])
                    return fail(SOBEL4X5_EINVAL,
                                "kernel %d is not antisymmetric under a half turn at tap (%d, %d)", k, i, j);
                sum += K[5 * i + j] < 0 ? -(int64_t)K[5 * i + j] : K[5 * i + j];
            }
        if (sum > limit)
            return fail(SOBEL4X5_EINVAL, "kernel %d: sum of |weights| = %lld exceeds %lld%s", k, (long long)sum,
                        (long long)limit, dir_type == SOBEL4X5_DIR_S16 ? " (int16 planes)" : "");
    }
    return ok();
}

int sobel4x5_family_weights(int32_t a, int32_t ab, int32_t an, int32_t am, int32_t anb, int32_t amb,
                            int32_t *out)
{
    if (!out) return fail(SOBEL4X5_EINVAL, "weights_out is NULL");
    if (a <= 0 || ab <= 0 || an <= 0 || am <= 0 || anb <= 0 || amb <= 0)
        return fail(SOBEL4X5_EINVAL, "the six family weights must be positive");
    if ((int64_t)an * ab != (int64_t)a * anb || (int64_t)am * ab != (int64_t)a * amb)
        return fail(SOBEL4X5_EINVAL, "inconsistent family weights: need (a*n)(a*b) = a(a*n*b), (a*m)(a*b) = a(a*m*b)");
    // K_x = a [1 n m n 1]^T x [-1 -b 0 b 1]; K_y its transpose
    const int32_t col[5] = {a, an, am, an, a};          // a * [1 n m n 1]
    const int32_t colb[5] = {ab, anb, amb, anb, ab};    // a * b * [1 n m n 1]
    int32_t Kx[5][5], Kd[5][5];
    for (int i = 0; i < 5; ++i) {
        Kx[i][0] = -col[i];
        Kx[i][1] = -colb[i];
        Kx[i][2] = 0;
        Kx[i][3] = colb[i];
        Kx[i][4] = col[i];
    }
    // K_d as printed in Eq. (sobel5_param)
    const int32_t d[5][5] = {{-am, -an, -a, -ab, 0},
                             {-an, -amb, -anb, 0, ab},
                             {-a, -anb, 0, anb, a},
                             {-ab, 0, anb, amb, an},
                             {0, ab, a, an, am}};
    for (int i = 0; i < 5; ++i)
        for (int j = 0; j < 5; ++j) Kd[i][j] = d[i][j];
    for (int i = 0; i < 5; ++i)
        for (int j = 0; j < 5; ++j) {
            out[0 * 25 + 5 * i + j] = Kx[i][j];           // 0 deg
            out[1 * 25 + 5 * i + j] = Kd[i][j];           // 45 deg
            out[2 * 25 + 5 * i + j] = Kx[j][i];           // 90 deg: transpose
            out[3 * 25 + 5 * i + j] = Kd[i][4 - j];       // 135 deg: left-right mirror
        }
    return ok();
}

int sobel4x5_u8_weighted(const uint8_t *src, int32_t width, int32_t height, int64_t src_pitch, int32_t border,
                         const int32_t *weights, const sobel4x5_outputs *out, void *stream)
{
    int32_t Wo, Ho;
    if (int rc = validate_u8(src, width, height, src_pitch, border, out, &Wo, &Ho)) return rc;
    if (int rc = sobel4x5_validate_weights(weights, out->dir_type)) return rc;
    // weights that fit int8 (the family K(a, b, n, m) with small weights,
    // Eq. (sobel5_1) among them): the matrix cores.  Larger ones take the
    // vector kernel, which multiplies in 16 bits.
    if (env_int("SOBEL4X5_W_MFMA", 1) == 1 && mfma_weights_fit(weights)) {
        const U8Job mj = make_job(src, width, height, src_pitch, Wo, Ho, out->mag, out->mag_pitch,
                                  out->dir_type ? out->dir : nullptr, out->dir_pitch, out->dir_type);
        hipError_t e = guard(launch_u8_mfma_weighted(mj, border, weights, env_int("SOBEL4X5_U8_WAVES", 0),
                                                     static_cast<hipStream_t>(stream)));
        return e == hipSuccess ? ok() : hip_fail(e, "sobel4x5_u8_weighted launch");
    }
    WJob j{};
    j.src = src;
    j.mag = out->mag;
    for (int k = 0; k < 4; ++k) j.dir[k] = out->dir_type ? out->dir[k] : nullptr;
    j.src_pitch = src_pitch;
    j.mag_pitch = out->mag_pitch;
    j.dir_pitch = out->dir_pitch;
    j.W = width;
    j.H = height;
    j.Wo = Wo;
    j.Ho = Ho;
    j.off = border == SOBEL4X5_BORDER_VALID ? 2 : 0;
    j.bmode = border == SOBEL4X5_BORDER_ZERO ? 1 : (border == SOBEL4X5_BORDER_REFLECT101 ? 2 : 0);
    j.dir_type = out->dir_type;
    // upper-half taps (0, 0..4), (1, 0..4), (2, 0), (2, 1)
    for (int k = 0; k < 4; ++k)
        for (int t = 0; t < 12; ++t) {
            const int i = t < 5 ? 0 : (t < 10 ? 1 : 2), jj = t < 10 ? t % 5 : t - 10;
            j.coef[k][t] = weights[25 * k + 5 * i + jj];
        }
    hipError_t e = launch_u8_weighted(j, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? ok() : hip_fail(e, "sobel4x5_u8_weighted launch");
}

int sobel4x5_debug_inject_failure(int32_t nth_call)
{
    if (nth_call < 0) return fail(SOBEL4X5_EINVAL, "nth_call must be >= 0");
    g_inject.store(nth_call, std::memory_order_relaxed);
    return ok();
}

int sobel4x5_debug_copy(const void *src, void *dst, int64_t nbytes, void *stream)
{
    if (nbytes < 0 || (nbytes % 16) || (nbytes > 0 && (!src || !dst)) ||
        ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 15u))
        return fail(SOBEL4X5_EINVAL, "copy needs 16-byte aligned pointers and a multiple of 16 bytes");
    hipError_t e = launch_copy16(src, dst, nbytes / 16, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? ok() : hip_fail(e, "sobel4x5_debug_copy launch");
}

int sobel4x5_debug_round_mag_ex(const int32_t *S, uint8_t *out, int64_t n, int32_t method, void *stream)
{
    if (n < 0 || (n > 0 && (!S || !out))) return fail(SOBEL4X5_EINVAL, "bad arguments");
    if (method != 0 && method != 1) return fail(SOBEL4X5_EINVAL, "method must be 0 or 1, got %d", method);
    hipError_t e = launch_round_mag(S, out, n, method, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? ok() : hip_fail(e, "sobel4x5_debug_round_mag launch");
}

int sobel4x5_debug_round_mag(const int32_t *S, uint8_t *out, int64_t n, void *stream)
{
    return sobel4x5_debug_round_mag_ex(S, out, n, 0, stream);
}

int sobel4x5_debug_round_quad(const int16_t *q, uint8_t *out, int64_t n, void *stream)
{
    if (n < 0 || (n > 0 && (!q || !out))) return fail(SOBEL4X5_EINVAL, "bad arguments");
    if (n > (INT64_MAX / 8)) return fail(SOBEL4X5_EINVAL, "n too large");
    hipError_t e = launch_round_quad(q, out, n, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? ok() : hip_fail(e, "sobel4x5_debug_round_quad launch");
}

int sobel4x5_pipe_create(int32_t max_width, int32_t max_height, int32_t depth, sobel4x5_pipe *out)
{
    if (!out) return fail(SOBEL4X5_EINVAL, "out is NULL");
    *out = nullptr;
    if (max_width < 1 || max_height < 1) return fail(SOBEL4X5_EINVAL, "max sizes must be >= 1");
    if (depth < 1 || depth > 16) return fail(SOBEL4X5_EINVAL, "depth must be in [1, 16], got %d", depth);
    auto *p = new (std::nothrow) sobel4x5_pipe_s;
    if (!p) return fail(SOBEL4X5_ENOMEM, "host allocation failed");
    p->max_w = max_width;
    p->max_h = max_height;
    p->slots.resize(depth);
    const int64_t pitch = (max_width + 255) / 256 * 256;
    const size_t bytes = (size_t)pitch * (size_t)max_height;
    for (auto &sl : p->slots) {
        sl.pitch = pitch;
        hipError_t e;
        if ((e = hipStreamCreateWithFlags(&sl.st, hipStreamNonBlocking)) != hipSuccess ||
            (e = hipMalloc(&sl.d_src, bytes)) != hipSuccess || (e = hipMalloc(&sl.d_mag, bytes)) != hipSuccess ||
            (e = hipHostMalloc(&sl.h_src, bytes, hipHostMallocDefault)) != hipSuccess ||
            (e = hipHostMalloc(&sl.h_mag, bytes, hipHostMallocDefault)) != hipSuccess) {
            pipe_free(p);
            delete p;
            return fail(SOBEL4X5_ENOMEM, "pipeline allocation failed: %s", hipGetErrorString(e));
        }
    }
    *out = p;
    return ok();
}

int sobel4x5_pipe_run(sobel4x5_pipe p, const sobel4x5_image *imgs, int32_t count, int32_t border)
{
    if (!p) return fail(SOBEL4X5_EINVAL, "pipe is NULL");
    if (count < 0 || (count > 0 && !imgs)) return fail(SOBEL4X5_EINVAL, "bad image array");
    for (int32_t i = 0; i < count; ++i) {
        const sobel4x5_image &m = imgs[i];
        int32_t Wo, Ho;
        if (int rc = out_dims(m.width, m.height, border, &Wo, &Ho)) return rc;
        if (!m.src || !m.mag) return fail(SOBEL4X5_EINVAL, "image %d: NULL pointer", i);
        if (m.width > p->max_w || m.height > p->max_h)
            return fail(SOBEL4X5_EINVAL, "image %d (%d x %d) exceeds the pipeline's %d x %d", i, m.width, m.height,
                        p->max_w, p->max_h);
        if (int rc = check_pitch("src", m.src_pitch, m.width, m.height)) return rc;
        if (int rc = check_pitch("mag", m.mag_pitch, Wo, Ho)) return rc;
    }
    const int depth = (int)p->slots.size();
    // A slot's `pending` indexes THIS call's image array.  Every return path
    // leaves every slot idle: on an error, wait for whatever the slots still
    // have queued (a copy into a caller's pinned buffer must not land after
    // the return) and drop the pending images without copying them out, so
    // that a later call, with another array, never finishes an image of
    // this one.
    auto abandon = [&](int rc) {
        for (auto &sl : p->slots) {
            if (sl.st) (void)hipStreamSynchronize(sl.st);
            sl.pending = -1;
            sl.staged_out = false;
        }
        return rc;
    };
    for (auto &sl : p->slots)   // idle after every earlier call; keep it so
        if (sl.pending >= 0) abandon(SOBEL4X5_OK);
    auto drain = [&](PipeSlot &sl) -> hipError_t {
        if (sl.pending < 0) return hipSuccess;
        hipError_t e = guard(hipStreamSynchronize(sl.st));
        if (e == hipSuccess) pipe_finish(sl, imgs, border);
        return e;
    };
    for (int32_t i = 0; i < count; ++i) {
        PipeSlot &sl = p->slots[i % depth];
        if (hipError_t e = drain(sl); e != hipSuccess) return abandon(hip_fail(e, "pipeline wait"));
        const sobel4x5_image &m = imgs[i];
        int32_t Wo, Ho;
        out_dims(m.width, m.height, border, &Wo, &Ho);
        // host to device (pageable sources go through the slot's pinned
        // staging buffer, so that the copy itself is asynchronous)
        const uint8_t *hs = m.src;
        int64_t hp = m.src_pitch;
        if (!pipe_direct(m.src, m.src_pitch, m.width, m.height)) {
            for (int32_t r = 0; r < m.height; ++r)
                std::memcpy(sl.h_src + r * sl.pitch, m.src + r * m.src_pitch, (size_t)m.width);
            hs = sl.h_src;
            hp = sl.pitch;
        }
        // the slot owns image i from its first enqueued operation on
        sl.pending = i;
        sl.staged_out = false;
        const int64_t sp = pipe_pitch(sl, hp, m.width);
        hipError_t e = guard(pipe_copy(sl.d_src, sp, hs, hp, m.width, m.height, hipMemcpyHostToDevice, sl.st));
        if (e != hipSuccess) return abandon(hip_fail(e, "pipeline host-to-device copy"));
        sl.staged_out = !pipe_direct(m.mag, m.mag_pitch, Wo, Ho);
        uint8_t *hm = sl.staged_out ? sl.h_mag : m.mag;
        const int64_t op = sl.staged_out ? sl.pitch : m.mag_pitch, dp = pipe_pitch(sl, op, Wo);
        U8Job j = make_job(sl.d_src, m.width, m.height, sp, Wo, Ho, sl.d_mag, dp, nullptr, 0, 0);
        if ((e = guard(launch_u8_single(j, border, U8Shape{}, sl.st))) != hipSuccess)
            return abandon(hip_fail(e, "pipeline launch"));
        e = guard(pipe_copy(hm, op, sl.d_mag, dp, Wo, Ho, hipMemcpyDeviceToHost, sl.st));
        if (e != hipSuccess) return abandon(hip_fail(e, "pipeline device-to-host copy"));
    }
    for (auto &sl : p->slots)
        if (hipError_t e = drain(sl); e != hipSuccess) return abandon(hip_fail(e, "pipeline wait"));
    return ok();
}

int sobel4x5_pipe_destroy(sobel4x5_pipe p)
{
    if (!p) return fail(SOBEL4X5_EINVAL, "pipe is NULL");
    pipe_free(p);
    delete p;
    return ok();
}

}  // extern "C"
