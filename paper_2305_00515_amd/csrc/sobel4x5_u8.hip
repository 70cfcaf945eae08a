// A plain copy kernel that serves as the bandwidth reference, the
// autotuner's fingerprint of output planes, and the diagnostics of the uint8
// roundings.

#include "u8_band.hpp"

namespace s4x5 {
namespace {

// Plain streaming copy: the reference point for the achievable HBM
// bandwidth and for calibrating the memory-traffic counters.  Each
// workgroup copies one contiguous 16 KiB block, four 16-byte loads per lane
// in flight before the stores (measured 5.7 TB/s on 1 GiB, against 4.6 TB/s
// for a grid-stride loop).
__global__ __launch_bounds__(256) void k_copy16(const uint4 *__restrict__ src, uint4 *__restrict__ dst, int64_t n16)
{
    const int64_t base = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    uint4 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (base + 256 * k < n16) v[k] = src[base + 256 * k];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (base + 256 * k < n16) dst[base + 256 * k] = v[k];
}

// Order-independent fingerprint of one output plane (the autotuner's check
// that a candidate tile shape reproduces the reference bytes): the byte at
// (row r, column c) contributes mix(r, c, byte), with the splitmix64
// finaliser as the mix; each workgroup sums (mod 2^64) the contributions of
// kFpRows rows into out[blockIdx.x].
constexpr int kFpRows = 16;

__global__ __launch_bounds__(256) void k_fingerprint(const uint8_t *__restrict__ base, int64_t pitch,
                                                     int64_t row_bytes, int64_t rows, uint64_t *__restrict__ out)
{
    const int64_t r0 = (int64_t)blockIdx.x * kFpRows;
    const int64_t r1 = r0 + kFpRows < rows ? r0 + kFpRows : rows;
    uint64_t acc = 0;
    for (int64_t r = r0; r < r1; ++r) {
        const uint8_t *row = base + r * pitch;
        for (int64_t c = threadIdx.x; c < row_bytes; c += 256) {
            uint64_t v = ((uint64_t)r << 40) ^ ((uint64_t)c << 8) ^ (uint64_t)row[c];
            v = (v ^ (v >> 30)) * 0xbf58476d1ce4e5b9ull;
            v = (v ^ (v >> 27)) * 0x94d049bb133111ebull;
            acc += v ^ (v >> 31);
        }
    }
    __shared__ uint64_t red[256];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x] = red[0];
}

// The kernels' rounding of a magnitude (method 0), and the same by an integer
// root (method 1).
__global__ void k_round_mag(const int32_t *S, uint8_t *out, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = (uint8_t)mag_byte(S[i], 0, 0);
}

// round(sqrt(S)) is the number of r in 1..255 with (r - 1/2)^2 < S, that is
// r^2 - r < S for whole S: a bitwise search.
__global__ void k_round_mag_int(const int32_t *S, uint8_t *out, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int r = 0;
    for (int b = 128; b > 0; b >>= 1)
        if ((r + b) * (r + b - 1) < S[i]) r += b;
    out[i] = (uint8_t)r;
}

// Quadruples (E1, E2, Hp, Hm) of int16, S = 2 (E1^2 + E2^2 + Hp^2 + Hm^2): the
// clamp, the 24-bit squares and the rounding of the kernels, on a form of S that
// no kernel forms itself.  The halves
// E1 = (Gx + Gy) / 2, ... reach sqrt(S / 2), so they are clamped at 256 like
// a response: one that is larger saturates the magnitude alone.
__global__ __launch_bounds__(256) void k_round_quad(const int16_t *q, uint8_t *out, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int G[4] = {q[4 * i], q[4 * i + 1], q[4 * i + 2], q[4 * i + 3]};
    out[i] = (uint8_t)mag_byte(2 * sum_squares<4, true>(G), 0, 0);
}

}  // namespace

hipError_t launch_copy16(const void *src, void *dst, int64_t n16, hipStream_t st)
{
    if (n16 <= 0) return hipSuccess;
    const int64_t blocks = (n16 + 1023) / 1024;
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_copy16, dim3((unsigned)blocks), dim3(256), 0, st, static_cast<const uint4 *>(src),
                       static_cast<uint4 *>(dst), n16);
    return hipGetLastError();
}

int64_t fingerprint_blocks(int64_t rows) { return (rows + kFpRows - 1) / kFpRows; }

hipError_t launch_fingerprint(const void *base, int64_t pitch, int64_t row_bytes, int64_t rows, uint64_t *partials,
                              hipStream_t st)
{
    const int64_t blocks = fingerprint_blocks(rows);
    if (blocks <= 0 || row_bytes <= 0) return hipSuccess;
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_fingerprint, dim3((unsigned)blocks), dim3(256), 0, st, static_cast<const uint8_t *>(base),
                       pitch, row_bytes, rows, partials);
    return hipGetLastError();
}

hipError_t launch_round_quad(const int16_t *q, uint8_t *out, int64_t n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const int64_t blocks = (n + 255) / 256;
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_round_quad, dim3((unsigned)blocks), dim3(256), 0, st, q, out, n);
    return hipGetLastError();
}

hipError_t launch_round_mag(const int32_t *S, uint8_t *out, int64_t n, int method, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const int64_t blocks = (n + 255) / 256;
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    if (method == 1)
        hipLaunchKernelGGL(k_round_mag_int, dim3((unsigned)blocks), dim3(256), 0, st, S, out, n);
    else
        hipLaunchKernelGGL(k_round_mag, dim3((unsigned)blocks), dim3(256), 0, st, S, out, n);
    return hipGetLastError();
}

}  // namespace s4x5
