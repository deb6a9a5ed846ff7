// Integration-buffer kernels: the float64 dump of tile partials, the int8
// calibration scales, the read-out transpose and a plain fill.
#include "dump_dev.h"

namespace corr {
namespace {

// The first workgroup also clears the F-stage's tile tickets for the next
// launch (a launch of its own before each F-stage took 2 to 5 us of a chunk).
template <typename P, bool FRESH>
__global__ __launch_bounds__(256) void dump_kernel(const P *partial, double2 *acc, int nsplit, int64_t n,
                                                   unsigned *tickets) {
    if (blockIdx.x == 0 && threadIdx.x < 8) tickets[threadIdx.x * kTicketStride] = 0;
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e < n) dump_one<P, FRESH>(partial, acc, nsplit, n, e);
}

__global__ __launch_bounds__(256) void scales_kernel(const float *power, int nparts, int N, int a_pad,
                                                     int K, int W, const unsigned *w_valid,
                                                     float codes_per_rms, float *scales, float *scales_p) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    const int w = w_valid ? (int)*w_valid : W;
    if (e >= N * K) return;
    const float sc = scale_one(power, nparts, a_pad, K, w, e, codes_per_rms);
    scales[e] = sc;
    if (scales_p) scales_p[reg_scale_index(K, e / K, e % K)] = sc;
}

// dst[bl][f] = acc[f][bl]; acc = 0.  Bound by memory: 48 bytes an element.  A
// tile of 64 baselines by 16 channels is turned through LDS, so that a
// wavefront reads (and clears) 1 KB of a channel's row and writes 256 bytes of
// a baseline's; written straight, each lane of a wavefront wrote to a line of
// its own.  The tiles of a channel row follow each other on one XCD (workgroup
// b runs on XCD b % 8), since rows of nb 16-byte elements start inside a line.
// N = 256, K = 512: 416 -> 161 us (5.0 TB/s, a large copy's rate; 176 us
// without the order of tiles, 170 us in 64 x 32 tiles, 212 us in 16 x 64);
// N = 44, K = 256: 5.4 -> 3.5 us.
// As float2 the sums leave in float, divided by their antennas' scales where
// there are any: in double, as a host loop over the doubles did.
constexpr int kFinB = 64, kFinF = 16;

// First antenna of baseline bl of N antennas (row a starts at a N - a (a - 1) / 2).
__device__ __forceinline__ int first_antenna(int bl, int N) {
    int a = (int)((2 * N + 1 - sqrtf((float)((2 * N + 1) * (2 * N + 1) - 8 * bl))) * 0.5f);
    while (a > 0 && a * N - a * (a - 1) / 2 > bl) --a;
    while ((a + 1) * N - (a + 1) * a / 2 <= bl) ++a;
    return a;
}

template <typename T, bool CLEAR>
__global__ __launch_bounds__(256) void finalize_kernel(double2 *acc, T *dst, const float *scales, int N, int K, int nb,
                                                       int ntb, int ntiles) {
    __shared__ T tile[kFinF][kFinB + 1];
    const int lb = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    if (lb >= ntiles) return;
    const int b0 = lb % ntb * kFinB, f0 = lb / ntb * kFinF;
    constexpr int R = kFinB * kFinF / 256, RF = 256 / kFinB, RB = 256 / kFinF;
    const int x = threadIdx.x % kFinB, y = threadIdx.x / kFinB;
    if (b0 + x < nb) {
        double2 *p = acc + (int64_t)(f0 + y) * nb + b0 + x;
        double2 v[R];
#pragma unroll
        for (int i = 0; i < R; ++i) v[i] = p[(int64_t)i * RF * nb];
        if constexpr (sizeof(T) == sizeof(float2)) {
            if (scales) {
                const int a = first_antenna(b0 + x, N), b = b0 + x - (a * N - a * (a - 1) / 2) + a;
                const float *sa = scales + (int64_t)a * K + f0 + y, *sb = scales + (int64_t)b * K + f0 + y;
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    const double d = (double)sa[i * RF] * (double)sb[i * RF];
                    v[i].x /= d;
                    v[i].y /= d;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
            if constexpr (sizeof(T) == sizeof(float2))
                tile[y + i * RF][x] = make_float2((float)v[i].x, (float)v[i].y);
            else
                tile[y + i * RF][x] = v[i];
            if (CLEAR) p[(int64_t)i * RF * nb] = make_double2(0.0, 0.0);
        }
    }
    __syncthreads();
    const int f = threadIdx.x % kFinF, b = threadIdx.x / kFinF;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int bl = b0 + b + i * RB;
        if (bl < nb) dst[(int64_t)bl * K + f0 + f] = tile[f][b + i * RB];
    }
}

__global__ __launch_bounds__(256) void fill_zero_kernel(uint4 *p, int64_t n16) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += (int64_t)gridDim.x * 256)
        p[i] = make_uint4(0u, 0u, 0u, 0u);
}

}  // namespace

namespace {

template <typename P>
hipError_t launch_dump_as(const void *partial, double2 *acc, int nsplit, int K, int nb, bool fresh, unsigned *tickets,
                          hipStream_t st) {
    const int64_t n = (int64_t)K * nb;
    const int grid = (int)((n + 255) / 256);
    if (fresh)
        hipLaunchKernelGGL((dump_kernel<P, true>), dim3(grid), dim3(256), 0, st, reinterpret_cast<const P *>(partial), acc,
                           nsplit, n, tickets);
    else
        hipLaunchKernelGGL((dump_kernel<P, false>), dim3(grid), dim3(256), 0, st, reinterpret_cast<const P *>(partial), acc,
                           nsplit, n, tickets);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_dump(int prec, const void *partial, double2 *acc, int nsplit, int K, int nb, bool fresh,
                       unsigned *tickets, hipStream_t st) {
    if (prec == kINT8) return launch_dump_as<int2>(partial, acc, nsplit, K, nb, fresh, tickets, st);
    if (prec == kINT16) return launch_dump_as<double2>(partial, acc, nsplit, K, nb, fresh, tickets, st);
    return launch_dump_as<float2>(partial, acc, nsplit, K, nb, fresh, tickets, st);
}

hipError_t launch_scales(const float *power, int nparts, int N, int a_pad, int K, int W,
                         const unsigned *w_valid, float codes_per_rms, float *scales, float *scales_p,
                         hipStream_t st) {
    const int grid = (N * K + 255) / 256;
    hipLaunchKernelGGL(scales_kernel, dim3(grid), dim3(256), 0, st, power, nparts, N, a_pad, K, W, w_valid,
                       codes_per_rms, scales, scales_p);
    return hipGetLastError();
}

namespace {

template <typename T, bool CLEAR = true>
hipError_t launch_finalize_as(double2 *acc, T *dst, const float *scales, int N, int K, int nb, hipStream_t st) {
    static_assert(128 % kFinF == 0, "K, a multiple of 128, is whole tiles");
    const int ntb = (nb + kFinB - 1) / kFinB, ntiles = ntb * (K / kFinF);
    const int grid = 8 * ((ntiles + 7) / 8);  // workgroups past the end exit
    hipLaunchKernelGGL((finalize_kernel<T, CLEAR>), dim3(grid), dim3(256), 0, st, acc, dst, scales, N, K, nb, ntb, ntiles);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_finalize(double2 *acc, double2 *dst, int K, int nb, hipStream_t st) {
    return launch_finalize_as<double2>(acc, dst, nullptr, 0, K, nb, st);
}

hipError_t launch_finalize_keep(double2 *acc, double2 *dst, int K, int nb, hipStream_t st) {
    return launch_finalize_as<double2, false>(acc, dst, nullptr, 0, K, nb, st);
}

hipError_t launch_finalize_float(double2 *acc, float2 *dst, const float *scales, int N, int K, int nb, hipStream_t st) {
    return launch_finalize_as<float2>(acc, dst, scales, N, K, nb, st);
}

hipError_t launch_fill_zero(void *p, size_t bytes, hipStream_t st) {
    if (bytes % 16) return hipErrorInvalidValue;
    const int64_t n16 = (int64_t)(bytes / 16);
    if (n16 == 0) return hipSuccess;
    int64_t grid = (n16 + 255) / 256;
    if (grid > 4096) grid = 4096;
    hipLaunchKernelGGL(fill_zero_kernel, dim3((int)grid), dim3(256), 0, st, reinterpret_cast<uint4 *>(p), n16);
    return hipGetLastError();
}

}  // namespace corr
