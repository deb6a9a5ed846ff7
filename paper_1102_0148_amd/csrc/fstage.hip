// Single-job F-stage kernels over the device functions of fstage_dev.h.
#include "fstage_reg_dev.h"

namespace corr {
namespace {

// Persistent workgroups; workgroup b runs on XCD b % 8 (round-robin
// dispatch), and the tiles of XCD x are the range [x t8, (x+1) t8), dealt one
// by one by that XCD's ticket counter (zero at launch: the dump that follows
// the last launch cleared it): tiles in flight on one XCD are
// neighbours (consecutive antenna groups of nearby time records) whose
// partial lines meet in one L2.
template <int M, int PREC, int GA, bool TRACK>
__device__ __forceinline__ void f_records(const FArgs &args, float2 *zbuf, uint32_t *bbuf) {
    __shared__ int s_tk[2];
    const int t8 = (args.ntiles + 7) / 8;
    const int x = blockIdx.x % 8;
    const int lo = x * t8, hi = min(lo + t8, args.ntiles);
    f_tiles_dyn<M, PREC, GA, TRACK>(args, lo, hi, args.ticket + kTicketStride * x, s_tk, zbuf, bbuf);
}

template <int M, int PREC, int GA, bool POWER>
__global__ __launch_bounds__(kThreads) void fstage_kernel(FArgs kargs) {
    using Sh = FShape<M, PREC, GA, POWER>;
    // a replayed graph passes the input through a device slot that the host
    // rewrites before each replay; a chunk starts s_base spectra into it.
    // The cast through the global address space keeps the input loads
    // global: from a generic pointer they would be flat loads, which also
    // count against lgkmcnt, so every wait for LDS would wait for the next
    // tile's prefetch too.
    typedef const __attribute__((address_space(1))) uint8_t *gptr;
    FArgs args = kargs;
    if (args.in_slot)
        args.in = (const uint8_t *)*reinterpret_cast<const gptr *>(args.in_slot) + (int64_t)args.s_base * args.N * M;
    static_assert(Sh::LDS <= 160 * 1024, "LDS budget");
    __shared__ float2 zbuf[Sh::NF * Sh::SLOT];
    __shared__ __attribute__((aligned(16))) uint32_t bbuf[Sh::FPR * (M / 4)];
    if constexpr (!POWER) {
        f_records<M, PREC, GA, false>(args, zbuf, bbuf);
    } else {
        f_power_block<M>(args, blockIdx.x, zbuf, bbuf);
    }
}

// Records with delay and phase tracking: a kernel of its own, so the kernels
// without tracking are exactly the ones above.
template <int M, int PREC, int GA>
__global__ __launch_bounds__(kThreads) void fstage_track_kernel(FArgs args) {
    using Sh = FShape<M, PREC, GA, false>;
    __shared__ float2 zbuf[Sh::NF * Sh::SLOT];
    __shared__ __attribute__((aligned(16))) uint32_t bbuf[Sh::FPR * (M / 4)];
    f_records<M, PREC, GA, true>(args, zbuf, bbuf);
}

// Records by the register transform: two workgroups per CU (two wavefronts a SIMD, 256
// registers each; the workgroup's 74 KB of operands).
template <int M, int PREC, bool TRACK>
__global__ __launch_bounds__(kThreads, 2) void fstage_reg_kernel(FArgs kargs) {
    // as in fstage_kernel
    typedef const __attribute__((address_space(1))) uint8_t *gptr;
    FArgs args = kargs;
    if (args.in_slot)
        args.in = (const uint8_t *)*reinterpret_cast<const gptr *>(args.in_slot) + (int64_t)args.s_base * args.N * M;
    __shared__ __attribute__((aligned(16))) uint4 lds[kRegLds];
    __shared__ int s_tk[2];
    const int sets = args.ntiles / 4;  // a chunk has a multiple of 4 time records
    const int t8 = (sets + 7) / 8;
    const int x = blockIdx.x % 8, rank = blockIdx.x / 8, wgs = gridDim.x / 8;
    const int lo = x * t8, hi = min(lo + t8, sets);
    unsigned *const ctr = args.ticket + kTicketStride * x;
    if constexpr (TRACK && M == 512) {
        // (short of registers: what follows spills more here, N = 44, 4096 spectra int8
        // 231 -> 242 us)
        reg_load_ops<M>(args, lds);
        __syncthreads();
        reg_units_dyn<M, PREC, TRACK>(args, lo, hi, ctr, s_tk, lds);
        return;
    }
    // A workgroup's first two sets go by its rank on the XCD, so that their tickets,
    // the samples and the operands are not fetched one after another.  Calls queued
    // back to back, before and so (us; with the LDS transform of up to 16 sequences a
    // workgroup, which this one replaced, in brackets): K = 256, N = 4, 444 spectra
    // fp16 19.3 and 17.5 (25.0), int8 36.7 and 36.0 (37.1), int16 39.2 and 39.0 (37.5: 16
    // sequences in one wavefront take longer than in four); K = 512, N = 16, 64 spectra
    // int16 41.4 and 40.7 (40.4); N = 44, K = 256, 4096 spectra int8 117.4 and 114.6
    // (141.9).  Few units keep this transform all the same: the codes of an
    // integration do not depend on the chunks it is cut into.
    const int set = lo + rank;
    if (set >= hi) return;
    u32x4 raw[4];
    reg_load_set<M, PREC>(args, set, raw);
    reg_load_ops<M>(args, lds);  // waits for the samples too
    __syncthreads();
    reg_sets<M, PREC, TRACK>(args, set, set + wgs, lo + 2 * wgs, hi, ctr, s_tk, lds, raw);
}

template <int M, int PREC, bool TRACK>
hipError_t launch_reg(const FArgs &a, hipStream_t st) {
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    // two workgroups per CU, no more than one per set of units
    const int cap = 2 * cus / 8 > 0 ? 2 * cus / 8 : 1;
    const int need = (a.ntiles + 31) / 32;
    const int grid = 8 * (need < cap ? need : cap);
    hipLaunchKernelGGL((fstage_reg_kernel<M, PREC, TRACK>), dim3(grid), dim3(kThreads), 0, st, a);
    return hipGetLastError();
}

template <int M, int PREC, int GA, bool POWER>
hipError_t launch_one(const FArgs &a, int grid, hipStream_t st) {
    if constexpr (FShape<M, PREC, GA, POWER>::LDS > 160 * 1024) {
        return hipErrorInvalidValue;
    } else {
        const bool track = !POWER && a.track;
        if (!POWER) {
            // as many workgroups (a multiple of 8) as stay resident, at most one
            // per tile
            int per_cu = 0, dev = 0, cus = 0;
            hipError_t e = track ? hipOccupancyMaxActiveBlocksPerMultiprocessor(
                                       &per_cu, fstage_track_kernel<M, PREC, GA>, kThreads, 0)
                                 : hipOccupancyMaxActiveBlocksPerMultiprocessor(
                                       &per_cu, fstage_kernel<M, PREC, GA, POWER>, kThreads, 0);
            if (e == hipSuccess) e = hipGetDevice(&dev);
            if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
            if (e != hipSuccess) return e;
            const int cap = per_cu * cus / 8 > 0 ? per_cu * cus / 8 : 1;
            const int need = (a.ntiles + 7) / 8;
            grid = 8 * (need < cap ? need : cap);
        }
        if (track)
            hipLaunchKernelGGL((fstage_track_kernel<M, PREC, GA>), dim3(grid), dim3(kThreads), 0, st, a);
        else
            hipLaunchKernelGGL((fstage_kernel<M, PREC, GA, POWER>), dim3(grid), dim3(kThreads), 0, st, a);
        return hipGetLastError();
    }
}

template <int M, int PREC>
hipError_t launch_mp(int ga, int power, const FArgs &a, int grid, hipStream_t st) {
    if (power) return launch_one<M, kFP32, power_group(M), true>(a, grid, st);
    if constexpr (reg_fft<M, PREC>()) return a.track ? launch_reg<M, PREC, true>(a, st) : launch_reg<M, PREC, false>(a, st);
    else switch (ga) {
        case 1: return launch_one<M, PREC, 1, false>(a, grid, st);
        case 2: return launch_one<M, PREC, 2, false>(a, grid, st);
        case 4: return launch_one<M, PREC, 4, false>(a, grid, st);
        case 8: return launch_one<M, PREC, 8, false>(a, grid, st);
        case 16: return launch_one<M, PREC, 16, false>(a, grid, st);
    }
    return hipErrorInvalidValue;
}

template <int M>
hipError_t launch_m(int prec, int ga, int power, const FArgs &a, int grid, hipStream_t st) {
    switch (prec) {
        case kFP32: return launch_mp<M, kFP32>(ga, power, a, grid, st);
        case kFP16: return launch_mp<M, kFP16>(ga, power, a, grid, st);
        case kINT8: return launch_mp<M, kINT8>(ga, power, a, grid, st);
        case kINT16: return launch_mp<M, kINT16>(ga, power, a, grid, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace

int fstage_lds_bytes(int M, int prec, int ga) {
    const int L = M / 16, FPR = kThreads / L, SLOT = M + M / 16 + 1;
    return record_times(prec) * ga * SLOT * 8 + FPR * M;
}

int fstage_default_group(int M, int prec) {
    const int fpr = kThreads / (M / 16);
    const int g = fpr / record_times(prec);
    return g < 1 ? 1 : g;
}

// Twice the antennas where a tile then still leaves two workgroups to a CU (70 KB
// of LDS): the records of a tile fill whole lines, or more of one.  F-stage, one
// round of transforms and two (us): fp32 K = 1024, N = 37, 3001 spectra 452 and 271,
// N = 6, 16384 spectra 532 and 240; K = 512, N = 44, 8192 spectra 419 and 338, N = 200,
// 4096 spectra 1095 and 773; K = 256, N = 44, 16384 spectra 351 and 320; fp16 K = 1024,
// N = 37 322 and 212.  Not where padding to the larger group costs more (K = 256: N = 20
// 87 and 91, N = 24 85 and 90; a third more is won back from K = 512 on: N = 9 and its
// X-stage 501 and 500, K = 1024, N = 5 544 and 298), nor where the chip is not filled
// (K = 512, N = 8, 64 spectra 8.4 and 10.7).  int16 and int8 at K = 1024 gain nothing
// (N = 37 with the X-stage 377 and 381; 262 and 350).
int fstage_auto_group(int M, int prec, int N, int chunk) {
    const int g = fstage_default_group(M, prec);
    if (!(prec == kFP32 && M >= 256) && !(prec == kFP16 && M == 1024)) return g;
    const int64_t records = (chunk + record_times(prec) - 1) / record_times(prec);
    const int one = round_up(N, g), two = round_up(N, 2 * g);
    const bool padded = M == 256 ? two * 4 > one * 5 : two * 3 > one * 4;
    return padded || records * (two / (2 * g)) < 512 ? g : 2 * g;
}

hipError_t launch_fstage(int M, int prec, int ga, int power_mode, const FArgs &a, int grid,
                         hipStream_t st) {
    if (!power_mode && fstage_lds_bytes(M, prec, ga) > 160 * 1024) return hipErrorInvalidValue;
    switch (M) {
        case 128: return launch_m<128>(prec, ga, power_mode, a, grid, st);
        case 256: return launch_m<256>(prec, ga, power_mode, a, grid, st);
        case 512: return launch_m<512>(prec, ga, power_mode, a, grid, st);
        case 1024: return launch_m<1024>(prec, ga, power_mode, a, grid, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace corr
