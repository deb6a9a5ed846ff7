// The F-stage of the reduced-precision records at 512- and 1024-point real
// transforms (M = 256 and 512 channels): the whole transform in the registers of
// one wavefront, on the matrix cores, with no exchange through LDS and no barrier.
//
// A wavefront transforms 16 real sequences e_t[512] at a time: 16 blocks at M =
// 256; at M = 512 the even and the odd samples of 8 blocks (t = 2 block + parity).
// With n = 16 s + f (s < 32, f < 16), c < 16 and d < 16 the bins come in two
// matrix products:
//   Y[f][c]  = sum_s W512^(c (16 s + f)) e[16 s + f]        (c > 0)
//   E[c + 32 d] = sum_f W16^(f d) Y[f][c].
// The input is real, so c = 1 .. 15 gives every bin that is no multiple of 16 (E[c
// + 32 d] for d >= 8 as the conjugate of bin 512 - c - 32 d); there is no separate
// split of a half-length complex transform and no multiplication by twiddles, which
// the first product's matrix takes in (a matrix for each f).  Column c = 0 holds
// instead the folded samples p[r] = sum_t e[r + 32 t], as p[f] + i p[f + 16], and
// the second product takes them to the bins 16 d with a matrix of its own, the
// 32-point transform of real input.
//
// Layout, on v_mfma_f32_16x16x32_f16 (lane (j, g), j = lane mod 16, g = lane / 16,
// holds row j of the left operand and column j of the right one over contraction
// positions 8g .. 8g + 7, and gets rows 4g .. 4g + 3 of column j of the result):
//   first product, for each f: left rows c, right columns t, contraction s.  Lane
//     (t, g) needs the samples s = 8q + 2g + b of sequence t (position 4b + q), the
//     16 bytes at 64 q + 16 g of the block: four coalesced loads straight into
//     registers, and a transpose of bytes within the lane.  It gets Y[f][4g + i].
//   between them, for each i: the four lane groups and the four quarters of f change
//     places (two pairs of row swaps), so that lane (t, g) holds f = 4g .. 4g + 3 of
//     columns c = 4 gamma + i.
//   second product, for each c: left rows t, right columns d, contraction (f, re or
//     im).  Lane (d, g) gets sequences t = 4g .. 4g + 3 of bin c + 32 d: consecutive
//     spectra of one antenna, which is what a record holds.
//
// Precision: the samples are exact in f16, and each factor is a sum of f16 halves (W
// = hi + lo and Y = hi + lo, products exact in the f32 accumulator, the lo lo terms
// dropped): about 7e-8 of the spectrum's rms (the transform before it, a half-length
// complex one with twiddles and a split in f32, 1.6e-7).  p is a sum of 16 samples,
// exact in f16, and bins 0 and M / 2 meet only factors 0 and +-1: they stay exact.
//
// Bound: vector work (unpacking 13, halves 12, row swaps 8, quantising and packing
// about 20 instructions per sequence; 59 for int8, where the transform through LDS
// before it issued 120) beside 10 matrix products per sequence, and the record stores,
// of 16 to 64 bytes a piece.  The first product's 64 matrices (64 KB) are read from
// LDS, where a workgroup loads them once.  F-stage times, before and now, same box:
// N = 44, 512-point, 65536 spectra: fp16 0.99 -> 0.86 ms, int8 0.83 -> 0.64, int16 1.04
// -> 0.98 (without the stores fp16 takes 0.46, int8 0.55); N = 256, 1024-point, 16384
// spectra: int8 2.67 -> 2.36 ms (1.86 without the stores); N = 37, 1024-point, 16384
// spectra: fp16 0.76 -> 0.39 ms; N = 61, 5001 spectra: int16 0.34 -> 0.22 ms.
#pragma once
#include "fstage_dev.h"

namespace corr {
namespace {

// Sequences per block, and antennas of a unit of 16 sequences.
template <int M> constexpr int reg_seqs() { return M / 256; }
template <int M, int PREC> constexpr int reg_group() { return 16 / (reg_seqs<M>() * record_times(PREC)); }

// LDS of a workgroup: the operands (kRegOps of them), then W_2M^k in the order
// [c][d] of the lanes (M = 512).
constexpr int kRegTw2 = kRegOps, kRegLds = kRegTw2 + 128;
constexpr int kRegB16 = 16 * 4 * 64, kRegB0 = kRegB16 + 4 * 64;

// The bin of column c and lane column d, k < 256.
__device__ __forceinline__ int reg_bin(int c, int d) { return c == 0 ? 16 * d : d < 8 ? c + 32 * d : 512 - c - 32 * d; }

// Fill the workgroup's LDS; the caller synchronises.
template <int M>
__device__ __forceinline__ void reg_load_ops(const FArgs &args, uint4 *lds) {
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int i = w; i < kRegOps / 64; i += kThreads / 64)
        __builtin_amdgcn_global_load_lds(args.ops + i * 64 + lane, lds + i * 64, 16, 0, 0);
    if constexpr (reg_seqs<M>() == 2) {
        float2 *tw2 = reinterpret_cast<float2 *>(lds + kRegTw2);
        tw2[threadIdx.x] = args.tw[M + reg_bin(threadIdx.x >> 4, threadIdx.x & 15)];
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);
}

// Units are handed out in sets of four, one to each wavefront of a workgroup, which
// starts them together: the records of the set's antennas of a channel, two to eight
// lines' halves that would else be written by wavefronts far apart in time, meet in
// the L2 while they are fresh.  Unit u of a chunk is (time record tq, antenna group
// ga); a set stays within one time record but for the remainders of the groups over
// four, which are gathered from 2 or 4 time records (a chunk has a multiple of 4).
// N = 44, 65536 spectra, int8: 0.86 ms with units dealt to wavefronts one by one, 0.64
// so.  (Exchanging the four wavefronts' records through LDS, so that a store wrote 64 to
// 256 bytes a piece, cost more in barriers than it gave: int8 0.70, fp16 0.88 -> 1.0.)
__device__ __forceinline__ void reg_unit_at(int u, int ngroups, int &tq, int &ga) {
    const int rem = ngroups & 3, whole = ngroups - rem;
    const int rows = rem == 0 ? 1 : rem == 2 ? 2 : 4;
    const int block = u / (rows * ngroups), l = u % (rows * ngroups), m = l - rows * whole;
    const int of = m < 0 ? whole : rem, k = m < 0 ? l : m;
    tq = block * rows + k / of;
    ga = k % of + (m < 0 ? 0 : whole);
}

// The lane's 64 bytes of time record tq and antenna group ga, unconditionally: blocks
// past the chunk or past N come from the zero page.
template <int M, int PREC>
__device__ __forceinline__ void reg_load(const FArgs &args, int tq, int ga, u32x4 (&raw)[4]) {
    constexpr int P = reg_seqs<M>(), TS = record_times(PREC), GA = reg_group<M, PREC>();
    const int lane = threadIdx.x & 63, j = lane & 15, g = lane >> 4;
    const int blk = j / P;
    const int s = tq * TS + blk % TS, a = ga * GA + blk / TS;
    const uint8_t *zeros = reinterpret_cast<const uint8_t *>(args.tw + M + M / 2);
    const uint8_t *src = s < args.S && a < args.N ? args.in + ((int64_t)s * args.N + a) * M : zeros;
    src += P == 1 ? 16 * g : 32 * g + 16 * (j & 1);
#pragma unroll
    for (int q = 0; q < 4; ++q)
        raw[q] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src + 64 * P * q));
}

// Bytes b of d0 .. d3 to dword r[b].
__device__ __forceinline__ void byte_transpose(uint32_t d0, uint32_t d1, uint32_t d2, uint32_t d3, uint32_t (&r)[4]) {
    const uint32_t l01 = __builtin_amdgcn_perm(d1, d0, 0x05010400u), h01 = __builtin_amdgcn_perm(d1, d0, 0x07030602u);
    const uint32_t l23 = __builtin_amdgcn_perm(d3, d2, 0x05010400u), h23 = __builtin_amdgcn_perm(d3, d2, 0x07030602u);
    r[0] = __builtin_amdgcn_perm(l23, l01, 0x05040100u);
    r[1] = __builtin_amdgcn_perm(l23, l01, 0x07060302u);
    r[2] = __builtin_amdgcn_perm(h23, h01, 0x05040100u);
    r[3] = __builtin_amdgcn_perm(h23, h01, 0x07060302u);
}

// Low nibbles of two dwords' bytes as eight f16 values: offset nibbles u = n + 8 as
// 1024 + u (byte u under the exponent byte 0x64), then minus 1032: exact.
__device__ __forceinline__ h8_t nibbles_f16(uint32_t a, uint32_t b) {
    const uint32_t u[2] = {(a & 0x0f0f0f0fu) ^ 0x08080808u, (b & 0x0f0f0f0fu) ^ 0x08080808u};
    h8_t x;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const uint32_t bits = __builtin_amdgcn_perm(0x64646464u, u[w >> 1], w & 1 ? 0x04030402u : 0x04010400u);
        const h2_t v = __builtin_bit_cast(h2_t, bits) - h2_t{(_Float16)1032.0f, (_Float16)1032.0f};
        x[2 * w] = v[0];
        x[2 * w + 1] = v[1];
    }
    return x;
}

// Lane group g of register r[F] to lane group F of register r[g].
__device__ __forceinline__ void row_transpose(uint32_t &r0, uint32_t &r1, uint32_t &r2, uint32_t &r3) {
    const auto a = __builtin_amdgcn_permlane32_swap(r0, r2, false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(r1, r3, false, false);
    const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
    const auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
    r0 = c[0];
    r1 = c[1];
    r2 = d[0];
    r3 = d[1];
}

// Lane groups 2p and 2p + 1 swap: the odd group's x with the even group's y.  After it
// the even group holds both groups' x (its own in x, the odd one's in y), and the odd
// group both groups' y (the even one's in x, its own in y).
__device__ __forceinline__ void pair_exchange(uint32_t &x, uint32_t &y) {
    const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
    x = r[0];
    y = r[1];
}

// As quantise (fstage_dev.h), for NB bins of NV values with a scale each: one test for
// the lot.
template <int NB, int NV>
__device__ __forceinline__ void quantise_bins(const float (&x)[NB][NV], const float (&sc)[NB], float lim, unsigned &wsat,
                                              float (&qm)[NB][NV]) {
    constexpr float kMagic = 12582912.0f;
    float top = 0.0f;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        float m = 0.0f;
#pragma unroll
        for (int t = 0; t < NV; t += 2)
            m = __builtin_elementwise_maximum(__builtin_elementwise_maximum(m, fabsf(x[b][t])), fabsf(x[b][t + 1]));
        top = __builtin_elementwise_maximum(top, m * sc[b]);
#pragma unroll
        for (int t = 0; t < NV; ++t) qm[b][t] = __builtin_fmaf(x[b][t], sc[b], kMagic);
    }
    if (__ballot(top >= lim + 0.5f)) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int t = 0; t < NV; ++t) {
                wsat += (unsigned)__popcll(__ballot(fabsf(qm[b][t] - kMagic) > lim));
                qm[b][t] = __builtin_amdgcn_fmed3f(qm[b][t], kMagic - lim, kMagic + lim);
            }
    }
}

__device__ __forceinline__ uint32_t pack_bytes(uint32_t b0, uint32_t b1, uint32_t b2, uint32_t b3) {
    return __builtin_amdgcn_perm(b1, b0, 0x0c0c0400u) | __builtin_amdgcn_perm(b3, b2, 0x04000c0cu);
}
__device__ __forceinline__ uint32_t pack_f16(float a, float b) {
    return __builtin_bit_cast(uint32_t, h2_t{(_Float16)a, (_Float16)b});
}

// The records of one unit from the lane's bytes.
template <int M, int PREC, bool TRACK>
__device__ __forceinline__ void reg_unit(const FArgs &args, int tq, int ga, const u32x4 (&raw)[4], const uint4 *lds,
                                         unsigned &wsat) {
    constexpr int P = reg_seqs<M>(), TS = record_times(PREC), GA = reg_group<M, PREC>();
    constexpr int kSpan = 4 / P;  // consecutive spectra of an antenna in a lane
    const int lane = threadIdx.x & 63, j = lane & 15, g = lane >> 4;
    const h8_t *ops = reinterpret_cast<const h8_t *>(lds) + lane;

    // scales of the lane's bins, (c = 4 gamma + i, d) at [a][half][d][i][gamma], loaded an
    // i or more ahead and before the stores of the i at hand, which a wait for them would
    // else wait for too
    const int a = ga * GA + g * kSpan / TS;  // the lane's antenna
    float4 scales[4][P];
    auto load_scales = [&](int i) {
        if constexpr (is_quant(PREC)) {
            const float4 *src =
                reinterpret_cast<const float4 *>(args.scales_p) + ((int64_t)(a < args.N ? a : 0) * P * 16 + j) * 4 + i;
#pragma unroll
            for (int p = 0; p < P; ++p) scales[i][p] = src[p * 64];
        }
    };
    load_scales(0);

    // first product: halves of Y[f][4g + i], f = 4F + 2q' and + 1 in dwords [F][i][q']
    // (real parts) and [F][i][2 + q'] (imaginary parts)
    uint32_t hi[4][4][4], lo[4][4][4];
    float m1 = -1.0f;  // opaque: a known -1 turns the fma into a subtraction, which has no mixed-precision form
    asm volatile("" : "+v"(m1));
    // Step f: the operands of f + 1 are read, the samples of f + 1 unpacked and half of
    // the last finished pair of f split while the products of f run, so that no step
    // waits for LDS or for its own products.
    h8_t w[2][4], x[2];
    f4_t yr[4], yi[4];
    auto operands = [&](int f) {
#pragma unroll
        for (int o = 0; o < 4; ++o) w[f & 1][o] = ops[(4 * f + o) * 64];
    };
    auto split = [&](int f, const f4_t (&y)[4], int part) {  // of the pair f, f + 1
        const int F = f / 4, q = f / 2 % 2;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float u = y[f & 3][i], v = y[(f & 3) + 1][i];
            const h2_t h = __builtin_bit_cast(h2_t, __builtin_amdgcn_cvt_pkrtz(u, v));
            hi[F][i][2 * part + q] = __builtin_bit_cast(uint32_t, h);
            lo[F][i][2 * part + q] = __builtin_bit_cast(
                uint32_t, h2_t{(_Float16)__builtin_fmaf((float)h[0], m1, u), (_Float16)__builtin_fmaf((float)h[1], m1, v)});
        }
    };
    // P = 1: byte 8 s + f / 2 of a block; dword 2b + h of load q holds f = 8h .. 8h + 7 of
    // s = 8q + 2g + b.  P = 2: byte 16 s + f, the nibble the parity of the lane's
    // sequence; lanes j and j ^ 1 each loaded one of the two s of every q, and both take
    // both, nibble by nibble.  r: one f's (pair of f's) samples per dword.
    uint32_t r[2][4];
    const int sh = 4 * (j & 1);
    auto samples = [&](int f) {
        if constexpr (P == 1) {
            if (f % 8 == 0) {
                const int h = f / 8;
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    byte_transpose(raw[0][2 * b + h], raw[1][2 * b + h], raw[2][2 * b + h], raw[3][2 * b + h], r[b]);
            }
            const int k = f % 8 / 2, sf = 4 * (f & 1);
            x[f & 1] = nibbles_f16(r[0][k] >> sf, r[1][k] >> sf);
        } else {
            if (f % 4 == 0) {
                const int d = f / 4;
                uint32_t v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t even = __builtin_amdgcn_update_dpp(0, raw[q][d], 0xA0, 0xf, 0xf, true);
                    const uint32_t odd = __builtin_amdgcn_update_dpp(0, raw[q][d], 0xF5, 0xf, 0xf, true);
                    v[q] = ((even >> sh) & 0x0f0f0f0fu) | ((odd << (4 - sh)) & 0xf0f0f0f0u);
                }
                byte_transpose(v[0], v[1], v[2], v[3], r[0]);
            }
            x[f & 1] = nibbles_f16(r[0][f % 4], r[0][f % 4] >> 4);
        }
    };
    operands(0);
    samples(0);
#pragma unroll
    for (int f = 0; f < 16; ++f) {
        const f4_t zero = {0.0f, 0.0f, 0.0f, 0.0f};
        __builtin_amdgcn_sched_barrier(0);
        if (f + 1 < 16) operands(f + 1);
        const h8_t (&o)[4] = w[f & 1];
        f4_t &a = yr[f & 3], &b = yi[f & 3];
        a = mfma_h(o[1], x[f & 1], zero);
        b = mfma_h(o[3], x[f & 1], zero);
        a = mfma_h(o[0], x[f & 1], a);
        b = mfma_h(o[2], x[f & 1], b);
        if (f + 1 < 16) samples(f + 1);
        if (f >= 2) split((f - 2) & ~1, f & 1 ? yi : yr, f & 1);
        // operands first, then a product every few vector operations
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    split(14, yr, 0);
    split(14, yi, 1);
    h8_t b16[4];
#pragma unroll
    for (int o = 0; o < 4; ++o) b16[o] = ops[kRegB16 + o * 64];

    // where the records go: a buffer resource over the time block and offsets past its
    // range for padding antennas, as in tile_records
    const int n_store = (args.N + 7) & ~7;
    // The antennas after the last group have zeros already, but a line written in part
    // costs more than the stores that complete it at once: `tail` antennas of zeros after
    // this group (N = 44, 65536 spectra: fp16 0.97 -> 0.87 ms, int16 1.05 -> 0.97; N = 37, K =
    // 512, 16384 spectra: fp16 0.47 -> 0.39; written after the group's records and not
    // beside them, 0.95 and 0.43).  Not for the other forms, whose narrower groups would
    // need two or three such stores a record (N = 44 int8 0.64 -> 0.67).
    constexpr bool TAIL = GA >= 4 || PREC == kFP16;
    const int tail = TAIL && (ga + 1) * GA >= args.N ? (GA >= 4 ? n_store : (args.N + 3) & ~3) - (ga + 1) * GA : 0;
    const int tqb = __builtin_amdgcn_readfirstlane(tq / kTQB);
    const uint32_t rstep = (uint32_t)kTQB * (uint32_t)args.a_pad * kRecordBytes;  // from channel to channel
    const uint32_t span = (uint32_t)M * rstep;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        args.spec + (int64_t)tqb * M * kTQB * args.a_pad, 0, (int)span, kBufferRsrcFlags);
    const bool stored = a < n_store;
    const uint32_t row = ((uint32_t)(tq % kTQB) * (uint32_t)args.a_pad + (uint32_t)a) * kRecordBytes;
    // lane column d's bins are kd + sd c for c > 0 and 16 d for c = 0: byte offsets of them
    // (from an opaque lane column: what depends on it alone, as the channel numbers as
    // doubles that tracking takes, would be kept through all units, in registers that there
    // are none for, and reloaded behind the stores; tracked int8, N = 44: 0.31 -> 0.25 ms)
    int jo = j;
    asm volatile("" : "+v"(jo));
    const int kd = jo < 8 ? 32 * jo : 512 - 32 * jo, sd = jo < 8 ? 1 : -1;
    const uint32_t base = stored ? (uint32_t)kd * rstep + row : span, base0 = stored ? (uint32_t)(16 * j) * rstep + row : span;
    const int step = stored ? sd * (int)rstep : 0;
    const uint32_t mirror = stored ? 512u * rstep + 2u * row : 2u * span;  // bin 512 - k: at mirror - its offset
    TrackModel<M> model;
    if constexpr (TRACK) {
        const double4 *at = args.track + a;
        asm volatile("" : "+v"(at));  // not loaded before the first product, which needs the registers
        model.load(*at, args.s_base + tq * TS + g * kSpan % TS);
    }
    // y in odd lane groups, x in even ones (a select that stays one: from an array the
    // compiler would load at a selected address)
    auto odd_group = [&](uint32_t x, uint32_t y) { return x ^ ((x ^ y) & (uint32_t)-(g & 1)); };
    auto store = [&](uint4 rec, uint32_t off) {
        __builtin_amdgcn_raw_buffer_store_b128(u32x4{rec.x, rec.y, rec.z, rec.w}, rs, off, 0, 0);
        if constexpr (TAIL)
            for (int z = GA; z <= tail; z += GA)
                __builtin_amdgcn_raw_buffer_store_b128(u32x4{0, 0, 0, 0}, rs, off + (uint32_t)(z * kRecordBytes), 0, 0);
    };
    // second product of columns c = 8h + i and c + 4, n = 2i + h
    f4_t zr[2][2], zi[2][2];  // [n mod 2][column]
    auto second = [&](int n) {
        const int i = n >> 1, h = n & 1;
        if (h == 0) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                row_transpose(hi[0][i][q], hi[1][i][q], hi[2][i][q], hi[3][i][q]);
                row_transpose(lo[0][i][q], lo[1][i][q], lo[2][i][q], lo[3][i][q]);
            }
        }
        h8_t vh[2], vl[2], w0[4];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int gm = 2 * h + e;
            vh[e] = __builtin_bit_cast(h8_t, u32x4{hi[gm][i][0], hi[gm][i][1], hi[gm][i][2], hi[gm][i][3]});
            vl[e] = __builtin_bit_cast(h8_t, u32x4{lo[gm][i][0], lo[gm][i][1], lo[gm][i][2], lo[gm][i][3]});
        }
        if (n == 0) {
#pragma unroll
            for (int o = 0; o < 4; ++o) w0[o] = ops[kRegB0 + o * 64];
        }
        // (three products in turn: a product waits for no other one)
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const h8_t v = t == 0 ? vl[e] : vh[e];
                const int o = t == 1 ? 1 : 0;
                const f4_t zero = {0.0f, 0.0f, 0.0f, 0.0f};
                const h8_t wr = n == 0 && e == 0 ? w0[o] : b16[o], wi = n == 0 && e == 0 ? w0[2 + o] : b16[2 + o];
                zr[n & 1][e] = mfma_h(v, wr, t == 0 ? zero : zr[n & 1][e]);
                zi[n & 1][e] = mfma_h(v, wi, t == 0 ? zero : zi[n & 1][e]);
            }
    };

    // The next columns' products run beside a pair's vector work, but where their
    // registers would spill (N = 256, 1024-point, 16384 spectra: fp16 3.0 -> 2.5 ms; int8
    // 2.44, 2.36 without).
    constexpr bool AHEAD = !TRACK && !(P == 2 && PREC == kINT8);
    if constexpr (AHEAD) second(0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (i < 3) load_scales(i + 1);
        const float4 (&sc)[P] = scales[i];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if constexpr (!AHEAD) second(2 * i + h);
            else if (2 * i + h < 7) second(2 * i + h + 1);
            // bins [column][half], spectra of each, and where their records go
            float re[2][P][kSpan], im[2][P][kSpan], s[2][P];
            uint32_t at[2][P];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int gm = 2 * h + e, c = 4 * gm + i;
                const f4_t yr = zr[h][e], yi = zi[h][e];
                const int k = c == 0 ? 16 * jo : kd + sd * c;  // (tracking)
                at[e][0] = c == 0 ? base0 : base + (uint32_t)__mul24(c, step);
                if constexpr (P == 1) {
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        re[e][0][t] = yr[t];
                        // column 0 has bin 256 in bin 0's imaginary part
                        im[e][0][t] = c == 0 && j == 0 ? 0.0f : yi[t];
                    }
                    if constexpr (TRACK) model.template rotate<kSpan>((double)k, re[e][0], im[e][0]);
                } else {
                    // X[k] = E[k] + W O[k], X[512 - k] = conj(E[k] - W O[k]); bins 0 and 256
                    // of the sequences are real and lane (0, 0) has both
                    at[e][1] = mirror - at[e][0];
                    if (c == 0 && j == 0) at[e][1] = stored ? 256u * rstep + row : span;
                    const float2 w = reinterpret_cast<const float2 *>(lds + kRegTw2)[16 * c + j];
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const float2 E = make_float2(yr[2 * t], yi[2 * t]), O = make_float2(yr[2 * t + 1], yi[2 * t + 1]);
                        const float2 o = cmul(O, w);
                        re[e][0][t] = E.x + o.x;
                        im[e][0][t] = E.y + o.y;
                        re[e][1][t] = E.x - o.x;
                        im[e][1][t] = o.y - E.y;
                        if (c == 0 && j == 0) {
                            re[e][0][t] = E.x + O.x;
                            im[e][0][t] = 0.0f;
                            re[e][1][t] = E.y;
                            im[e][1][t] = -O.y;
                        }
                    }
                    if constexpr (TRACK) {
                        model.template rotate<kSpan>((double)k, re[e][0], im[e][0]);
                        model.template rotate<kSpan>((double)(c == 0 && j == 0 ? 256 : 512 - k), re[e][1], im[e][1]);
                    }
                }
#pragma unroll
                for (int p = 0; p < P; ++p)
                    if constexpr (is_quant(PREC)) s[e][p] = gm == 0 ? sc[p].x : gm == 1 ? sc[p].y : gm == 2 ? sc[p].z : sc[p].w;
            }
            if constexpr (PREC == kFP16) {
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    if constexpr (P == 1) {
                        store(make_uint4(pack_f16(re[e][0][0], re[e][0][1]), pack_f16(re[e][0][2], re[e][0][3]),
                                         pack_f16(im[e][0][0], im[e][0][1]), pack_f16(im[e][0][2], im[e][0][3])), at[e][0]);
                    } else {
                        uint32_t r0 = pack_f16(re[e][0][0], re[e][0][1]), r1 = pack_f16(re[e][1][0], re[e][1][1]);
                        uint32_t m0 = pack_f16(im[e][0][0], im[e][0][1]), mm = pack_f16(im[e][1][0], im[e][1][1]);
                        pair_exchange(r0, r1);
                        pair_exchange(m0, mm);
                        store(make_uint4(r0, r1, m0, mm), odd_group(at[e][0], at[e][1]));
                    }
                }
            } else if constexpr (PREC == kINT16) {
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    if constexpr (P == 1) {
                        store(make_record<kINT16, 4>(re[e][0], im[e][0], s[e][0], wsat), at[e][0]);
                    } else {
                        // per bin the digits' bytes of two spectra: high [re re im im], low the same
                        float x[2][4], qm[2][4];
                        uint32_t hd[2], ld[2];
#pragma unroll
                        for (int p = 0; p < 2; ++p) {
                            x[p][0] = re[e][p][0], x[p][1] = re[e][p][1];
                            x[p][2] = im[e][p][0], x[p][3] = im[e][p][1];
                        }
                        quantise_bins<2, 4>(x, s[e], (float)kI16Max, wsat, qm);
#pragma unroll
                        for (int p = 0; p < 2; ++p) {
                            uint32_t hb[4], lb[4];
#pragma unroll
                            for (int t = 0; t < 4; ++t) int16_digit_bits(qm[p][t], hb[t], lb[t]);
                            hd[p] = pack_bytes(hb[0], hb[1], hb[2], hb[3]);
                            ld[p] = pack_bytes(lb[0], lb[1], lb[2], lb[3]);
                        }
                        pair_exchange(hd[0], hd[1]);
                        pair_exchange(ld[0], ld[1]);
                        store(make_uint4(__builtin_amdgcn_perm(hd[1], hd[0], 0x05040100u),
                                         __builtin_amdgcn_perm(hd[1], hd[0], 0x07060302u),
                                         __builtin_amdgcn_perm(ld[1], ld[0], 0x05040100u),
                                         __builtin_amdgcn_perm(ld[1], ld[0], 0x07060302u)), odd_group(at[e][0], at[e][1]));
                    }
                }
            } else if constexpr (P == 1) {
                // int8: both columns' four spectra; the pair of lane groups of an antenna
                // (spectra 0-3 and 4-7) exchange, the even one for column c, the odd one for c + 4
                float x[2][8], qm[2][8], sb[2] = {s[0][0], s[1][0]};
                uint32_t rw[2], iw[2];
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int t = 0; t < 4; ++t) x[e][t] = re[e][0][t], x[e][4 + t] = im[e][0][t];
                quantise_bins<2, 8>(x, sb, 127.0f, wsat, qm);
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    // the low byte of 1.5 * 2^23 + q is q as two's complement
                    uint32_t b[8];
#pragma unroll
                    for (int t = 0; t < 8; ++t) b[t] = __float_as_uint(qm[e][t]);
                    rw[e] = pack_bytes(b[0], b[1], b[2], b[3]);
                    iw[e] = pack_bytes(b[4], b[5], b[6], b[7]);
                }
                pair_exchange(rw[0], rw[1]);
                pair_exchange(iw[0], iw[1]);
                store(make_uint4(rw[0], rw[1], iw[0], iw[1]), odd_group(at[0][0], at[1][0]));
            } else {
                // int8: two spectra of four bins in each lane group; the lane groups take a bin each
                float x[4][4], qm[4][4], sb[4];
                uint32_t v[4];
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const int e = b >> 1, p = b & 1;
                    x[b][0] = re[e][p][0], x[b][1] = re[e][p][1];
                    x[b][2] = im[e][p][0], x[b][3] = im[e][p][1];
                    sb[b] = s[e][p];
                }
                quantise_bins<4, 4>(x, sb, 127.0f, wsat, qm);
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    v[b] = pack_bytes(__float_as_uint(qm[b][0]), __float_as_uint(qm[b][1]), __float_as_uint(qm[b][2]),
                                      __float_as_uint(qm[b][3]));
                row_transpose(v[0], v[1], v[2], v[3]);
                store(make_uint4(__builtin_amdgcn_perm(v[1], v[0], 0x05040100u),
                                 __builtin_amdgcn_perm(v[3], v[2], 0x05040100u),
                                 __builtin_amdgcn_perm(v[1], v[0], 0x07060302u),
                                 __builtin_amdgcn_perm(v[3], v[2], 0x07060302u)),
                      g & 2 ? odd_group(at[1][0], at[1][1]) : odd_group(at[0][0], at[0][1]));
            }
        }
    }
}

template <int PREC>
__device__ __forceinline__ void reg_add_sat(const FArgs &args, unsigned wsat) {
    if constexpr (is_quant(PREC)) {
        if ((threadIdx.x & 63) == 0 && wsat) atomicAdd(args.sat, (unsigned long long)wsat);
    }
}

// Units [u0, u1), u0 and u1 multiples of 4, by a workgroup; the next set's bytes are
// loaded while one is transformed.
template <int M, int PREC>
__device__ __forceinline__ void reg_units(const FArgs &args, int u0, int u1, const uint4 *lds) {
    if (u0 >= u1) return;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int tq, ga, tn, gn;
    reg_unit_at(u0 + w, args.ngroups, tq, ga);
    u32x4 raw[4];
    reg_load<M, PREC>(args, tq, ga, raw);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // as in f_tiles
    unsigned wsat = 0;
    for (int u = u0; u < u1; u += 4) {
        u32x4 cur[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) cur[q] = raw[q];
        reg_unit_at((u + 4 < u1 ? u + 4 : u) + w, args.ngroups, tn, gn);
        reg_load<M, PREC>(args, tn, gn, raw);
        reg_unit<M, PREC, false>(args, tq, ga, cur, lds, wsat);
        tq = tn;
        ga = gn;
        __builtin_amdgcn_s_barrier();  // the wavefronts start a set together
    }
    reg_add_sat<PREC>(args, wsat);
}

// Sets of four units, first `set`, whose bytes raw holds, then `next`, then base + ticket
// for tickets of *ctr (zero at launch), below hi, as f_tiles_dyn deals tiles: thread 0
// holds a ticket ahead and publishes the next one in s_tk before the barrier that ends a
// set.
template <int M, int PREC, bool TRACK>
__device__ __forceinline__ void reg_sets(const FArgs &args, int set, int next, int base, int hi, unsigned *ctr, int *s_tk,
                                         const uint4 *lds, u32x4 (&raw)[4]) {
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tq, ga, tn, gn;
    reg_unit_at(4 * set + w, args.ngroups, tq, ga);
    unsigned wsat = 0, tk = 0;
    for (;;) {
        if (tid == 0) tk = atomicInc(ctr, 0xffffffffu);
        u32x4 cur[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) cur[q] = raw[q];
        // the last set re-reads its own bytes rather than branch around the load
        reg_unit_at(4 * (next < hi ? next : set) + w, args.ngroups, tn, gn);
        reg_load<M, PREC>(args, tn, gn, raw);
        reg_unit<M, PREC, TRACK>(args, tq, ga, cur, lds, wsat);
        if (tid == 0) s_tk[0] = (int)tk;
        __syncthreads();  // s_tk published; the wavefronts start a set together
        if (next >= hi) break;
        set = next;
        tq = tn;
        ga = gn;
        next = base + s_tk[0];
        __syncthreads();  // s_tk has been read
    }
    reg_add_sat<PREC>(args, wsat);
}

// Load the bytes of this wavefront's unit of a set.
template <int M, int PREC>
__device__ __forceinline__ void reg_load_set(const FArgs &args, int set, u32x4 (&raw)[4]) {
    int tq, ga;
    reg_unit_at(4 * set + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), args.ngroups, tq, ga);
    reg_load<M, PREC>(args, tq, ga, raw);
}

// Sets [lo, hi), every one by ticket.
template <int M, int PREC, bool TRACK>
__device__ __forceinline__ void reg_units_dyn(const FArgs &args, int lo, int hi, unsigned *ctr, int *s_tk,
                                              const uint4 *lds) {
    if (threadIdx.x == 0) {
        s_tk[0] = (int)atomicAdd(ctr, 1u);
        s_tk[1] = (int)atomicAdd(ctr, 1u);
    }
    __syncthreads();
    const int set = lo + s_tk[0], next = lo + s_tk[1];
    __syncthreads();  // s_tk[0] is rewritten below
    if (set >= hi) return;
    u32x4 raw[4];
    reg_load_set<M, PREC>(args, set, raw);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // as in f_tiles
    reg_sets<M, PREC, TRACK>(args, set, next, lo, hi, ctr, s_tk, lds, raw);
}

}  // namespace
}  // namespace corr
