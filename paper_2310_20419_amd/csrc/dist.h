// delta(a, b) = squared Euclidean distance of two rows of X (Eq. 3 with dist = squared L2),
// computed by a group of 8 consecutive lanes; all 8 receive the result.
//
//   uint8 rows : exact int32, sum of (a-b)^2 through three byte dot products per word.
//   16-bit rows: IEEE binary16 (DT_F16) or bfloat16 (DT_BF16) storage; every coordinate stands for the
//                float it converts to exactly, and the arithmetic is that of float rows (8 coordinates
//                per 16-byte chunk).
//   float rows : each lane accumulates (double)(a-b)^2 over its 16-byte chunks in chunk order,
//                the 8 partial sums are combined in a fixed xor tree, and the double is rounded
//                once to float.  (a-b)^2 == (b-a)^2 exactly, so delta(a,b) and delta(b,a) are the
//                same bits wherever they are computed.
// The result is returned as the 32 "dist_bits" of a key: the int32 value, or the float's bit pattern.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "wave_prims.h"

#define DT_U8 0
#define DT_F32 1
#define DT_F16 2
#define DT_BF16 3

// bytes of one coordinate
__host__ __device__ constexpr int dt_size(int dt) { return dt == DT_U8 ? 1 : (dt == DT_F16 || dt == DT_BF16) ? 2 : 4; }

// Sum over the 8 lanes of a group, every lane receiving it: partner 1, then 2, then 4 (a fixed order, so the
// double sums are the same bits wherever they are formed).  The exchanges inside a quad are DPP moves.
__device__ __forceinline__ int group8_sum(int v)
{
    v += (int)xor_lane_u32<1>((uint32_t)v);
    v += (int)xor_lane_u32<2>((uint32_t)v);
    v += (int)xor_lane_u32<4>((uint32_t)v);
    return v;
}
__device__ __forceinline__ double group8_sum(double v)
{
    v += __builtin_bit_cast(double, xor_lane_u64(__builtin_bit_cast(unsigned long long, v), 1));
    v += __builtin_bit_cast(double, xor_lane_u64(__builtin_bit_cast(unsigned long long, v), 2));
    v += __builtin_bit_cast(double, xor_lane_u64(__builtin_bit_cast(unsigned long long, v), 4));
    return v;
}

// The same sum in the first four lanes of a group only: what comes from lane l + 4 is a DPP shift by 4, not a trip through the LDS unit.
__device__ __forceinline__ int group8_sum_low(int v)
{
    v += (int)xor_lane_u32<1>((uint32_t)v);
    v += (int)xor_lane_u32<2>((uint32_t)v);
    v += __builtin_amdgcn_update_dpp(0, v, 0x104, 0xF, 0xF, true);      // row_shl:4
    return v;
}
__device__ __forceinline__ double group8_sum_low(double v)
{
    v += __builtin_bit_cast(double, xor_lane_u64(__builtin_bit_cast(unsigned long long, v), 1));
    v += __builtin_bit_cast(double, xor_lane_u64(__builtin_bit_cast(unsigned long long, v), 2));
    const u64 w = __builtin_bit_cast(u64, v);
    const u32 lo = (u32)__builtin_amdgcn_update_dpp(0, (int)(u32)w, 0x104, 0xF, 0xF, true);
    const u32 hi = (u32)__builtin_amdgcn_update_dpp(0, (int)(u32)(w >> 32), 0x104, 0xF, 0xF, true);
    v += __builtin_bit_cast(double, (u64)hi << 32 | lo);
    return v;
}

// a 16-bit stored coordinate as the float it stands for (exact)
template <int DT>
__device__ __forceinline__ float coord16_to_float(unsigned short bits)
{
    if (DT == DT_BF16) return __uint_as_float((uint32_t)bits << 16);
    return (float)__builtin_bit_cast(_Float16, bits);
}

// acc + the sum over 16 bytes of (a - b)^2 = a.a + b.b - 2 a.b; every term fits comfortably in 32 bits.  The products accumulate in the dot
// instructions themselves, and b.b is apart, so that it is formed once for several rows a.  (Together with group8_sum_low, the vector instructions of the
// uint8 search 1,013 -> 991 and 8 trips through the LDS unit less: 10,000 queries on 1M x 128, which are bound by issue, 871 -> 831 us.)
__device__ __forceinline__ int sqdiff_piece_u8(const uint4 &a, const uint4 &b, int acc)
{
    uint32_t bb = __builtin_amdgcn_udot4(b.x, b.x, 0u, false);
    bb = __builtin_amdgcn_udot4(b.y, b.y, bb, false);
    bb = __builtin_amdgcn_udot4(b.z, b.z, bb, false);
    bb = __builtin_amdgcn_udot4(b.w, b.w, bb, false);
    uint32_t ab = __builtin_amdgcn_udot4(a.x, b.x, 0u, false);
    ab = __builtin_amdgcn_udot4(a.y, b.y, ab, false);
    ab = __builtin_amdgcn_udot4(a.z, b.z, ab, false);
    ab = __builtin_amdgcn_udot4(a.w, b.w, ab, false);
    uint32_t aa = __builtin_amdgcn_udot4(a.x, a.x, (uint32_t)acc + bb, false);
    aa = __builtin_amdgcn_udot4(a.y, a.y, aa, false);
    aa = __builtin_amdgcn_udot4(a.z, a.z, aa, false);
    aa = __builtin_amdgcn_udot4(a.w, a.w, aa, false);
    return (int)(aa - 2u * ab);
}

// UF (float rows): 16-byte chunks per lane whose loads are issued together before the (ordered)
// accumulation; it changes how many loads are in flight, never the order of the arithmetic.  UF >= 2.
// TOGETHER (16-bit rows): inside the float16 merges the scheduler waits for one piece after the other, so that the conversions take fewer registers.  Rows of more than 128
// coordinates, which take several trips, there have a loop of their own in which a barrier keeps the loads before the arithmetic.  With two pieces a trip nothing spills (three: the same
// within 8 % either way); in that loop rows of up to 128 took 1-4 % longer.  8 rounds, R = 96, before / now, ms: 300,000 x 160 6.83 / 5.88, x 320 8.84 / 8.43, x 960 27.8 / 22.9,
// 20,000 x 768 2.08 / 1.51; 1M x 640, R = 32, 5 rounds 45.9 / 39.8.
template <int DT, int UF = 4, bool TOGETHER = false>
__device__ __forceinline__ uint32_t group8_dist_bits(const void *pa, const void *pb, int d,
                                                     int vec_ok, int sub)
{
    if (DT == DT_U8) {
        const uint8_t *a = (const uint8_t *)pa, *b = (const uint8_t *)pb;
        int acc = 0;
        if (vec_ok) {
            const int nchunk = d >> 4;
            for (int c = sub; c < nchunk; c += 8) {
                uint4 va = ((const uint4 *)a)[c], vb = ((const uint4 *)b)[c];
                acc = sqdiff_piece_u8(va, vb, acc);
            }
        } else {
            for (int e = sub; e < d; e += 8) {
                int t = (int)a[e] - (int)b[e];
                acc += t * t;
            }
        }
        acc = group8_sum(acc);
        return (uint32_t)acc;
    } else if (DT == DT_F16 || DT == DT_BF16) {
        const unsigned short *a = (const unsigned short *)pa, *b = (const unsigned short *)pb;
        typedef unsigned short us8 __attribute__((ext_vector_type(8)));
        double acc = 0.0;
        if (vec_ok) {
            const int nchunk = d >> 3;
            const us8 *pa8 = (const us8 *)a, *pb8 = (const us8 *)b;
            int c = sub;
            constexpr int TAIL = TOGETHER ? 2 : UF - 1;
            if (TOGETHER) {
                for (; nchunk > 8 * TAIL && c - sub < nchunk; c += 8 * UF) {
                    us8 va[UF], vb[UF];
                    if (c - sub + 8 * UF <= nchunk) {
#pragma unroll
                        for (int k = 0; k < UF; ++k) { va[k] = pa8[c + 8 * k]; vb[k] = pb8[c + 8 * k]; }
                    } else {
#pragma unroll
                        for (int k = 0; k < UF; ++k) {      // (as below)
                            const bool in = c + 8 * k < nchunk;
                            va[k] = in ? pa8[c + 8 * k] : (us8)(0);
                            vb[k] = in ? pb8[c + 8 * k] : (us8)(0);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int k = 0; k < UF; ++k)
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const double t = (double)coord16_to_float<DT>(va[k][e]) - (double)coord16_to_float<DT>(vb[k][e]);
                            acc = fma(t, t, acc);
                        }
                }
            } else {
                for (; c + 8 * (UF - 1) < nchunk; c += 8 * UF) {
                    us8 va[UF], vb[UF];
#pragma unroll
                    for (int k = 0; k < UF; ++k) { va[k] = pa8[c + 8 * k]; vb[k] = pb8[c + 8 * k]; }
#pragma unroll
                    for (int k = 0; k < UF; ++k)
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const double t = (double)coord16_to_float<DT>(va[k][e]) - (double)coord16_to_float<DT>(vb[k][e]);
                            acc = fma(t, t, acc);
                        }
                }
            }
            if (c < nchunk) {
                // the last, shorter trip: its loads are issued together as well; a chunk past the end reads as zeros,
                // and adding the square of 0 - 0 leaves the sum as it is, so the arithmetic is that of the short loop
                us8 va[TAIL > 0 ? TAIL : 1], vb[TAIL > 0 ? TAIL : 1];
#pragma unroll
                for (int k = 0; k < TAIL; ++k) {
                    const bool in = c + 8 * k < nchunk;
                    va[k] = in ? pa8[c + 8 * k] : (us8)(0);
                    vb[k] = in ? pb8[c + 8 * k] : (us8)(0);
                }
#pragma unroll
                for (int k = 0; k < TAIL; ++k)
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const double t = (double)coord16_to_float<DT>(va[k][e]) - (double)coord16_to_float<DT>(vb[k][e]);
                        acc = fma(t, t, acc);
                    }
            }
        } else {
            for (int e = sub; e < d; e += 8) {
                const double t = (double)coord16_to_float<DT>(a[e]) - (double)coord16_to_float<DT>(b[e]);
                acc = fma(t, t, acc);
            }
        }
        acc = group8_sum(acc);
        return __float_as_uint((float)acc);
    } else {
        const float *a = (const float *)pa, *b = (const float *)pb;
        double acc = 0.0;
        if (vec_ok) {
            const int nchunk = d >> 2;
            const float4 *pa4 = (const float4 *)a, *pb4 = (const float4 *)b;
            int c = sub;
            // UF chunks per trip, all 2 UF loads issued before the (ordered) accumulation
            for (; c + 8 * (UF - 1) < nchunk; c += 8 * UF) {
                float4 va[UF], vb[UF];
#pragma unroll
                for (int k = 0; k < UF; ++k) { va[k] = pa4[c + 8 * k]; vb[k] = pb4[c + 8 * k]; }
#pragma unroll
                for (int k = 0; k < UF; ++k) {
                    double t;
                    t = (double)va[k].x - (double)vb[k].x; acc = fma(t, t, acc);
                    t = (double)va[k].y - (double)vb[k].y; acc = fma(t, t, acc);
                    t = (double)va[k].z - (double)vb[k].z; acc = fma(t, t, acc);
                    t = (double)va[k].w - (double)vb[k].w; acc = fma(t, t, acc);
                }
            }
            if (c < nchunk) {
                // the last, shorter trip: its loads are issued together as well; a chunk past the end reads as zeros,
                // and adding the square of 0 - 0 leaves the sum as it is, so the arithmetic is that of the short loop
                float4 va[UF - 1 > 0 ? UF - 1 : 1], vb[UF - 1 > 0 ? UF - 1 : 1];
#pragma unroll
                for (int k = 0; k < UF - 1; ++k) {
                    const bool in = c + 8 * k < nchunk;
                    va[k] = in ? pa4[c + 8 * k] : make_float4(0.f, 0.f, 0.f, 0.f);
                    vb[k] = in ? pb4[c + 8 * k] : make_float4(0.f, 0.f, 0.f, 0.f);
                }
#pragma unroll
                for (int k = 0; k < UF - 1; ++k) {
                    double t;
                    t = (double)va[k].x - (double)vb[k].x; acc = fma(t, t, acc);
                    t = (double)va[k].y - (double)vb[k].y; acc = fma(t, t, acc);
                    t = (double)va[k].z - (double)vb[k].z; acc = fma(t, t, acc);
                    t = (double)va[k].w - (double)vb[k].w; acc = fma(t, t, acc);
                }
            }
        } else {
            for (int e = sub; e < d; e += 8) {
                double t = (double)a[e] - (double)b[e];
                acc = fma(t, t, acc);
            }
        }
        acc = group8_sum(acc);
        return __float_as_uint((float)acc);
    }
}
