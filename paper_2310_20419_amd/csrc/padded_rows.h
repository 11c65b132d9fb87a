// Copies of X whose rows have a length that the matrix-core scans take.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "half_rows.h"
#include "wave_prims.h"

// Rows the matrix instructions cannot take as they lie in X (a length that is no multiple of 64 bytes, or an X that is
// not 16-byte aligned): a copy with rows of rb bytes, a multiple of 128, zeros past the end of a row (they add nothing
// to a product or to a squared difference).  A distance must come out with the same bits as from X itself, because
// RandomGraph and the step-wise calls compute it there and equal edges must carry equal keys.  dist.h adds the
// coordinates of lane s of 8 in the order of the lane's 16-byte pieces s, s + 8, ... where X can be read in such pieces:
// then the copy keeps the order of the coordinates (permute = 0).  Otherwise lane s takes coordinates s, s + 8, ...
// one by one, and the copy puts the next coordinates of that sequence into the lane's next piece: piece 8 b + s holds
// coordinates V b + s, V b + s + 8, ... (V = 128 / size of a coordinate; permute = 1).  Distances and products do not
// depend on the order of the coordinates otherwise.  The copy streams (200,000 x 100: about 60 us); the build it makes
// possible: 200,000 x 100 float 95.7 -> 34.0 ms, S = 20, R = 96, 60 rounds.
template <typename T>      // uint32_t: float rows, unsigned short: 16-bit rows
__device__ __forceinline__ uint4 padded_piece(const T *x, int c, int d, int permute, u32 exponent, bool &odd)     // piece c of the copy of row x
{
    constexpr int V = 16 / (int)sizeof(T);      // coordinates per piece
    const int e0 = permute ? 8 * V * (c >> 3) + (c & 7) : V * c, step = permute ? 8 : 1;
    T t[V];
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const int e = e0 + k * step;
        t[k] = e < d ? x[e] : (T)0;
        odd = odd || ((u32)t[k] & exponent) == exponent;       // exponent bits all set: NaN or infinity
    }
    if constexpr (sizeof(T) == 4)
        return make_uint4(t[0], t[1], t[2], t[3]);
    else
        return make_uint4((u32)t[0] | (u32)t[1] << 16, (u32)t[2] | (u32)t[3] << 16, (u32)t[V - 4] | (u32)t[V - 3] << 16,
                          (u32)t[V - 2] | (u32)t[V - 1] << 16);
}

template <typename T>
__device__ __forceinline__ bool pad_all_rows(const T *__restrict__ X, long long N, int d, u32 rb, int permute, u32 exponent, uint4 *__restrict__ Xp)
{
    const u32 pieces = rb / 16u;
    bool odd = false;
    for (u64 i = (u64)blockIdx.x * 256u + threadIdx.x; i < (u64)N * pieces; i += (u64)gridDim.x * 256u) {
        const u64 u = i / pieces;
        Xp[i] = padded_piece<T>(X + u * (u64)d, (int)(i - u * pieces), d, permute, exponent, odd);
    }
    return odd;
}

template <typename T>
__global__ __launch_bounds__(256) void k_prepare_rows(const T *__restrict__ X, long long N, int d, u32 rb, int permute,
                                                      u32 exponent, uint4 *__restrict__ Xp, u32 *__restrict__ nonfinite)
{
    if (pad_all_rows<T>(X, N, d, rb, permute, exponent, Xp)) *nonfinite = 1u;
}

// centre[c] = mean of coordinate c over the sample, square[b] = sum of the squared deviations of the 64 coordinates of block b.
// Sixteen wavefronts share the sample's rows, 32 loads in flight each: a chain of 128 loads in four took 38 us, a
// hundredth of a 20,000-vertex build.
__global__ __launch_bounds__(1024) void k_half_centre(const float *__restrict__ X, long long N, int d, float *__restrict__ centre,
                                                      float *__restrict__ square, HalfPar *__restrict__ par)
{
    __shared__ double s1[16][64], s2[16][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = blockIdx.x * 64 + lane, n = (int)(N < HALF_SAMPLE ? N : HALF_SAMPLE);
    const float *col = X + (c < d ? c : d - 1);
    if (blockIdx.x == 0 && threadIdx.x == 0) par->share_bits = par->rest_bits = 0u;
    float v[HALF_SAMPLE / 16];
#pragma unroll
    for (int k = 0; k < HALF_SAMPLE / 16; ++k) {
        const int i = wave + 16 * k;
        v[k] = col[(size_t)((i < n ? i : 0) * N / n) * d];
    }
    double a = 0.0, b = 0.0;
#pragma unroll
    for (int k = 0; k < HALF_SAMPLE / 16; ++k) {
        const double x = wave + 16 * k < n && fabsf(v[k]) <= 3.0e38f ? (double)v[k] : 0.0;
        a += x;
        b = fma(x, x, b);
    }
    s1[wave][lane] = a;
    s2[wave][lane] = b;
    __syncthreads();
    if (wave == 0) {
        for (int w = 1; w < 16; ++w) {
            a += s1[w][lane];
            b += s2[w][lane];
        }
        const double mean = a / (double)n;
        if (c < d) centre[c] = (float)mean;
        double dev = b - mean * a;
        dev = c < d && dev > 0.0 ? dev : 0.0;
        for (int o = 32; o > 0; o >>= 1) dev += __builtin_bit_cast(double, shfl_xor_u64(__builtin_bit_cast(u64, dev), o));
        if (lane == 0) square[blockIdx.x] = (float)fmin(dev, 3.0e38);
    }
}

// L lanes per row, 8 coordinates (16 bytes of the copy) per lane and trip.
template <int L>
__global__ __launch_bounds__(256) void k_half_rows(const float *__restrict__ X, long long N, int d, int vec_ok, u32 rowbytes,
                                                   const float *__restrict__ centre, const float *__restrict__ square,
                                                   char *__restrict__ H, HalfPar *__restrict__ par)
{
    __shared__ float s[4][2];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, sub = lane & (L - 1);
    const int n = (int)(N < HALF_SAMPLE ? N : HALF_SAMPLE), nsq = (d + 63) / 64;
    double tot = 0.0;
    for (int k = lane; k < nsq; k += 64) tot += (double)square[k];
    for (int o = 32; o > 0; o >>= 1) tot += __builtin_bit_cast(double, shfl_xor_u64(__builtin_bit_cast(u64, tot), o));
    const float ms = (float)(tot / ((double)n * (double)d));
    int e = ms > 0.f && ms < 3.0e38f ? -4 - (ilogbf(ms) >> 1) : 0;
    e = e < -60 ? -60 : e > 60 ? 60 : e;
    if (blockIdx.x == 0 && threadIdx.x == 0) par->exponent = e;
    const float scale = ldexpf(1.f, e);
    const int pieces = (int)(rowbytes / 16u);
    const float small = (float)d * 0x1p-18f;
    float share = 0.f, rest = 0.f;
    for (u64 row = ((u64)blockIdx.x * 256u + threadIdx.x) / L; row < (u64)N; row += (u64)gridDim.x * (256u / L)) {
        const float *x = X + row * (u64)d;
        double err = 0.0;
        float nrm = 0.f;
        for (int p = sub; p < pieces; p += L) {
            v8h h;
            float v[8], m[8];
            if (vec_ok && 8 * p + 8 <= d) {
                *(float4 *)&v[0] = ((const float4 *)(x + 8 * p))[0];
                *(float4 *)&v[4] = ((const float4 *)(x + 8 * p))[1];
                *(float4 *)&m[0] = ((const float4 *)(centre + 8 * p))[0];
                *(float4 *)&m[4] = ((const float4 *)(centre + 8 * p))[1];
            } else {
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int c = 8 * p + k;
                    v[k] = c < d ? x[c] : 0.f;
                    m[k] = c < d ? centre[c] : 0.f;
                }
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float t = (v[k] - m[k]) * scale;
                h[k] = fabsf(t) <= 65504.f ? (_Float16)t : (_Float16)__uint_as_float(0x7FC00000u);
                const float hf = (float)h[k];
                const double r = ((double)v[k] - (double)m[k]) * (double)scale - (double)hf;
                err = fma(r, r, err);
                nrm = fmaf(hf, hf, nrm);
            }
            *(v8h *)(H + row * (u64)rowbytes + 16u * (u32)p) = h;
        }
#pragma unroll
        for (int o = L / 2; o > 0; o >>= 1) {
            err += __builtin_bit_cast(double, shfl_xor_u64(__builtin_bit_cast(u64, err), o));
            nrm += __shfl_xor(nrm, o);
        }
        // a row of NaN compares false and counts for neither
        if (nrm >= small) share = fmaxf(share, (float)sqrt(err / (double)nrm));
        else if (nrm < small) rest = fmaxf(rest, (float)sqrt(err));
    }
    for (int o = 32; o > 0; o >>= 1) {
        share = fmaxf(share, __shfl_xor(share, o));
        rest = fmaxf(rest, __shfl_xor(rest, o));
    }
    if (lane == 0) { s[wave][0] = share; s[wave][1] = rest; }
    __syncthreads();
    if (threadIdx.x < 2) {
        float m = fmaxf(fmaxf(s[0][threadIdx.x], s[1][threadIdx.x]), fmaxf(s[2][threadIdx.x], s[3][threadIdx.x]));
        if (m > 0.f) atomicMax(threadIdx.x ? &par->rest_bits : &par->share_bits, __float_as_uint(m));
    }
}
