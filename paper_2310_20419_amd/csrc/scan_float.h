// UpdateNeighbors scan (Alg. 4, the body of the vertex loop) for float rows on the 16-bit matrix cores: 16-bit rows as they are
// stored, float32 rows through their half-precision copy (see HalfRows).  The walk, the tiles and the masks are those of
// the uint8 scan (scan_mfma.h); what differs is that a tile only decides pairs beyond its error bound.
//
// With n_i the diagonal of the Gram tiles of v_mfma_f32_32x32x16_{f16,bf16} and D_i = delta(u, v_i), row i fails against column j
// iff D_i >= delta(v_i, w_j).  The tile gives
//     P_ij = 2 <x_i, x_j> - n_j + (D_i - n_i) = D_i - delta~(v_i, w_j) ,
// certain to fail where P_ij >= tol_i, certain to pass where P_ij < -tol_i, undecided between.  tol_i covers, for every
// column j of the list with n_j <= nmax:
//   - the block: one instruction adds 16 products and the accumulator; taking its error as at most 16 x 2^-24 of the sum of
//     their magnitudes (an in-bounds probe against double precision: 1.8 for operands of one size, 5.7 for operands spread over 20
//     binades), G and either norm are off by d 2^-24 of sqrt(n_i n_j) resp. n, hence (2 d + 20) 2^-24 (n_i + nmax), the
//     constant for the evaluation of P and the rounding of delta to float.  Subnormal halves enter such a sum with the
//     smallest normal exponent, which loses them up to 2^-24 of 2^-28 each (10.3 x 2^-24 measured): 2^-46 d on top for binary16;
//   - float32 rows, h_i in place of x_i: with r_i >= |x_i - h_i|, rho = r_i + rmax and b = |h_i - h_j| the distance
//     a = |x_i - x_j| is within rho of b.  a <= sqrt(D_i) where b^2 <= (sqrt(D_i) - rho)^2, a > sqrt(D_i) where
//     b^2 > (sqrt(D_i) + rho)^2, hence 2 sqrt(D_i) rho + rho^2;
//   - what falls below the smallest normal number.
// Rows or distances that are not finite, or beyond 10^36, leave all their pairs undecided.
//
// An undecided pair is resolved in double precision only if its outcome can matter: its column may be kept, and no column before it
// prunes the row for certain; a vertex, or a
// group of short-list vertices, with more than FLOAT_PAIR_CAP such pairs (ties in bulk) is left as it is, and scanned by the same
// wavefront at the end of its walk on double-precision tiles.  The redirected edges are stored without their delta(v,w): the merge at w computes it (close_keys), where the row
// of w serves every edge w receives, at twice the scan's occupancy and next to a sort that leaves the memory idle.
//
// Measured on 60-round builds (scan kernels, ms; against 16-row groups of whole float32 rows, which also computed the redirected
// distances: 119 and 871): 1M x 96 58 ms, vector units 0.57 busy, 6.0 TB/s fetched; 1M x 960 300 ms, 5.9 TB/s; 300,000 x 768 bfloat16
// 70 ms, 6.2 TB/s.  Random rows in 128-byte chunks reach 6.9 TB/s.
#pragma once
#include "round.h"
#include "scan_mfma.h"
#include "half_rows.h"
#include "dist.h"
#include "scan_mfma_f32.h"

typedef float v16f __attribute__((ext_vector_type(16)));

#define FLOAT_PAIR_CAP 256

template <int NG>
struct alignas(16) FloatScanSmem {
    float gt[NG > 1 ? 1024 * NG : 32 * GT_STRIDE];      // the rows on their way; a diagonal Gram tile; later the undecided pairs: row << 8 | column, then their distances
    float nrm[32 * NG];            // n_j by list position
    int id[32 * NG];               // vertex id by list position
    int left;                      // see leave_vertex
};

// The rows of the exact routine and what the tolerance is made of; the same for every vertex of a launch.
struct FloatRows {
    const char *X;                 // rows of d coordinates, 16-byte pieces
    int d;
    const HalfPar *par;            // float32 rows
    int *left;                     // [N] see leave_vertex; null: vertices go to `redo` instead
    int *redo;                     // [N] vertices left to a launch that follows: all, or those with more than 96 entries ...
    u32 *n_redo;                   // ... and how many
    long long N;
};

// The vertices that a wavefront leaves alone (lists of up to 96 entries), to be scanned in double precision at the end of its walk: a
// chain from the last one to the first through an array by vertex.  Its head is in LDS, so that the walk keeps nothing for it.
__device__ __forceinline__ void leave_vertex(int u, const FloatRows &fr, int *head, bool first_lane, bool longest)
{
    if (longest || !fr.left) {
        if (first_lane) fr.redo[atomicAdd(fr.n_redo, 1u)] = u;
    } else if (first_lane) {
        fr.left[u] = *head;
        *head = u;
    }
}

__device__ __forceinline__ u32 both_halves(u64 b) { return (u32)b | (u32)(b >> 32); }

// maximum over the 32 lanes of a half-wave (both halves hold the same values), v >= 0
__device__ __forceinline__ float half_wave_max(float v)
{
    v = fmaxf(v, __uint_as_float(xor_lane_u32<1>(__float_as_uint(v))));
    v = fmaxf(v, __uint_as_float(xor_lane_u32<2>(__float_as_uint(v))));
    v = fmaxf(v, __uint_as_float(xor_lane_u32<4>(__float_as_uint(v))));
    v = fmaxf(v, __uint_as_float(xor_lane_u32<8>(__float_as_uint(v))));
    v = fmaxf(v, __uint_as_float(xor_lane_u32<16>(__float_as_uint(v))));
    return v;
}

template <int DT, bool HALF>
struct FloatOp {
    static_assert(HALF == (DT == DT_F32), "float32 rows through the copy, 16-bit rows as stored");
    typedef v16f tile_t;
    template <int NG> using Smem = FloatScanSmem<NG>;
    FloatRows fr;
    mutable u32 n_open = 0;      // of this wavefront
    float eps, tiny, gam, bet;
    double spread;     // relative difference that two orders of summation in double precision may make
    int e2;

    __device__ __forceinline__ FloatOp(const FloatRows &rows, u32 rowbytes) : fr(rows)
    {
        eps = (2.f * (float)(rowbytes / 2u) + 20.f) * 5.9604644775390625e-08f;
        gam = bet = 0.f;
        e2 = 0;
        spread = (2.0 * (double)rows.d + 32.0) * 1.1102230246251565e-16;
        if constexpr (HALF) {
            // rounded up: what the sums of k_half_rows and the square roots here may have lost, and the root of a norm n that comes from
            // the tile, d 2^-24 n off at most (see above): d 2^-25
            const float up = 1.0001f + (float)(rowbytes / 2u) * 0x1p-24f;
            gam = up * __uint_as_float(rows.par->share_bits);
            bet = up * __uint_as_float(rows.par->rest_bits);
            e2 = 2 * rows.par->exponent;
            tiny = (float)(rowbytes / 2u) * 0x1p-46f + ldexpf(1.f, -120 + (e2 > 0 ? e2 : 0));
        } else {
            tiny = DT == DT_F16 ? (float)rows.d * 0x1p-46f : (float)(8 * rows.d + 8) * 1.17549435e-38f;
        }
    }

    // one wavefront in OPEN_SAMPLE (an add of each to one address takes 10 ns, 20 us a round)
    static __device__ __forceinline__ bool sampled() { return (blockIdx.x & 7) == 0 && __builtin_amdgcn_readfirstlane(threadIdx.x) == 0; }
    __device__ __forceinline__ void report(RoundCtr *ctr) const
    {
        if (n_open && sampled() && threadIdx.x == 0) atomicAdd(&ctr->n_open, n_open);
    }

    static __device__ __forceinline__ v16f mac(const v4i &a, const v4i &b, const v16f &c)
    {
        if constexpr (DT == DT_BF16)
            return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
        else
            return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), c, 0, 0, 0);
    }

    // delta(u, v) in the block's scale
    __device__ __forceinline__ float scaled(u32 dist_bits) const
    {
        return HALF ? ldexpf(__uint_as_float(dist_bits), e2) : __uint_as_float(dist_bits);
    }
    __device__ __forceinline__ float slack(float n) const { return fmaf(gam, __builtin_amdgcn_sqrtf(n), bet); }
    __device__ __forceinline__ float tolerance(float D, float n, float nmax) const
    {
        float t = fmaf(eps, n + nmax, tiny);
        if constexpr (HALF) {
            const float rho = slack(n) + slack(nmax);
            t = fmaf(rho, rho, t);
            t = fmaf(2.00001f * __builtin_amdgcn_sqrtf(D), rho, t);
        }
        return t;
    }

    // n of the 32 rows of a diagonal tile, through LDS; lane l32 of either half gets row l32's
    static __device__ __forceinline__ float diagonal(const v16f &G, float *gt_, int l32, int half)
    {
        float4 *gt = (float4 *)(gt_ + l32 * GT_STRIDE + 4 * half);
        gt[0] = make_float4(G[0], G[1], G[2], G[3]);
        gt[2] = make_float4(G[4], G[5], G[6], G[7]);
        gt[4] = make_float4(G[8], G[9], G[10], G[11]);
        gt[6] = make_float4(G[12], G[13], G[14], G[15]);
        wave_sync();
        return gt_[l32 * GT_STRIDE + l32];
    }

    // bit a -> column 8 (a / 4) + 4 half + a % 4
    static __device__ __forceinline__ u32 column_bits(u32 w, int half)
    {
        w = (w | (w << 8)) & 0x00FF00FFu;
        w = (w | (w << 4)) & 0x0F0F0F0Fu;
        return w << (4 * half);
    }

    // the columns (of this half-wave's 16) that the row of this lane passes for certain, and that it does not fail for certain
    static __device__ __forceinline__ void outcomes(const v16f &G, const float *nrm, int half, float cs, float cm, u32 &pass, u32 &notfail)
    {
        u32 p = 0, q = 0;
#pragma unroll
        for (int b = 3; b >= 0; --b) {
            const float4 nj = ((const float4 *)nrm)[2 * b + half];
            const float t3 = fmaf(2.f, G[4 * b + 3], -nj.w), t2 = fmaf(2.f, G[4 * b + 2], -nj.z);
            const float t1 = fmaf(2.f, G[4 * b + 1], -nj.y), t0 = fmaf(2.f, G[4 * b + 0], -nj.x);
            p = __builtin_amdgcn_alignbit(p, __float_as_uint(t3 + cm), 31);
            q = __builtin_amdgcn_alignbit(q, __float_as_uint(t3 + cs), 31);
            p = __builtin_amdgcn_alignbit(p, __float_as_uint(t2 + cm), 31);
            q = __builtin_amdgcn_alignbit(q, __float_as_uint(t2 + cs), 31);
            p = __builtin_amdgcn_alignbit(p, __float_as_uint(t1 + cm), 31);
            q = __builtin_amdgcn_alignbit(q, __float_as_uint(t1 + cs), 31);
            p = __builtin_amdgcn_alignbit(p, __float_as_uint(t0 + cm), 31);
            q = __builtin_amdgcn_alignbit(q, __float_as_uint(t0 + cs), 31);
        }
        pass = column_bits(p, half);
        notfail = column_bits(q, half);
    }

    // The squared distance of two rows by L consecutive lanes, summed in an order of its own; every lane receives it.
    static __device__ __forceinline__ double wide_distance(const char *a, const char *b, int pieces, int sub, int L)
    {
        double acc = 0.0;
#pragma unroll 1
        for (int c = sub; c < pieces; c += 2 * L) {
            const int c1 = c + L < pieces ? c + L : c;
            const uint4 a0 = ((const uint4 *)a)[c], b0 = ((const uint4 *)b)[c], a1 = ((const uint4 *)a)[c1], b1 = ((const uint4 *)b)[c1];
            acc += piece_distance(a0, b0);
            if (c + L < pieces) acc += piece_distance(a1, b1);
        }
#pragma unroll 1
        for (int o = 1; o < L; o <<= 1) acc += __builtin_bit_cast(double, shfl_xor_u64(__builtin_bit_cast(u64, acc), o));
        return acc;
    }
    static __device__ __forceinline__ double piece_distance(const uint4 &a, const uint4 &b)
    {
        double acc = 0.0;
        const u32 x[4] = {a.x, a.y, a.z, a.w}, y[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if constexpr (DT == DT_F32) {
                const double t = (double)__uint_as_float(x[k]) - (double)__uint_as_float(y[k]);
                acc = fma(t, t, acc);
            } else {
                const double t0 = (double)coord16_to_float<DT>((unsigned short)x[k]) - (double)coord16_to_float<DT>((unsigned short)y[k]);
                const double t1 = (double)coord16_to_float<DT>((unsigned short)(x[k] >> 16)) - (double)coord16_to_float<DT>((unsigned short)(y[k] >> 16));
                acc = fma(t0, t0, acc);
                acc = fma(t1, t1, acc);
            }
        }
        return acc;
    }

    // The pairs (row of this lane, columns open[J]) are resolved: those that fail join F[J].  false: too many.
    // All lanes of 16, 32 or 64 take a row's pieces at once, one trip to memory for most rows where the 8 lanes of the exact
    // routine need one per 32 coordinates or so, and often there is a single pair.  Where the sum, which differs from the exact
    // routine's in its order only, is within `spread` of a rounding boundary of float (ties between such sums are not:
    // both round alike) the exact routine is asked.
    template <int NB>
    __device__ __forceinline__ bool resolve(const u32 (&open)[NB], u32 (&F)[NB], int row, u32 dist_bits, float *gt, const int *id, int lane) const
    {
        uint16_t *pair = (uint16_t *)gt;
        u32 *dd = (u32 *)gt + FLOAT_PAIR_CAP / 2;
        int mine = 0;
#pragma unroll
        for (int J = 0; J < NB; ++J) mine += __popc(open[J]);
        int incl = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(incl, o);
            if (lane >= o) incl += up;
        }
        const int total = __builtin_amdgcn_readlane(incl, 63);
        if (total > FLOAT_PAIR_CAP) {
            n_open += (u32)total;
            return false;
        }
        wave_sync();
        int at = incl - mine;
#pragma unroll
        for (int J = 0; J < NB; ++J)
#pragma unroll 1
            for (u32 bits = open[J]; bits; bits &= bits - 1u) pair[at++] = (uint16_t)((row << 8) | (32 * J + __builtin_ctz(bits)));
        wave_sync();
        const size_t rb = (size_t)fr.d * dt_size(DT);
        const int pieces = (int)(rb >> 4);
        const int L = pieces <= 16 ? 16 : pieces <= 32 ? 32 : 64, sh = L == 16 ? 4 : L == 32 ? 5 : 6, sub = lane & (L - 1);
        bool unsure = false;
#pragma unroll 1
        for (int p = lane >> sh; p - (lane >> sh) < total; p += 64 >> sh) {
            const u32 pr = pair[p < total ? p : 0];
            const double e = wide_distance(fr.X + (size_t)id[(pr >> 8) & 127u] * rb, fr.X + (size_t)id[pr & 127u] * rb, pieces, sub, L);
            const float lo = (float)(e - e * spread), hi = (float)(e + e * spread);
            const bool certain = lo == hi;      // (not where e is not a number: its sign depends on the order of the sum)
            if (sub == 0 && p < total) dd[p] = certain ? __float_as_uint(lo) : 0xFFFFFFFFu;
            unsure = unsure || !certain;
        }
        wave_sync();
        if (__builtin_amdgcn_ballot_w64(unsure) != 0ull) {
            const int grp = lane >> 3, s8 = lane & 7;
#pragma unroll 1
            for (int base = 0; base < total; base += 8) {
                const int p = base + grp;
                if (p < total && dd[p] == 0xFFFFFFFFu) {
                    const u32 pr = pair[p];
                    const u32 db = group8_dist_bits<DT, 2>(fr.X + (size_t)id[(pr >> 8) & 127u] * rb, fr.X + (size_t)id[pr & 127u] * rb, fr.d, 1, s8);
                    if (s8 == 0) dd[p] = db;
                }
            }
            wave_sync();
        }
        at = incl - mine;
        int ties = 0;
#pragma unroll
        for (int J = 0; J < NB; ++J)
#pragma unroll 1
            for (u32 bits = open[J]; bits; bits &= bits - 1u, ++at) {
                // as bits, like the pair-at-a-time kernel: the same order for numbers, a defined one for NaN
                if (dist_bits >= dd[at]) F[J] |= bits & (0u - bits);
                ties += dist_bits == dd[at];
            }
        // equal distances (rows that repeat) are undecided in either form: they count a quarter (8 rounds, tiles throughout / from GROUP_OPEN such
        // pairs on groups: every row four times, 20,000 x 96 float16 1.52 / 1.86 ms; a hundred times, 200,000 x 100 float32 16.0 / 15.4)
        if (sampled()) {
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) ties += __shfl_xor(ties, o);
            n_open += (u32)(total - ties + (ties >> 2));
        }
        wave_sync();
        return true;
    }

    template <int NG, typename GRAM, typename HOLD>
    __device__ __forceinline__ void list(const ScanItem &cur, const GRAM &gram, FloatScanSmem<NG> &sm, int R, u64 *__restrict__ keys,
                                         int *__restrict__ deg, EdgeOut &out, int lane,
                                         u64 &tiles, u64 &rows, u64 &nprops_total, u32 &ev_lane, HOLD hold) const
    {
        const int l32 = lane & 31, half = lane >> 5;
        const int u = __builtin_amdgcn_readfirstlane(cur.u);
        int m = __builtin_amdgcn_readfirstlane(cur.m);
        if (m > 32 * NG) m = 32 * NG;   // cannot happen: the list is built per degree class
        if (m > R) m = R;
        u64 *row = keys + (size_t)u * R;
        u64 kreg[2];
        kreg[0] = lane < m ? cur.k[0] : KEY_PAD;
        kreg[1] = (NG > 2 && lane + 64 < m) ? cur.k[1] : KEY_PAD;
        u64 newm[2];
        newm[0] = __builtin_amdgcn_ballot_w64(lane < m && (kreg[0] & 1ull));
        newm[1] = __builtin_amdgcn_ballot_w64(NG > 2 && lane + 64 < m && (kreg[1] & 1ull));
        const bool any_new = (newm[0] | newm[1]) != 0;
        bool left = false;
        u32 eid[NG], etgt[NG];
        int eplace[NG];
        u32 Kw[NG], badc[NG];
#pragma unroll
        for (int I = 0; I < NG; ++I) eplace[I] = -1, Kw[I] = 0, badc[I] = 0, eid[I] = 0, etgt[I] = 0;
        int np_base = 0;
        u32 ev_all = 0;
        float nmax = 0.f;
        if (any_new) {
            wave_sync();
            if (lane < 32 * NG) sm.id[lane] = (int)key_id(kreg[0]);
            if (NG > 2 && lane + 64 < 32 * NG) sm.id[64 + lane] = (int)key_id(kreg[1]);
            rows += m;
            const u32 hm = 0x0F0F0F0Fu << (4 * half);
#pragma unroll
            for (int I = 0; I < NG; ++I) {
                if (32 * I < m && !left) {      // wave-uniform
                    const v16f G = gram.tile(I, I);
                    const float ni = diagonal(G, sm.gt, l32, half);
                    if (half == 0) sm.nrm[32 * I + l32] = ni;
                    wave_sync();
                    const u64 kb = shfl_u64(kreg[I >> 1], 32 * (I & 1) + l32);
                    const bool validi = 32 * I + l32 < m;
                    const bool newi = kb & 1ull;
                    const float D = scaled(key_dist(kb));
                    const bool far = !(ni <= 1e36f);
                    badc[I] = (u32)__builtin_amdgcn_ballot_w64(validi && far);
                    nmax = half_wave_max(fmaxf(nmax, validi && !far ? ni : 0.f));
                    const float tol = tolerance(D, ni, nmax), c0 = D - ni, cs = c0 - tol, cm = c0 + tol;
                    const bool badr = far || !(D <= 1e36f);
                    const bool odd = __builtin_amdgcn_ballot_w64(validi && badr) != 0ull;
                    const u32 new_I = (u32)(newm[I >> 1] >> (32 * (I & 1)));
                    u32 F[NG], U[NG], E[NG];
                    bool some = false;
#pragma unroll
                    for (int J = 0; J < NG; ++J) F[J] = U[J] = E[J] = 0;
#pragma unroll
                    for (int J = 0; J <= I; ++J) {
                        // a tile without a new row and without a new column holds only old/old pairs, which Alg. 4 skips
                        const u32 new_J = (u32)(newm[J >> 1] >> (32 * (J & 1)));
                        if ((new_I | new_J) == 0) continue;
                        tiles += 1;
                        u32 e = newi ? 0xFFFFFFFFu : new_J;
                        if (J == I) e &= (1u << l32) - 1u;
                        if (!validi) e = 0;
                        E[J] = e & hm;
                        v16f acc = G;
                        if (J < I) acc = gram.tile(I, J);
                        u32 pass, notfail;
                        outcomes(acc, sm.nrm + 32 * J, half, cs, cm, pass, notfail);
                        F[J] = E[J] & ~notfail;
                        U[J] = E[J] & notfail & ~pass;
                        if (odd || badc[J]) {
                            U[J] = badr ? E[J] : (U[J] | (E[J] & badc[J]));
                            F[J] &= ~U[J];
                        }
                        some = some || (J < I ? (U[J] & Kw[J]) : U[J]) != 0;
                    }
                    const u32 rem = (u32)(m - 32 * I);
                    const u32 vmask = rem >= 32u ? 0xFFFFFFFFu : ((1u << rem) - 1u);
                    if (__builtin_amdgcn_ballot_w64(some) != 0ull) {
                        // the pairs that can matter (see the top of the file): hi = rows not pruned for certain, lo = rows kept for certain
                        bool sure = false, may = false;
#pragma unroll
                        for (int J = 0; J < I; ++J) {
                            sure = sure || (F[J] & Kw[J]) != 0;
                            may = may || ((F[J] | U[J]) & Kw[J]) != 0;
                        }
                        const u32 hmax = vmask & ~both_halves(__builtin_amdgcn_ballot_w64(sure));
                        const u32 lmax = vmask & ~both_halves(__builtin_amdgcn_ballot_w64(may));
                        u32 hi = hmax, lo = 0;
#pragma unroll 1
                        for (int sweep = 0; sweep < 33; ++sweep) {
                            lo = lmax & ~both_halves(__builtin_amdgcn_ballot_w64(((F[I] | U[I]) & hi) != 0));
                            const u32 h = hmax & ~both_halves(__builtin_amdgcn_ballot_w64((F[I] & lo) != 0));
                            if (h == hi) break;
                            hi = h;
                        }
                        int first = 0x7FFFFFFF;
#pragma unroll
                        for (int J = I; J >= 0; --J) {
                            const u32 fk = F[J] & (J < I ? Kw[J] : lo);
                            if (fk) first = 32 * J + __builtin_ctz(fk);
                        }
                        {
                            const int other = __shfl_xor(first, 32);
                            first = other < first ? other : first;
                        }
                        u32 open[NG];
                        bool any = false;
#pragma unroll
                        for (int J = 0; J < NG; ++J) open[J] = 0;
#pragma unroll
                        for (int J = 0; J <= I; ++J) {
                            const int rel = first - 32 * J;
                            const u32 before = rel >= 32 ? 0xFFFFFFFFu : rel <= 0 ? 0u : ((1u << rel) - 1u);
                            open[J] = U[J] & (J < I ? Kw[J] : hi) & before;
                            any = any || open[J] != 0;
                        }
                        if (__builtin_amdgcn_ballot_w64(any) != 0ull)
                            left = !resolve<NG>(open, F, 32 * I + l32, key_dist(kb), sm.gt, sm.id, lane);
                    }
                    if (!left) {
                        bool pre = false;
#pragma unroll
                        for (int J = 0; J < I; ++J) pre = pre || ((F[J] & Kw[J]) != 0);
                        const u32 Kmax = vmask & ~both_halves(__builtin_amdgcn_ballot_w64(pre));
                        u32 Kcur = Kmax;
#pragma unroll 1
                        for (int sweep = 0; sweep < 33; ++sweep) {
                            const u32 Knew = Kmax & ~both_halves(__builtin_amdgcn_ballot_w64((F[I] & Kcur) != 0));
                            if (Knew == Kcur) break;
                            Kcur = Knew;
                        }
                        Kw[I] = Kcur;
                        const bool kept = (Kcur >> l32) & 1u;
                        const bool pruned = validi && !kept && half == 0;
                        int tgt = 0x7FFFFFFF;
#pragma unroll
                        for (int J = I; J >= 0; --J) {
                            const u32 fk = F[J] & Kw[J];
                            if (fk) tgt = 32 * J + __builtin_ctz(fk);
                        }
                        {
                            const int other = __shfl_xor(tgt, 32);
                            tgt = other < tgt ? other : tgt;
                        }
#pragma unroll
                        for (int J = 0; J <= I; ++J) {
                            const int rel = tgt - 32 * J;
                            const u32 upto = rel >= 31 ? 0xFFFFFFFFu : (rel < 0 ? 0u : ((2u << rel) - 1u));
                            ev_all += (u32)__popc(E[J] & Kw[J] & upto);
                        }
                        const u64 pm = __builtin_amdgcn_ballot_w64(pruned);
                        if (pruned) {
                            eid[I] = key_id(kb);
                            etgt[I] = (u32)sm.id[tgt];
                            eplace[I] = (np_base + __popcll(pm & lanes_below(lane))) | tgt << 8;
                        }
                        np_base += __popcll(pm);
                        if (I + 1 < NG) wave_sync();   // before the next block overwrites the tile
                    }
                }
            }
        }
        hold();     // every store of the trip comes after this point
        out.flush(lane);
        if (left) {
            leave_vertex(u, fr, &sm.left, lane == 0, NG > 3);
            return;
        }
        ev_lane += ev_all;
        u64 ekey[NG];
#pragma unroll
        for (int I = 0; I < NG; ++I) ekey[I] = make_key(OPEN_DIST, eid[I], 1u);
        out.template list<NG>(ekey, etgt, eplace, np_base, u, lane, sm.gt);
        const u64 K0 = (u64)Kw[0] | (NG > 1 ? ((u64)Kw[NG > 1 ? 1 : 0] << 32) : 0ull);
        const u64 K1 = NG > 2 ? ((u64)Kw[NG > 2 ? 2 : 0] | (NG > 3 ? ((u64)Kw[NG > 3 ? 3 : 0] << 32) : 0ull)) : 0ull;
        const int nk0 = __popcll(K0);
        if ((K0 >> lane) & 1ull) row[__popcll(K0 & lanes_below(lane))] = kreg[0] & ~1ull;
        if (NG > 2 && ((K1 >> lane) & 1ull)) row[nk0 + __popcll(K1 & lanes_below(lane))] = kreg[1] & ~1ull;
        if (lane == 0 && any_new) deg[u] = nk0 + __popcll(K1);
        nprops_total += np_base;
    }

    template <int P, typename GRAM, typename HOLD>
    __device__ __forceinline__ void pack(const PackItem &cur, const GRAM &gram, FloatScanSmem<1> &sm, int R, u64 *__restrict__ keys,
                                         int *__restrict__ deg, EdgeOut &out, int lane,
                                         u32 &tiles, u32 &rows, u32 &nprops_total, u32 &ev_lane, HOLD hold) const
    {
        constexpr int W = 32 / P;
        const int l32 = lane & 31, half = lane >> 5, seg = l32 / W, pos = l32 % W;
        const int u = cur.u;
        int m = cur.m;
        if (m > W) m = W;   // cannot happen: the list is built per degree class
        if (m > R) m = R;
        const bool valid = u >= 0 && pos < m;
        const u64 kb = valid ? cur.k : KEY_PAD;
        const bool newi = valid && (kb & 1ull);
        const bool leader = u >= 0 && pos == 0 && half == 0;
        const u32 new32 = (u32)__builtin_amdgcn_ballot_w64(newi && half == 0);
        const bool any_new = new32 != 0;
        const u32 segmask = (W == 32 ? 0xFFFFFFFFu : ((1u << (W & 31)) - 1u) << (seg * W));
        const u32 below = (1u << l32) - 1u;
        bool pruned = false, kept = false, left = false;
        u32 Kcur = 0, pm = 0, tgt_id = 0;
        int tgt_pos = 0;
        if (any_new) {
            const u32 vmask = (u32)__builtin_amdgcn_ballot_w64(valid && half == 0);
            wave_sync();
            if (half == 0) sm.id[l32] = (int)key_id(kb);
            const v16f G = gram.tile(0, 0);
            const float ni = diagonal(G, sm.gt, l32, half);
            if (half == 0) sm.nrm[l32] = ni;
            rows += __popc(vmask);
            tiles += 1;
            wave_sync();
            const float D = scaled(key_dist(kb));
            const bool far = !(ni <= 1e36f), badr = far || !(D <= 1e36f);
            const float nmax = half_wave_max(valid && !far ? ni : 0.f);
            const float tol = tolerance(D, ni, nmax), c0 = D - ni, cs = c0 - tol, cm = c0 + tol;
            const u32 hm = 0x0F0F0F0Fu << (4 * half);
            u32 E = newi ? segmask : (new32 & segmask);
            E &= below;
            if (!valid) E = 0;
            E &= hm;
            u32 pass, notfail;
            outcomes(G, sm.nrm, half, cs, cm, pass, notfail);
            u32 F[1], U = E & notfail & ~pass;
            F[0] = E & ~notfail;
            if (__builtin_amdgcn_ballot_w64(valid && badr) != 0ull) {
                U = badr ? E : (U | (E & (u32)__builtin_amdgcn_ballot_w64(valid && far)));
                F[0] &= ~U;
            }
            if (__builtin_amdgcn_ballot_w64(U != 0) != 0ull) {
                u32 hi = vmask, lo = 0;
#pragma unroll 1
                for (int sweep = 0; sweep < 33; ++sweep) {
                    lo = vmask & ~both_halves(__builtin_amdgcn_ballot_w64(((F[0] | U) & hi) != 0));
                    const u32 h = vmask & ~both_halves(__builtin_amdgcn_ballot_w64((F[0] & lo) != 0));
                    if (h == hi) break;
                    hi = h;
                }
                int first = 32;
                if (F[0] & lo) first = __builtin_ctz(F[0] & lo);
                {
                    const int other = __shfl_xor(first, 32);
                    first = other < first ? other : first;
                }
                u32 open[1] = {U & hi & (first >= 32 ? 0xFFFFFFFFu : ((1u << first) - 1u))};
                if (__builtin_amdgcn_ballot_w64(open[0] != 0) != 0ull) left = !resolve<1>(open, F, l32, key_dist(kb), sm.gt, sm.id, lane);
            }
            if (!left) {
                Kcur = vmask;
#pragma unroll 1
                for (int sweep = 0; sweep < 33; ++sweep) {
                    const u32 Knew = vmask & ~both_halves(__builtin_amdgcn_ballot_w64((F[0] & Kcur) != 0));
                    if (Knew == Kcur) break;
                    Kcur = Knew;
                }
                kept = (Kcur >> l32) & 1u;
                pruned = valid && !kept && half == 0;
                int tgt = 0x7FFFFFFF;
                {
                    const u32 fk = F[0] & Kcur;
                    if (fk) tgt = __builtin_ctz(fk);
                    const int other = __shfl_xor(tgt, 32);
                    tgt = other < tgt ? other : tgt;
                }
                {
                    const u32 upto = tgt >= 31 ? 0xFFFFFFFFu : ((2u << tgt) - 1u);
                    ev_lane += (u32)__popc(E & Kcur & upto);
                }
                pm = (u32)__builtin_amdgcn_ballot_w64(pruned);
                if (pruned) {
                    tgt_id = (u32)sm.id[tgt];
                    tgt_pos = tgt;
                }
                nprops_total += __popc(pm);
            }
        }
        hold();     // every store of the trip comes after this point
        out.flush(lane);
        if (left) {
            for (u64 lm = __builtin_amdgcn_ballot_w64(leader); lm; lm &= lm - 1ull) {
                leave_vertex(__builtin_amdgcn_readlane(u, __builtin_ctzll(lm)), fr, &sm.left, lane == 0, false);
            }
            return;
        }
        out.pack(make_key(OPEN_DIST, key_id(kb), 1u), tgt_id, tgt_pos, u, __popc(pm & segmask & below), pm, leader, segmask, lane, sm.gt);
        if (kept && half == 0) keys[(size_t)u * R + __popc(Kcur & segmask & below)] = kb & ~1ull;
        if (leader && any_new) deg[u] = __popc(Kcur & segmask);
    }
};

// One wavefront a list: eight pairs of eight of its entries, spread over it, against the tolerance that the tiles would have, 8 lanes a
// pair.
#define SAMPLE_BLOCKS 64
template <int DT>
__global__ __launch_bounds__(256) void k_float_sample(const char *__restrict__ G, u32 rowbytes, FloatRows fr, int R, const u64 *__restrict__ keys,
                                                      const int *__restrict__ deg, const int *__restrict__ lists, u32 enough, RoundCtr *ctr)
{
    __shared__ u32 s_pairs, s_open;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, grp = lane >> 3, sub = lane & 7;
    u32 active = 0, below[NDEG];
#pragma unroll
    for (int k = 0; k < NDEG; ++k) {
        below[k] = active;
        active += ctr->n_active[k];
    }
    if (active < enough) return;
    if (threadIdx.x == 0) s_pairs = s_open = 0u;
    // a vertex of the active lists, by a multiplicative hash of the wavefront's number
    const u32 i = (u32)(((u64)((blockIdx.x * 4u + (u32)wave) * 0x9E3779B1u + 0x7F4A7C15u) * active) >> 32);
    size_t at = i;
#pragma unroll
    for (int k = 1; k < NDEG; ++k)
        if (i >= below[k]) at = (size_t)k * fr.N + (i - below[k]);
    const int u = lists[at];
    // the list is read without waiting for the degree; lane l holds slots l and 64 + l
    const u64 *row = keys + (size_t)u * R;
    const u64 k0 = row[lane < R ? lane : R - 1], k1 = row[lane + 64 < R ? lane + 64 : R - 1];
    const int m = deg[u] < R ? deg[u] : R, t = m < 8 ? m : 8;
    const int ti = (int)(0x77654321u >> (4 * grp)) & 15, tj = (int)(0x52302110u >> (4 * grp)) & 15;
    const int ei = ti * (m - 1) / 7, ej = tj * (m - 1) / 7;      // (the farthest entry is one of them: rows far larger than the others are there)
    const u64 ki = ei < 64 ? shfl_u64(k0, ei & 63) : shfl_u64(k1, ei & 63), kj = ej < 64 ? shfl_u64(k0, ej & 63) : shfl_u64(k1, ej & 63);
    const FloatOp<DT, DT == DT_F32> op(fr, rowbytes);
    const bool have = t == 8 && ((ki | kj) & 1ull);
    float n = 0.f, delta = 0.f;
    if (have) {
        const char *g = G + (size_t)key_id(ki) * rowbytes;
        for (u32 c = 16u * sub; c < rowbytes; c += 128u) {
            const uint4 p = *(const uint4 *)(g + c);
            const u32 x[4] = {p.x, p.y, p.z, p.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                constexpr int T = DT == DT_BF16 ? DT_BF16 : DT_F16;
                const float a = coord16_to_float<T>((unsigned short)x[k]), b = coord16_to_float<T>((unsigned short)(x[k] >> 16));
                n = fmaf(a, a, n);
                n = fmaf(b, b, n);
            }
        }
        const size_t rb = (size_t)fr.d * dt_size(DT);
        delta = op.scaled(group8_dist_bits<DT, 4>(fr.X + (size_t)key_id(ki) * rb, fr.X + (size_t)key_id(kj) * rb, fr.d, 1, sub));
        n += __uint_as_float(xor_lane_u32<1>(__float_as_uint(n)));
        n += __uint_as_float(xor_lane_u32<2>(__float_as_uint(n)));
        n += __uint_as_float(xor_lane_u32<4>(__float_as_uint(n)));
    }
    __syncthreads();
    const float nhalf = half_wave_max(n <= 1e36f ? n : 0.f), nmax = fmaxf(nhalf, __shfl_xor(nhalf, 32));
    const float D = op.scaled(key_dist(ki));
    const bool open = have && !(n <= 1e36f && fabsf(D - delta) > op.tolerance(D, n, nmax));
    const u64 pairs = __builtin_amdgcn_ballot_w64(have && sub == 0), opens = __builtin_amdgcn_ballot_w64(open && sub == 0);
    if (lane == 0 && pairs) {
        atomicAdd(&s_pairs, (u32)__popcll(pairs));
        atomicAdd(&s_open, (u32)__popcll(opens));
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_pairs) {
        atomicAdd(&ctr->sample_pairs, s_pairs);
        atomicAdd(&ctr->sample_open, s_open);
    }
}

// This wavefront's vertices of a class, up to 16 NRC entries each, in groups of 16 rows; vertex i of the class is at(i).
template <int DT, int NG, int NRC, int SMEM, typename AT>
__device__ __forceinline__ void group_lists(const FloatRows &fr, int R, u64 *keys, int *deg, AT at, u32 gw, u32 nw, int &head, u32 n, const EdgeSink &sink,
                                            RoundCtr *ctr, char *sm)
{
    static_assert(sizeof(F32ScanSmem<NRC>) <= SMEM, "the group form works in the LDS of the tile form");
    const bool first_lane = (threadIdx.x & 63) == 0;
    f32_scan_body<NG, 1, NRC, true, DT>(fr.X, fr.d, R, keys, deg, at, gw, nw, n, sink.props, sink.nprop, ctr,
                                        [&](int u) {
                                            if (!fr.left) {
                                                if (first_lane) {
                                                    sink.nprop[u] = 0;
                                                    fr.redo[atomicAdd(fr.n_redo, 1u)] = u;
                                                }
                                            } else {
                                                if (first_lane) fr.left[u] = head;
                                                head = u;
                                            }
                                        },
                                        *reinterpret_cast<F32ScanSmem<NRC> *>(sm));
}

// ... and what it has left, in double precision.  scatter: with the edges of these vertices.
template <int DT, int NG, int NRC, int SMEM>
__device__ __forceinline__ void finish_left(const FloatRows &fr, int R, u64 *keys, int *deg, int head, const EdgeSink &sink, RoundCtr *ctr, char *sm,
                                            bool scatter)
{
    static_assert(sizeof(F32ScanSmem<NRC>) <= SMEM, "the group form works in the LDS of the tile form");
    int next = __builtin_amdgcn_readfirstlane(head);
    if (__builtin_expect(next < 0, 1)) return;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");      // the chain is read by other lanes than wrote it
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    u32 n = 0;
    for (int u = next; u >= 0; u = fr.left[u]) ++n;
    const auto at = [&](u32) {      // asked in order
        const int u = next;
        next = fr.left[u];
        return u;
    };
    f32_scan_body<NG, 1, NRC, false, DT>(fr.X, fr.d, R, keys, deg, at, 0, 1, n, sink.props, sink.nprop, ctr, [](int) {}, *reinterpret_cast<F32ScanSmem<NRC> *>(sm));
    next = __builtin_amdgcn_readfirstlane(head);
    if (scatter) scatter_chain(sink, at, n, R);
}

// Lists of at most 8, 16, 32 entries (blockIdx.y = degree class): 4, 2, 1 vertices per wavefront.
template <int DT>
__global__ __launch_bounds__(256, 4) void k_scan_float_small(
    const int8_t *__restrict__ G, u32 rowbytes, FloatRows fr, int R, u64 *__restrict__ keys, int *__restrict__ deg,
    const int *__restrict__ lists, EdgeSink sink, RoundCtr *ctr)
{
    typedef FloatOp<DT, DT == DT_F32> OP;
    constexpr int SMEM = sizeof(FloatScanSmem<1>);
    __shared__ FloatScanSmem<1> smem[4];
    __shared__ PendingEdges pend[4];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    FloatScanSmem<1> &sm = smem[wave];
    const int y = blockIdx.y, rb = (int)rowbytes;
    const int *list = lists + (size_t)y * fr.N;
    const u32 n = ctr->n_active[y];
    const OP op(fr, rowbytes);
    const bool groups = group_form(ctr);
    stamp_scan_start(ctr);
    int head = -1;
    if (__builtin_expect(groups, 0)) {
        const auto at = [=](u32 i) { return list[i]; };
        if (y < 2) group_lists<DT, 1, 1, SMEM>(fr, R, keys, deg, at, blockIdx.x * 4 + wave, gridDim.x * 4, head, n, sink, ctr, (char *)&sm);
        else group_lists<DT, 1, 2, SMEM>(fr, R, keys, deg, at, blockIdx.x * 4 + wave, gridDim.x * 4, head, n, sink, ctr, (char *)&sm);
    } else {
        EdgeOut out(sink, pend[wave], R);
        sm.left = -1;
        wave_sync();
        if (y == 0) scan_packed_stream_body<OP, 4>(op, G, rb, R, keys, deg, list, n, out, ctr, sm, blockIdx.x, gridDim.x);
        else if (y == 1) scan_packed_stream_body<OP, 2>(op, G, rb, R, keys, deg, list, n, out, ctr, sm, blockIdx.x, gridDim.x);
        else scan_packed_stream_body<OP, 1>(op, G, rb, R, keys, deg, list, n, out, ctr, sm, blockIdx.x, gridDim.x);
        op.report(ctr);
        head = sm.left;
    }
    finish_left<DT, 1, 2, SMEM>(fr, R, keys, deg, head, sink, ctr, (char *)&sm, !groups);
    if (__builtin_expect(groups, 0)) scatter_walk(sink, [=](u32 i) { return list[i]; }, blockIdx.x * 4 + wave, gridDim.x * 4, n, R);
}

// Classes C0 .. NC - 1 in one launch, the grid's blocks divided among them by their work (as k_update_scan_mfma_u8_all).
// FINISH: what is left is scanned at the end (see finish_left), else in a launch that follows (fr.left is null).
template <int DT, int NC, int C0, bool FINISH>
__global__ __launch_bounds__(256, (NC == 6 ? 1 : 2)) void k_scan_float_all(
    const int8_t *__restrict__ G, u32 rowbytes, FloatRows fr, int R, u64 *__restrict__ keys, int *__restrict__ deg,
    const int *__restrict__ lists, EdgeSink sink, RoundCtr *ctr)
{
    typedef FloatOp<DT, DT == DT_F32> OP;
    __shared__ PendingEdges pend[4];
    constexpr int NGMAX = NC - 2, SMEM = sizeof(FloatScanSmem<NGMAX>);
    static_assert(NC == 5 || NC == 6, "short lists plus two or three long-list classes");
    static_assert(C0 == 0 || C0 == 3, "with the short lists or without");
    __shared__ FloatScanSmem<NGMAX> smem[4];
    u32 n[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) n[c] = c >= C0 ? ctr->n_active[c] : 0u;
    const OP op(fr, rowbytes);
    const bool groups = group_form(ctr);
    if (C0 == 0) stamp_scan_start(ctr);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), rb = (int)rowbytes;
    const size_t N = (size_t)fr.N;
    constexpr u32 tile_weight[6] = {6u, 12u, 24u, 46u, 78u, 112u}, group_weight[6] = {16u, 16u, 24u, 44u, 72u, 0u};
    u32 weight[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) weight[c] = groups ? group_weight[c] : tile_weight[c];
    const u32 n0 = n[0];
    if (groups) {
        if (C0 == 0) n[1] += n0, n[0] = 0u;      // classes 0 and 1 as one
        if (NC > 5) n[NC > 5 ? 5 : 0] = 0u;      // (the group form takes lists of up to 96 entries: see launch_float_scan)
    }
    u32 block, mine;
    const int cls = share_blocks<NC>(n, weight, block, mine);
    if (cls < 0) return;
    int head = -1;
    char *sm = (char *)&smem[wave];
    if (__builtin_expect(groups, 0)) {
        const int *list = lists + (size_t)cls * N;
        const auto at = [=](u32 i) { return list[i]; };
        if (C0 == 0 && cls == 1)
            group_lists<DT, 1, 1, SMEM>(fr, R, keys, deg, [=](u32 i) { return i < n0 ? lists[i] : list[i - n0]; }, block * 4 + wave, mine * 4, head, n[1], sink, ctr, sm);
        else if (C0 == 0 && cls == 2) group_lists<DT, 1, 2, SMEM>(fr, R, keys, deg, at, block * 4 + wave, mine * 4, head, n[2], sink, ctr, sm);
        else if (cls == 3) group_lists<DT, 2, 4, SMEM>(fr, R, keys, deg, at, block * 4 + wave, mine * 4, head, n[3], sink, ctr, sm);
        else group_lists<DT, 3, 6, SMEM>(fr, R, keys, deg, at, block * 4 + wave, mine * 4, head, n[4], sink, ctr, sm);
    } else {
        const int *list = lists + (size_t)cls * N;
        EdgeOut out(sink, pend[wave], R);
        FloatScanSmem<1> &sm1 = *reinterpret_cast<FloatScanSmem<1> *>(sm);
        if (C0 == 0 && cls < 3) {
            sm1.left = -1;
            wave_sync();
            if (cls == 0) scan_packed_stream_body<OP, 4>(op, G, rb, R, keys, deg, list, n[0], out, ctr, sm1, block, mine);
            else if (cls == 1) scan_packed_stream_body<OP, 2>(op, G, rb, R, keys, deg, list, n[1], out, ctr, sm1, block, mine);
            else scan_packed_stream_body<OP, 1>(op, G, rb, R, keys, deg, list, n[2], out, ctr, sm1, block, mine);
            head = sm1.left;
        } else if (cls == 3) {
            FloatScanSmem<2> &sm2 = *reinterpret_cast<FloatScanSmem<2> *>(sm);
            sm2.left = -1;
            wave_sync();
            scan_list_stream_body<OP, 2>(op, G, rb, R, keys, deg, list, n[3], out, ctr, sm2, block, mine);
            head = sm2.left;
        } else if (cls == 4) {
            FloatScanSmem<3> &sm3 = *reinterpret_cast<FloatScanSmem<3> *>(sm);
            sm3.left = -1;
            wave_sync();
            scan_list_stream_body<OP, 3>(op, G, rb, R, keys, deg, list, n[4], out, ctr, sm3, block, mine);
            head = sm3.left;
        } else if (NC > 5 && cls == 5) {
            scan_list_stream_body<OP, NGMAX>(op, G, rb, R, keys, deg, list, n[NC > 5 ? 5 : 0], out, ctr, smem[wave], block, mine);
        }
        op.report(ctr);
    }
    if constexpr (FINISH) {
        if (C0 == 0 && cls < 3) finish_left<DT, 1, 2, SMEM>(fr, R, keys, deg, head, sink, ctr, sm, !groups);
        else if (cls == 3) finish_left<DT, 2, 4, SMEM>(fr, R, keys, deg, head, sink, ctr, sm, !groups);
        else if (cls == 4) finish_left<DT, 3, 6, SMEM>(fr, R, keys, deg, head, sink, ctr, sm, !groups);
    }
    if (__builtin_expect(groups, 0)) {
        u32 nc = 0;
#pragma unroll
        for (int c = C0; c < NC; ++c) nc = c == cls ? n[c] : nc;
        const int *list = lists + (size_t)cls * N;
        const u32 joined = C0 == 0 && cls == 1 ? n0 : 0u;      // (classes 0 and 1 as one)
        scatter_walk(sink, [=](u32 i) { return i < joined ? lists[i] : list[i - joined]; }, block * 4 + wave, mine * 4, nc, R);
    }
}
