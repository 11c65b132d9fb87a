// UpdateNeighbors scan (Alg. 4, the body of the vertex loop) for uint8 rows on the matrix cores.
//
// One wavefront owns one vertex u with m <= 32*NG list entries.  The rows x_v of its whole list are
// gathered straight into MFMA operand registers, rows of more than 128 bytes through LDS (lane l: row l%32 of a 32-row group, bytes
// [32s + 16(l/32), +16) of K-step s) from a copy of X made once per build in which every byte is
// the int8 x-128 (this leaves every difference, hence every delta, unchanged).  n_v = |x_v - 128|^2
// is read off the diagonal of the Gram tile of v's block with itself.
// For a block I of 32 list positions (rows v_i) and a block J <= I (candidates w_j) the tile
//     T_ij = 2 <x_i, x_j> - n_j - t_i ,   t_i = n_i - delta(u, v_i)
// is formed from the Gram tile G(I, J) of v_mfma_i32_32x32x32_i8 (for J = I the one that gave the norms) by
// one shift-add per entry.  The first operand is block J, the second block I, so a lane holds ROW i = l%32 of the tile
// and 16 of its columns, j = 8(a/4) + 4(l/32) + a%4: by the symmetry of the Gram matrix no transpose
// is needed.  Both operands use the same byte order, so however the hardware pairs the K bytes, the
// two sides pair alike.  With delta(v_i, w_j) = n_i + n_j - 2<x_i, x_j> (exact in int32):
//     the prune test fires  <=>  delta(u, v_i) >= delta(v_i, w_j)  <=>  T_ij >= 0 ,
// Each half-wave collects the outcomes for its 16 columns as bits of one word per row.  The loop over v
// then run on bit masks: the kept set U' is the unique solution K of
//     K_i = not exists j < i : F_ij and K_j
// (F already masked by the old/old skip), found per 32-row block by iterating
// K <- Phi(K) from "all kept" until it stops changing (row i is final after i+1 sweeps).  A pruned
// row's redirect target is the first set bit of F_i & K, and delta(v,w) for the new edge comes from
// the tile kept in LDS:  delta(v_i, w_j) = delta(u, v_i) - T_ij.
#pragma once
#include "scan_mfma.h"

typedef int v16i __attribute__((ext_vector_type(16)));

template <int NG>
struct alignas(16) MfmaScanSmem {
    int gt[NG * 32 * GT_STRIDE];   // tiles T(I, J) of the current block I: [(32J + i) * GT_STRIDE + j]
    int nrm[32 * NG];              // n_j by list position
    int id[32 * NG];               // vertex id by list position
};

// Once per build: Xs <- X - 128 as int8 (n bytes, a multiple of 16).
__global__ __launch_bounds__(256) void k_prepare_u8(const uint8_t *__restrict__ X, size_t n,
                                                    int8_t *__restrict__ Xs)
{
    const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 16;
    if (i < n) {
        v4i x = *(const v4i *)(X + i);
        x ^= (int)0x80808080;
        *(v4i *)(Xs + i) = x;
    }
}

// The same for rows the tiles do not fit: row u of Xs is dp bytes (dp >= d, a multiple of 4): the d bytes of x_u minus
// 128, then zeros, which add nothing to a product of two rows.  X may have any alignment, so it is read by single
// bytes, a wavefront taking 256 consecutive ones of a row.
__global__ __launch_bounds__(256) void k_prepare_u8_rows(const uint8_t *__restrict__ X, long long N, int d, int dp,
                                                         int8_t *__restrict__ Xs)
{
    const u32 words = (u32)dp / 4u;
    for (u64 i = (u64)blockIdx.x * 256u + threadIdx.x; i < (u64)N * words; i += (u64)gridDim.x * 256u) {
        const u64 u = i / words;
        const int e = 4 * (int)(i - u * words);
        const uint8_t *x = X + u * (u64)d + e;
        u32 w = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (e + k < d) w |= ((u32)x[k] ^ 0x80u) << (8 * k);
        *(u32 *)(Xs + 4 * i) = w;
    }
}

// The body of Alg. 4's vertex loop for the vertex in `cur`, whose Gram tiles `gram` yields.  hold() names the
// registers in flight for the trips after this one (see arrived).
template <int NG, typename GRAM, typename OUT, typename HOLD>
__device__ __forceinline__ void scan_vertex_u8(const ScanItem &cur, const GRAM &gram, MfmaScanSmem<NG> &sm, int R, u64 *__restrict__ keys,
                                               int *__restrict__ deg, OUT &out, int lane, u64 &tiles, u64 &rows,
                                               u64 &nprops_total, u32 &ev_lane, HOLD hold)
{
    const int l32 = lane & 31, half = lane >> 5;
    const int u = __builtin_amdgcn_readfirstlane(cur.u);      // same in every lane: keep it scalar
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
    const bool any_new = (newm[0] | newm[1]) != 0;   // else every pair was tested before
    // what the scan leaves to be stored: per block one redirected edge per lane, and the kept set
    u64 ekey[NG];
    u32 etgt[NG];
    int eplace[NG];
    u32 Kw[NG];                             // U' as bit masks over list positions, 32 per word (uniform)
#pragma unroll
    for (int I = 0; I < NG; ++I) eplace[I] = -1, Kw[I] = 0, ekey[I] = 0, etgt[I] = 0;
    int np_base = 0;
    if (any_new) {
    wave_sync();   // the previous vertex is done with the LDS tables
    if (lane < 32 * NG) sm.id[lane] = (int)key_id(kreg[0]);
    if (NG > 2 && lane + 64 < 32 * NG) sm.id[64 + lane] = (int)key_id(kreg[1]);
    rows += m;
    const u32 hm = 0x0F0F0F0Fu << (4 * half);   // the columns this half-wave holds

#pragma unroll
    for (int I = 0; I < NG; ++I) {
        if (32 * I < m) {                   // wave-uniform
            // the Gram tile of the block with itself; n of its rows is the diagonal, read back through
            // LDS (rows past the list hold row 0 of X; no mask ever selects them)
            const v16i G = gram.tile(I, I);
            {
                int4 *gt = (int4 *)(sm.gt + (32 * I + l32) * GT_STRIDE + 4 * half);
                gt[0] = make_int4(G[0], G[1], G[2], G[3]);
                gt[2] = make_int4(G[4], G[5], G[6], G[7]);
                gt[4] = make_int4(G[8], G[9], G[10], G[11]);
                gt[6] = make_int4(G[12], G[13], G[14], G[15]);
            }
            wave_sync();
            const int nrI = sm.gt[(32 * I + l32) * GT_STRIDE + l32];
            if (half == 0) sm.nrm[32 * I + l32] = nrI;
            wave_sync();
            // this block's rows in lane-per-row form (lane l32 <-> list position 32 I + l32), in both halves
            const u64 kb = shfl_u64(kreg[I >> 1], 32 * (I & 1) + l32);
            const int posi = 32 * I + l32;
            const bool validi = posi < m;
            const bool newi = kb & 1ull;
            const int di = (int)key_dist(kb);
            const int negt = di - nrI;
            const u32 new_I = (u32)(newm[I >> 1] >> (32 * (I & 1)));
            u32 F[NG], E[NG];
#pragma unroll
            for (int J = 0; J < NG; ++J) F[J] = E[J] = 0;
#pragma unroll
            for (int J = 0; J <= I; ++J) {
                // a tile without a new row and without a new column holds only old/old pairs, which Alg. 4 skips
                const u32 new_J = (u32)(newm[J >> 1] >> (32 * (J & 1)));
                if ((new_I | new_J) == 0) continue;
                tiles += 1;
                // the old/old skip: a pair is tested only if v or w is new; only w before v count
                u32 e = newi ? 0xFFFFFFFFu : new_J;
                if (J == I) e &= (1u << l32) - 1u;
                if (!validi) e = 0;
                E[J] = e & hm;
                // lane: row l32 of block I; acc[a]: column 8(a/4) + 4 half + a%4 of block J
                v16i acc = G;
                if (J < I) acc = gram.tile(I, J);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int4 nj = ((const int4 *)sm.nrm)[8 * J + 2 * q + half];
                    acc[4 * q + 0] = (acc[4 * q + 0] << 1) + (negt - nj.x);
                    acc[4 * q + 1] = (acc[4 * q + 1] << 1) + (negt - nj.y);
                    acc[4 * q + 2] = (acc[4 * q + 2] << 1) + (negt - nj.z);
                    acc[4 * q + 3] = (acc[4 * q + 3] << 1) + (negt - nj.w);
                }
                int4 *gt = (int4 *)(sm.gt + (32 * J + l32) * GT_STRIDE + 4 * half);
                gt[0] = make_int4(acc[0], acc[1], acc[2], acc[3]);
                gt[2] = make_int4(acc[4], acc[5], acc[6], acc[7]);
                gt[4] = make_int4(acc[8], acc[9], acc[10], acc[11]);
                gt[6] = make_int4(acc[12], acc[13], acc[14], acc[15]);
                // bit a of ok: T < 0, v passes the prune test against column a
                u32 ok = 0;
#pragma unroll
                for (int a = 15; a >= 0; --a) ok = __builtin_amdgcn_alignbit(ok, (u32)acc[a], 31);
                // bit 4q + k  ->  column 8q + 4 half + k
                ok = (ok | (ok << 8)) & 0x00FF00FFu;
                ok = (ok | (ok << 4)) & 0x0F0F0F0Fu;
                ok <<= 4 * half;
                F[J] = E[J] & ~ok;
            }
            // the loop over v on masks; what the two half-waves find for a row is joined through ballots
            bool pre = false;
#pragma unroll
            for (int J = 0; J < I; ++J) pre = pre || ((F[J] & Kw[J]) != 0);
            const u64 preb = __builtin_amdgcn_ballot_w64(pre);
            const u32 rem = (u32)(m - 32 * I);
            const u32 vmask = rem >= 32u ? 0xFFFFFFFFu : ((1u << rem) - 1u);
            const u32 Kmax = vmask & ~((u32)preb | (u32)(preb >> 32));
            u32 Kcur = Kmax;
            for (int sweep = 0; sweep < 33; ++sweep) {
                const u64 hit = __builtin_amdgcn_ballot_w64((F[I] & Kcur) != 0);
                const u32 Knew = Kmax & ~((u32)hit | (u32)(hit >> 32));
                if (Knew == Kcur) break;
                Kcur = Knew;
            }
            Kw[I] = Kcur;
            const bool kept = (Kcur >> l32) & 1u;
            const bool pruned = validi && !kept && half == 0;
            // first failing w over both halves
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
            // the evaluations Alg. 4 makes for this row: tested candidates up to and including w
            int ev = 0;
#pragma unroll
            for (int J = 0; J <= I; ++J) {
                const int rel = tgt - 32 * J;
                const u32 upto = rel >= 31 ? 0xFFFFFFFFu : (rel < 0 ? 0u : ((2u << rel) - 1u));
                ev += __popc(E[J] & Kw[J] & upto);
            }
            ev_lane += (u32)ev;
            wave_sync();   // the tiles are in LDS
            const u64 pm = __builtin_amdgcn_ballot_w64(pruned);
            if (pruned) {
                const int tv = sm.gt[((tgt & ~31) + l32) * GT_STRIDE + (tgt & 31)];
                const u32 dvw = (u32)(di - tv);
                // the redirect: v enters w's list
                ekey[I] = make_key(dvw, key_id(kb), 1u);
                etgt[I] = (u32)sm.id[tgt];
                eplace[I] = (np_base + __popcll(pm & lanes_below(lane))) | tgt << 8;
            }
            np_base += __popcll(pm);
            if (I + 1 < NG) wave_sync();   // before the next block overwrites the tiles
        }
    }
    }
    hold();     // every store of the trip comes after this point
    out.flush(lane);
    out.template list<NG>(ekey, etgt, eplace, np_base, u, lane, sm.gt);
    // kept entries, flag old, compacted back into the row
    const u64 K0 = (u64)Kw[0] | (NG > 1 ? ((u64)Kw[NG > 1 ? 1 : 0] << 32) : 0ull);
    const u64 K1 = NG > 2 ? ((u64)Kw[NG > 2 ? 2 : 0] | (NG > 3 ? ((u64)Kw[NG > 3 ? 3 : 0] << 32) : 0ull)) : 0ull;
    const int nk0 = __popcll(K0);
    if ((K0 >> lane) & 1ull) row[__popcll(K0 & lanes_below(lane))] = kreg[0] & ~1ull;
    if (NG > 2 && ((K1 >> lane) & 1ull)) row[nk0 + __popcll(K1 & lanes_below(lane))] = kreg[1] & ~1ull;
    if (lane == 0 && any_new) deg[u] = nk0 + __popcll(K1);
    nprops_total += np_base;
}

template <int P, typename GRAM, typename OUT, typename HOLD>
__device__ __forceinline__ void pack_vertices_u8(const PackItem &cur, const GRAM &gram, MfmaScanSmem<1> &sm, int R,
                                                 u64 *__restrict__ keys, int *__restrict__ deg, OUT &out, int lane,
                                                 u32 &tiles, u32 &rows, u32 &nprops_total, u32 &ev_lane, HOLD hold)
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
    const bool any_new = new32 != 0;   // else nothing is new in any of the P lists: every pair was tested before
    const u32 segmask = (W == 32 ? 0xFFFFFFFFu : ((1u << (W & 31)) - 1u) << (seg * W));
    const u32 below = (1u << l32) - 1u;
    // what the scan leaves to be stored
    bool pruned = false, kept = false;
    u32 Kcur = 0, pm = 0, dvw = 0, tgt_id = 0;
    int tgt_pos = 0;
    if (any_new) {
        const u32 vmask = (u32)__builtin_amdgcn_ballot_w64(valid && half == 0);
        wave_sync();   // the previous group is done with the LDS tables
        if (half == 0) sm.id[l32] = (int)key_id(kb);
        // n of every row: the diagonal of the Gram tile, through LDS (rows past a list hold row 0 of X;
        // no mask ever selects them)
        // lane: row l32; G[a]: <x_row, x_col> for column 8(a/4) + 4 half + a%4
        const v16i G = gram.tile(0, 0);
        {
            int4 *gt = (int4 *)(sm.gt + l32 * GT_STRIDE + 4 * half);
            gt[0] = make_int4(G[0], G[1], G[2], G[3]);
            gt[2] = make_int4(G[4], G[5], G[6], G[7]);
            gt[4] = make_int4(G[8], G[9], G[10], G[11]);
            gt[6] = make_int4(G[12], G[13], G[14], G[15]);
        }
        wave_sync();
        const int ni = sm.gt[l32 * GT_STRIDE + l32];
        if (half == 0) sm.nrm[l32] = ni;
        rows += __popc(vmask);
        tiles += 1;
        wave_sync();

        const int di = (int)key_dist(kb);
        const int negt = di - ni;
        const u32 hm = 0x0F0F0F0Fu << (4 * half);   // the columns this half-wave holds
        // the old/old skip: a pair is tested only if v or w is new; only w before v (in v's own list) count
        u32 E = newi ? segmask : (new32 & segmask);
        E &= below;
        if (!valid) E = 0;
        E &= hm;
        // T = 2 G - n_j - t_i from the Gram tile that gave the norms
        v16i acc;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int4 nj = ((const int4 *)sm.nrm)[2 * q + half];
            acc[4 * q + 0] = (G[4 * q + 0] << 1) + (negt - nj.x);
            acc[4 * q + 1] = (G[4 * q + 1] << 1) + (negt - nj.y);
            acc[4 * q + 2] = (G[4 * q + 2] << 1) + (negt - nj.z);
            acc[4 * q + 3] = (G[4 * q + 3] << 1) + (negt - nj.w);
        }
        {
            int4 *gt = (int4 *)(sm.gt + l32 * GT_STRIDE + 4 * half);
            gt[0] = make_int4(acc[0], acc[1], acc[2], acc[3]);
            gt[2] = make_int4(acc[4], acc[5], acc[6], acc[7]);
            gt[4] = make_int4(acc[8], acc[9], acc[10], acc[11]);
            gt[6] = make_int4(acc[12], acc[13], acc[14], acc[15]);
        }
        // bit a of ok: T < 0, v passes the prune test against column a
        u32 ok = 0;
#pragma unroll
        for (int a = 15; a >= 0; --a) ok = __builtin_amdgcn_alignbit(ok, (u32)acc[a], 31);
        // bit 4q + k  ->  column 8q + 4 half + k
        ok = (ok | (ok << 8)) & 0x00FF00FFu;
        ok = (ok | (ok << 4)) & 0x0F0F0F0Fu;
        ok <<= 4 * half;
        const u32 F = E & ~ok;
        // the loop over v on masks; what the two half-waves find for a row is joined through ballots
        Kcur = vmask;
        for (int sweep = 0; sweep < 33; ++sweep) {
            const u64 hit = __builtin_amdgcn_ballot_w64((F & Kcur) != 0);
            const u32 Knew = vmask & ~((u32)hit | (u32)(hit >> 32));
            if (Knew == Kcur) break;
            Kcur = Knew;
        }
        kept = (Kcur >> l32) & 1u;
        pruned = valid && !kept && half == 0;
        // first failing w over both halves
        int tgt = 0x7FFFFFFF;
        {
            const u32 fk = F & Kcur;
            if (fk) tgt = __builtin_ctz(fk);
            const int other = __shfl_xor(tgt, 32);
            tgt = other < tgt ? other : tgt;
        }
        // the evaluations Alg. 4 makes for this row: tested candidates up to and including w
        {
            const u32 upto = tgt >= 31 ? 0xFFFFFFFFu : ((2u << tgt) - 1u);
            ev_lane += (u32)__popc(E & Kcur & upto);
        }
        wave_sync();   // the tile is in LDS
        pm = (u32)__builtin_amdgcn_ballot_w64(pruned);
        if (pruned) {
            dvw = (u32)(di - sm.gt[l32 * GT_STRIDE + tgt]);
            tgt_id = (u32)sm.id[tgt];
            tgt_pos = tgt;
        }
        nprops_total += __popc(pm);
    }
    hold();     // every store of the trip comes after this point
    // the redirect: v enters w's list
    out.flush(lane);
    out.pack(make_key(dvw, key_id(kb), 1u), tgt_id, tgt_pos, u, __popc(pm & segmask & below), pm, leader, segmask, lane, sm.gt);
    // kept entries, flag old, compacted back into the row
    if (kept && half == 0) keys[(size_t)u * R + __popc(Kcur & segmask & below)] = kb & ~1ull;
    if (leader && any_new) deg[u] = __popc(Kcur & segmask);
}

// What the walks below do with the rows of a vertex: uint8 rows.
struct U8Op {
    typedef v16i tile_t;
    template <int NG> using Smem = MfmaScanSmem<NG>;
    static __device__ __forceinline__ v16i mac(const v4i &a, const v4i &b, const v16i &c)
    {
        return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
    }
    template <int NG, typename... ARGS>
    __device__ __forceinline__ void list(ARGS &&...args) const { scan_vertex_u8<NG>(static_cast<ARGS &&>(args)...); }
    template <int P, typename... ARGS>
    __device__ __forceinline__ void pack(ARGS &&...args) const { pack_vertices_u8<P>(static_cast<ARGS &&>(args)...); }
};

// (four groups of streamed rows: 160 accumulator registers, so one block per CU)
template <int NG, int KS, typename OUT>
__global__ __launch_bounds__(256, (NG == 1 ? 5 : NG == 2 ? 3 : KS == 0 && NG == 4 ? 1 : 2)) void k_update_scan_mfma_u8(
    const int8_t *__restrict__ X, int d, int R, u64 *__restrict__ keys,
    int *__restrict__ deg, const int *__restrict__ list, const u32 *__restrict__ n_list,
    EdgeSink sink, RoundCtr *__restrict__ ctr)
{
    __shared__ MfmaScanSmem<NG> smem[4];
    __shared__ typename OUT::Pending pend[4];
    OUT out(sink, pend[threadIdx.x >> 6], R);
    scan_list_any<U8Op, NG, KS>(U8Op(), X, d, R, keys, deg, list, *n_list, out, ctr, smem[threadIdx.x >> 6], blockIdx.x, gridDim.x);
}

// The three short-list classes in one launch: blockIdx.y = degree class (lists of at most 8, 16, 32
// entries: 4, 2, 1 vertices per wavefront).  Each class is walked by the gridDim.x blocks of its row.
template <int KS, typename OUT>
__global__ __launch_bounds__(256, 4) void k_update_scan_mfma_u8_small(
    const int8_t *__restrict__ X, int d, int R, u64 *__restrict__ keys, int *__restrict__ deg,
    const int *__restrict__ lists, long long N, EdgeSink sink, RoundCtr *__restrict__ ctr)
{
    __shared__ MfmaScanSmem<1> smem[4];
    __shared__ typename OUT::Pending pend[4];
    OUT out(sink, pend[threadIdx.x >> 6], R);
    MfmaScanSmem<1> &sm = smem[threadIdx.x >> 6];
    const int y = blockIdx.y;
    const int *list = lists + (size_t)y * N;
    const u32 n = ctr->n_active[y];
    stamp_scan_start(ctr);
    if (y == 0) scan_packed_any<U8Op, 4, KS>(U8Op(), X, d, R, keys, deg, list, n, out, ctr, sm, blockIdx.x, gridDim.x);
    else if (y == 1) scan_packed_any<U8Op, 2, KS>(U8Op(), X, d, R, keys, deg, list, n, out, ctr, sm, blockIdx.x, gridDim.x);
    else scan_packed_any<U8Op, 1, KS>(U8Op(), X, d, R, keys, deg, list, n, out, ctr, sm, blockIdx.x, gridDim.x);
}

// Classes C0 .. NC - 1 in one launch, all of them resident together: the grid's blocks are divided among the
// classes in proportion to their work (active lists x matrix tiles per list), one block at least for a class
// that has any; every block derives the same division from the round's counters.  The classes then share the
// start-up and the tail that each launch of its own pays.  NC classes: 3 short-list ones, then lists of at
// most 64, 96, 128 entries.  Every block carries the registers and the LDS of the longest class (two blocks
// per CU).  C0 = 0, every class: for inputs so small that no class alone has enough lists to fill the chip
// (the short-list classes lose occupancy: with many active lists their own launch is faster).  C0 = 3, the
// long-list classes only, next to k_update_scan_mfma_u8_small: for large inputs.
template <int KS, typename OUT, int NC, int C0 = 0>
__global__ __launch_bounds__(256, (KS == 0 && NC == 6 ? 1 : 2)) void k_update_scan_mfma_u8_all(
    const int8_t *__restrict__ X, int d, int R, u64 *__restrict__ keys, int *__restrict__ deg,
    const int *__restrict__ lists, long long N, EdgeSink sink, RoundCtr *__restrict__ ctr)
{
    constexpr int NGMAX = NC - 2;
    static_assert(NC >= 4 && NC <= 6, "short lists plus one to three long-list classes");
    __shared__ MfmaScanSmem<NGMAX> smem[4];
    __shared__ typename OUT::Pending pend[4];
    OUT out(sink, pend[threadIdx.x >> 6], R);
    if (C0 == 0) stamp_scan_start(ctr);
    // work per list: 4, 2, 1 lists share a tile; among the longer classes in proportion to their NG (NG + 1) / 2
    // tiles (3 : 6 : 10; the division is sensitive there: 3 : 4.5 or 3 : 8 costs the 1M build 4 % of its scan time),
    // and a 64-entry list weighted 2.25 short tiles (measured on 100,000 vertices: 1.5 -> 1.60 ms, 2 -> 1.51, 2.25 ->
    // 1.49, 3 -> 1.53, 4 -> 1.70 ms of scan time per build)
    // streamed rows (KS = 0): the rows' bytes dominate, and a list of a class holds 6, 12, 24, 46, 78, 112 of them or so
    constexpr u32 weight[6] = {4u, 8u, 16u, KS ? 36u : 30u, KS ? 72u : 50u, KS ? 120u : 72u};
    u32 n[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) n[c] = c >= C0 ? ctr->n_active[c] : 0u;
    u32 block, mine;
    const int cls = share_blocks<NC>(n, weight, block, mine);
    if (cls < 0) return;
    const int *list = lists + (size_t)cls * N;
    const int wave = threadIdx.x >> 6;
    MfmaScanSmem<1> &sm1 = *reinterpret_cast<MfmaScanSmem<1> *>(&smem[wave]);
    if (C0 == 0 && cls == 0) scan_packed_any<U8Op, 4, KS>(U8Op(), X, d, R, keys, deg, list, n[0], out, ctr, sm1, block, mine);
    else if (C0 == 0 && cls == 1) scan_packed_any<U8Op, 2, KS>(U8Op(), X, d, R, keys, deg, list, n[1], out, ctr, sm1, block, mine);
    else if (C0 == 0 && cls == 2) scan_packed_any<U8Op, 1, KS>(U8Op(), X, d, R, keys, deg, list, n[2], out, ctr, sm1, block, mine);
    else if (cls == 3)
        scan_list_any<U8Op, 2, KS>(U8Op(), X, d, R, keys, deg, list, n[3], out, ctr, *reinterpret_cast<MfmaScanSmem<2> *>(&smem[wave]), block, mine);
    else if (NC > 4 && cls == 4)
        scan_list_any<U8Op, 3, KS>(U8Op(), X, d, R, keys, deg, list, n[NC > 4 ? 4 : 0], out, ctr, *reinterpret_cast<MfmaScanSmem<3> *>(&smem[wave]), block, mine);
    else if (NC > 5 && cls == 5)
        scan_list_any<U8Op, 4, KS>(U8Op(), X, d, R, keys, deg, list, n[NC > 5 ? 5 : 0], out, ctr, *reinterpret_cast<MfmaScanSmem<4> *>(&smem[wave]), block, mine);
}
