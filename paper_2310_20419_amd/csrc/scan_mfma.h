// The walk of the matrix-core scans over a round's active lists, and how a list's rows reach the matrix instructions: lane l of
// a wavefront holds 16 bytes, piece 2 s + l / 32, of row l % 32 of each group of 32 list entries, for step s of an instruction
// that takes 32 bytes of every row.  What is done with a vertex's Gram tiles is the business of the class OP (uint8 rows:
// scan_u8.h, float rows: scan_float.h):
//     tile_t, mac           accumulator of a 32 x 32 tile and the matrix instruction
//     Smem<NG>              LDS of a wavefront; its gt, of 4 KB per 32 rows at least, is free until the Gram tiles are complete
//     list<NG>, pack<P>     the body of Alg. 4's vertex loop for one vertex of up to 32 NG entries, for P vertices of up to 32 / P; its
//                           edges go to an EdgeOut, which has delivered those of the trip before once hold() has been called, or an EdgesLeft
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "round.h"
#include "scatter.h"
#include "wave_prims.h"

typedef int v4i __attribute__((ext_vector_type(4)));

#define GT_STRIDE 36   // dwords per row of a tile in LDS (32 + 4: conflict-free b128 stores)

// What the scan holds in registers for one vertex of its work list before it is that vertex's turn.
struct ScanItem {
    int u;          // vertex, -1 past the end of the list
    int m;          // its degree
    u64 k[2];       // its list: positions lane and lane + 64
};

template <int NG>
__device__ __forceinline__ ScanItem scan_item_load(int u, const u64 *__restrict__ keys,
                                                   const int *__restrict__ deg, int R, int lane)
{
    // the list is read without waiting for the degree: slots past it exist (rows are R wide) and are masked later
    // past the end of the work list (u < 0) vertex 0 is read instead and given degree 0: loads without branches
    ScanItem it;
    const u64 *row = keys + (size_t)(u >= 0 ? u : 0) * R;
    const int m = deg[u >= 0 ? u : 0];
    it.u = u;
    it.m = u >= 0 ? m : 0;
    it.k[0] = row[lane < R ? lane : R - 1];                                  // positions past the degree are masked later
    it.k[1] = NG > 2 ? row[lane + 64 < R ? lane + 64 : R - 1] : KEY_PAD;
    return it;
}

// Issues the loads of one vertex's rows of X into MFMA operand layout (no arithmetic on them yet).
template <int NG, int KS>
__device__ __forceinline__ void scan_gather(const int8_t *__restrict__ X, const ScanItem &it, int l32,
                                            int half, v4i (&A)[NG][KS])
{
    constexpr int d = KS * 32;
    const int m = it.m < 32 * NG ? it.m : 32 * NG;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const u32 idr = key_id(it.k[g >> 1]);
        const int id = __shfl((int)idr, 32 * (g & 1) + l32);
        // a lane without a list entry reads row 0 of X (every load unconditional: no registers to clear, no
        // branch); what such a row contributes is never selected by a mask
        const bool valid = it.u >= 0 && 32 * g + l32 < m;
        const int8_t *p = X + (size_t)(valid ? id : 0) * d + half * 16;
#pragma unroll
        for (int s = 0; s < KS; ++s) A[g][s] = *(const v4i *)(p + s * 32);
    }
}

// What a trip has in flight for the trips after it: the rows of the next vertex (or group) and the
// list of the one after.  The memory counter of a wavefront is in order and counts stores as well, so a
// wait for these loads that stood after the trip's stores would also wait for the stores to be
// acknowledged; naming the registers as inputs of an empty statement just before the stores puts the
// wait there, where the loads are a whole trip old and the stores are not yet issued.
__device__ __forceinline__ void arrived(const v4i &x) { asm volatile("" ::"v"(x)); }
__device__ __forceinline__ void arrived(u64 x) { asm volatile("" ::"v"(x)); }
__device__ __forceinline__ void arrived(int x) { asm volatile("" ::"v"(x)); }

// The same number, of which the compiler knows nothing: what a trip derives from it (masks, LDS addresses) is computed again in
// every trip instead of waiting in registers, of which the streamed scans have none to spare (a spilled one is read back
// through the same in-order memory counter as the rows in flight, which then have to arrive first).
__device__ __forceinline__ int afresh(int x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// Where a vertex's Gram tiles come from: formed on demand from rows that are held whole in registers (rows of 32 KS
// bytes) ...
template <typename OP, int NG, int KS>
struct RowsGram {
    const v4i (&A)[NG][KS];
    __device__ __forceinline__ typename OP::tile_t tile(int I, int J) const
    {
        typename OP::tile_t G = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < KS; ++s) G = OP::mac(A[J][s], A[I][s], G);
        return G;
    }
};
// ... or accumulated beforehand while longer rows were streamed through the registers (stream_gram)
template <typename OP, int NG>
struct StreamedGram {
    const typename OP::tile_t (&G)[NG * (NG + 1) / 2];
    __device__ __forceinline__ typename OP::tile_t tile(int I, int J) const { return G[I * (I + 1) / 2 + J]; }
};

// Rows that registers do not hold whole are streamed, 128 bytes of every row (a chunk) at a time, while the accumulators of all
// the vertex's tiles stay (16 registers per tile).  Loads in the operand layout would give every lane a piece of another row, and
// such an instruction keeps the address unit busy for 64 cycles: at most 9.7 TB/s of lanes, used or not (measured on rows that sit in the
// L2), which lists that fill 20 of 32 slots cannot afford next to 6.9 TB/s of memory.  So 8 neighbouring lanes take a row's 128 bytes (32
// TB/s), and the chunk goes through LDS into the operand layout; piece q of row r lies in slot q ^ (r % 8) of its 128
// bytes, which neither side's accesses conflict on.  A chunk of 64 bytes per row in flight, or one line in two instructions
// a chunk apart, reaches 5.3 TB/s where 128 reach 6.9.  A wavefront's LDS traffic is in order, so one buffer serves every
// chunk.  Rows of an odd number of 64 bytes end in half a chunk.
// A tile costs 32 cycles per 32 bytes of its rows, a sixth of what its rows cost in memory time, so every tile is
// formed, needed or not.
template <int NG>
__device__ __forceinline__ void stage_fetch(const int8_t *const (&rp)[4 * NG], int c, int rowbytes, int lane, v4i (&x)[4 * NG])
{
    int off = 128 * c;
    if (off + 128 > rowbytes && (lane & 4)) off -= 64;      // half a chunk: its lanes twice
#pragma unroll
    for (int i = 0; i < 4 * NG; ++i) x[i] = *(const v4i *)(rp[i] + off);
}

template <int NG>
__device__ __forceinline__ void stage_store(char *stage, int lane, const v4i (&x)[4 * NG])
{
    char *p = stage + (lane >> 3) * 128 + (((lane & 7) ^ (lane >> 3)) << 4);
#pragma unroll
    for (int i = 0; i < 4 * NG; ++i) *(v4i *)(p + 1024 * i) = x[i];
    wave_sync();
}

template <typename OP, int NG, int S0, int S1>
__device__ __forceinline__ void stage_steps(const char *stage, int lane, typename OP::tile_t (&G)[NG * (NG + 1) / 2])
{
    const int l32 = lane & 31, half = lane >> 5;
#pragma unroll
    for (int s = S0; s < S1; ++s) {
        v4i a[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) a[g] = *(const v4i *)(stage + 4096 * g + l32 * 128 + (((2 * s + half) ^ (l32 & 7)) << 4));
#pragma unroll
        for (int I = 0; I < NG; ++I)
#pragma unroll
            for (int J = 0; J <= I; ++J) G[I * (I + 1) / 2 + J] = OP::mac(a[J], a[I], G[I * (I + 1) / 2 + J]);
    }
}

template <typename OP, int NG>
__device__ __forceinline__ void stage_tiles(const char *stage, int c, int rowbytes, int lane, typename OP::tile_t (&G)[NG * (NG + 1) / 2])
{
    stage_steps<OP, NG, 0, 2>(stage, lane, G);
    if (128 * c + 128 <= rowbytes) stage_steps<OP, NG, 2, 4>(stage, lane, G);      // wave-uniform
    wave_sync();
}

// NBUF chunks are in flight: chunks 0 .. NBUF - 1 (in x0, x1) have been asked for; the buffers are free afterwards.  Loads past
// the end re-read the last chunk.
template <typename OP, int NG, int NBUF>
__device__ __forceinline__ void stream_gram(const int8_t *const (&rp)[4 * NG], int rowbytes, int lane, char *stage, v4i (&x0)[4 * NG],
                                            v4i (&x1)[4 * NG], typename OP::tile_t (&G)[NG * (NG + 1) / 2])
{
    const int nchunk = (rowbytes + 127) / 128, last = nchunk - 1;
#pragma unroll
    for (int t = 0; t < NG * (NG + 1) / 2; ++t) G[t] = (typename OP::tile_t)(0);
    wave_sync();
#pragma unroll 1
    for (int c = 0; c < nchunk; c += NBUF) {
        stage_store<NG>(stage, lane, x0);
        __builtin_amdgcn_sched_barrier(0);
        stage_fetch<NG>(rp, c + NBUF < last ? c + NBUF : last, rowbytes, lane, x0);
        __builtin_amdgcn_sched_barrier(0);
        stage_tiles<OP, NG>(stage, c, rowbytes, lane, G);
        if (NBUF == 2 && c + 1 < nchunk) {
            stage_store<NG>(stage, lane, x1);
            __builtin_amdgcn_sched_barrier(0);
            stage_fetch<NG>(rp, c + 3 < last ? c + 3 : last, rowbytes, lane, x1);
            __builtin_amdgcn_sched_barrier(0);
            stage_tiles<OP, NG>(stage, c + 1, rowbytes, lane, G);
        }
    }
}

// The work list is walked with a two-deep software pipeline: while vertex i is computed, the rows of
// vertex i+1 are already in flight and the list of vertex i+2 is being fetched, so that the chain
// list -> degree/list entries -> rows of X is paid once per wavefront, not once per vertex.  The loop
// body is written out twice so that the two row buffers swap roles without being copied.
// block `block` of `nblocks` walks the work list
template <typename OP, int NG, int KS, typename OUT>
__device__ __forceinline__ void scan_list_body(const OP &op, const int8_t *__restrict__ X, int R, u64 *__restrict__ keys,
                                               int *__restrict__ deg, const int *__restrict__ list, u32 n_active,
                                               OUT &out,
                                               RoundCtr *__restrict__ ctr, typename OP::template Smem<NG> &sm, u32 block, u32 nblocks)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // scalar: the loop control stays on the scalar unit
    const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    const u32 gw = block * 4 + wave, nw = nblocks * 4;
    u64 tiles = 0, rows = 0, nprops_total = 0;   // tiles: 32x32 blocks of pair distances computed
    u32 ev_lane = 0;   // per-lane share of the algorithmic evaluation count, summed at the end

    if (gw >= n_active) return;
    ScanItem cur = scan_item_load<NG>(list[gw], keys, deg, R, lane);
    ScanItem nxt = scan_item_load<NG>(gw + nw < n_active ? list[gw + nw] : -1, keys, deg, R, lane);
    int u_after = gw + 2 * nw < n_active ? list[gw + 2 * nw] : -1;
    v4i A0[NG][KS], A1[NG][KS];
    scan_gather<NG, KS>(X, cur, l32, half, A0);
    // once per wavefront: the loop starts with nothing in flight
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int s = 0; s < KS; ++s) arrived(A0[g][s]);
    arrived(nxt.k[0]), arrived(nxt.k[1]), arrived(nxt.m), arrived(u_after);
    auto hold = [&](const v4i (&An)[NG][KS], const ScanItem &aft) {
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int s = 0; s < KS; ++s) arrived(An[g][s]);
        arrived(aft.k[0]), arrived(aft.m), arrived(u_after);
        if (NG > 2) arrived(aft.k[1]);
    };

    u32 it = gw;
    while (true) {
        // ---- even trip: `cur` lives in A0, the next vertex is fetched into A1
        scan_gather<NG, KS>(X, nxt, l32, half, A1);
        ScanItem aft = scan_item_load<NG>(u_after, keys, deg, R, lane);
        {
            const unsigned long long j = (unsigned long long)it + 3ull * nw;
            u_after = j < n_active ? list[j] : -1;
        }
        op.template list<NG>(cur, RowsGram<OP, NG, KS>{A0}, sm, R, keys, deg, out, lane, tiles, rows, nprops_total,
                           ev_lane, [&] { hold(A1, aft); });
        cur = nxt;
        nxt = aft;
        if ((unsigned long long)it + nw >= n_active) break;
        it += nw;
        // ---- odd trip: roles of the two buffers exchanged
        scan_gather<NG, KS>(X, nxt, l32, half, A0);
        aft = scan_item_load<NG>(u_after, keys, deg, R, lane);
        {
            const unsigned long long j = (unsigned long long)it + 3ull * nw;
            u_after = j < n_active ? list[j] : -1;
        }
        op.template list<NG>(cur, RowsGram<OP, NG, KS>{A1}, sm, R, keys, deg, out, lane, tiles, rows, nprops_total,
                           ev_lane, [&] { hold(A0, aft); });
        cur = nxt;
        nxt = aft;
        if ((unsigned long long)it + nw >= n_active) break;
        it += nw;
    }
    out.flush(lane);
    u64 evals_algo = ev_lane;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) evals_algo += shfl_xor_u64(evals_algo, o);
    if (lane == 0 && rows) add_round_stats(ctr, evals_algo, tiles * 1024ull, rows, nprops_total);
}

// The same walk for rows of d > 128 bytes (d a multiple of 64).  The first chunk of the next vertex's rows (of lists of up to 32 entries:
// the first two) is asked for as soon as the current one's matrix work is done, so it travels during its prune test and its stores.
template <typename OP, int NG, typename OUT>
__device__ __forceinline__ void scan_list_stream_body(const OP &op, const int8_t *__restrict__ X, int d, int R, u64 *__restrict__ keys,
                                                      int *__restrict__ deg, const int *__restrict__ list, u32 n_active,
                                                      OUT &out,
                                                      RoundCtr *__restrict__ ctr, typename OP::template Smem<NG> &sm, u32 block, u32 nblocks)
{
    // (two chunks for longer lists as well: 60,000 x 784 uint8 4.60 -> 4.79 ms, 1M x 96 101 -> 119, whose registers spill)
    constexpr int NBUF = NG == 1 ? 2 : 1;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int lane = threadIdx.x & 63;
    const u32 gw = block * 4 + wave, nw = nblocks * 4;
    const int last = (d + 127) / 128 - 1;
    char *stage = (char *)sm.gt;
    u64 tiles = 0, rows = 0, nprops_total = 0;
    u32 ev_lane = 0;

    if (gw >= n_active) return;
    // 16 bytes, piece lane % 8, of rows 8 i + lane / 8
    auto row_pointers = [&](const ScanItem &it, const int8_t *(&rp)[4 * NG]) {
        const int m = it.m < 32 * NG ? it.m : 32 * NG;
#pragma unroll
        for (int i = 0; i < 4 * NG; ++i) {
            const int r = 8 * i + (lane >> 3), id = __shfl((int)key_id(it.k[i >> 3]), r & 63);
            const bool valid = it.u >= 0 && r < m;      // else row 0 (see scan_gather)
            rp[i] = X + (size_t)(valid ? id : 0) * (size_t)d + 16 * (lane & 7);
        }
    };
    ScanItem cur = scan_item_load<NG>(list[gw], keys, deg, R, lane);
    ScanItem nxt = scan_item_load<NG>(gw + nw < n_active ? list[gw + nw] : -1, keys, deg, R, lane);
    int u_after = gw + 2 * nw < n_active ? list[gw + 2 * nw] : -1;
    const int8_t *rp[4 * NG];
    v4i x0[4 * NG], x1[4 * NG];
    row_pointers(cur, rp);
    stage_fetch<NG>(rp, 0, d, lane, x0);
    if (NBUF == 2) stage_fetch<NG>(rp, last < 1 ? last : 1, d, lane, x1);

    for (u32 it = gw;; it += nw) {
        lane = afresh(lane);
        typename OP::tile_t G[NG * (NG + 1) / 2];
        stream_gram<OP, NG, NBUF>(rp, d, lane, stage, x0, x1, G);
        row_pointers(nxt, rp);
        stage_fetch<NG>(rp, 0, d, lane, x0);
        if (NBUF == 2) stage_fetch<NG>(rp, last < 1 ? last : 1, d, lane, x1);
        ScanItem aft = scan_item_load<NG>(u_after, keys, deg, R, lane);
        {
            const unsigned long long j = (unsigned long long)it + 3ull * nw;
            u_after = j < n_active ? list[j] : -1;
        }
        op.template list<NG>(cur, StreamedGram<OP, NG>{G}, sm, R, keys, deg, out, lane, tiles, rows, nprops_total,
                           ev_lane, [&] {
#pragma unroll
                               for (int i = 0; i < 4 * NG; ++i) {
                                   arrived(x0[i]);
                                   if (NBUF == 2) arrived(x1[i]);
                               }
                               arrived(aft.k[0]), arrived(aft.m), arrived(u_after);
                               if (NG > 2) arrived(aft.k[1]);
                           });
        cur = nxt;
        nxt = aft;
        if ((unsigned long long)it + nw >= n_active) break;
    }
    out.flush(lane);
    u64 evals_algo = ev_lane;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) evals_algo += shfl_xor_u64(evals_algo, o);
    if (lane == 0 && rows) add_round_stats(ctr, evals_algo, tiles * 1024ull, rows, nprops_total);
}

// KS = 0: rows of d > 128 bytes, streamed
template <typename OP, int NG, int KS, typename OUT>
__device__ __forceinline__ void scan_list_any(const OP &op, const int8_t *__restrict__ X, int d, int R, u64 *__restrict__ keys,
                                              int *__restrict__ deg, const int *__restrict__ list, u32 n_active,
                                              OUT &out,
                                              RoundCtr *__restrict__ ctr, typename OP::template Smem<NG> &sm, u32 block, u32 nblocks)
{
    if constexpr (KS == 0) scan_list_stream_body<OP, NG>(op, X, d, R, keys, deg, list, n_active, out, ctr, sm, block, nblocks);
    else scan_list_body<OP, NG, KS>(op, X, R, keys, deg, list, n_active, out, ctr, sm, block, nblocks);
}

// ---------------------------------------------------------------------------------------------
// Lists of at most 32 entries: P = 1, 2 or 4 vertices share a wavefront, each owning W = 32/P of
// the 32 rows of one tile (rows [W p, W p + W) belong to the p-th vertex of the group).  The Gram tile
// then holds P independent diagonal blocks; the masks keep every row inside its own block, so the
// fixed-point sweeps of all P vertices run together on one 32-bit word.  Every lane (both
// half-waves) holds the list entry of its row.
struct PackItem {
    int u;          // vertex of this lane's segment, -1 past the end of the list
    int m;          // its degree
    u64 k;          // the list entry at this lane's position (KEY_PAD past R)
};

template <int P>
__device__ __forceinline__ PackItem pack_item_load(int u, const u64 *__restrict__ keys,
                                                   const int *__restrict__ deg, int R, int pos)
{
    // past the end of the work list (u < 0) vertex 0 is read instead and given degree 0: loads without branches
    PackItem it;
    const int m = deg[u >= 0 ? u : 0];
    it.u = u;
    it.m = u >= 0 ? m : 0;
    it.k = keys[(size_t)(u >= 0 ? u : 0) * R + (pos < R ? pos : R - 1)];   // slots past the degree exist and are masked later
    return it;
}

template <int P, int KS>
__device__ __forceinline__ void pack_gather(const int8_t *__restrict__ X, const PackItem &it, int pos,
                                            int half, v4i (&A)[1][KS])
{
    constexpr int d = KS * 32, W = 32 / P;
    // a lane without a list entry reads row 0 of X (see scan_gather)
    const bool valid = it.u >= 0 && pos < (it.m < W ? it.m : W);
    const int8_t *p = X + (size_t)(valid ? key_id(it.k) : 0u) * d + half * 16;
#pragma unroll
    for (int s = 0; s < KS; ++s) A[0][s] = *(const v4i *)(p + s * 32);
}

// Same two-deep software pipeline as k_update_scan_mfma_u8; trip g of a wavefront takes list entries
// [P g, P g + P).
template <typename OP, int P, int KS, typename OUT>
__device__ __forceinline__ void scan_packed_body(const OP &op, const int8_t *__restrict__ X, int R, u64 *__restrict__ keys,
                                                 int *__restrict__ deg, const int *__restrict__ list,
                                                 u32 n_active, OUT &out, RoundCtr *__restrict__ ctr,
                                                 typename OP::template Smem<1> &sm, u32 block, u32 nblocks)
{
    constexpr int W = 32 / P;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // scalar: the loop control stays on the scalar unit
    const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    const int seg = l32 / W, pos = l32 % W;
    const u32 gw = block * 4 + wave, nw = nblocks * 4;
    const u32 n_groups = (n_active + (u32)P - 1u) / (u32)P;
    u32 tiles = 0, rows = 0, nprops_total = 0;   // per wavefront: far below 2^32
    u32 ev_lane = 0;

    if (gw >= n_groups) return;
    auto vertex_of = [&](unsigned long long g) -> int {
        const unsigned long long idx = g * P + (unsigned)seg;
        return (g < n_groups && idx < n_active) ? list[idx] : -1;
    };
    PackItem cur = pack_item_load<P>(vertex_of(gw), keys, deg, R, pos);
    PackItem nxt = pack_item_load<P>(vertex_of((unsigned long long)gw + nw), keys, deg, R, pos);
    int u_after = vertex_of((unsigned long long)gw + 2ull * nw);
    v4i A0[1][KS], A1[1][KS];
    pack_gather<P, KS>(X, cur, pos, half, A0);
    // once per wavefront: the loop starts with nothing in flight
#pragma unroll
    for (int s = 0; s < KS; ++s) arrived(A0[0][s]);
    arrived(nxt.k), arrived(nxt.m), arrived(u_after);
    auto hold = [&](const v4i (&An)[1][KS], const PackItem &aft) {
#pragma unroll
        for (int s = 0; s < KS; ++s) arrived(An[0][s]);
        arrived(aft.k), arrived(aft.m), arrived(u_after);
    };

    u32 it = gw;
    while (true) {
        // ---- even trip: `cur` lives in A0, the next group is fetched into A1
        pack_gather<P, KS>(X, nxt, pos, half, A1);
        PackItem aft = pack_item_load<P>(u_after, keys, deg, R, pos);
        u_after = vertex_of((unsigned long long)it + 3ull * nw);
        op.template pack<P>(cur, RowsGram<OP, 1, KS>{A0}, sm, R, keys, deg, out, lane, tiles, rows, nprops_total, ev_lane,
                            [&] { hold(A1, aft); });
        cur = nxt;
        nxt = aft;
        if ((unsigned long long)it + nw >= n_groups) break;
        it += nw;
        // ---- odd trip: roles of the two buffers exchanged
        pack_gather<P, KS>(X, nxt, pos, half, A0);
        aft = pack_item_load<P>(u_after, keys, deg, R, pos);
        u_after = vertex_of((unsigned long long)it + 3ull * nw);
        op.template pack<P>(cur, RowsGram<OP, 1, KS>{A1}, sm, R, keys, deg, out, lane, tiles, rows, nprops_total, ev_lane,
                            [&] { hold(A0, aft); });
        cur = nxt;
        nxt = aft;
        if ((unsigned long long)it + nw >= n_groups) break;
        it += nw;
    }
    out.flush(lane);
    u64 evals_algo = ev_lane;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) evals_algo += shfl_xor_u64(evals_algo, o);
    if (lane == 0 && rows) add_round_stats(ctr, evals_algo, (u64)tiles * 1024ull, rows, nprops_total);
}

// The same for rows of d > 128 bytes (see scan_list_stream_body).
template <typename OP, int P, typename OUT>
__device__ __forceinline__ void scan_packed_stream_body(const OP &op, const int8_t *__restrict__ X, int d, int R, u64 *__restrict__ keys,
                                                        int *__restrict__ deg, const int *__restrict__ list,
                                                        u32 n_active, OUT &out, RoundCtr *__restrict__ ctr,
                                                        typename OP::template Smem<1> &sm, u32 block, u32 nblocks)
{
    constexpr int W = 32 / P;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int lane = threadIdx.x & 63;
    const u32 gw = block * 4 + wave, nw = nblocks * 4;
    const u32 n_groups = (n_active + (u32)P - 1u) / (u32)P;
    const int last = (d + 127) / 128 - 1;
    char *stage = (char *)sm.gt;
    u32 tiles = 0, rows = 0, nprops_total = 0;
    u32 ev_lane = 0;

    if (gw >= n_groups) return;
    auto vertex_of = [&](unsigned long long g) -> int {
        const unsigned long long idx = g * P + (unsigned)((lane & 31) / W);
        return (g < n_groups && idx < n_active) ? list[idx] : -1;
    };
    // lane l32 of either half holds the list entry of row l32; 16 bytes, piece lane % 8, of rows 8 i + lane / 8
    auto row_pointers = [&](const PackItem &it, const int8_t *(&rp)[4]) {
        const bool valid = it.u >= 0 && (lane & 31) % W < (it.m < W ? it.m : W);      // else row 0 (see scan_gather)
        const int mine = valid ? (int)key_id(it.k) : 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) rp[i] = X + (size_t)__shfl(mine, 8 * i + (lane >> 3)) * (size_t)d + 16 * (lane & 7);
    };
    PackItem cur = pack_item_load<P>(vertex_of(gw), keys, deg, R, (lane & 31) % W);
    PackItem nxt = pack_item_load<P>(vertex_of((unsigned long long)gw + nw), keys, deg, R, (lane & 31) % W);
    int u_after = vertex_of((unsigned long long)gw + 2ull * nw);
    const int8_t *rp[4];
    v4i x0[4], x1[4];
    row_pointers(cur, rp);
    stage_fetch<1>(rp, 0, d, lane, x0);
    stage_fetch<1>(rp, last < 1 ? last : 1, d, lane, x1);

    for (u32 it = gw;; it += nw) {
        lane = afresh(lane);
        typename OP::tile_t G[1];
        stream_gram<OP, 1, 2>(rp, d, lane, stage, x0, x1, G);
        row_pointers(nxt, rp);
        stage_fetch<1>(rp, 0, d, lane, x0);
        stage_fetch<1>(rp, last < 1 ? last : 1, d, lane, x1);
        PackItem aft = pack_item_load<P>(u_after, keys, deg, R, (lane & 31) % W);
        u_after = vertex_of((unsigned long long)it + 3ull * nw);
        op.template pack<P>(cur, StreamedGram<OP, 1>{G}, sm, R, keys, deg, out, lane, tiles, rows, nprops_total, ev_lane,
                            [&] {
#pragma unroll
                                for (int i = 0; i < 4; ++i) arrived(x0[i]), arrived(x1[i]);
                                arrived(aft.k), arrived(aft.m), arrived(u_after);
                            });
        cur = nxt;
        nxt = aft;
        if ((unsigned long long)it + nw >= n_groups) break;
    }
    out.flush(lane);
    u64 evals_algo = ev_lane;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) evals_algo += shfl_xor_u64(evals_algo, o);
    if (lane == 0 && rows) add_round_stats(ctr, evals_algo, (u64)tiles * 1024ull, rows, nprops_total);
}

template <typename OP, int P, int KS, typename OUT>
__device__ __forceinline__ void scan_packed_any(const OP &op, const int8_t *__restrict__ X, int d, int R, u64 *__restrict__ keys,
                                                int *__restrict__ deg, const int *__restrict__ list, u32 n_active,
                                                OUT &out,
                                                RoundCtr *__restrict__ ctr, typename OP::template Smem<1> &sm, u32 block, u32 nblocks)
{
    if constexpr (KS == 0) scan_packed_stream_body<OP, P>(op, X, d, R, keys, deg, list, n_active, out, ctr, sm, block, nblocks);
    else scan_packed_body<OP, P, KS>(op, X, R, keys, deg, list, n_active, out, ctr, sm, block, nblocks);
}

// Divides the grid's blocks among NC classes in proportion to their work, n[c] lists of weight[c] each; the grid has
// more blocks than there are classes (and < 2^24).  Returns the class of this block, which is number `block` of the
// `mine` blocks that class got, or -1 if there is no work at all.
// A class gets one block plus its share of the rest: the shares are differences of one non-decreasing
// function of the running sum that ends at `spare` exactly (total / total = 1), so they add up to the grid
// whatever the rounding of the single-precision quotient; every block computes the same numbers.
template <int NC, int NWEIGHT>
__device__ __forceinline__ int share_blocks(const u32 (&n)[NC], const u32 (&weight)[NWEIGHT], u32 &block, u32 &mine)
{
    u64 total = 0;
    u32 nonempty = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        total += (u64)n[c] * weight[c];
        nonempty += n[c] != 0u;
    }
    if (total == 0) return -1;
    const u32 spare = gridDim.x - nonempty;
    const float scale = (float)spare, ftotal = (float)total;
    u32 first = 0, below = 0;
    int cls = -1;
    u64 cum = 0;
    mine = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        cum += (u64)n[c] * weight[c];
        const u32 upto = (u32)(scale * ((float)cum / ftotal));
        const u32 nb = n[c] ? 1u + upto - below : 0u;
        below = upto;
        if (cls < 0 && blockIdx.x < first + nb) {
            cls = c;
            mine = nb;
        }
        if (cls < 0) first += nb;
    }
    block = blockIdx.x - first;
    return cls;      // (-1 cannot happen here: the shares add up to the grid)
}
