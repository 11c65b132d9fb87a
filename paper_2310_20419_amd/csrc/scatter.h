// How redirected edges reach their targets: inboxes, and the chains of what arrives past them.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "round.h"
#include "wave_prims.h"

#define INBOX_CAP 64   // redirected edges a vertex can receive per round without the overflow path

// Bit j set iff lane j of this lane's row of 16 holds the same value, for the lanes reached by rotations R .. 15.
template <int R>
__device__ __forceinline__ u32 same_target_mask(u32 tgt, int sub)
{
    if constexpr (R >= 16) {
        return 0u;
    } else {
        const u32 t = (u32)__builtin_amdgcn_update_dpp(0, (int)tgt, 0x120 + R, 0xF, 0xF, true);     // row_ror:R
        const u32 here = (t == tgt ? 1u : 0u) << ((sub - R) & 15);
        return here | same_target_mask<R + 1>(tgt, sub);
    }
}

// Redirected edges that arrive past their target's inbox ("late") stay where they are, in props, and are chained: a
// target has LATE_LISTS lists, arrival number a is on list (a - inbox) mod LATE_LISTS, so the lists are of equal
// length and a wavefront walks all of them at once.  The heads need no clearing: how many edges are on a list follows
// from the target's count.  They lie in the bin array (8 R bytes per vertex, 4 LATE_LISTS needed); rows of fewer than 32
// slots have no room for them there and receive fewer edges, so they use 32 of their 64 inbox slots and keep the heads in the
// other 32.  (A second pass over all active vertices, once bins had been handed out, used to move them: one launch more
// per round and 1.06 of 26 ms at 1M x 128.  Whole builds: 5,000 x 32 381 -> 354 us, 100,000 x 128 4.61 -> 4.33
// ms, 1M x 128 26.0 -> 25.5 ms.  A round in which one vertex receives 700,000 edges, second pass / as many lists as fit 4 R
// bytes / now: rows of 8 slots 19.5 / 78.6 / 19.7 ms, of 16 19.5 / 40.4 / 19.7, of 96 19.5 / 20.8 / 19.8, the last because the links
// of a chunk are asked for while the one before it is sorted; 7,000 edges, 8 slots: 0.29 / 0.87 / 0.28.)
#define LATE_LISTS 64
#define LATE_OPEN 512     // float rows: late edges of a vertex whose distances its merge computes
static __host__ __device__ inline int round_inbox(int R) { return R < 32 ? 32 : INBOX_CAP; }

// list head l of vertex x is at [x * stride + l]
struct LateHeads {
    u32 *base;
    u32 stride;
};
static __host__ __device__ inline LateHeads late_heads(u64 *inbox, u64 *bins, int R)
{
    LateHeads h;
    h.base = R < 32 ? (u32 *)(inbox + 32) : (u32 *)bins;
    h.stride = R < 32 ? 2u * INBOX_CAP : (u32)LATE_LISTS;
    return h;
}

// Where the edges of a round go.
struct EdgeSink {
    int *count;        // [N] edges received; null: the scan leaves its edges in props, how many in nprop, for k_scatter
    u64 *inbox;
    LateHeads heads;
    Prop *props;       // [N * R] slots u * R .. are vertex u's
    int *nprop;        // [N]
};

// The edge numbered `place` among those its target receives; `slot` is a place in props that no other edge has.
__device__ __forceinline__ void deliver(const EdgeSink &s, int cap, u64 key, u32 tgt, int place, u32 slot)
{
    if (place < cap) {
        s.inbox[(size_t)tgt * INBOX_CAP + place] = key;
    } else {
        s.props[slot].key = key;
        s.props[slot].next = atomicExch(&s.heads.base[(size_t)tgt * s.heads.stride + ((u32)(place - cap) & (LATE_LISTS - 1u))], slot);
    }
}

struct PendingEdges {
    u64 key[64];
    u32 tgt[64];       // (groups of short lists: slots in the upper half)
    uint8_t pos[64];
};

// The scatter of the tile scans.  At the end of a trip a wavefront asks for the arrival numbers of the edges it has redirected, lanes that share
// a target with one atomic, and at the end of the next one, when they have long been there, it writes the edges to their inboxes, so no edge is stored and read again.  (As a
// kernel of its own after the scan the same work was bound by the atomics, of which the part does 2.7 x 10^10 a second and no more.  uint8 rows: they run under the gathers in part,
// 1M x 128 scans 12.2 + scatter 3.7 ms as two kernels, 14.3 as one.  1M x 96 float32: hardly, 59.3 + 8.2 ms against 67.4, whole builds
// 102.6 against 100.6.  At the end of a wavefront's walk it kept too few in flight: 100,000 x 128 a heavy round 63 + 23 -> 94 us.)
// What waits from trip to trip is the key and the target of an edge in LDS, one edge per lane, and two registers.
struct EdgeOut {
    typedef PendingEdges Pending;
    const EdgeSink &s;
    PendingEdges &pend;
    int R, cap;
    u64 waiting = 0;    // lanes with an edge that waits (uniform)
    u32 slot0 = 0;      // slot of the edge of lane 0, the others follow; all ones: slots in pend.tgt[32 ..]
    int first = 0;      // the arrival number that the lane got for all edges that share its target
    u32 how = 0;        // place among those | lane that has the number << 8

    __device__ __forceinline__ EdgeOut(const EdgeSink &sink, PendingEdges &p, int R_) : s(sink), pend(p), R(R_), cap(round_inbox(R_)) {}

    // All lanes.  No edge waits afterwards.
    __device__ __forceinline__ void flush(int lane)
    {
        if (waiting == 0ull) return;
        const int place = __shfl(first, (int)(how >> 8)) + (int)(how & 255u);
        if ((waiting >> lane) & 1ull) {
            u32 slot = slot0 + (u32)lane;
            if (slot0 == 0xFFFFFFFFu) slot = pend.tgt[32 + (lane & 31)];
            deliver(s, cap, pend.key[lane], pend.tgt[lane], place, slot);
        }
        waiting = 0ull;
    }

    // The edges of one vertex u: the lane holds those with place[I] >= 0, `np` in all, their targets by id, and as place their number and the target's
    // position in the list << 8.
    // scratch: 256 bytes per 32 entries.
    template <int NG>
    __device__ __forceinline__ void list(const u64 (&key)[NG], const u32 (&tgt)[NG], const int (&place)[NG], int np, int u, int lane, void *scratch)
    {
        if (!s.count) {
#pragma unroll
            for (int I = 0; I < NG; ++I)
                if (place[I] >= 0) emit_redirect(key[I], tgt[I], s.props + (size_t)u * R + (place[I] & 255));
            if (lane == 0) s.nprop[u] = np;
            return;
        }
        if (np == 0) return;
        u32 *cnt = (u32 *)scratch, *lead = cnt + 32 * NG;
        if (NG > 2 && np > 64) {      // more edges than lanes: not worth a second round of registers, so these numbers are waited for
            wave_sync();
            if (lane < 32 * NG) cnt[lane] = 0u;
            if (lane + 64 < 32 * NG) cnt[lane + 64] = 0u;
            wave_sync();
            u32 rank[NG];
#pragma unroll
            for (int I = 0; I < NG; ++I) rank[I] = place[I] >= 0 ? atomicAdd(&cnt[place[I] >> 8], 1u) : 1u;
            wave_sync();
#pragma unroll
            for (int I = 0; I < NG; ++I)
                if (rank[I] == 0u) lead[place[I] >> 8] = (u32)atomicAdd(&s.count[tgt[I]], (int)cnt[place[I] >> 8]);
            wave_sync();
#pragma unroll
            for (int I = 0; I < NG; ++I)
                if (place[I] >= 0) deliver(s, cap, key[I], tgt[I], (int)(lead[place[I] >> 8] + rank[I]), (u32)u * (u32)R + (u32)(place[I] & 255));
            return;
        }
        wave_sync();
#pragma unroll
        for (int I = 0; I < NG; ++I)
            if (place[I] >= 0) {
                const int e = place[I] & 255;
                pend.key[e] = key[I];
                pend.tgt[e] = tgt[I];
                pend.pos[e] = (uint8_t)(place[I] >> 8);
            }
        if (lane < 32 * NG) cnt[lane] = 0u;
        if (NG > 2 && lane + 64 < 32 * NG) cnt[lane + 64] = 0u;
        wave_sync();
        const u32 t = pend.tgt[lane];
        const u32 q = lane < np ? pend.pos[lane] : 0u;
        u32 rank = 0u;
        if (lane < np) {
            rank = atomicAdd(&cnt[q], 1u);
            if (rank == 0u) lead[q] = (u32)lane;
        }
        wave_sync();
        const u32 l = lead[q], together = cnt[q];
        if (lane < np && rank == 0u) first = atomicAdd(&s.count[t], (int)together);
        how = rank | l << 8;
        waiting = np < 64 ? (1ull << np) - 1ull : ~0ull;
        slot0 = (u32)u * (u32)R;
    }

    // The edges of a group of short lists: at most one per lane, those of the lanes in `pm` (below 32), slot: in the vertex's own; `leader`: a lane
    // for each vertex, all its lanes in segmask.  scratch: 256 bytes.
    __device__ __forceinline__ void pack(u64 key, u32 tgt, int pos, int u, int slot, u32 pm, bool leader, u32 segmask, int lane, void *scratch)
    {
        const bool have = lane < 32 && ((pm >> (lane & 31)) & 1u);
        if (!s.count) {
            if (have) emit_redirect(key, tgt, s.props + (size_t)u * R + slot);
            if (leader) s.nprop[u] = __popc(pm & segmask);
            return;
        }
        if (pm == 0u) return;
        u32 *cnt = (u32 *)scratch, *lead = cnt + 32;
        wave_sync();
        if (lane < 32) cnt[lane] = 0u;
        wave_sync();
        u32 rank = 0u;
        if (have) {
            pend.key[lane] = key;
            pend.tgt[lane] = tgt;
            pend.tgt[32 + lane] = (u32)u * (u32)R + (u32)slot;
            rank = atomicAdd(&cnt[pos], 1u);
            if (rank == 0u) lead[pos] = (u32)lane;
        }
        wave_sync();
        const u32 l = lead[pos], together = cnt[pos];
        if (have && rank == 0u) first = atomicAdd(&s.count[tgt], (int)together);
        how = rank | l << 8;
        waiting = (u64)pm;
        slot0 = 0xFFFFFFFFu;
    }
};

// What a tile scan takes in place of an EdgeOut to leave all its edges in props: a kernel that has the registers of one block per CU (uint8 rows streamed, lists of
// up to 128 entries) pays for the other's code even where it does not scatter.
struct EdgesLeft {
    struct Pending {};
    const EdgeSink &s;
    int R;

    __device__ __forceinline__ EdgesLeft(const EdgeSink &sink, Pending &, int R_) : s(sink), R(R_) {}
    __device__ __forceinline__ void flush(int) {}
    template <int NG>
    __device__ __forceinline__ void list(const u64 (&key)[NG], const u32 (&tgt)[NG], const int (&place)[NG], int np, int u, int lane, void *)
    {
#pragma unroll
        for (int I = 0; I < NG; ++I)
            if (place[I] >= 0) emit_redirect(key[I], tgt[I], s.props + (size_t)u * R + (place[I] & 255));
        if (lane == 0) s.nprop[u] = np;
    }
    __device__ __forceinline__ void pack(u64 key, u32 tgt, int, int u, int slot, u32 pm, bool leader, u32 segmask, int lane, void *)
    {
        if (lane < 32 && ((pm >> (lane & 31)) & 1u)) emit_redirect(key, tgt, s.props + (size_t)u * R + slot);
        if (leader) s.nprop[u] = __popc(pm & segmask);
    }
};

// The edges in props[u * R ..], nprop[u] of them, of the vertices at(i), i = first, first + step, ... below `end`, LANES (16 or 64) lanes per vertex.  Lanes of a row of 16 that share a
// target take their arrival numbers with one atomic (a vertex usually redirects several entries to the same kept neighbour).  The loads of the next vertex (its count and its first
// LANES edges) are issued before the atomics of the current one; the list entry of the vertex after that is fetched one trip earlier still.  The atomics of C times LANES edges are on
// their way together.
template <int LANES, int C, typename AT>
__device__ __forceinline__ void scatter_vertices(const EdgeSink &s, AT at, unsigned long long first, unsigned long long step, u32 end, int R)
{
    const int cap = round_inbox(R), lane = threadIdx.x & 63, e = lane & (LANES - 1), sub = lane & 15, gbase = lane & ~15;
    if (first >= end) return;
    auto vertex_at = [&](unsigned long long i) -> int { return i < end ? at((u32)i) : -1; };
    auto first_edges = [&](int u, int &np, Prop &pr) {
        np = 0;
        pr.key = 0; pr.tgt = 0xFFFFFFFFu; pr.next = 0;
        if (u >= 0) {
            np = s.nprop[u];
            if (e < R) pr = s.props[(size_t)u * R + e];   // slots past np exist; masked below
        }
    };
    int u = vertex_at(first), np;
    Prop pr0;
    first_edges(u, np, pr0);
    int u_next = vertex_at(first + step);
    for (unsigned long long it = first; it < end; it += step) {
        int np_next;
        Prop pr_next;
        first_edges(u_next, np_next, pr_next);
        const int u_after = vertex_at(it + 2ull * step);

        for (int p0 = 0; p0 < np; p0 += LANES * C) {      // same trip count for all lanes of a vertex
            Prop pr[C];
            u32 same[C];
            int base[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const int p = p0 + LANES * c + e;
                pr[c] = pr0;
                if ((c > 0 || p0 > 0) && p < np) pr[c] = s.props[(size_t)u * R + p];
                if (p >= np) pr[c].tgt = 0xFFFFFFFFu;
            }
#pragma unroll
            for (int c = 0; c < C; ++c) {
                // lanes of my row with my target: rotation r of the row brings the target of lane (sub - r) mod 16
                same[c] = (1u << sub) | same_target_mask<1>(pr[c].tgt, sub);
                base[c] = 0;
                if (p0 + LANES * c + e < np && sub == __builtin_ctz(same[c])) base[c] = atomicAdd(&s.count[pr[c].tgt], __popc(same[c]));
            }
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const int p = p0 + LANES * c + e, place = __shfl(base[c], gbase + __builtin_ctz(same[c])) + __popc(same[c] & ((1u << sub) - 1u));
                if (p < np) {
                    if (place < cap) {
                        s.inbox[(size_t)pr[c].tgt * INBOX_CAP + place] = pr[c].key;
                    } else {
                        const size_t slot = (size_t)u * R + p;
                        s.props[slot].next = atomicExch(&s.heads.base[(size_t)pr[c].tgt * s.heads.stride + ((u32)(place - cap) & (LATE_LISTS - 1u))], (u32)slot);
                    }
                }
            }
        }
        u = u_next; np = np_next; pr0 = pr_next;
        u_next = u_after;
    }
}

// The edges that a form without tiles has left in props, for its vertices at(gw), at(gw + nw), ... below `end`.  These kernels keep fewer wavefronts in flight than k_scatter, so each
// takes four vertices and 32 edges of them at once, unless it has no more than two.  8 rounds, k_scatter / a vertex at a time / now, ms, float32 with norms over 12 binades: 1M x 96
// 23.6 / 24.8 / 23.8, 1M x 32, R = 32, 9.21 / 10.56 / 9.41, 200,000 x 100, R = 32, 3.85 / 4.01 / 3.83, R = 128 14.3 / 14.4 / 14.2 (16 edges of each: 9.41, 3.82, 14.3; 64: 9.55, 3.86, 14.2).
template <typename AT>
__device__ __forceinline__ void scatter_walk(const EdgeSink &s, AT at, u32 gw, u32 nw, u32 end, int R)
{
    if (!s.count || gw >= end) return;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");      // the edges are read by other lanes than wrote them
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    if (end - gw <= 2u * nw) scatter_vertices<64, 1>(s, at, gw, nw, end, R);
    else scatter_vertices<16, 2>(s, at, gw + (unsigned long long)((threadIdx.x & 63) >> 4) * nw, 4ull * nw, end, R);
}
// ... and for n of them that are asked in order, by all lanes together.
template <typename AT>
__device__ __forceinline__ void scatter_chain(const EdgeSink &s, AT at, u32 n, int R)
{
    if (!s.count) return;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    const int group = (threadIdx.x & 63) >> 4;
    for (u32 i = 0; i < n; i += 4u) {
        int mine = -1;
        for (int q = 0; q < 4 && i + (u32)q < n; ++q) {
            const int u = at(i + (u32)q);
            if (group == q) mine = u;
        }
        scatter_vertices<16, 2>(s, [=](u32) { return mine; }, 0ull, 1ull, mine >= 0 ? 1u : 0u, R);
    }
}
