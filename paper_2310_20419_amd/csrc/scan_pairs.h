// UpdateNeighbors scan (Alg. 4, the body of the vertex loop), pair at a time: any row length and type, every decision from
// the routine all stored distances come from.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dist.h"
#include "wave_prims.h"

// One vertex u by one wavefront, in the algorithm's own order: v runs over the sorted list of m entries (entry lane in k0,
// entry lane + 64 in k1); the kept set U' so far is a bit mask; the delta(v,w) of up to 8 eligible w (kept,
// not old/old) are evaluated at once by 8-lane groups in ascending w, and the first failing one
// prunes v and redirects it.  Kept entries are written back in place with the flag cleared.
// sk, pkey, ptgt: LDS of the wavefront's own, at least m entries each.  Returns the number of redirected edges (also in
// *n_edges), -1 (0 there) for a list without a new entry.
template <int DT>
__device__ __forceinline__ int scan_vertex_pairs(const void *X, int d, int vec_ok, int R, int u, int m, u64 k0, u64 k1,
                                                 u64 *row, int *deg, Prop *props, int *n_edges, u64 *sk, u64 *pkey, u32 *ptgt,
                                                 int lane, u64 &evals_algo, u64 &evals_exec)
{
    const int sub = lane & 7, grp = lane >> 3;
    const size_t rowbytes = (size_t)d * dt_size(DT);
    wave_sync();
    if (lane < m) sk[lane] = k0;
    if (lane + 64 < m) sk[lane + 64] = k1;
    const u64 new0 = __builtin_amdgcn_ballot_w64(lane < m && (k0 & 1ull));
    const u64 new1 = __builtin_amdgcn_ballot_w64(lane + 64 < m && (k1 & 1ull));
    wave_sync();
    if ((new0 | new1) == 0) {
        if (lane == 0) *n_edges = 0;
        return -1;
    }
    u64 K0 = 0, K1 = 0;   // U' as positions in the sorted list
    int np = 0;
    for (int i = 0; i < m; ++i) {
        const u64 ki = sk[i];
        const u32 di = key_dist(ki), idv = key_id(ki);
        const bool newv = ki & 1ull;
        u64 e0 = newv ? K0 : (K0 & new0);   // old/old pairs are skipped
        u64 e1 = newv ? K1 : (K1 & new1);
        bool pruned = false;
        const char *xv = (const char *)X + (size_t)idv * rowbytes;
        while ((e0 | e1) != 0 && !pruned) {
            int mypos = -1, nb = 0;
#pragma unroll
            for (int g = 0; g < 8; ++g) {
                int p = -1;
                if (e0) { p = __builtin_ctzll(e0); e0 &= e0 - 1; }
                else if (e1) { p = 64 + __builtin_ctzll(e1); e1 &= e1 - 1; }
                if (p >= 0) ++nb;
                if (grp == g) mypos = p;
            }
            const u32 idw = key_id(sk[mypos >= 0 ? mypos : 0]);
            u32 db = 0;
            if (mypos >= 0)
                db = group8_dist_bits<DT>(xv, (const char *)X + (size_t)idw * rowbytes, d, vec_ok, sub);
            const bool fail = mypos >= 0 && di >= db;   // the prune test
            const u64 fm = __builtin_amdgcn_ballot_w64(fail && sub == 0);
            if (fm) {
                const int fl = __builtin_ctzll(fm);     // first failing w in list order
                const u32 fdb = __shfl(db, fl), fidw = __shfl(idw, fl);
                if (lane == 0) {                        // the edge update: (u,v) leaves, (w,v) enters
                    pkey[np] = make_key(fdb, idv, 1u);
                    ptgt[np] = fidw;
                }
                ++np;
                evals_algo += (fl >> 3) + 1;
                pruned = true;
            } else {
                evals_algo += nb;
            }
            evals_exec += nb;
        }
        if (!pruned) {
            if (i < 64) K0 |= 1ull << i; else K1 |= 1ull << (i - 64);   // v joins U'
        }
    }
    // kept entries, flag old, compacted back into the row
    const int nk0 = __popcll(K0);
    if ((K0 >> lane) & 1ull) row[__popcll(K0 & lanes_below(lane))] = k0 & ~1ull;
    if ((K1 >> lane) & 1ull) row[nk0 + __popcll(K1 & lanes_below(lane))] = k1 & ~1ull;
    if (lane == 0) {
        deg[u] = nk0 + __popcll(K1);
        *n_edges = np;
    }
    wave_sync();
    for (int p = lane; p < np; p += 64) emit_redirect(pkey[p], ptgt[p], props + (size_t)u * R + p);
    return np;
}
