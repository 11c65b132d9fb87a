// librnnd: Relative NN-Descent graph construction (arXiv 2310.20419, Alg. 4-6) on gfx950.
//
// A wavefront, or a group of 16, 32 or 64 of its lanes, owns one vertex in every per-vertex kernel.
// A round is synchronous:
//   scan     every active vertex (one holding a "new" entry) runs the body of Alg. 4's vertex loop on its own list,
//            writes its kept entries back in place and leaves its redirected edges in its slot of `props`
//   scatter  every redirected edge takes an arrival number at its target (the round's only atomic per
//            edge) and moves into the target's inbox (up to INBOX_CAP slots per vertex); later arrivals are chained.
//            The scans by tiles do it themselves, in their trips (see EdgeOut); a kernel of its own serves the others
//   classify vertices that received edges form the `touched` lists, by the size of the merge they need
//   merge    every touched list becomes the first R distinct keys of (kept entries + inbox + later arrivals)
//   compact  touched vertices whose new list holds a "new" entry form the next active lists,
//            one per degree class (see degree_class)
// (small inputs: the last three in one launch, see k_merge_blocks)
// Between outer rounds AddReverseEdges (Alg. 5) uses the same inboxes and bins (launch_reverse).
// Counters that many wavefronts would hit at one address are aggregated per block first.
// search.h holds the graph search of Alg. 1 (rnnd_search).
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>
#include <mutex>

#include "../../include/rnnd.h"
#include "wave_prims.h"
#include "round.h"

#define WAVES_PER_BLOCK 4
#define BLOCK (64 * WAVES_PER_BLOCK)
#define GOLDEN64 0x9E3779B97F4A7C15ull
#define RNND_MAX_SLOTS 0x7FFFFF00ull   // N * (slots per row): bin offsets are ints, -1 = no bin
#define RNND_MAX_RUN_SLOTS 131072      // rounds (x runs per pass): one small counter block each

#include "dist.h"
#include "scatter.h"
#include "scan_u8.h"
#include "scan_pairs.h"
#include "padded_rows.h"
#include "launch.h"
#include "search.h"

__global__ void k_stamp(u64 *dst) { if (threadIdx.x == 0) *dst = wall_clock64(); }

// Degree class of a list of m entries: which scan kernel takes it.  use_classes 0: one list for all
// (generic scan).  2 (uint8 and 16-bit matrix-core scans): classes 0, 1, 2 = at most 8, 16, 32 entries (four, two,
// one vertex per wavefront), 3, 4, 5 = at most 64, 96, 128 (two, three, four 32-row blocks).
// 1 (scan of whole float32 rows, 16-row groups): classes 0..6 = at most 8, 16, 32, 48, 64, 80, 96 entries
// (1, 1, 2, 3, 4, 5, 6 groups), 7 = more (generic scan).
__device__ __forceinline__ int degree_class(int m, int use_classes)
{
    if (!use_classes) return 0;
    if (m <= 16) return m <= 8 ? 0 : 1;
    if (use_classes == 2) return m <= 32 ? 2 : 2 + ((m - 1) >> 5);
    return m <= 96 ? 1 + ((m - 1) >> 4) : 7;
}

// ------------------------------------------------------------------ RandomGraph
// Alg. 6, RandomGraph: S distinct random neighbours (wave_random_ids), their distances, sorted.
template <int DT>
__global__ __launch_bounds__(BLOCK) void k_random_graph(const void *X, long long N, int d, int vec_ok,
                                                        int S, int R, u64 seed, u64 *keys, int *deg,
                                                        int8_t *vcls, int use_classes)
{
    static_assert(SEARCH_MAX_L >= RNND_MAX_R, "the id / distance tables of the search hold a whole list");
    __shared__ SearchSmem s_tab[WAVES_PER_BLOCK];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const long long u = (long long)blockIdx.x * WAVES_PER_BLOCK + wave;
    if (u >= N) return;
    int *ids = s_tab[wave].id;
    const size_t rowbytes = (size_t)d * dt_size(DT);
    wave_random_ids(seed, N, u, S, ids, lane);
    wave_sync();
    // delta(u, id), 8 lanes per row; short uint8 rows: the loads of up to 32 rows in flight together
    search_eval<DT>(X, (const char *)X + (size_t)u * rowbytes, d, vec_ok, rowbytes, s_tab[wave], S, lane);
    wave_sync();
    u64 *row = keys + (size_t)u * R;
    if (S <= 32) {     // the upper half of the wavefront sorts padding
        u64 k = lane < S ? make_key(s_tab[wave].dist[lane], (u32)ids[lane], 1u) : KEY_PAD;
        k = group_sort<32>(k);
        if (lane < S) row[lane] = k;
    } else if (S <= 64) {
        u64 k[1];
        k[0] = lane < S ? make_key(s_tab[wave].dist[lane], (u32)ids[lane], 1u) : KEY_PAD;
        wave_sort<1>(k);
        if (lane < S) row[lane] = k[0];
    } else {
        u64 k[2];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            int e = r * 64 + lane;
            k[r] = e < S ? make_key(s_tab[wave].dist[e], (u32)ids[e], 1u) : KEY_PAD;
        }
        wave_sort<2>(k);
        if (lane < S) row[lane] = k[0];
        if (lane + 64 < S) row[lane + 64] = k[1];
    }
    if (lane == 0) {
        deg[u] = S;
        if (vcls) vcls[u] = (int8_t)degree_class(S, use_classes);   // every vertex starts with "new" entries
    }
}

// ------------------------------------------------- UpdateNeighbors: scan (generic kernel)
// The body of Alg. 4's vertex loop (scan_vertex_pairs) for one vertex per wavefront.
struct WorkList {
    const int *list;
    const u32 *n;
    const int *list2 = nullptr;      // the list instead of it where *second is not 0
    const u32 *n2 = nullptr, *second = nullptr;
};
template <int DT>
__global__ __launch_bounds__(BLOCK) void k_update_scan(const void *X, int d, int vec_ok, int R,
                                                       u64 *keys, int *deg, WorkList work, EdgeSink sink, RoundCtr *ctr)
{
    __shared__ u64 s_key[WAVES_PER_BLOCK][RNND_MAX_R];
    __shared__ u64 s_pkey[WAVES_PER_BLOCK][RNND_MAX_R];
    __shared__ u32 s_ptgt[WAVES_PER_BLOCK][RNND_MAX_R];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const u32 gw = blockIdx.x * WAVES_PER_BLOCK + wave, nw = gridDim.x * WAVES_PER_BLOCK;
    const bool second = work.second && *work.second != 0u;
    const int *list = second ? work.list2 : work.list;
    const u32 n_active = second ? *work.n2 : *work.n;
    stamp_scan_start(ctr);
    u64 evals_algo = 0, evals_exec = 0, rows = 0, nprops_total = 0;
    for (u32 it = gw; it < n_active; it += nw) {
        const int u = list[it];
        int m = deg[u];
        if (m > R) m = R;
        u64 *row = keys + (size_t)u * R;
        u64 k0 = lane < m ? row[lane] : KEY_PAD;
        u64 k1 = lane + 64 < m ? row[lane + 64] : KEY_PAD;
        const int np = scan_vertex_pairs<DT>(X, d, vec_ok, R, u, m, k0, k1, row, deg, sink.props, sink.nprop + u, s_key[wave], s_pkey[wave], s_ptgt[wave],
                                             lane, evals_algo, evals_exec);
        if (np < 0) continue;
        rows += m;
        nprops_total += np;
    }
    if (lane == 0 && rows) add_round_stats(ctr, evals_algo, evals_exec, rows, nprops_total);
    scatter_walk(sink, [=](u32 i) { return list[i]; }, gw, nw, n_active, R);
}

// ------------------------------------------------------ UpdateNeighbors: merge
// Vertices x with cnt[x] > list_min are appended to `list`; those with cnt[x] > bin_min get a bin of
// cnt[x] - bin_sub keys starting at binoff[x] (others: binoff = -1).  One pair of atomics per 1024
// vertices.  Optionally clears zero_a[] and zero_b[], sets thr[] to "keep all", marks in cand[]
// the vertices with deg[x] + cnt[x] > cand_R, and lists in flagged[] those with flag[x] >= 0.
__global__ __launch_bounds__(1024) void k_assign_bins(long long N, const int *cnt, int list_min, int bin_min,
                                                      int bin_sub, int *binoff, u32 *bin_cursor, int *list,
                                                      u32 *n_list, int *zero_a, int *zero_b, u64 *thr,
                                                      const int *deg, int cand_R, int8_t *cand, const int8_t *flag, int *flagged, u32 *n_flagged)
{
    __shared__ u32 s_sum[16], s_num[16], s_flag[16], s_base[3];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long long x = (long long)blockIdx.x * 1024 + threadIdx.x;
    int c = 0;
    if (x < N) {
        c = cnt[x];
        if (zero_a) zero_a[x] = 0;
        if (zero_b) zero_b[x] = 0;
        if (thr) thr[x] = KEY_PAD;
        if (cand) cand[x] = (int8_t)(deg[x] + c > cand_R);
    }
    const bool in_list = c > list_min;
    const u32 mine = c > bin_min ? (u32)(c - bin_sub) : 0u;
    u32 incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        u32 v = __shfl_up(incl, o);
        if (lane >= o) incl += v;
    }
    const u64 hb = __builtin_amdgcn_ballot_w64(in_list);
    const bool is_flagged = flag && x < N && flag[x] >= 0;
    const u64 fb = __builtin_amdgcn_ballot_w64(is_flagged);
    if (lane == 63) { s_sum[wave] = incl; s_num[wave] = (u32)__popcll(hb); s_flag[wave] = (u32)__popcll(fb); }
    __syncthreads();
    if (threadIdx.x == 0) {
        u32 ts = 0, tn = 0, tf = 0;
        for (int w = 0; w < 16; ++w) {
            const u32 a = s_sum[w], b = s_num[w], c = s_flag[w];
            s_sum[w] = ts; s_num[w] = tn; s_flag[w] = tf;
            ts += a; tn += b; tf += c;
        }
        const u32 b0 = ts ? atomicAdd(bin_cursor, ts) : 0u, b1 = tn ? atomicAdd(n_list, tn) : 0u, b2 = tf ? atomicAdd(n_flagged, tf) : 0u;
        s_base[0] = b0; s_base[1] = b1; s_base[2] = b2;
    }
    __syncthreads();
    if (x < N) {
        binoff[x] = mine ? (int)(s_base[0] + s_sum[wave] + incl - mine) : -1;
        if (in_list) list[s_base[1] + s_num[wave] + __popcll(hb & lanes_below(lane))] = (int)x;
        if (is_flagged) flagged[s_base[2] + s_flag[wave] + __popcll(fb & lanes_below(lane))] = (int)x;
    }
}

// The active lists of a round's first ncl degree classes walked as one: start[k] = entries of the classes before k.
struct ActiveLists {
    const int *lists;
    long long N;
    u32 start[NDEG + 1];
};

__device__ __forceinline__ ActiveLists active_lists(const int *lists, long long N, const RoundCtr *ctr, int ncl)
{
    ActiveLists a;
    a.lists = lists;
    a.N = N;
    u32 sum = 0;
#pragma unroll
    for (int k = 0; k < NDEG; ++k) {
        a.start[k] = sum;
        sum += k < ncl ? ctr->n_active[k] : 0u;
    }
    a.start[NDEG] = sum;
    return a;
}

// entry i of the concatenation, i < start[NDEG]
__device__ __forceinline__ int active_vertex(const ActiveLists &a, u32 i)
{
    u32 c = 0, off = i;
#pragma unroll
    for (int k = 1; k < NDEG; ++k)
        if (i >= a.start[k]) {
            c = (u32)k;
            off = i - a.start[k];
        }
    return a.lists[(size_t)c * (size_t)a.N + off];
}

// The padded copy for a single round (see k_prepare_rows).  Where fewer than one vertex in LISTED_SHARE is active only the
// rows their lists name are copied, by one wavefront for 8 entries; a row named twice is written twice, with the same bytes.
// On a snapshot that is nearly converged the copy of all rows costs more than the round: 200,000 x 100 float32, 690
// vertices active, call with all rows / these rows / no copy and the generic kernel: 197 / 148 / 149 us; 1M x 100, 9,251
// active: 590 / 450 / 464; 28,399 active, where either copy reads about as much: 640 / - / 612; 100,000 x 901, 252: 315 / 173 / 512.
#define LISTED_SHARE 64
#define LISTED_MIN_N 32768       // below, the copy of all rows is a launch's worth of time
template <typename T>
__global__ __launch_bounds__(256) void k_prepare_listed_rows(const T *__restrict__ X, long long N, int d, u32 rb, int permute,
                                                             uint4 *__restrict__ Xp, const int *lists, const RoundCtr *ctr,
                                                             const u64 *__restrict__ keys, const int *__restrict__ deg, int R)
{
    const ActiveLists al = active_lists(lists, N, ctr, NDEG);
    const u32 n = al.start[NDEG], pieces = rb / 16u;
    if ((u64)n * LISTED_SHARE >= (u64)N) {
        (void)pad_all_rows<T>(X, N, d, rb, permute, 0u, Xp);
        return;
    }
    const u32 parts = ((u32)R + 7u) / 8u;
    const int lane = threadIdx.x & 63;
    for (u64 w = ((u64)blockIdx.x * 256u + threadIdx.x) >> 6; w < (u64)n * parts; w += (u64)gridDim.x * 4u) {
        const int u = active_vertex(al, (u32)(w / parts)), first = 8 * (int)(w % parts);
        int m = deg[u] - first;
        if (first + m > R) m = R - first;
        if (m > 8) m = 8;
        if (m <= 0) continue;
        const u32 mine = key_id(keys[(size_t)u * R + first + (lane < m ? lane : 0)]), total = (u32)m * pieces;
        bool odd = false;
        for (u32 base = 0; base < total; base += 64u) {
            const u32 i = base + (u32)lane, e = i < total ? i / pieces : 0u;
            const size_t id = (u32)__shfl((int)mine, (int)e);      // (every lane takes part)
            if (i < total) Xp[id * pieces + (i - e * pieces)] = padded_piece<T>(X + id * (size_t)d, (int)(i - e * pieces), d, permute, 0u, odd);
        }
    }
}

// Redirected edges of the float scans arrive without their distances (OPEN_DIST).  Computes them for the lanes whose key (of a
// vertex in the list of vertex x) is open, in 8-lane groups, in the order the wavefront holds them; every lane of the
// wavefront takes part.  DT_U8: nothing is ever open.
struct OpenEdges {
    union {
        uint2 edge[64];
        uint8_t lane[128];      // see repeats
    };
    u32 dist[64];
};
// From the second pass on 15-40 % of the redirected edges name an edge that another vertex redirects in the same round or that the list holds already;
// their distances need not be computed where the merge would drop the second of two equal keys.  Lanes whose open key names the vertex of a key that some lane of
// the same G holds in `list` or, of several open ones, all but one: found through a table of 128 lanes by vertex, in which the last one to write wins (a lane that loses its place to
// another vertex counts as no repeat).  Equal vertices are equal keys only if the distances have the same bits.  Those of open keys do: one routine forms them, operands in the same order.
// A listed one does (same_bits) where this library has formed it on the same rows, in either order, unless it is a NaN, whose sign is that of the operand it came
// with or the other; a caller's snapshot may hold distances summed in another order, so there lists are not looked at.  Merge with / without: 1M x 96 float32 25.6 / 26.3 ms, 1M x 960 182 / 188; whole builds 1M x 960 513 / 524,
// 300,000 x 768 bfloat16 97.6 / 99.8, 200,000 x 960 84.7 / 86.7, 200,000 x 16 10.83 / 10.84 (open keys only: 523, 99.3, 86.5, 10.92). Not in
// k_merge_blocks (merge of 20,000 x 96 float32 0.935 / 0.890, whole builds of 96 bfloat16 20,000 2.51 / 2.47, 60,000 5.92 / 5.87), although long rows would gain there too: float32 20,000 x 960
// 8.74 / 9.16, 60,000 x 384 12.2 / 12.5, 130,000 x 960 67.4 / 69.9, bfloat16 130,000 x 768 40.7 / 41.7.
template <int G>
__device__ __forceinline__ bool repeats(u64 key, bool open, u64 list, bool listed, OpenEdges *s, int lane)
{
    constexpr u32 SLOTS = 2 * G;
    const u32 base = (u32)(lane / G) * SLOTS;
    const u32 at = base + ((key_id(key) * 0x9E3779B1u) >> 16) % SLOTS, lat = base + ((key_id(list) * 0x9E3779B1u) >> 16) % SLOTS;
    wave_sync();
    if (open) s->lane[at] = (uint8_t)lane;
    wave_sync();
    if (listed) s->lane[lat] = (uint8_t)(64 + lane);
    wave_sync();
    const u32 w = open ? s->lane[at] : (u32)lane;
    const u32 of_open = (u32)__shfl((int)key_id(key), (int)(w & 63u)), of_list = (u32)__shfl((int)key_id(list), (int)(w & 63u));
    return open && w != (u32)lane && (w >= 64u ? of_list : of_open) == key_id(key);
}
template <int DT, int G, bool SEEK>
__device__ __forceinline__ u64 close_keys(u64 key, int x, bool have, u64 list, bool listed, int same_bits, OpenEdges *s, const char *__restrict__ X, int d, int lane)
{
    if constexpr (DT == DT_U8) {
        return key;
    } else {
        bool open = have && key_dist(key) == OPEN_DIST;
        if (__builtin_amdgcn_ballot_w64(open) == 0ull) return key;
        if (SEEK && repeats<G>(key, open, list, same_bits && listed && key_dist(list) <= INFINITE_DIST, s, lane)) {
            key = KEY_PAD;
            open = false;
        }
        const u64 om = __builtin_amdgcn_ballot_w64(open);
        const int total = __popcll(om);
        const size_t rb = (size_t)d * dt_size(DT);
        const int mine = __popcll(om & lanes_below(lane)), grp = lane >> 3, sub = lane & 7;
        wave_sync();
        if (open) s->edge[mine] = make_uint2(key_id(key), (u32)x);
        wave_sync();
        for (int b = 0; b < total; b += 8) {
            const int e = b + grp;
            if (e < total) {
                const uint2 vw = s->edge[e];
                const u32 db = group8_dist_bits<DT, DT == DT_F16 ? 2 : 3, DT == DT_F16>(X + (size_t)vw.x * rb, X + (size_t)vw.y * rb, d, 1, sub);
                if (sub == 0) s->dist[e] = db;
            }
        }
        wave_sync();
        return open ? make_key(s->dist[mine], key_id(key), 1u) : key;
    }
}

// For scans that leave their edges in props (see scan_scatters): every active vertex moves its redirected edges to their targets.  Arrivals below round_inbox(R) go to
// the target's inbox, later ones onto one of its lists (see LATE_LISTS).
__global__ __launch_bounds__(BLOCK) void k_scatter(long long N, const int *lists, int ncl, RoundCtr *ctr, EdgeSink sink, int R, u32 enough)
{
    const u32 g = (blockIdx.x * BLOCK + threadIdx.x) >> 4, ng = (gridDim.x * BLOCK) >> 4;
    // the classes' lists as one: the grid is shared by their entries, however they are spread over the classes
    const ActiveLists al = active_lists(lists, N, ctr, ncl);
    const u32 n = al.start[NDEG];
    if (n < RNND_MAX_SLOTS) stamp_scan_stop(ctr);      // (always: the clock is read once the scan's counters are here)
    if (enough && blockIdx.x == 0 && threadIdx.x == 0) decide_next_form(ctr, n, enough);
    scatter_vertices<16, 1>(sink, [&](u32 i) { return active_vertex(al, i); }, g, ng, n, R);
}

// What k_scatter does besides scattering, for a round whose scan has scattered: by one thread.
__device__ __forceinline__ void end_scan(RoundCtr *ctr, u32 enough)
{
    u32 active = 0;
#pragma unroll
    for (int k = 0; k < NDEG; ++k) active += ctr->n_active[k];
    if (active < RNND_MAX_SLOTS) ctr->t_scan_stop = wall_clock64();      // (always: the clock is read once the scan's counters are here)
    if (enough) decide_next_form(ctr, active, enough);
}

// Computes the open distances of the late edges of vertex x; each group of 8 lanes of the block walks its share of the lists.
template <int DT>
__device__ __attribute__((noinline)) void close_late(long long x, int late, LateHeads heads, Prop *props, const char *X, int d)
{
    const int sub = threadIdx.x & 7;
    const size_t rb = (size_t)d * dt_size(DT);
    for (u32 l = threadIdx.x >> 3; l < LATE_LISTS; l += blockDim.x >> 3) {
        u32 at = heads.base[(size_t)x * heads.stride + l];
        for (int left = (late - (int)l + LATE_LISTS - 1) / LATE_LISTS; left > 0; --left) {
            const u64 key = props[at].key;
            const u32 next = props[at].next;
            if (key_dist(key) == OPEN_DIST) {
                const u32 db = group8_dist_bits<DT, 2>(X + (size_t)key_id(key) * rb, X + (size_t)x * rb, d, 1, sub);
                if (sub == 0) props[at].key = make_key(db, key_id(key), 1u);
            }
            at = next;
        }
    }
}

// Merge class of a vertex that holds nb entries and received c: how wide a sort its merge needs.  cap = round_inbox(R):
// the first three read received edges from the inbox only.
__device__ __forceinline__ int merge_class(int nb, int c, int cap)
{
    const int total = nb + c;
    return c > cap ? 3 : total <= 16 ? 0 : total <= 32 ? 1 : total <= 64 ? 2 : 3;
}

// Every vertex x that received edges (cnt[x] > 0) is appended to the touched list of its merge class.  A block covers
// TC_TILES x 1024 vertices and takes its space with one atomic per class.  Four tiles per block
// keep the atomics of a 1M-vertex round few; on small inputs two tiles (twice the blocks, a shorter chain in
// each) are faster: 100,000 vertices 4.68 -> 4.55 ms per build, 1M 26.0 -> 26.1 ms.
// Float rows: a hub's merge walks its late edges with one wavefront, which would also compute their open distances; for hubs
// of more than LATE_OPEN late edges the block does that here, 8 lanes for each of the hub's lists.
template <int TC_TILES, int DT>
__global__ __launch_bounds__(1024) void k_touch_classify(long long N, int cap, const int *cnt, const int *deg, RoundCtr *ctr, int *tlists,
                                                         LateHeads heads, Prop *props, const char *__restrict__ X, int d, int scattered, u32 enough)
{
    if (scattered && blockIdx.x == 0 && threadIdx.x == 0) end_scan(ctr, enough);
    __shared__ u32 s_cnt[TC_TILES][16][NMRG], s_base[NMRG];
    bool hub = false;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int mc[TC_TILES];
    u32 rank[TC_TILES];
#pragma unroll
    for (int k = 0; k < TC_TILES; ++k) {
        const long long x = ((long long)blockIdx.x * TC_TILES + k) * 1024 + threadIdx.x;
        mc[k] = -1;
        if (x < N) {
            const int c = cnt[x];
            if (c > 0) mc[k] = merge_class(deg[x], c, cap);
            if (DT != DT_U8) hub = hub || c > cap + LATE_OPEN;
        }
        rank[k] = 0;
#pragma unroll
        for (int q = 0; q < NMRG; ++q) {
            const u64 b = __builtin_amdgcn_ballot_w64(mc[k] == q);
            if (mc[k] == q) rank[k] = (u32)__popcll(b & lanes_below(lane));
            if (lane == 0) s_cnt[k][wave][q] = (u32)__popcll(b);
        }
    }
    __syncthreads();
    if (wave == 0) {
        // exclusive prefix over the TC_TILES x 16 wavefront totals, in (tile, wavefront) order: lane = tile * 16 + wavefront
        static_assert(TC_TILES * 16 <= 64, "one lane of the first wavefront per (tile, wavefront)");
        const bool used = lane < TC_TILES * 16;
        const int k = used ? lane >> 4 : 0, w = lane & 15;
#pragma unroll
        for (int q = 0; q < NMRG; ++q) {
            const u32 a = !used ? 0u : s_cnt[k][w][q];
            u32 in = a;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                u32 v = __shfl_up(in, o);
                if (lane >= o) in += v;
            }
            if (used) s_cnt[k][w][q] = in - a;
            if (lane == 63) s_base[q] = in;
        }
        wave_sync();
        if (lane < NMRG) {     // the block's atomics are in flight together
            const u32 tot = s_base[lane];
            s_base[lane] = tot ? atomicAdd(&ctr->n_touched[lane], tot) : 0u;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < TC_TILES; ++k) {
        const long long x = ((long long)blockIdx.x * TC_TILES + k) * 1024 + threadIdx.x;
        if (x < N && mc[k] >= 0)
            tlists[(size_t)mc[k] * N + s_base[mc[k]] + s_cnt[k][wave][mc[k]] + rank[k]] = (int)x;
    }
    if constexpr (DT != DT_U8) {
        __shared__ int s_hub[TC_TILES * 1024], s_hubs;
        if (__syncthreads_or(hub) == 0) return;
        if (threadIdx.x == 0) s_hubs = 0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < TC_TILES; ++k) {
            const long long x = ((long long)blockIdx.x * TC_TILES + k) * 1024 + threadIdx.x;
            if (x < N && cnt[x] > cap + LATE_OPEN) s_hub[atomicAdd(&s_hubs, 1)] = (int)x;
        }
        __syncthreads();
        const int n = s_hubs;
        for (int h = 0; h < n; ++h) close_late<DT>(s_hub[h], cnt[s_hub[h]] - cap, heads, props, X, d);
    }
}

// Merge of the touched vertices whose kept entries + received edges number at most G: one vertex per
// group of G lanes.  list <- first R distinct keys; tcls[it] <- degree class if a "new" entry survives, else -1.
// Lane `sub` of a group holds list slot `sub` and inbox slot G-1-sub, so what to load depends only on
// the vertex; the loads of the next vertex and the list entry of the one after are issued before the
// current vertex is sorted.
struct MergeItem {
    int x;        // vertex, -1 past the end of the list
    int nb, c;    // kept entries, received entries
    u64 kr, ki;   // list slot `sub`, inbox slot G-1-sub (either may be garbage: masked by nb, c)
};

template <int G>
__device__ __forceinline__ MergeItem merge_item_load(int x, int R, const u64 *keys, const int *deg,
                                                     const int *cnt, const u64 *inbox, int sub)
{
    // past the end of the list (x < 0) vertex 0 is read instead and given no entries: loads without branches
    MergeItem m;
    const size_t xx = (size_t)(x >= 0 ? x : 0);
    const int nb = deg[xx], c = cnt[xx];
    m.x = x;
    m.nb = x >= 0 ? nb : 0;
    m.c = x >= 0 ? c : 0;
    m.kr = keys[xx * R + (sub < R ? sub : R - 1)];
    m.ki = inbox[xx * INBOX_CAP + (G - 1 - sub)];
    return m;
}

// Wavefront `first` of `nwaves` that share the list tlist[0 .. n).
template <int G, int DT, bool SEEK>
__device__ __forceinline__ void merge_group_body(int R, u64 *keys, int *deg, const int *tlist, u32 n, u32 first, u32 nwaves,
                                                 int *cnt, const u64 *inbox, int8_t *tcls, int use_classes, RoundCtr *ctr,
                                                 int same_bits, OpenEdges *s_open, const char *__restrict__ X, int d)
{
    int dropped = 0;
    static_assert(G <= INBOX_CAP, "a group merge reads the received edges from the inbox only");
    int lane = threadIdx.x & 63, sub = lane & (G - 1), shift = lane & ~(G - 1);
    const u64 gmask = G == 64 ? ~0ull : ((1ull << (G & 63)) - 1ull);
    const u32 gid = first * (64 / G) + (u32)(lane / G), ngrp = nwaves * (64 / G);
    if (gid - (DT == DT_U8 ? 0u : (u32)(lane / G)) >= n) return;
    // list indices fit 32 bits with room to spare: n <= 2^31 and three strides of the grid are far below 2^31
    auto vertex_at = [&](u32 i) -> int { const int v = tlist[i < n ? i : n - 1u]; return i < n ? v : -1; };
    MergeItem cur = merge_item_load<G>(vertex_at(gid), R, keys, deg, cnt, inbox, sub);
    int x_next = vertex_at(gid + ngrp);
    int x_after = vertex_at(gid + 2u * ngrp);
    // (open distances are computed by the whole wavefront: it leaves the loop as one, groups past the end hold no vertex)
    const u32 lead = DT == DT_U8 ? 0u : (u32)(lane / G);
    for (u32 it = gid; it - lead < n; it += ngrp) {
        if constexpr (DT != DT_U8) {
            lane = afresh(lane);
            sub = lane & (G - 1);
            shift = lane & ~(G - 1);
        }
        const MergeItem nxt = merge_item_load<G>(x_next, R, keys, deg, cnt, inbox, sub);
        x_next = x_after;
        x_after = vertex_at(it + 3u * ngrp);

        const int x = cur.x, nb = cur.nb, c = cur.c;
        u64 *row = keys + (size_t)x * R;
        u64 k = KEY_PAD;
        if (sub < nb) k = cur.kr;
        else if (G - 1 - sub < c) k = cur.ki;
        k = close_keys<DT, G, SEEK>(k, x, sub >= nb && G - 1 - sub < c, k, sub < nb, same_bits, s_open, X, d, lane);
        k = group_sort<G>(k);
        u64 prev = shfl_up1_u64(k);
        if (sub == 0) prev = KEY_PAD;
        const bool keep = (k != KEY_PAD) && ((k >> 1) != (prev >> 1));
        const u64 m = (__builtin_amdgcn_ballot_w64(keep) >> shift) & gmask;
        const int pos = __popcll(m & lanes_below(sub));
        const bool w = keep && pos < R;
        if (w) row[pos] = k;
        const u64 nm = (__builtin_amdgcn_ballot_w64(w && (k & 1ull)) >> shift) & gmask;
        if (sub == 0 && (DT == DT_U8 || x >= 0)) {
            int nd = __popcll(m);
            if (nd > R) { dropped += nd - R; nd = R; }
            deg[x] = nd;
            cnt[x] = 0;
            tcls[it] = nm ? (int8_t)degree_class(nd, use_classes) : (int8_t)-1;
        }
        cur = nxt;
    }
    if (dropped) atomicAdd(&ctr->stat[blockIdx.x & (STAT_SLOTS - 1)][4], (u64)dropped);
}

// General merge (any size): one touched vertex per wavefront; kept entries + inbox + late edges.
// The common case (no late edges, at most 128 keys in all) is sorted in registers from
// loads issued one vertex ahead: lane l holds list slots l and l + 64 and inbox slot 63 - l.
struct WideItem {
    int x, nb, c;
    u64 r0, r1, in;
};

__device__ __forceinline__ WideItem wide_item_load(int x, int R, const u64 *keys, const int *deg, const int *cnt,
                                                   const u64 *inbox, int lane)
{
    WideItem m;
    const size_t xx = (size_t)(x >= 0 ? x : 0);      // as in merge_item_load
    const int nb = deg[xx], c = cnt[xx];
    m.x = x;
    m.nb = x >= 0 ? nb : 0;
    m.c = x >= 0 ? c : 0;
    m.r0 = keys[xx * R + (lane < R ? lane : R - 1)];
    m.r1 = keys[xx * R + (lane + 64 < R ? lane + 64 : R - 1)];
    m.in = inbox[xx * INBOX_CAP + (INBOX_CAP - 1 - lane)];
    return m;
}

// The edge at props[at] of one of a vertex's late lists (see LATE_LISTS), if there is one.
struct LateEdge {
    u64 key;
    u32 next;
};
__device__ __forceinline__ LateEdge late_edge(const Prop *props, u32 at, bool have)
{
    LateEdge e;
    e.key = KEY_PAD;
    e.next = 0;
    if (have) {
        e.key = props[at].key;
        e.next = props[at].next;
    }
    return e;
}

template <int DT, bool SEEK>
__device__ __forceinline__ void merge_general_body(int R, u64 *keys, int *deg, const int *tlist, u32 n, u32 first, u32 nwaves,
                                                   int *cnt, const u64 *inbox,
                                                   LateHeads heads, const Prop *props, int8_t *tcls,
                                                   int use_classes, u64 (*s_stage)[RNND_MAX_R], RoundCtr *ctr,
                                                   int same_bits, OpenEdges *s_open, const char *__restrict__ X, int d)
{
    int dropped = 0;
    static_assert(INBOX_CAP == 64 && LATE_LISTS == 64, "lane l prefetches inbox slot 63 - l and walks list l");
    const int cap = round_inbox(R);
    const int wave = threadIdx.x >> 6;
    int lane = threadIdx.x & 63;
    const u32 gw = first, nw = nwaves;
    if (gw >= n) return;
    auto vertex_at = [&](u32 i) -> int { const int v = tlist[i < n ? i : n - 1u]; return i < n ? v : -1; };
    WideItem cur = wide_item_load(vertex_at(gw), R, keys, deg, cnt, inbox, lane);
    int x_next = vertex_at(gw + nw);
    int x_after = vertex_at(gw + 2u * nw);
    for (u32 it = gw; it < n; it += nw) {
        if constexpr (DT != DT_U8) lane = afresh(lane);
        const WideItem nxt = wide_item_load(x_next, R, keys, deg, cnt, inbox, lane);
        x_next = x_after;
        x_after = vertex_at(it + 3u * nw);

        const int x = __builtin_amdgcn_readfirstlane(cur.x);
        const int nb = __builtin_amdgcn_readfirstlane(cur.nb), c = __builtin_amdgcn_readfirstlane(cur.c);
        cur.in = close_keys<DT, 64, SEEK>(cur.in, x, 63 - lane < (c < cap ? c : cap), cur.r0, lane < nb, same_bits, s_open, X, d, lane);
        bool any_new = false;
        int nd;
        if (c <= cap && nb + c <= 128) {
            u64 k[2];
            k[0] = lane < nb ? cur.r0 : KEY_PAD;
            k[1] = lane + 64 < nb ? cur.r1 : (63 - lane < c ? cur.in : KEY_PAD);
            wave_sort<2>(k);
            nd = wave_unique_prefix<2>(k, lane, R, keys + (size_t)x * R, &any_new, &dropped);
        } else {
            const int ca = c < cap ? c : cap, late = c - ca;
            const u32 *head = heads.base + (size_t)x * heads.stride;
            u64 *row = keys + (size_t)x * R;
            if (nb + late <= 64) {
                // a full inbox, and at most one late edge per list: the lists from the top lane down, above the kept entries
                u64 k[2];
                k[0] = lane < nb ? cur.r0 : late_edge(props, 63 - lane < late ? head[63 - lane] : 0u, 63 - lane < late).key;
                k[0] = close_keys<DT, 64, SEEK>(k[0], x, lane >= nb && 63 - lane < late, k[0], lane < nb, same_bits, s_open, X, d, lane);
                k[1] = 63 - lane < ca ? cur.in : KEY_PAD;
                wave_sort<2>(k);
                nd = wave_unique_prefix<2>(k, lane, R, row, &any_new, &dropped);
            } else {
                // inbox and late edges in chunks of 128 against the best R found so far; lane l walks list l, and the two
                // records of the next chunk travel while this one is sorted and cut
                const LateEdge first = late_edge(props, lane < late ? head[lane] : 0u, lane < late);
                u64 k[4];
                k[0] = lane < nb ? cur.r0 : KEY_PAD;
                k[1] = lane + 64 < nb ? cur.r1 : KEY_PAD;
                k[2] = 63 - lane < ca ? cur.in : KEY_PAD;
                k[3] = close_keys<DT, 64, SEEK>(first.key, x, lane < late, k[0], lane < nb, same_bits, s_open, X, d, lane);
                LateEdge a = late_edge(props, first.next, LATE_LISTS + lane < late);
                for (int at = LATE_LISTS;; at += 2 * LATE_LISTS) {      // edges taken so far; `a` is the next one of my list
                    wave_sort<4>(k);
                    const LateEdge b = late_edge(props, a.next, at + LATE_LISTS + lane < late);
                    nd = wave_unique_prefix<4>(k, lane, R, s_stage[wave], &any_new, &dropped);
                    wave_sync();
                    k[0] = lane < nd ? s_stage[wave][lane] : KEY_PAD;
                    k[1] = lane + 64 < nd ? s_stage[wave][lane + 64] : KEY_PAD;
                    wave_sync();
                    if (at >= late) break;
                    k[2] = close_keys<DT, 64, SEEK>(a.key, x, at + lane < late, k[0], lane < nd, same_bits, s_open, X, d, lane);
                    k[3] = close_keys<DT, 64, SEEK>(b.key, x, at + LATE_LISTS + lane < late, k[0], lane < nd, same_bits, s_open, X, d, lane);
                    a = late_edge(props, b.next, at + 2 * LATE_LISTS + lane < late);
                }
                if (lane < nd) row[lane] = k[0];
                if (lane + 64 < nd) row[lane + 64] = k[1];
            }
        }
        if (lane == 0) {
            deg[x] = nd;
            cnt[x] = 0;
            tcls[it] = any_new ? (int8_t)degree_class(nd, use_classes) : (int8_t)-1;
        }
        cur = nxt;
    }
    if (lane == 0 && dropped) atomicAdd(&ctr->stat[blockIdx.x & (STAT_SLOTS - 1)][4], (u64)dropped);
}

// All four merge classes in one launch: blockIdx.y = merge class (touched list y, tcls + y*N).
template <int DT>
__global__ __launch_bounds__(BLOCK, (DT == DT_U8 ? 1 : 5)) void k_merge(long long N, int R, u64 *keys, int *deg, const int *tlists,
                                                 const u32 *n_touched, int *cnt, const u64 *inbox,
                                                 LateHeads heads, const Prop *props, int8_t *tcls,
                                                 int use_classes, int same_bits, RoundCtr *ctr, const char *__restrict__ X, int d)
{
    __shared__ u64 s_stage[WAVES_PER_BLOCK][RNND_MAX_R];
    static_assert(sizeof(OpenEdges) <= sizeof(u64) * RNND_MAX_R, "the open edges lie in the stage, which is free until they are closed");
    OpenEdges *so = reinterpret_cast<OpenEdges *>(&s_stage[threadIdx.x >> 6]);
    const int y = blockIdx.y;
    const int *tlist = tlists + (size_t)y * N;
    int8_t *tc = tcls + (size_t)y * N;
    const u32 n = n_touched[y], first = blockIdx.x * WAVES_PER_BLOCK + (threadIdx.x >> 6), nwaves = gridDim.x * WAVES_PER_BLOCK;
    if (y == 0) merge_group_body<16, DT, true>(R, keys, deg, tlist, n, first, nwaves, cnt, inbox, tc, use_classes, ctr, same_bits, so, X, d);
    else if (y == 1) merge_group_body<32, DT, true>(R, keys, deg, tlist, n, first, nwaves, cnt, inbox, tc, use_classes, ctr, same_bits, so, X, d);
    else if (y == 2) merge_group_body<64, DT, true>(R, keys, deg, tlist, n, first, nwaves, cnt, inbox, tc, use_classes, ctr, same_bits, so, X, d);
    else merge_general_body<DT, true>(R, keys, deg, tlist, n, first, nwaves, cnt, inbox, heads, props, tc, use_classes, s_stage, ctr, same_bits, so, X, d);
}

// Classify, merge and compact of a round in one launch, for inputs whose rounds wait for launches (4-6 us each) rather than for
// their work: a block takes `span` vertices (at most one per thread), sorts those that received edges into the merge classes in
// LDS, merges them, and appends the ones that hold a "new" entry to the next active lists with one atomic per degree class.
template <int DT>
__global__ __launch_bounds__(BLOCK, (DT == DT_U8 ? 1 : 5)) void k_merge_blocks(long long N, int span, int R, u64 *keys, int *deg, int *cnt,
                                                                               const u64 *inbox, LateHeads heads, Prop *props, int use_classes,
                                                                               RoundCtr *ctr, int *lists, u32 *n_next,
                                                                               const char *__restrict__ X, int d, int scattered, u32 enough)
{
    __shared__ u64 s_stage[WAVES_PER_BLOCK][RNND_MAX_R];
    __shared__ int s_list[NMRG][BLOCK];
    __shared__ int8_t s_cls[NMRG][BLOCK];
    __shared__ u32 s_n[NMRG], s_out[NDEG], s_base[NDEG];
    if (scattered && blockIdx.x == 0 && threadIdx.x == 0) end_scan(ctr, enough);
    const int wave = threadIdx.x >> 6;
    OpenEdges *so = reinterpret_cast<OpenEdges *>(&s_stage[wave]);
    const int cap = round_inbox(R);
    if (threadIdx.x < NMRG) s_n[threadIdx.x] = 0;
    if (threadIdx.x < NDEG) s_out[threadIdx.x] = 0;
    __syncthreads();
    const long long x = (long long)blockIdx.x * span + threadIdx.x;
    int c = 0;
    if ((int)threadIdx.x < span && x < N) c = cnt[x];
    if (c > 0) {
        const int q = merge_class(deg[x], c, cap);
        s_list[q][atomicAdd(&s_n[q], 1u)] = (int)x;
    }
    __syncthreads();
    if (DT != DT_U8) {
        for (u32 i = 0; i < s_n[3]; ++i) {
            const int v = s_list[3][i], late = cnt[v] - cap;
            if (late > LATE_OPEN) close_late<DT>(v, late, heads, props, X, d);
        }
        __syncthreads();
    }
    // (the classes start with different wavefronts)
    merge_group_body<16, DT, false>(R, keys, deg, s_list[0], s_n[0], wave, 4, cnt, inbox, s_cls[0], use_classes, ctr, 0, so, X, d);
    merge_group_body<32, DT, false>(R, keys, deg, s_list[1], s_n[1], (wave + 3) & 3, 4, cnt, inbox, s_cls[1], use_classes, ctr, 0, so, X, d);
    merge_group_body<64, DT, false>(R, keys, deg, s_list[2], s_n[2], (wave + 2) & 3, 4, cnt, inbox, s_cls[2], use_classes, ctr, 0, so, X, d);
    merge_general_body<DT, false>(R, keys, deg, s_list[3], s_n[3], (wave + 1) & 3, 4, cnt, inbox, heads, props, s_cls[3], use_classes, s_stage, ctr, 0, so, X, d);
    __syncthreads();
    // at most `span` items in all: one per thread
    int k = -1, item = 0;
    u32 at = 0, i = threadIdx.x;
#pragma unroll
    for (int q = 0; q < NMRG; ++q) {
        if (k == -1 && i < s_n[q]) {
            item = s_list[q][i];
            k = s_cls[q][i];
            if (k < 0) k = -2;
        } else if (k == -1) {
            i -= s_n[q];
        }
    }
    if (k >= 0) at = atomicAdd(&s_out[k], 1u);
    __syncthreads();
    if (threadIdx.x < NDEG) {
        const u32 n = s_out[threadIdx.x];
        s_base[threadIdx.x] = n ? atomicAdd(&n_next[threadIdx.x], n) : 0u;
    }
    __syncthreads();
    if (k >= 0) lists[(size_t)k * N + s_base[k] + at] = item;
}

// Items i < n with cls[first + i] >= 0 are appended to list cls[first + i]; item i stands for vertex idx[i]
// (or first + i).  blockIdx.y = s selects source list s: n_ptr[s], idx + s*N, cls + s*N.  One atomic per class
// per 1024 items.  With `taken`, the class of every listed item is then cleared there (taken may be cls).
__global__ __launch_bounds__(1024) void k_compact_classes(const u32 *n_ptr, u32 n_fixed, const int *idx,
                                                          const int8_t *cls, int *lists, long long N,
                                                          u32 *n_out, u32 first, int8_t *taken)
{
    __shared__ u32 s_cnt[16][NDEG], s_base[NDEG];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const u32 n = n_ptr ? n_ptr[blockIdx.y] : n_fixed;
    if (idx) idx += (size_t)blockIdx.y * N;
    cls += (size_t)blockIdx.y * N;
    for (u32 base = blockIdx.x * 1024u; base < n; base += gridDim.x * 1024u) {
        const u32 i = base + threadIdx.x;
        const int c = i < n ? (int)cls[first + i] : -1;
        u64 b[NDEG];
#pragma unroll
        for (int k = 0; k < NDEG; ++k) b[k] = __builtin_amdgcn_ballot_w64(c == k);
        if (lane == 0) {
#pragma unroll
            for (int k = 0; k < NDEG; ++k) s_cnt[wave][k] = (u32)__popcll(b[k]);
        }
        __syncthreads();
        if (threadIdx.x < NDEG) {
            u32 tot = 0;
            for (int w = 0; w < 16; ++w) { u32 a = s_cnt[w][threadIdx.x]; s_cnt[w][threadIdx.x] = tot; tot += a; }
            s_base[threadIdx.x] = tot ? atomicAdd(&n_out[threadIdx.x], tot) : 0u;
        }
        __syncthreads();
        if (c >= 0 && c < NDEG) {
            u64 mine = b[0];
#pragma unroll
            for (int k = 1; k < NDEG; ++k) mine = (c == k) ? b[k] : mine;
            const u32 off = s_base[c] + s_cnt[wave][c] + (u32)__popcll(mine & lanes_below(lane));
            lists[(size_t)c * N + off] = idx ? idx[i] : (int)(first + i);
            if (taken) taken[first + i] = (int8_t)-1;
        }
        __syncthreads();
    }
}

// Block-sequential passes keep the class of every vertex that holds a "new" entry in vcls[] between runs:
// after a run's merge, vcls[x] <- tcls of every touched vertex x (blockIdx.y = merge class).
__global__ __launch_bounds__(256) void k_store_classes(const u32 *n_touched, const int *tlists, const int8_t *tcls,
                                                       long long N, int8_t *vcls)
{
    const u32 n = n_touched[blockIdx.y];
    const int *tl = tlists + (size_t)blockIdx.y * N;
    const int8_t *tc = tcls + (size_t)blockIdx.y * N;
    for (u32 i = blockIdx.x * 256u + threadIdx.x; i < n; i += gridDim.x * 256u) vcls[tl[i]] = tc[i];
}

// ------------------------------------------------------------ AddReverseEdges
// The first kernel of a call clears the call's cursors and the lengths of the next round's lists (n_next may be null), which only kernels after it use.
__device__ __forceinline__ void clear_cursors(u32 *misc, u32 *n_next)
{
    if (blockIdx.x == 0 && threadIdx.x < 16) {
        misc[threadIdx.x] = 0u;
        if (n_next && threadIdx.x < NDEG) n_next[threadIdx.x] = 0u;
    }
}

// The union and the out-degree cut of Alg. 5 need, for every x, the edges that point to x.  Every edge (u, v) takes an arrival
// number at v (one atomic on fill[v]); the first INBOX_CAP arrivals are written to v's inbox as
// key(delta, u, new).  A later arrival is remembered with its edge (late[] holds its number, over[u]
// one bit per list position of u, mark[u] says that u has any) and k_reverse_surplus places it in
// v's bin once bins exist.
// 16 lanes per vertex (lists are mostly short: a wavefront per vertex would leave most lanes idle and the
// kernel is bound by its three dependent trips to memory: degree, list entry, arrival number).
__global__ __launch_bounds__(BLOCK) void k_reverse_scatter(long long N, int R, const u64 *keys, const int *deg,
                                                           int *fill, u64 *inbox, u32 *late, u64 *over,
                                                           int8_t *mark, u32 *misc, u32 *n_next)
{
    clear_cursors(misc, n_next);
    const int lane = threadIdx.x & 63, sub = lane & 15, gsh = lane & ~15;
    const long long u = ((long long)blockIdx.x * BLOCK + threadIdx.x) >> 4;
    const bool valid = u < N;
    const int m = valid ? deg[u] : 0;
    // the same number of trips for the four vertices of a wavefront (the ballot below is the wavefront's)
    int mmax = m;
    mmax = max(mmax, __shfl_xor(mmax, 16));
    mmax = max(mmax, __shfl_xor(mmax, 32));
    u64 ov[2] = {0ull, 0ull};
    for (int e0 = 0; e0 < mmax; e0 += 16) {
        const int e = e0 + sub;
        bool is_late = false;
        if (e < m) {
            const u64 k = keys[(size_t)u * R + e];
            const u32 v = key_id(k);
            const int a = atomicAdd(&fill[v], 1);
            if (a < INBOX_CAP) {
                inbox[(size_t)v * INBOX_CAP + a] = make_key(key_dist(k), (u32)u, 1u);
            } else {
                late[(size_t)u * R + e] = (u32)a;
                is_late = true;
            }
        }
        const u64 bits = (__builtin_amdgcn_ballot_w64(is_late) >> gsh) & 0xFFFFull;     // my vertex's 16 positions
        ov[e0 >> 6] |= bits << (e0 & 63);
    }
    if (valid && sub == 0) {
        const bool any = (ov[0] | ov[1]) != 0;
        mark[u] = (int8_t)any;
        if (any) { over[2 * u] = ov[0]; over[2 * u + 1] = ov[1]; }
    }
}

// The late arrivals of k_reverse_scatter go to their targets' bins (which hold arrivals INBOX_CAP, ...).
__global__ __launch_bounds__(BLOCK) void k_reverse_surplus(long long N, int R, const u64 *keys, const u32 *late,
                                                           const u64 *over, const int8_t *mark,
                                                           const int *binoff, u64 *bins, const u32 *n_binned)
{
    if (*n_binned == 0u) return;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const long long u = (long long)blockIdx.x * WAVES_PER_BLOCK + wave;
    if (u >= N || !mark[u]) return;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const u64 ov = over[2 * u + r];
        if ((ov >> lane) & 1ull) {
            const int e = 64 * r + lane;
            const u64 k = keys[(size_t)u * R + e];
            const u32 v = key_id(k);
            bins[(size_t)binoff[v] + (late[(size_t)u * R + e] - INBOX_CAP)] = make_key(key_dist(k), (u32)u, 1u);
        }
    }
}

// ---- the same transposition without one device-scope atomic per edge (large N) -------------------------
// Targets are cut into ranges of RANGE_TARGETS consecutive ids.  Every block of BIN_CHUNK source vertices
// counts its edges per range in LDS (k_bin_count); a column-wise prefix over the blocks turns the counts into
// the place of every (block, range) run in one edge array ordered by range (k_bin_offsets, k_bin_bases: no
// atomics, the layout is a pure function of the graph); the blocks copy their edges there, taking ranks from
// LDS counters (k_bin_partition); then one workgroup per range, which alone owns its targets, counts the edges
// of each target in LDS, hands out the surplus bins, and moves every edge into its target's inbox or bin with
// arrival numbers from the LDS counters (k_bin_place).  What k_reverse_scatter, the first k_assign_bins and
// k_reverse_surplus leave behind -- fill[], inbox, binoff[], bins, cand[], zeroed cnt[] and cnt_in[] -- is
// left in the same form (slot order inside an inbox is arbitrary in both; every consumer sorts).
#define RANGE_BITS 11
#define RANGE_TARGETS (1 << RANGE_BITS)
#define RANGE_MAX 16384       // ranges a block can histogram in LDS (64 KB): N <= RANGE_MAX * RANGE_TARGETS
#define BIN_CHUNK 2048        // source vertices per block of the count and partition kernels
#define BIN_THREADS 1024

// Walks the edges of the block's BIN_CHUNK source vertices: thread t of a pass takes list position t % 16 of
// vertex t / 16 (lists are short on average; longer ones take further trips), four vertices per thread in
// flight.  f(u, key) is called once per edge.
template <typename F>
__device__ __forceinline__ void for_each_edge_of_chunk(long long N, int W, const u64 *__restrict__ keys,
                                                       const int *__restrict__ deg, F f)
{
    const int sub = threadIdx.x & 15, grp = threadIdx.x >> 4;      // 64 groups of 16 lanes
    const long long u0 = (long long)blockIdx.x * BIN_CHUNK;
    constexpr int GROUPS = BIN_THREADS / 16, UNROLL = 4;
    for (int i = grp; i < BIN_CHUNK; i += GROUPS * UNROLL) {
        long long u[UNROLL];
        int m[UNROLL];
        u64 k[UNROLL];
#pragma unroll
        for (int j = 0; j < UNROLL; ++j) {
            u[j] = u0 + i + j * GROUPS;
            m[j] = (i + j * GROUPS < BIN_CHUNK && u[j] < N) ? deg[u[j]] : 0;
        }
#pragma unroll
        for (int j = 0; j < UNROLL; ++j) k[j] = sub < m[j] ? keys[(size_t)u[j] * W + sub] : 0ull;
#pragma unroll
        for (int j = 0; j < UNROLL; ++j) {
            if (sub < m[j]) f(u[j], k[j]);
            for (int e = sub + 16; e < m[j]; e += 16) f(u[j], keys[(size_t)u[j] * W + e]);
        }
    }
}

__global__ __launch_bounds__(BIN_THREADS) void k_bin_count(long long N, int W, const u64 *__restrict__ keys,
                                                           const int *__restrict__ deg, u32 nranges, u32 *__restrict__ blockhist,
                                                           u32 *misc, u32 *n_next)
{
    __shared__ u32 hist[RANGE_MAX];
    clear_cursors(misc, n_next);
    for (u32 r = threadIdx.x; r < nranges; r += BIN_THREADS) hist[r] = 0;
    __syncthreads();
    for_each_edge_of_chunk(N, W, keys, deg, [&](long long, u64 k) { atomicAdd(&hist[key_id(k) >> RANGE_BITS], 1u); });
    __syncthreads();
    u32 *out = blockhist + (size_t)blockIdx.x * nranges;
    for (u32 r = threadIdx.x; r < nranges; r += BIN_THREADS) out[r] = hist[r];
}

// blockhist[b][r] <- edges of range r in the blocks before b; range_tot[r] <- edges of range r in all.
// A workgroup takes 64 ranges; its 16 wavefronts each take a slice of consecutive blocks (a wavefront reads
// 64 consecutive counters of one block at a time), sum it, and after a prefix over the slices walk it again.
__global__ __launch_bounds__(1024) void k_bin_offsets(u32 nblocks, u32 nranges, u32 *__restrict__ blockhist,
                                                      u32 *__restrict__ range_tot)
{
    __shared__ u32 s_sum[16][64];
    const u32 col = threadIdx.x & 63, slice = threadIdx.x >> 6;
    const u32 r = blockIdx.x * 64 + col;
    const bool have = r < nranges;
    const u32 per = (nblocks + 15) / 16;
    const u32 b0 = slice * per < nblocks ? slice * per : nblocks, b1 = b0 + per < nblocks ? b0 + per : nblocks;
    u32 sum = 0;
    if (have) {
        u32 b = b0;
        for (; b + 4 <= b1; b += 4) {
            const u32 c0 = blockhist[(size_t)b * nranges + r], c1 = blockhist[(size_t)(b + 1) * nranges + r];
            const u32 c2 = blockhist[(size_t)(b + 2) * nranges + r], c3 = blockhist[(size_t)(b + 3) * nranges + r];
            sum += c0 + c1 + c2 + c3;
        }
        for (; b < b1; ++b) sum += blockhist[(size_t)b * nranges + r];
    }
    s_sum[slice][col] = sum;
    __syncthreads();
    u32 run = 0, all = 0;
    for (u32 sl = 0; sl < 16; ++sl) {
        const u32 v = s_sum[sl][col];
        run += sl < slice ? v : 0u;
        all += v;
    }
    if (have) {
        if (slice == 0) range_tot[r] = all;
        u32 b = b0;
        for (; b + 4 <= b1; b += 4) {
            const u32 c0 = blockhist[(size_t)b * nranges + r], c1 = blockhist[(size_t)(b + 1) * nranges + r];
            const u32 c2 = blockhist[(size_t)(b + 2) * nranges + r], c3 = blockhist[(size_t)(b + 3) * nranges + r];
            blockhist[(size_t)b * nranges + r] = run;
            blockhist[(size_t)(b + 1) * nranges + r] = run + c0;
            blockhist[(size_t)(b + 2) * nranges + r] = run + c0 + c1;
            blockhist[(size_t)(b + 3) * nranges + r] = run + c0 + c1 + c2;
            run += c0 + c1 + c2 + c3;
        }
        for (; b < b1; ++b) {
            const u32 c = blockhist[(size_t)b * nranges + r];
            blockhist[(size_t)b * nranges + r] = run;
            run += c;
        }
    }
}

// range_base[r] <- edges of the ranges before r (one block; nranges <= RANGE_MAX); range_base[nranges] <- all.
__global__ __launch_bounds__(1024) void k_bin_bases(u32 nranges, const u32 *__restrict__ range_tot, u32 *__restrict__ range_base)
{
    __shared__ u32 s_w[16];
    constexpr int PER = RANGE_MAX / 1024;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    u32 v[PER], mine = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const u32 r = threadIdx.x * PER + k;
        v[k] = r < nranges ? range_tot[r] : 0u;
        mine += v[k];
    }
    u32 incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const u32 t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
    }
    if (lane == 63) s_w[wave] = incl;
    __syncthreads();
    u32 before = 0;
    for (int w = 0; w < wave; ++w) before += s_w[w];
    u32 run = before + incl - mine;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const u32 r = threadIdx.x * PER + k;
        if (r < nranges) range_base[r] = run;
        run += v[k];
    }
    if (threadIdx.x == 1023) range_base[nranges] = run;
}

// Edge (u, v) -> part[place of (my block, range of v) + rank inside it] = { key(delta, u, new), v }.
__global__ __launch_bounds__(BIN_THREADS) void k_bin_partition(long long N, int W, const u64 *__restrict__ keys,
                                                               const int *__restrict__ deg, u32 nranges,
                                                               const u32 *__restrict__ blockhist,
                                                               const u32 *__restrict__ range_base, Prop *__restrict__ part)
{
    __shared__ u32 cursor[RANGE_MAX];
    const u32 *mine = blockhist + (size_t)blockIdx.x * nranges;
    for (u32 r = threadIdx.x; r < nranges; r += BIN_THREADS) cursor[r] = range_base[r] + mine[r];
    __syncthreads();
    for_each_edge_of_chunk(N, W, keys, deg, [&](long long u, u64 k) {
        const u32 v = key_id(k);
        const u32 at = atomicAdd(&cursor[v >> RANGE_BITS], 1u);
        Prop pr;
        pr.key = make_key(key_dist(k), (u32)u, 1u);
        pr.tgt = v;
        pr.next = 0;
        part[at] = pr;
    });
}

// One workgroup per range of targets.  One sweep over the range's edges numbers the arrivals per target in LDS
// and writes the first INBOX_CAP of each target straight into its inbox; later arrivals (hubs: rare) wait in an
// LDS stash until the sweep has counted every target and the surplus bins are handed out.  A range whose
// stash overflows is swept again with the bins known, rewriting every place.
#define PLACE_THREADS 512
#define PLACE_STASH 2048
__global__ __launch_bounds__(PLACE_THREADS) void k_bin_place(long long N, int R, const Prop *__restrict__ part,
                                                             const u32 *__restrict__ range_base, const int *__restrict__ deg,
                                                             int *__restrict__ fill, u64 *__restrict__ inbox,
                                                             int *__restrict__ binoff, u64 *__restrict__ bins,
                                                             u32 *__restrict__ bin_cursor, int *__restrict__ zero_a,
                                                             int *__restrict__ zero_b, int8_t *__restrict__ cand)
{
    __shared__ u32 arr[RANGE_TARGETS], bin_at[RANGE_TARGETS];
    __shared__ u64 st_key[PLACE_STASH];
    __shared__ u32 st_tgt[PLACE_STASH], st_arr[PLACE_STASH];
    __shared__ u32 s_w[PLACE_THREADS / 64], s_base, s_stash;
    constexpr int PER = RANGE_TARGETS / PLACE_THREADS, NW = PLACE_THREADS / 64, UNROLL = 4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const u32 first = blockIdx.x << RANGE_BITS;          // first target of my range
    const u32 e0 = range_base[blockIdx.x], e1 = range_base[blockIdx.x + 1];
#pragma unroll
    for (int k = 0; k < PER; ++k) arr[threadIdx.x * PER + k] = 0;
    if (threadIdx.x == 0) s_stash = 0;
    __syncthreads();
    // pass == 0: arrivals below INBOX_CAP to the inbox, later ones to the stash.  pass == 1 (only after a stash
    // overflow): every edge again, surplus straight to the bins.
    auto sweep = [&](const int pass) {
        for (u32 e = e0 + threadIdx.x; e < e1; e += PLACE_THREADS * UNROLL) {
            Prop pr[UNROLL];
#pragma unroll
            for (int j = 0; j < UNROLL; ++j) {
                pr[j].tgt = 0xFFFFFFFFu;
                if (e + j * PLACE_THREADS < e1) pr[j] = part[e + j * PLACE_THREADS];
            }
#pragma unroll
            for (int j = 0; j < UNROLL; ++j) {
                if (pr[j].tgt == 0xFFFFFFFFu) continue;
                const u32 t = pr[j].tgt - first;
                const u32 a = atomicAdd(&arr[t], 1u);
                if (a < (u32)INBOX_CAP) {
                    inbox[(size_t)pr[j].tgt * INBOX_CAP + a] = pr[j].key;
                } else if (pass == 1) {
                    bins[(size_t)bin_at[t] + (a - INBOX_CAP)] = pr[j].key;
                } else {
                    const u32 at = atomicAdd(&s_stash, 1u);
                    if (at < (u32)PLACE_STASH) { st_key[at] = pr[j].key; st_tgt[at] = t; st_arr[at] = a; }
                }
            }
        }
    };
    sweep(0);
    __syncthreads();
    // per target: the count, the candidate mark of the in-degree cut, cleared counters, a bin for the surplus
    u32 c[PER], surplus[PER], mine = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        c[k] = arr[threadIdx.x * PER + k];
        surplus[k] = c[k] > (u32)INBOX_CAP ? c[k] - (u32)INBOX_CAP : 0u;
        mine += surplus[k];
    }
    u32 incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const u32 t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
    }
    if (lane == 63) s_w[wave] = incl;
    __syncthreads();
    if (threadIdx.x == 0) {
        u32 tot = 0;
        for (int w = 0; w < NW; ++w) { const u32 a = s_w[w]; s_w[w] = tot; tot += a; }
        s_base = tot ? atomicAdd(bin_cursor, tot) : 0u;
    }
    __syncthreads();
    u32 run = s_base + s_w[wave] + incl - mine;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const long long v = (long long)first + threadIdx.x * PER + k;
        if (v < N) {
            fill[v] = (int)c[k];
            zero_a[v] = 0;
            zero_b[v] = 0;
            cand[v] = (int8_t)(deg[v] + (int)c[k] > R);
            binoff[v] = surplus[k] ? (int)run : -1;
        }
        bin_at[threadIdx.x * PER + k] = run;     // where the target's bin starts (if it has one)
        run += surplus[k];
    }
    __syncthreads();
    const u32 stashed = s_stash;
    if (stashed <= (u32)PLACE_STASH) {
        for (u32 i = threadIdx.x; i < stashed; i += PLACE_THREADS)
            bins[(size_t)bin_at[st_tgt[i]] + (st_arr[i] - INBOX_CAP)] = st_key[i];
    } else {
#pragma unroll
        for (int k = 0; k < PER; ++k) arr[threadIdx.x * PER + k] = 0;
        __syncthreads();
        sweep(1);
    }
}

// For every edge (u, v) of a flagged list whose v owns a bin: bins[v] <- key(delta, u, flag).  The flagged
// vertices come as a list (one wavefront per vertex).  Nothing to do when no bin was handed out (*n_binned == 0).
__global__ __launch_bounds__(BLOCK) void k_fill_bins(int R, const u64 *keys, const int *deg, const int *flagged,
                                                     const u32 *n_flagged, const int *binoff, int *fill,
                                                     u64 *bins, u32 flag, const u32 *n_binned)
{
    if (*n_binned == 0u) return;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const u32 n = *n_flagged, nw = gridDim.x * WAVES_PER_BLOCK;
    for (u32 it = blockIdx.x * WAVES_PER_BLOCK + wave; it < n; it += nw) {
        const int u = flagged[it];
        const int m = deg[u];
        for (int e = lane; e < m; e += 64) {
            const u64 k = keys[(size_t)u * R + e];
            const u32 v = key_id(k);
            const int off = binoff[v];
            if (off >= 0) bins[(size_t)off + atomicAdd(&fill[v], 1)] = make_key(key_dist(k), (u32)u, flag);
        }
    }
}

// Alg. 5, union and out-degree cut: list(x) <- first R distinct of list(x) + reversed edges into x (flag new).
// Then the edges of the new list are counted at those targets that can end up with more than R
// incoming edges (cand[v]: |list(v)| + |edges into v| > R before the union; for every other vertex
// the union itself bounds the in-degree by R); rowflag[x] = 0 if the list has such an edge, else -1.
// vcls[x] <- degree class if the list holds a "new" entry, else -1.
struct RevItem {       // what a half-wave holds of its vertex before it is that vertex's turn
    int c, nb;         // reversed edges received, entries held
    u64 kr, ki;        // list slot l32, inbox slot 31 - l32 (either may be garbage: masked by nb, c)
};

__device__ __forceinline__ RevItem rev_item_load(long long x, long long N, int W, const u64 *keys, const int *deg,
                                                 const int *fill, const u64 *inbox, int l32)
{
    // past the last vertex, vertex 0 is read instead and given nothing: loads without branches
    RevItem it;
    const size_t xx = x < N ? (size_t)x : 0;
    const int c = fill[xx], nb = deg[xx];
    it.c = x < N ? c : 0;
    it.nb = x < N ? nb : 0;
    it.kr = keys[xx * W + (l32 < W ? l32 : W - 1)];
    it.ki = inbox[xx * INBOX_CAP + (31 - l32)];
    return it;
}

__global__ __launch_bounds__(BLOCK) void k_reverse_merge(long long N, int W, int R, u64 *keys, int *deg, int *fill,
                                                         const u64 *inbox, const int *binoff, const u64 *bins,
                                                         const int8_t *cand, int *cnt_in, int8_t *rowflag,
                                                         int8_t *vcls, int use_classes)
{   // rows are W slots apart (W >= R); lists are cut to R
    __shared__ u64 s_stage[WAVES_PER_BLOCK][RNND_MAX_R];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    // a wavefront takes two vertices at a time, one per half: lists are short on average, and when both unions
    // have at most 32 keys they are formed side by side (32-lane sorts); otherwise one after the other.  The
    // grid is persistent: what the next pair needs in the short case is loaded before the current pair is sorted.
    const long long npairs = (N + 1) / 2;
    const long long gw = (long long)blockIdx.x * WAVES_PER_BLOCK + wave, nw = (long long)gridDim.x * WAVES_PER_BLOCK;
    if (gw >= npairs) return;
    RevItem cur = rev_item_load(2 * gw + half, N, W, keys, deg, fill, inbox, l32);
    for (long long pair = gw; pair < npairs; pair += nw) {
        const RevItem nxt = rev_item_load(2 * (pair + nw) + half, pair + nw < npairs ? N : 0, W, keys, deg, fill, inbox, l32);
        const long long x0 = 2 * pair, xh = x0 + half;
        const bool have = xh < N;
        const int ch = cur.c, nbh = cur.nb;
        const bool small = __builtin_amdgcn_ballot_w64(nbh + ch > 32) == 0;
        if (small) {
            u64 *row = keys + (size_t)xh * W;
            u64 k = KEY_PAD;
            if (have) {
                if (l32 < nbh) k = cur.kr;
                else if (31 - l32 < ch) k = cur.ki;
            }
            k = group_sort<32>(k);
            u64 prev = shfl_up1_u64(k);
            if (l32 == 0) prev = KEY_PAD;
            const bool keep = (k != KEY_PAD) && ((k >> 1) != (prev >> 1));
            const u32 m = (u32)(__builtin_amdgcn_ballot_w64(keep) >> (32 * half));
            const int pos = __popc(m & ((1u << l32) - 1u));
            const bool w = keep && pos < R;
            if (w) row[pos] = k;
            bool cd = false;
            if (w) {
                const u32 v = key_id(k);
                if (cand[v]) {
                    atomicAdd(&cnt_in[v], 1);
                    cd = true;
                }
            }
            const u32 nm = (u32)(__builtin_amdgcn_ballot_w64(w && (k & 1ull)) >> (32 * half));
            const u32 cm = (u32)(__builtin_amdgcn_ballot_w64(cd) >> (32 * half));
            if (have && l32 == 0) {
                int nd = __popc(m);
                if (nd > R) nd = R;
                deg[xh] = nd;
                fill[xh] = 0;
                rowflag[xh] = (int8_t)(cm != 0 ? 0 : -1);      // class 0 of a compaction = the flagged vertices
                vcls[xh] = nm ? (int8_t)degree_class(nd, use_classes) : (int8_t)-1;
            }
        } else {
            for (int h = 0; h < 2; ++h) {
                const long long x = x0 + h;
                if (x >= N) break;
                u64 *row = keys + (size_t)x * W;
                const int c = __shfl(ch, 32 * h);
                int nd = __shfl(nbh, 32 * h);
                if (c == 0 && nd > R) nd = R;   // Alg. 5 cuts every out-list to its R shortest; the row is sorted and distinct
                if (c > 0) {
                    bool any_new;
                    const int ca = c < INBOX_CAP ? c : INBOX_CAP;
                    wave_sync();    // the staging area may still be read by the previous vertex
                    nd = wave_merge_row(row, nd, inbox + (size_t)x * INBOX_CAP, ca, bins + (c > ca ? binoff[x] : 0), c - ca, R,
                                        s_stage[wave], lane, &any_new);
                    wave_sync();    // the list is read back below by other lanes of this wavefront
                }
                bool nw_ = false, cd = false;
                for (int e = lane; e < nd; e += 64) {
                    const u64 k = row[e];
                    nw_ = nw_ || (k & 1ull);
                    const u32 v = key_id(k);
                    if (cand[v]) {
                        atomicAdd(&cnt_in[v], 1);
                        cd = true;
                    }
                }
                const u64 bn = __builtin_amdgcn_ballot_w64(nw_), bc = __builtin_amdgcn_ballot_w64(cd);
                if (lane == 0) {
                    deg[x] = nd;
                    fill[x] = 0;
                    rowflag[x] = (int8_t)(bc != 0 ? 0 : -1);
                    vcls[x] = bn ? (int8_t)degree_class(nd, use_classes) : (int8_t)-1;
                }
            }
        }
        cur = nxt;
    }
}

// Alg. 5, in-degree cut, first half: thr[v] <- the R-th smallest (delta, source) among the edges into v.
__global__ __launch_bounds__(BLOCK) void k_incap_threshold(int R, const int *list, const u32 *n_list,
                                                           const int *cnt, const int *binoff,
                                                           const u64 *bins, u64 *thr)
{
    __shared__ u64 s_stage[WAVES_PER_BLOCK][RNND_MAX_R];
    __shared__ u64 s_row[WAVES_PER_BLOCK][RNND_MAX_R];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const u32 gw = blockIdx.x * WAVES_PER_BLOCK + wave, nw = gridDim.x * WAVES_PER_BLOCK;
    const u32 n = *n_list;
    for (u32 it = gw; it < n; it += nw) {
        const int v = list[it];
        bool any_new;
        wave_sync();
        const int nd = wave_merge_row(s_row[wave], 0, bins + binoff[v], cnt[v], bins, 0, R, s_stage[wave],
                                      lane, &any_new);
        wave_sync();
        if (lane == 0) thr[v] = s_row[wave][nd - 1];
    }
}

// Alg. 5, in-degree cut, second half: edge (u, v) survives iff (delta, u) <= thr[v]; vcls[u] follows the
// new degree.  Only the flagged lists (those with an edge to a candidate) can lose an edge; they come as a list.
// Nothing to do when no vertex has more than R incoming edges (*n_hubs == 0).
__global__ __launch_bounds__(BLOCK) void k_incap_filter(int R, u64 *keys, int *deg, const u64 *thr,
                                                        const int *flagged, const u32 *n_flagged, int8_t *vcls,
                                                        int use_classes, const u32 *n_hubs)
{
    if (*n_hubs == 0u) return;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const u32 n = *n_flagged, nw = gridDim.x * WAVES_PER_BLOCK;
    for (u32 it = blockIdx.x * WAVES_PER_BLOCK + wave; it < n; it += nw) {
        const int u = flagged[it];
        const int m = deg[u];
        u64 *row = keys + (size_t)u * R;
        u64 k[2];
        bool keep[2];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            int e = r * 64 + lane;
            k[r] = e < m ? row[e] : KEY_PAD;
            keep[r] = e < m && make_key(key_dist(k[r]), (u32)u, 0u) <= thr[key_id(k[r])];
        }
        const u64 m0 = __builtin_amdgcn_ballot_w64(keep[0]), m1 = __builtin_amdgcn_ballot_w64(keep[1]);
        const u64 n0 = __builtin_amdgcn_ballot_w64(keep[0] && (k[0] & 1ull));
        const u64 n1 = __builtin_amdgcn_ballot_w64(keep[1] && (k[1] & 1ull));
        const int c0 = __popcll(m0);
        if (keep[0]) row[__popcll(m0 & lanes_below(lane))] = k[0];
        if (keep[1]) row[c0 + __popcll(m1 & lanes_below(lane))] = k[1];
        if (lane == 0) {
            const int nd = c0 + __popcll(m1);
            deg[u] = nd;
            vcls[u] = (n0 | n1) ? (int8_t)degree_class(nd, use_classes) : (int8_t)-1;
        }
    }
}

__global__ void k_zero_u32(u32 *p, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0;
}

// vcls[u] for a snapshot handed in by the caller
__global__ __launch_bounds__(BLOCK) void k_classify(long long N, int R, const u64 *keys, const int *deg,
                                                    int8_t *vcls, int use_classes)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const long long u = (long long)blockIdx.x * WAVES_PER_BLOCK + wave;
    if (u >= N) return;
    int m = deg[u];
    if (m > R) m = R;
    bool nw = false;
    for (int e = lane; e < m; e += 64) nw = nw || (keys[(size_t)u * R + e] & 1ull);
    const u64 b = __builtin_amdgcn_ballot_w64(nw);
    if (lane == 0) vcls[u] = b ? (int8_t)degree_class(m, use_classes) : (int8_t)-1;
}

__global__ void k_export(long long N, int R, const u64 *keys, const int *deg, int *graph_out,
                         int *degree_out)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N * R) return;
    long long u = i / R;
    int e = (int)(i - u * R);
    int m = deg[u];
    graph_out[i] = e < m ? (int)key_id(keys[i]) : -1;
    if (e == 0) degree_out[u] = m;
}

// The same, four slots per thread (R a multiple of 4, graph_out 16-byte aligned).
__global__ __launch_bounds__(256) void k_export4(long long N, int R4, const u64 *keys, const int *deg, int4 *graph_out,
                                                 int *degree_out)
{
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;      // group of four slots
    if (i >= N * R4) return;
    const long long u = i / R4;
    const int e = 4 * (int)(i - u * R4);
    const int m = deg[u];
    int4 o = make_int4(-1, -1, -1, -1);
    if (e < m) {
        const ulonglong2 a = ((const ulonglong2 *)keys)[2 * i], b = ((const ulonglong2 *)keys)[2 * i + 1];
        o.x = (int)key_id(a.x);
        if (e + 1 < m) o.y = (int)key_id(a.y);
        if (e + 2 < m) o.z = (int)key_id(b.x);
        if (e + 3 < m) o.w = (int)key_id(b.y);
    }
    graph_out[i] = o;
    if (e == 0) degree_out[u] = m;
}

static void launch_export(long long N, int R, const u64 *keys, const int *deg, int *graph_out, int *degree_out,
                          hipStream_t st)
{
    if (R % 4 == 0 && ((uintptr_t)graph_out & 15) == 0 && ((uintptr_t)keys & 15) == 0)
        hipLaunchKernelGGL(k_export4, dim3((unsigned)(((size_t)N * (R / 4) + 255) / 256)), dim3(256), 0, st, N, R / 4, keys,
                           deg, (int4 *)graph_out, degree_out);
    else
        hipLaunchKernelGGL(k_export, dim3((unsigned)(((size_t)N * R + 255) / 256)), dim3(256), 0, st, N, R, keys, deg,
                           graph_out, degree_out);
}

// Measurement aid: random row gathers and nothing else.  Every wavefront draws row numbers from the
// counter generator and reads whole rows, LPR lanes per row with 16 bytes per lane and piece, four
// rows' worth of loads per lane in flight; the values are folded into one word per thread so that
// the loads cannot be dropped.  This is the access pattern of the scan kernels without their work.
template <int LPR>
__global__ __launch_bounds__(256) void k_probe_gather(const uint4 *X, u32 n_rows, u32 pieces, u64 trips, u64 seed, u32 *sink)
{
    constexpr int RPI = 64 / LPR;       // rows per load instruction
    const int lane = threadIdx.x & 63, r = lane / LPR, q = lane % LPR;
    const u64 gw = ((u64)blockIdx.x * 256 + threadIdx.x) >> 6, nw = ((u64)gridDim.x * 256) >> 6;
    u32 acc = 0;
    for (u64 t = gw; t < trips; t += nw) {
        const uint4 *p[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const u64 z = splitmix_finish(seed + 0x9E3779B97F4A7C15ull * (t * (4 * RPI) + (u64)(k * RPI + r) + 1));
            const u32 row = (u32)(((z >> 32) * (u64)n_rows) >> 32);
            p[k] = X + (size_t)row * pieces + q;
        }
        for (u32 c = 0; c < pieces; c += LPR) {
            uint4 v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = p[k][c];
#pragma unroll
            for (int k = 0; k < 4; ++k) acc ^= v[k].x + v[k].y + v[k].z + v[k].w;
        }
    }
    sink[(size_t)blockIdx.x * 256 + threadIdx.x] = acc;
}

// The same with the lane -> address map as the only variable: LPR lanes per row, each reading its PPL pieces
// of the row (16 bytes, LPR pieces apart), 8 / PPL rows per lane: 8 loads of 16 bytes per lane in flight
// whatever the map, all issued before the first is used.
template <int LPR, int PPL>
__global__ __launch_bounds__(256) void k_probe_gather_map(const uint4 *X, u32 n_rows, u64 trips, u64 seed, u32 *sink)
{
    constexpr int RPI = 64 / LPR, ROWS = 8 / PPL;
    const int lane = threadIdx.x & 63, r = lane / LPR, q = lane % LPR;
    const u64 gw = ((u64)blockIdx.x * 256 + threadIdx.x) >> 6, nw = ((u64)gridDim.x * 256) >> 6;
    u32 acc = 0;
    for (u64 t = gw; t < trips; t += nw) {
        uint4 v[ROWS][PPL];
#pragma unroll
        for (int k = 0; k < ROWS; ++k) {
            const u64 z = splitmix_finish(seed + 0x9E3779B97F4A7C15ull * (t * (ROWS * RPI) + (u64)(k * RPI + r) + 1));
            const u32 row = (u32)(((z >> 32) * (u64)n_rows) >> 32);
            const uint4 *p = X + (size_t)row * (LPR * PPL) + q;
#pragma unroll
            for (int j = 0; j < PPL; ++j) v[k][j] = p[j * LPR];
        }
#pragma unroll
        for (int k = 0; k < ROWS; ++k)
#pragma unroll
            for (int j = 0; j < PPL; ++j) acc ^= v[k][j].x + v[k][j].y + v[k][j].z + v[k][j].w;
    }
    sink[(size_t)blockIdx.x * 256 + threadIdx.x] = acc;
}

// ===================================================================== host side
#define HIPCHK(x)                                                                  \
    do {                                                                           \
        hipError_t e_ = (x);                                                       \
        if (e_ != hipSuccess) {                                                    \
            snprintf(g_last_hip_error, sizeof g_last_hip_error, "%s: %s", #x, hipGetErrorString(e_)); \
            rc = (e_ == hipErrorOutOfMemory) ? RNND_ERR_OOM : RNND_ERR_HIP;        \
            (void)hipGetLastError();   /* reported here: must not surface again in a later call */ \
            goto done;                                                             \
        }                                                                          \
    } while (0)

static char g_last_hip_error[512];
static int g_kernel_variant = 0;
static int g_event_timing = 0;    // 1: per-round times of the statistics from HIP events attached to the launches
static int g_transpose_path = 0;   // AddReverseEdges' transposition: 0 by size, 1 atomics, 2 binned
static int g_scan_launches = 0;    // uint8 matrix-core scan: 0 by size, 1 short lists + one launch per longer class, 2 one launch for all, 3 short lists + one launch for all longer classes
#define SMALL_INPUT_MAX_N 524288   // up to here one launch for all classes is the fastest form (measured, whole build against
                                   // launches per class: 0.75 x at 50,000 vertices, 0.78 x at 100,000, 0.90 x at 300,000, 0.955 x
                                   // at 500,000; 1.02 x at 1M, where it wins only in rounds with fewer than 250,000 active lists).
                                   // Above: the short-list launch and one launch for all longer classes (0.99 x at 1M)
#define LONG_SHARED_MAX_N 2097152  // ... up to here (1.00 x at 2M, 1.01 x at 4M, 1.00 x at 8M, 1.01 x at 20M: no start-up left to
                                   // share, and each class alone gets the occupancy that suits it); above: a launch per class
                                   // (bench.py names the round's scan launches by the same rule; include/rnnd.h states it)
#define BIN_MIN_N 262144            // below this the binned transposition's extra launches cost more than its atomics save

static size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

struct Workspace {
    char *base = nullptr;
    size_t bytes = 0;
    u64 *keys = nullptr;    // [N*R]   (unless the caller supplies a snapshot)
    int *deg = nullptr;     // [N]
    Prop *props = nullptr;  // [N*R]   slot u*R.. holds the edges vertex u redirected this round
    u64 *inbox = nullptr;   // [N*INBOX_CAP] redirected edges received this round, by target
    u64 *bins = nullptr;    // [N*R]   a round's heads of late edges; AddReverseEdges' bins
    u64 *thr = nullptr;     // [N]
    int *cnt = nullptr, *binoff = nullptr, *fill = nullptr, *touched = nullptr, *hubs = nullptr, *nprop = nullptr;
    // (touched: [NMRG*N]; until the scatter, the vertices that a float scan leaves)
    char *half = nullptr;     // half-precision copy of float32 rows
    int8_t *xs = nullptr;     // copy of X (see ScanPlan): X - 128 as int8 for the uint8 MFMA scan, or padded rows
    int *lists = nullptr;   // [NDEG*N] active lists by degree class
    int8_t *vcls = nullptr, *tcls = nullptr;   // [N], [NMRG*N]
    RoundCtr *ctr = nullptr;   // [n_ctr]
    u32 *misc = nullptr;       // [16]: small cursors for AddReverseEdges
    u32 *blockhist = nullptr;  // binned transposition: [blocks of BIN_CHUNK vertices][ranges], null when N is out of its range
    u32 *range_tot = nullptr, *range_base = nullptr;   // [RANGE_MAX + 1] each
    int n_ctr = 0;
    // cnt[], fill[] and ctr[] must read zero when a call starts; they lie next to each other so that one
    // fill kernel clears them (ws_clear)
    u32 *zero_begin = nullptr;
    size_t zero_words = 0;
};

static size_t bin_blocks(long long N) { return (size_t)((N + BIN_CHUNK - 1) / BIN_CHUNK); }
static size_t bin_ranges(long long N) { return (size_t)((N + RANGE_TARGETS - 1) >> RANGE_BITS); }

static size_t ws_layout(Workspace &w, long long N, int R, int n_ctr, bool own_graph, size_t xs_bytes)
{
    size_t off = 0;
    auto take = [&](size_t b) { size_t o = off; off += align_up(b); return o; };
    size_t o_keys = own_graph ? take((size_t)N * R * 8) : 0;
    size_t o_deg = own_graph ? take((size_t)N * 4) : 0;
    size_t o_inbox = take((size_t)N * INBOX_CAP * 8);
    size_t o_props = take((size_t)N * R * sizeof(Prop));
    size_t o_bins = take((size_t)N * R * 8);
    size_t o_thr = take((size_t)N * 8);
    size_t o_binoff = take((size_t)N * 4);
    size_t o_touched = take((size_t)N * 4 * NMRG), o_hubs = take((size_t)N * 4), o_nprop = take((size_t)N * 4);
    size_t o_xs = take(xs_bytes);
    size_t o_lists = take((size_t)N * 4 * NDEG);
    size_t o_vcls = take((size_t)N), o_tcls = take((size_t)N * NMRG);
    size_t o_misc = take(16 * 4);
    const bool binnable = N >= 2 && (unsigned long long)N <= (unsigned long long)RANGE_MAX * RANGE_TARGETS;
    size_t o_range = take(binnable ? (size_t)2 * (RANGE_MAX + 1) * 4 : 0);
    size_t o_blockhist = take(binnable ? bin_blocks(N) * bin_ranges(N) * 4 : 0);
    size_t o_cnt = take((size_t)N * 4), o_fill = take((size_t)N * 4);      // the zeroed span: cnt, fill, ctr
    size_t o_ctr = take((size_t)n_ctr * sizeof(RoundCtr));
    if (w.base) {
        if (own_graph) { w.keys = (u64 *)(w.base + o_keys); w.deg = (int *)(w.base + o_deg); }
        w.inbox = (u64 *)(w.base + o_inbox);
        w.props = (Prop *)(w.base + o_props);
        w.nprop = (int *)(w.base + o_nprop);
        w.bins = (u64 *)(w.base + o_bins);
        w.thr = (u64 *)(w.base + o_thr);
        w.cnt = (int *)(w.base + o_cnt);
        w.binoff = (int *)(w.base + o_binoff);
        w.fill = (int *)(w.base + o_fill);
        w.touched = (int *)(w.base + o_touched);
        w.hubs = (int *)(w.base + o_hubs);
        w.xs = (int8_t *)(w.base + o_xs);
        w.lists = (int *)(w.base + o_lists);
        w.vcls = (int8_t *)(w.base + o_vcls);
        w.tcls = (int8_t *)(w.base + o_tcls);
        w.ctr = (RoundCtr *)(w.base + o_ctr);
        w.misc = (u32 *)(w.base + o_misc);
        w.blockhist = binnable ? (u32 *)(w.base + o_blockhist) : nullptr;
        w.range_tot = (u32 *)(w.base + o_range);
        w.range_base = w.range_tot + (RANGE_MAX + 1);
        w.n_ctr = n_ctr;
        w.zero_begin = (u32 *)(w.base + o_cnt);
        w.zero_words = (off - o_cnt) / 4;
    }
    return off;
}

// Every entry point clears the counters of its workspace with this before its first kernel: a fill kernel,
// not a memset node, so that the same sequence stays valid inside a captured graph.
static void ws_clear(const Workspace &w, hipStream_t st)
{
    const size_t n = w.zero_words;
    const unsigned blocks = (unsigned)((n + 1023) / 1024 < 2048 ? (n + 1023) / 1024 : 2048);
    hipLaunchKernelGGL(k_zero_u32, dim3(blocks ? blocks : 1), dim3(256), 0, st, w.zero_begin, n);
}

static int check_data_args(const void *X, long long N, int d, int dtype, int metric, int R)
{
    if (!X) return RNND_ERR_NULL;
    if (dtype != RNND_U8 && dtype != RNND_F32 && dtype != RNND_F16 && dtype != RNND_BF16) return RNND_ERR_UNSUPPORTED;
    if (metric != RNND_L2SQ) return RNND_ERR_UNSUPPORTED;
    if (N < 2 || N > 2147483646LL || d < 1) return RNND_ERR_BAD_SHAPE;
    if (dtype == RNND_U8 && d > 33025) return RNND_ERR_BAD_SHAPE;
    if (R < 1 || R > RNND_MAX_R) return RNND_ERR_BAD_PARAM;
    // list slots are counted in 32-bit device counters, and a bin offset is an int with -1 for "no bin"
    if ((unsigned long long)N * (unsigned long long)R > RNND_MAX_SLOTS) return RNND_ERR_BAD_SHAPE;
    return RNND_OK;
}

static int vec_ok_for(const void *X, int d, int dtype)
{
    size_t rowbytes = (size_t)d * dt_size(dtype);
    return (rowbytes % 16 == 0) && (((uintptr_t)X) % 16 == 0);
}

// How UpdateNeighbors scans for this input.
//   variant   1 = generic kernel, 2 = int8 MFMA Gram kernel (uint8 rows), 3 = matrix-core Gram kernel for float or 16-bit
//             rows (fp32 / f16 / bf16 MFMA first, f64 MFMA for what it leaves)
//   copy      what the workspace's copy of X holds: nothing (the scan reads X), the bytes minus 128 of uint8 rows that
//             fit the tiles, or rows padded to a length the tiles take (dp coordinates; see k_prepare_*_rows)
// The first two are what a call needs; padded rows are an extra a call does without (generic kernel) where there is
// no room for them.
// Row length in bytes of the half-precision copy of d coordinates: a multiple of 128, so that no row shares a cache line; 64 and 192
// where a half or a third of 128 or 256 would be padding.
static u32 half_row_bytes(int d) { return d <= 32 ? 64u : d <= 64 ? 128u : d <= 128 ? ((u32)d + 31u) / 32u * 64u : ((u32)d + 63u) / 64u * 128u; }
// From how many vertices on a build's float32 scans take their Gram blocks from that copy: always but for the smallest inputs,
// whose lists the two launches that make it would hold up (60-round builds without / with it, R = 96: 300 x 96 1.64 / 1.21 ms, 2,000 x 33
// 1.60 / 1.55, 20,000 x 96 3.87 / 3.15, 1M x 960 915 / 526).
#define HALF_MIN_N 256
enum CopyKind { COPY_NONE = 0, COPY_U8, COPY_U8_ROWS, COPY_ROWS, COPY_ROWS_PERMUTED };
struct ScanPlan {
    int variant = 1, dp = 0;
    CopyKind copy = COPY_NONE;
    size_t copy_bytes = 0;
    u32 half_rb = 0;            // row length of the half-precision copy of float32 rows (see HalfRows), 0 = none
    size_t half_bytes = 0;      // what it takes: rows, centre, sums, parameters
    bool tiles16 = false;       // variant 3: 16-bit rows go to the 16-bit matrix instructions as they are
    // which degree classes the scan works by (see degree_class)
    int classes() const { return variant == 2 ? 2 : variant == 3 ? (tiles16 || half_rb ? 2 : 1) : 0; }
    bool extra() const { return copy > COPY_U8 || half_rb; }
};

// From how many vertices on padded rows are worth their copy, measured on whole builds (generic kernel against padded
// rows, S = 20, R = 96, 60 rounds):
//   uint8   always: d = 8: 1.8 -> 1.6 ms at 300 vertices, 4.8 -> 2.2 ms at 20,000; d = 100: 3.5 -> 1.6 and 15.7 -> 2.7 ms
//   float   d = 33: 2.2 -> 1.9 ms at 300 vertices, d = 100: 3.0 -> 1.9; d = 7: 1.8 -> 1.9 ms at 300, 2.4 -> 2.0 at 2,048
#define PAD_MIN_N_FLOAT 256
#define PAD_MIN_N_SHORT_FLOAT 2048      // rows of fewer than 16 coordinates
// UpdateNeighbors by itself: a call on fewer vertices scans X as it is, with no copy made for it.  A copy pays where there is
// work (2,000 x 100 float32, generic / padded: 170 / 111 us with 1,976 vertices active; 500 x 100: 152 / 107 with 493) and costs a launch
// or two where there is none (75 / 90 us), which small snapshots reach soonest.
#define PAD_MIN_N_STEP 2048
#define PAD_MAX_D 65536         // (row lengths in bytes stay far below 2^31)

static bool worth_padding(long long N, int d, int dtype, bool step)
{
    if (d > PAD_MAX_D || (step && N < PAD_MIN_N_STEP)) return false;
    return dtype == RNND_U8 || N >= (d < 16 ? PAD_MIN_N_SHORT_FLOAT : PAD_MIN_N_FLOAT);
}

static size_t half_layout(char *base, long long N, int d, u32 rb, struct HalfLayout *l);
static ScanPlan scan_plan_for(const void *X, long long N, int d, int dtype, bool may_pad, bool may_half = false)
{
    ScanPlan p;
    p.dp = d;
    if (g_kernel_variant == 1) return p;
    const bool aligned = (((uintptr_t)X) % 16 == 0);
    if (aligned && dtype == RNND_U8 && (d == 32 || d == 64 || d == 128)) {
        p.variant = 2;
        p.copy = COPY_U8;
        p.copy_bytes = (size_t)N * d;
    } else if (aligned && ((dtype == RNND_F32 && d % 16 == 0) || ((dtype == RNND_F16 || dtype == RNND_BF16) && d % 32 == 0))) {
        p.variant = 3;      // rows of a multiple of 64 bytes, as they are
    } else if (may_pad) {
        if (dtype == RNND_U8) {
            p.variant = 2;
            p.copy = COPY_U8_ROWS;
            p.dp = d <= 32 ? 32 : d <= 64 ? 64 : d <= 128 ? 128 : (d + 63) / 64 * 64;
            p.copy_bytes = (size_t)N * p.dp;
        } else {
            const int per = 128 / dt_size(dtype);
            p.variant = 3;
            p.copy = vec_ok_for(X, d, dtype) ? COPY_ROWS : COPY_ROWS_PERMUTED;
            p.dp = (int)(((long long)d + per - 1) / per * per);
            p.copy_bytes = (size_t)N * p.dp * dt_size(dtype);
        }
    }
    p.tiles16 = p.variant == 3 && dtype != RNND_F32 && g_kernel_variant == 0;
    if (may_half && N >= HALF_MIN_N && p.variant == 3 && dtype == RNND_F32 && g_kernel_variant == 0) {
        p.half_rb = half_row_bytes(d);
        p.half_bytes = half_layout(nullptr, N, d, p.half_rb, nullptr);
    }
    return p;
}

static inline int vertex_blocks(long long N) { return (int)((N + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK); }

// Events tied to kernels of one round (null: not wanted).  They are attached to the launches
// themselves, which costs no extra packet on the stream.
struct RoundEvents {
    hipEvent_t scan_start = nullptr;   // start of the first scan kernel
    hipEvent_t scan_stop = nullptr;    // end of the last scan kernel
    hipEvent_t round_stop = nullptr;   // end of the round's last kernel
};

static EdgeSink edge_sink(const Workspace &w, int R) { return EdgeSink{w.fill, w.inbox, late_heads(w.inbox, w.bins, R), w.props, w.nprop}; }

template <int NG, int KS, typename OUT>
static void launch_mfma_scan(const Workspace &w, int d, int R, u64 *keys, int *deg, long long N, RoundCtr *c,
                             hipStream_t st, hipEvent_t e_stop, const EdgeSink &sink)
{
    static const int per_cu = resident_blocks_per_cu(k_update_scan_mfma_u8<NG, KS, OUT>, NG == 2 ? 3 : 2);
    hipExtLaunchKernelGGL((k_update_scan_mfma_u8<NG, KS, OUT>), dim3(capped(cu_count() * per_cu, N)), dim3(256), 0, st, nullptr,
                          e_stop, 0, (const int8_t *)w.xs, d, R, keys, deg, w.lists + (size_t)(NG + 1) * N,
                          &c->n_active[NG + 1], sink, c);
}

// Fills w.xs, the copy of X the plan asks for.
// `round` (one round on this snapshot, its active lists made): padded float rows may be copied for its lists only.
struct SnapshotRound {
    const u64 *keys;
    const int *deg;
    int R;
};
static void launch_prepare(const Workspace &w, const ScanPlan &p, const void *X, long long N, int d, int dtype, const SnapshotRound *round,
                           hipStream_t st)
{
    const u32 exponent = dtype == RNND_F32 ? 0x7F800000u : dtype == RNND_F16 ? 0x7C00u : 0x7F80u;
    if (p.copy == COPY_NONE) return;
    if (p.copy == COPY_U8) {
        const size_t n = (size_t)N * d;
        hipLaunchKernelGGL(k_prepare_u8, dim3((unsigned)((n / 16 + 255) / 256)), dim3(256), 0, st, (const uint8_t *)X, n, w.xs);
        return;
    }
    const size_t threads = p.copy == COPY_U8_ROWS ? p.copy_bytes / 4 : p.copy_bytes / 16;
    const size_t need = (threads + 255) / 256, most = (size_t)cu_count() * 32;
    const dim3 grid((unsigned)(need < most ? need : most));
    const u32 rb = (u32)((size_t)p.dp * dt_size(dtype));
    const int permute = p.copy == COPY_ROWS_PERMUTED;
    if (p.copy == COPY_U8_ROWS)
        hipLaunchKernelGGL(k_prepare_u8_rows, grid, dim3(256), 0, st, (const uint8_t *)X, N, d, p.dp, w.xs);
    else if (round && dtype == RNND_F32)
        hipLaunchKernelGGL(k_prepare_listed_rows<u32>, grid, dim3(256), 0, st, (const u32 *)X, N, d, rb, permute, (uint4 *)w.xs,
                           (const int *)w.lists, (const RoundCtr *)w.ctr, round->keys, round->deg, round->R);
    else if (round)
        hipLaunchKernelGGL(k_prepare_listed_rows<unsigned short>, grid, dim3(256), 0, st, (const unsigned short *)X, N, d, rb, permute,
                           (uint4 *)w.xs, (const int *)w.lists, (const RoundCtr *)w.ctr, round->keys, round->deg, round->R);
    else if (dtype == RNND_F32)
        hipLaunchKernelGGL(k_prepare_rows<u32>, grid, dim3(256), 0, st, (const u32 *)X, N, d, rb, permute, exponent,
                           (uint4 *)w.xs, &w.ctr->nonfinite);
    else
        hipLaunchKernelGGL(k_prepare_rows<unsigned short>, grid, dim3(256), 0, st, (const unsigned short *)X, N, d, rb, permute,
                           exponent, (uint4 *)w.xs, &w.ctr->nonfinite);
}

// The rows every kernel but the uint8 matrix-core scan reads: X, or the padded copy of float or 16-bit rows; and the
// half-precision copy of float32 rows, if there is one.
struct RowsView {
    const void *X = nullptr;
    int d = 0, vec_ok = 0;
    HalfRows half;
    bool own_lists = false;     // the lists hold distances that this library has formed on these rows, and no others
};

// Where the parts of a half-precision copy lie.
struct HalfLayout {
    char *rows;
    float *centre, *square;
    HalfPar *par;
};
static size_t half_layout(char *base, long long N, int d, u32 rb, HalfLayout *l)
{
    size_t off = 0;
    auto take = [&](size_t b) { size_t o = off; off += align_up(b); return o; };
    const size_t o_rows = take((size_t)N * rb), o_centre = take((size_t)d * 4 + 32), o_square = take(((size_t)d + 63) / 64 * 4), o_par = take(sizeof(HalfPar));
    if (l) *l = HalfLayout{base + o_rows, (float *)(base + o_centre), (float *)(base + o_square), (HalfPar *)(base + o_par)};
    return off;
}

static void launch_half_rows(char *base, const void *X, long long N, int d, int vec_ok, u32 rb, hipStream_t st, HalfRows *out)
{
    HalfLayout l;
    half_layout(base, N, d, rb, &l);
    hipLaunchKernelGGL(k_half_centre, dim3((unsigned)((d + 63) / 64)), dim3(1024), 0, st, (const float *)X, N, d, l.centre, l.square, l.par);
    const int lanes = rb <= 512 ? 16 : 64;
    const size_t need = ((size_t)N * lanes + 255) / 256, most = (size_t)persistent_blocks();
    const dim3 grid((unsigned)(need < most ? need : most));
    if (lanes == 16)
        hipLaunchKernelGGL(k_half_rows<16>, grid, dim3(256), 0, st, (const float *)X, N, d, vec_ok, rb, (const float *)l.centre,
                           (const float *)l.square, l.rows, l.par);
    else
        hipLaunchKernelGGL(k_half_rows<64>, grid, dim3(256), 0, st, (const float *)X, N, d, vec_ok, rb, (const float *)l.centre,
                           (const float *)l.square, l.rows, l.par);
    out->rows = l.rows;
    out->rowbytes = rb;
    out->par = l.par;
}

// Makes the copy the plan asks for and says what the kernels are to read.  The matrix-core scan leaves every pair of rows
// that are not finite to the exact routine, so it gives the generic kernel's graph for them too, slowly where there are many.
// A build asks: where padded float rows hold a NaN or an infinity the plan falls back to the generic kernel on X.  That
// answer is waited for, about 20 us; UpdateNeighbors by itself (step), where a round may take no longer than that, does without it
// (20,000 x 40 float32, a call with two active vertices: 97 -> 86 us, 77 with no copy and the generic kernel; 1,625 active:
// 105 -> 92, 102).
static hipError_t prepare_rows(const Workspace &w, ScanPlan &p, const void *X, long long N, int d, int dtype, hipStream_t st, bool step,
                               const SnapshotRound *round, RowsView *rv)
{
    rv->X = X;
    rv->d = d;
    rv->vec_ok = vec_ok_for(X, d, dtype);
    rv->own_lists = !step;
    if (p.half_rb) launch_half_rows(w.half, X, N, d, rv->vec_ok, p.half_rb, st, &rv->half);
    launch_prepare(w, p, X, N, d, dtype, round, st);
    if (p.copy != COPY_ROWS && p.copy != COPY_ROWS_PERMUTED) return hipGetLastError();
    u32 nonfinite = 0;
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && !step) e = hipMemcpyAsync(&nonfinite, &w.ctr->nonfinite, sizeof nonfinite, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess && !step) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return e;
    if (nonfinite) {
        p = ScanPlan();
        p.dp = d;
        rv->half = HalfRows();
    } else {
        rv->X = w.xs;
        rv->d = p.dp;
        rv->vec_ok = 1;
    }
    return hipSuccess;
}

template <int KS, typename OUT>
static void launch_mfma_scan_classes(const Workspace &w, int d, int R, u64 *keys, int *deg, long long N, RoundCtr *c,
                                     hipStream_t st, const RoundEvents &re, const EdgeSink &sink)
{
    static const int per_cu = resident_blocks_per_cu(k_update_scan_mfma_u8_small<KS, OUT>, 4);
    const int n_big = (R > 32) + (R > 64) + (R > 96);   // launches after the short-list kernel
    // small inputs: every class in one launch (see k_update_scan_mfma_u8_all)
    if (n_big > 0 && (g_scan_launches == 2 || (g_scan_launches == 0 && N <= SMALL_INPUT_MAX_N))) {
        unsigned gx = capped((long long)cu_count() * 2, N);
        if (gx < 8) gx = 8;      // a block at least for every class
        if (n_big == 1)
            hipExtLaunchKernelGGL((k_update_scan_mfma_u8_all<KS, OUT, 4>), dim3(gx), dim3(256), 0, st, re.scan_start, re.scan_stop, 0,
                                  (const int8_t *)w.xs, d, R, keys, deg, w.lists, N, sink, c);
        else if (n_big == 2)
            hipExtLaunchKernelGGL((k_update_scan_mfma_u8_all<KS, OUT, 5>), dim3(gx), dim3(256), 0, st, re.scan_start, re.scan_stop, 0,
                                  (const int8_t *)w.xs, d, R, keys, deg, w.lists, N, sink, c);
        else
            hipExtLaunchKernelGGL((k_update_scan_mfma_u8_all<KS, OUT, 6>), dim3(gx), dim3(256), 0, st, re.scan_start, re.scan_stop, 0,
                                  (const int8_t *)w.xs, d, R, keys, deg, w.lists, N, sink, c);
        return;
    }
    const int ny = 1 + (R > 8) + (R > 16);
    hipExtLaunchKernelGGL((k_update_scan_mfma_u8_small<KS, OUT>), dim3(capped(cu_count() * per_cu, N), ny), dim3(256), 0, st,
                          re.scan_start, n_big == 0 ? re.scan_stop : nullptr, 0, (const int8_t *)w.xs, d, R, keys, deg,
                          w.lists, N, sink, c);
    // large inputs: the short-list launch above, then the longer classes in one launch
    if (n_big >= 2 && (g_scan_launches == 3 || (g_scan_launches == 0 && N <= LONG_SHARED_MAX_N))) {
        unsigned gx = capped((long long)cu_count() * 2, N);
        if (gx < 8) gx = 8;      // a block at least for every class
        if (n_big == 2)
            hipExtLaunchKernelGGL((k_update_scan_mfma_u8_all<KS, OUT, 5, 3>), dim3(gx), dim3(256), 0, st, nullptr, re.scan_stop, 0,
                                  (const int8_t *)w.xs, d, R, keys, deg, w.lists, N, sink, c);
        else
            hipExtLaunchKernelGGL((k_update_scan_mfma_u8_all<KS, OUT, 6, 3>), dim3(gx), dim3(256), 0, st, nullptr, re.scan_stop, 0,
                                  (const int8_t *)w.xs, d, R, keys, deg, w.lists, N, sink, c);
        return;
    }
    if (R > 32) launch_mfma_scan<2, KS, OUT>(w, d, R, keys, deg, N, c, st, n_big == 1 ? re.scan_stop : nullptr, sink);
    if (R > 64) launch_mfma_scan<3, KS, OUT>(w, d, R, keys, deg, N, c, st, n_big == 2 ? re.scan_stop : nullptr, sink);
    if (R > 96) launch_mfma_scan<4, KS, OUT>(w, d, R, keys, deg, N, c, st, n_big == 3 ? re.scan_stop : nullptr, sink);
}

template <int DT>
static void launch_generic_scan_dt(const Workspace &w, const void *X, int d, int vec_ok, int R, u64 *keys, int *deg, long long N,
                                   const WorkList &work, const EdgeSink &sink, unsigned blocks, RoundCtr *c, hipStream_t st, hipEvent_t e_start, hipEvent_t e_stop)
{
    hipExtLaunchKernelGGL(k_update_scan<DT>, dim3(blocks), dim3(BLOCK), 0, st, e_start, e_stop, 0, X, d, vec_ok, R, keys, deg,
                          work, sink, c);
}

// The generic scan over one list.
static void launch_generic_scan(const Workspace &w, const void *X, int d, int dtype, int vec_ok, int R, u64 *keys, int *deg,
                                long long N, const WorkList &work, const EdgeSink &sink, unsigned blocks, RoundCtr *c, hipStream_t st, hipEvent_t e_start,
                                hipEvent_t e_stop)
{
    if (dtype == RNND_U8) launch_generic_scan_dt<DT_U8>(w, X, d, vec_ok, R, keys, deg, N, work, sink, blocks, c, st, e_start, e_stop);
    else if (dtype == RNND_F16) launch_generic_scan_dt<DT_F16>(w, X, d, vec_ok, R, keys, deg, N, work, sink, blocks, c, st, e_start, e_stop);
    else if (dtype == RNND_BF16) launch_generic_scan_dt<DT_BF16>(w, X, d, vec_ok, R, keys, deg, N, work, sink, blocks, c, st, e_start, e_stop);
    else launch_generic_scan_dt<DT_F32>(w, X, d, vec_ok, R, keys, deg, N, work, sink, blocks, c, st, e_start, e_stop);
}

// dt (here and below): the type of the rows that open distances are computed from, DT_U8 where none are open
template <int DT>
static void launch_classify_dt(hipStream_t st, long long N, int R, const Workspace &w, const int *deg, RoundCtr *c, const void *X, int d, bool scattered, u32 enough)
{
    const LateHeads heads = late_heads(w.inbox, w.bins, R);
    if (N <= SMALL_INPUT_MAX_N)
        hipLaunchKernelGGL((k_touch_classify<2, DT>), dim3((unsigned)((N + 2047) / 2048)), dim3(1024), 0, st, N, round_inbox(R), w.fill, deg, c,
                           w.touched, heads, w.props, (const char *)X, d, scattered ? 1 : 0, enough);
    else
        hipLaunchKernelGGL((k_touch_classify<4, DT>), dim3((unsigned)((N + 4095) / 4096)), dim3(1024), 0, st, N, round_inbox(R), w.fill, deg, c,
                           w.touched, heads, w.props, (const char *)X, d, scattered ? 1 : 0, enough);
}

template <int DT>
static void launch_merge_dt(hipStream_t st, long long N, int R, const Workspace &w, u64 *keys, int *deg, int use_classes, bool same_bits, RoundCtr *c, const void *X, int d)
{
    static const int per_cu = resident_blocks_per_cu(k_merge<DT>, 6);
    hipLaunchKernelGGL(k_merge<DT>, dim3(capped(cu_count() * per_cu, N), NMRG), dim3(BLOCK), 0, st, N, R, keys, deg, w.touched, c->n_touched,
                       w.fill, w.inbox, late_heads(w.inbox, w.bins, R), (const Prop *)w.props, w.tcls, use_classes, same_bits ? 1 : 0, c, (const char *)X, d);
}

static void launch_classify(int dt, hipStream_t st, long long N, int R, const Workspace &w, const int *deg, RoundCtr *c, const void *X, int d, bool scattered, u32 enough)
{
    const auto go = dt == RNND_F32 ? launch_classify_dt<DT_F32> : dt == RNND_F16 ? launch_classify_dt<DT_F16> : dt == RNND_BF16 ? launch_classify_dt<DT_BF16> : launch_classify_dt<DT_U8>;
    go(st, N, R, w, deg, c, X, d, scattered, enough);
}
// Up to here classify, merge and compact are one launch, of up to 128 vertices a block, fewer where that gives fewer than 512
// blocks.  Three launches / one, ms: 5,000 x 32 uint8 0.355 / 0.302, 20,000 x 96 float32 3.14 / 2.92, 60,000 x 784 uint8 5.12 / 4.86,
// 100,000 x 128 uint8 4.39 / 4.15, 200,000 x 100 float32 21.5 / 22.2, 300,000 x 768 bfloat16 103.0 / 103.6; 64 vertices a block
// 3.08 ms at 20,000, 4.51 at 100,000, 256 vertices 3.05 and 4.30.
#define MERGE_BLOCKS_MAX_N 131072
#define MERGE_SPAN 128
#define MERGE_BLOCKS_MIN 512
template <int DT>
static void launch_merge_blocks_dt(hipStream_t st, long long N, int R, const Workspace &w, u64 *keys, int *deg, int use_classes, RoundCtr *c, const void *X, int d,
                                   bool scattered, u32 enough)
{
    int span = MERGE_SPAN;
    while (span > 16 && N / span < MERGE_BLOCKS_MIN) span >>= 1;
    hipLaunchKernelGGL(k_merge_blocks<DT>, dim3((unsigned)((N + span - 1) / span)), dim3(BLOCK), 0, st, N, span, R, keys, deg, w.fill, w.inbox,
                       late_heads(w.inbox, w.bins, R), w.props, use_classes, c, w.lists, (c + 1)->n_active, (const char *)X, d, scattered ? 1 : 0, enough);
}
static void launch_merge_blocks(int dt, hipStream_t st, long long N, int R, const Workspace &w, u64 *keys, int *deg, int use_classes, RoundCtr *c, const void *X, int d,
                                bool scattered, u32 enough)
{
    const auto go = dt == RNND_F32 ? launch_merge_blocks_dt<DT_F32> : dt == RNND_F16 ? launch_merge_blocks_dt<DT_F16> : dt == RNND_BF16 ? launch_merge_blocks_dt<DT_BF16> : launch_merge_blocks_dt<DT_U8>;
    go(st, N, R, w, keys, deg, use_classes, c, X, d, scattered, enough);
}
static void launch_merge(int dt, hipStream_t st, long long N, int R, const Workspace &w, u64 *keys, int *deg, int use_classes, bool same_bits, RoundCtr *c, const void *X, int d)
{
    const auto go = dt == RNND_F32 ? launch_merge_dt<DT_F32> : dt == RNND_F16 ? launch_merge_dt<DT_F16> : dt == RNND_BF16 ? launch_merge_dt<DT_BF16> : launch_merge_dt<DT_U8>;
    go(st, N, R, w, keys, deg, use_classes, same_bits, c, X, d);
}

// One run of consecutive vertex ids of a block-sequential pass: ids first .. first + count - 1.
struct VertexRun {
    u32 first = 0, count = 0;
};

// A round of fewer active vertices than this, or than a sixteenth of all, does not decide which form the float scan of the next
// one takes (see decide_next_form): 32 sampled wavefronts.
#define DECIDE_MIN_ACTIVE 1024u

// Whether the scan by tiles (and what follows it) scatters the edges itself (see EdgeOut).  Scans that hold rows whole always do: 1M x 128
// uint8 25.6 -> 23.6 ms, 3M x 128 (16 rounds) 36.5 -> 32.2, 1M x 64 (16 rounds, R = 64) 11.2 -> 9.3.  Streamed rows of up to OWN_SCATTER_ROW_BYTES do as well, longer ones
// as long as rows and inboxes stay below OWN_SCATTER_MAX_BYTES: beyond, an arrival number takes longer to come than the next rows, which wait behind it.  k_scatter after
// scans that have no scatter in them / k_scatter / in the scan, ms (60 rounds, * 15): float32 1M x 96 102.6 / 106.4 / 100.6, x 256 190.1 / 190.9 / 186.0, x 512 300.5 / 295.6 / 292.1, x 960 523.1 / 514.0 / 519.3;
// 3M x 128 396 / 407 / 394; 6M x 32 548 / 583 / 538; 2M x 512 * 244.8 / 245.5 / 245.3; 300,000 x 960 134.0 / 130.9 / 128.7; bfloat16 1M x 256 149.3 / 148.4 / 144.4, x 512 275.6 / 272.8 / 270.9,
// x 768 408.8 / 404.2 / 408.2; uint8 1M x 784 52.3 / 52.5 / 50.6, 2M x 784 112.0 / 112.1 / 109.7, 2M x 1024 * 67.1 / 66.9 / 66.3, 2M x 1536 * 98.1 / 96.4 / 98.0, 4M x 256 113.5 / 117.4 / 111.9,
// 1.2M x 2048 * 71.1 / 71.2 / 71.7.  (The device's placement of a buffer moves such a figure by up to 2 %, at 2M rows.)
#define OWN_SCATTER_ROW_BYTES 1024
#define OWN_SCATTER_MAX_BYTES 1750000000ll
// Streamed uint8 rows in lists of up to 128 entries: that scan has the registers of one block per CU, and the scatter costs it more than k_scatter takes once the launch saved
// (4 of about 40 us a round) counts for less.  R = 128, left to k_scatter / in the scan, 16 rounds, 60 rounds, ms: 5,000 x 320 0.897 / 0.789, 2.25 / 1.97; 20,000 x 320 1.319 / 1.261, 3.21 / 2.97;
// 40,000 x 320 1.796 / 1.802, 4.06 / 3.90; 60,000 x 200 2.37 / 2.43, 5.13 / 5.10; 60,000 x 784 3.01 / 3.05, 6.12 / 6.04; 100,000 x 200 3.47 / 3.64, 7.13 / 7.31;
// 300,000 x 320 8.49 / 9.08, 16.1 / 17.0; 3M x 200 72.9 / 74.8, -.
#define OWN_SCATTER_WIDE_U8_MAX_N 49152
static bool scan_scatters(const ScanPlan &plan, const RowsView &rv, long long N, int dtype, int R)
{
    if (plan.variant == 2 && plan.dp > 128 && R > 96 && N > OWN_SCATTER_WIDE_U8_MAX_N) return false;
    const long long rowbytes = plan.variant == 2 ? plan.dp : rv.half.rows ? rv.half.rowbytes : (long long)rv.d * dt_size(dtype);
    return rowbytes <= OWN_SCATTER_ROW_BYTES || N * (rowbytes + 8 * INBOX_CAP) <= OWN_SCATTER_MAX_BYTES;
}

// One synchronous round over the active lists of counter slot t (run == nullptr), or one run of a
// block-sequential pass: the run's active lists are taken from vcls[] first, and the classes of the
// vertices its merge touched go back to vcls[] instead of into the next slot's lists.
static hipError_t launch_update_round(const Workspace &w, const RowsView &rv, long long N, const ScanPlan &plan, int dtype,
                                      int R, u64 *keys, int *deg, int t,
                                      hipStream_t st, const RoundEvents &re = RoundEvents(),
                                      const VertexRun *run = nullptr)
{
    const unsigned pb = capped(persistent_blocks(), N);
    const void *X = rv.X;
    const int variant = plan.variant, use_classes = plan.classes();
    const int d = variant == 2 ? plan.dp : rv.d, vec_ok = rv.vec_ok;
    RoundCtr *c = w.ctr + t;
    const int open_dt = variant == 3 && use_classes == 2 ? dtype : RNND_U8;      // whose redirected edges come without distances
    const long long vertices = run ? (long long)run->count : N;
    const u32 enough = vertices / 16 > DECIDE_MIN_ACTIVE ? (u32)(vertices / 16) : DECIDE_MIN_ACTIVE;
    const bool own_scatter = use_classes == 2 && scan_scatters(plan, rv, N, dtype, R);
    const EdgeSink all = edge_sink(w, R);
    EdgeSink sink = all;
    if (!own_scatter) sink.count = nullptr;
    if (run) {
        const unsigned cb = (run->count + 1023u) / 1024u;
        hipLaunchKernelGGL(k_compact_classes, dim3(cb < 256u ? cb : 256u, 1), dim3(1024), 0, st, (const u32 *)nullptr,
                           run->count, (const int *)nullptr, (const int8_t *)w.vcls, w.lists, N, c->n_active,
                           run->first, w.vcls);
    }
    if (variant == 2) {
        if (d == 32) launch_mfma_scan_classes<1, EdgeOut>(w, d, R, keys, deg, N, c, st, re, sink);
        else if (d == 64) launch_mfma_scan_classes<2, EdgeOut>(w, d, R, keys, deg, N, c, st, re, sink);
        else if (d == 128) launch_mfma_scan_classes<4, EdgeOut>(w, d, R, keys, deg, N, c, st, re, sink);
        else if (own_scatter) launch_mfma_scan_classes<0, EdgeOut>(w, d, R, keys, deg, N, c, st, re, sink);
        else launch_mfma_scan_classes<0, EdgesLeft>(w, d, R, keys, deg, N, c, st, re, sink);
    } else if (variant == 3) {
        const bool generic_tail = R > 96;
        ScanLaunch l = {X, d, R, keys, deg, N, w.lists, sink, c, w.touched, st, re.scan_start,
                        generic_tail ? (hipEvent_t) nullptr : re.scan_stop, t, vertices, enough};
        if (use_classes == 2) {
            // lists of up to 128 entries; the generic kernel takes what the scan leaves of the longest, all of them where it takes groups
            const bool copy = rv.half.rows != nullptr;
            launch_float_scan(l, dtype, copy ? rv.half.rows : X, copy ? rv.half.rowbytes : (u32)(d * dt_size(dtype)), rv.half.par);
            if (generic_tail)
                launch_generic_scan(w, X, d, dtype, vec_ok, R, keys, deg, N, WorkList{l.redo, &c->n_redo, w.lists + (size_t)5 * N, &c->n_active[5], &c->groups}, sink, pb, c, st,
                                    nullptr, re.scan_stop);
        } else {
            // degree classes 0..6: lists of at most 8, 16, 32, 48, 64, 80, 96 entries = 1, 1, 2, 3, 4, 5, 6 groups of 16
            // rows; class 7 (97..128 entries: too many accumulator tiles) goes to the generic kernel
            if (g_kernel_variant != 2) {
                launch_f32_scan(l);
                launch_f64_redo(l, dtype);
            } else {
                launch_f64_classes(l, dtype);
            }
            if (generic_tail) launch_generic_scan(w, X, d, dtype, vec_ok, R, keys, deg, N, WorkList{w.lists + (size_t)7 * N, &c->n_active[7]}, sink, pb, c, st, nullptr, re.scan_stop);
        }
    } else {
        launch_generic_scan(w, X, d, dtype, vec_ok, R, keys, deg, N, WorkList{w.lists, &c->n_active[0]}, sink, pb, c, st, re.scan_start, re.scan_stop);
    }
    // from here on `fill` plays the role of the per-target count of this round
    const int ncl = use_classes ? NDEG : 1;
    const u32 decide = open_dt != RNND_U8 ? enough : 0u;
    if (!own_scatter)
        hipLaunchKernelGGL(k_scatter, dim3(pb), dim3(BLOCK), 0, st, N, (const int *)w.lists, ncl, c, all, R, decide);
    if (!run && !re.round_stop && N <= MERGE_BLOCKS_MAX_N) {
        launch_merge_blocks(open_dt, st, N, R, w, keys, deg, use_classes, c, X, d, own_scatter, decide);
        return hipGetLastError();
    }
    launch_classify(open_dt, st, N, R, w, deg, c, X, d, own_scatter, decide);
    launch_merge(open_dt, st, N, R, w, keys, deg, use_classes, rv.own_lists, c, X, d);
    if (run)
        hipLaunchKernelGGL(k_store_classes, dim3(64, NMRG), dim3(256), 0, st, (const u32 *)c->n_touched,
                           (const int *)w.touched, (const int8_t *)w.tcls, N, w.vcls);
    else
        hipExtLaunchKernelGGL(k_compact_classes, dim3(128, NMRG), dim3(1024), 0, st, nullptr, re.round_stop, 0,
                              (const u32 *)c->n_touched, 0u, (const int *)w.touched, (const int8_t *)w.tcls, w.lists,
                              N, (c + 1)->n_active, 0u, (int8_t *)nullptr);
    return hipGetLastError();
}

// One block-sequential pass: `blocks` runs of ceil(N / blocks) consecutive ids, in id order, counter slots
// t0, t0 + 1, ...  Returns the number of slots used through *used.
static hipError_t launch_update_pass_blocks(const Workspace &w, const RowsView &rv, long long N, const ScanPlan &plan, int dtype,
                                            int R, u64 *keys, int *deg, int t0,
                                            long long blocks, hipStream_t st, int *used)
{
    const long long bs = (N + blocks - 1) / blocks;
    int k = 0;
    for (long long lo = 0; lo < N; lo += bs, ++k) {
        VertexRun run;
        run.first = (u32)lo;
        run.count = (u32)(lo + bs < N ? bs : N - lo);
        hipError_t e = launch_update_round(w, rv, N, plan, dtype, R, keys, deg, t0 + k, st, RoundEvents(),
                                           &run);
        if (e != hipSuccess) return e;
    }
    *used = k;
    return hipSuccess;
}

// slots a pass of `blocks` runs uses
static long long runs_per_pass(long long N, long long blocks)
{
    const long long bs = (N + blocks - 1) / blocks;
    return (N + bs - 1) / bs;
}

// vcls[] (class of every vertex holding a "new" entry) -> active lists of round t_next
static void launch_compact_all(const Workspace &w, long long N, int t_next, hipStream_t st,
                               hipEvent_t e_stop = nullptr)
{
    hipExtLaunchKernelGGL(k_compact_classes, dim3(256, 1), dim3(1024), 0, st, nullptr, e_stop, 0,
                          (const u32 *)nullptr, (u32)N, (const int *)nullptr, (const int8_t *)w.vcls, w.lists, N,
                          w.ctr[t_next].n_active, 0u, (int8_t *)nullptr);
}

// AddReverseEdges; the active lists for round t_next are rebuilt from scratch (t_next < 0: only vcls[], the
// class of every vertex that holds a "new" entry, is written).  Expects fill[] == 0
// and leaves it so.  Between rounds nprop[], tcls[], props[] and touched[] are free: they serve as the
// second in-edge count, the per-vertex marks, the late arrival numbers and their position masks.  misc: [0] bin cursor, [1] vertices with a bin (union and out-degree cut), [4] flagged lists,
// [2] bin cursor, [3] vertices with more than R incoming edges (in-degree cut).
static hipError_t launch_reverse(const Workspace &w, long long N, int R, int use_classes, u64 *keys, int *deg,
                                 int t_next, hipStream_t st, hipEvent_t e_stop = nullptr, int W = 0)
{
    if (W == 0) W = R;      // rows are W slots apart; R is Alg. 5's bound on out- and in-degree
    const int vb = vertex_blocks(N), tb = (int)((N + 1023) / 1024);
    int *cnt_in = w.nprop;
    int8_t *cand = w.tcls, *rowflag = w.tcls + N, *mark = w.tcls + 2 * N;
    u32 *late = (u32 *)w.props;          // one word per list slot (props is 16 bytes per slot)
    u64 *over = (u64 *)w.touched;        // two words per vertex (touched is 16 bytes per vertex)
    u32 *n_next = t_next >= 0 ? w.ctr[t_next].n_active : nullptr;
    // union with reversed edges, out-lists cut to R
    // the transposition: one arrival-number atomic per edge, or (large N, see k_bin_count) binned by target range
    const bool binned = w.blockhist && g_transpose_path != 1 && (g_transpose_path == 2 || N >= BIN_MIN_N);
    if (binned) {
        const unsigned nb = (unsigned)bin_blocks(N), nr = (unsigned)bin_ranges(N);
        hipLaunchKernelGGL(k_bin_count, dim3(nb), dim3(BIN_THREADS), 0, st, N, W, (const u64 *)keys, (const int *)deg, nr, w.blockhist, w.misc, n_next);
        hipLaunchKernelGGL(k_bin_offsets, dim3((nr + 63) / 64), dim3(1024), 0, st, nb, nr, w.blockhist, w.range_tot);
        hipLaunchKernelGGL(k_bin_bases, dim3(1), dim3(1024), 0, st, nr, (const u32 *)w.range_tot, w.range_base);
        hipLaunchKernelGGL(k_bin_partition, dim3(nb), dim3(BIN_THREADS), 0, st, N, W, (const u64 *)keys, (const int *)deg, nr,
                           (const u32 *)w.blockhist, (const u32 *)w.range_base, w.props);
        hipLaunchKernelGGL(k_bin_place, dim3(nr), dim3(PLACE_THREADS), 0, st, N, R, (const Prop *)w.props, (const u32 *)w.range_base,
                           (const int *)deg, w.fill, w.inbox, w.binoff, w.bins, w.misc + 0, w.cnt, cnt_in, cand);
    } else {
        hipLaunchKernelGGL(k_reverse_scatter, dim3((unsigned)((N * 16 + BLOCK - 1) / BLOCK)), dim3(BLOCK), 0, st, N, W, keys, deg,
                           w.fill, w.inbox, late, over, mark, w.misc, n_next);
        hipLaunchKernelGGL(k_assign_bins, dim3(tb), dim3(1024), 0, st, N, w.fill, INBOX_CAP, INBOX_CAP, INBOX_CAP,
                           w.binoff, w.misc + 0, w.hubs, w.misc + 1, w.cnt, cnt_in, (u64 *)nullptr, deg, R, cand,
                           (const int8_t *)nullptr, (int *)nullptr, (u32 *)nullptr);
        hipLaunchKernelGGL(k_reverse_surplus, dim3(vb), dim3(BLOCK), 0, st, N, W, keys, late, over, mark, w.binoff,
                           w.bins, w.misc + 1);
    }
    static const int rmerge_per_cu = resident_blocks_per_cu(k_reverse_merge, 6);
    const int rm_blocks = cu_count() * rmerge_per_cu;
    hipLaunchKernelGGL(k_reverse_merge, dim3(rm_blocks < (vb + 1) / 2 ? rm_blocks : (vb + 1) / 2), dim3(BLOCK), 0, st, N, W, R, keys,
                       deg, w.fill, w.inbox, w.binoff, w.bins, cand, cnt_in, rowflag, w.vcls, use_classes);
    // in-lists cut to R; only vertices with more than R incoming edges need a bin, and only the flagged lists
    // (class 0 of rowflag[]) are walked: the launch that hands out the bins lists them in the first active list, which is free until
    // the lists of the next round are rebuilt at the end
    int *flagged = w.lists;
    hipLaunchKernelGGL(k_assign_bins, dim3(tb), dim3(1024), 0, st, N, cnt_in, R, R, 0, w.binoff, w.misc + 2, w.hubs,
                       w.misc + 3, w.cnt, (int *)nullptr, w.thr, (const int *)nullptr, 0, (int8_t *)nullptr, (const int8_t *)rowflag, flagged, w.misc + 4);
    hipLaunchKernelGGL(k_fill_bins, dim3(capped(persistent_blocks(), N)), dim3(BLOCK), 0, st, W, (const u64 *)keys, (const int *)deg,
                       (const int *)flagged, (const u32 *)(w.misc + 4), w.binoff, w.cnt, w.bins, 0u, w.misc + 3);
    hipLaunchKernelGGL(k_incap_threshold, dim3(capped(persistent_blocks(), N)), dim3(BLOCK), 0, st, R, w.hubs, w.misc + 3,
                       cnt_in, w.binoff, w.bins, w.thr);
    hipLaunchKernelGGL(k_incap_filter, dim3(capped(persistent_blocks(), N)), dim3(BLOCK), 0, st, W, keys, deg, w.thr,
                       (const int *)flagged, (const u32 *)(w.misc + 4), w.vcls, use_classes, w.misc + 3);
    if (t_next >= 0) launch_compact_all(w, N, t_next, st, e_stop);
    else if (e_stop) (void)hipEventRecord(e_stop, st);
    return hipGetLastError();
}

static void fill_round_stats(rnnd_stats *s, const RoundCtr *h, int rounds)
{
    s->rounds = rounds;
    for (int t = 0; t < rounds; ++t) s->group_scans += h[t].groups != 0u;
    for (int t = 0; t < rounds && t < RNND_MAX_ROUNDS; ++t) {
        s->active[t] = 0;
        for (int c = 0; c < NDEG; ++c) s->active[t] += h[t].n_active[c];
        for (int k = 0; k < STAT_SLOTS; ++k) {
            s->algo_evals[t] += (int64_t)h[t].stat[k][0];
            s->exec_evals[t] += (int64_t)h[t].stat[k][1];
            s->gathered_rows[t] += (int64_t)h[t].stat[k][2];
            s->proposals[t] += (int64_t)h[t].stat[k][3];
            s->dropped[t] += (int64_t)h[t].stat[k][4];
        }
    }
}

// --------------------------------------------------------------- where a call's workspace comes from
// 1. the block the library keeps per device between calls (allocated by the first call that needs it, grown
//    when a later call needs more, handed back by rnnd_release_workspace): repeated builds pay no allocation;
// 2. a fresh allocation, freed when the call ends, if another thread's call holds that block;
// 3. for rnnd_build_static only: the file-scope array below, which needs no allocation at all.
// The padded copy of X has a block of its own (1. and 2.), because a call can do without it: asking for it must not cost
// the block the call cannot do without, and it is the first to go when that block cannot be had.
#define RNND_MAX_DEVICES 64
#define SEARCH_MAX_BLOCKS 16384     // queries a search has in flight at most

static __device__ __align__(256) unsigned char scratch[RNND_STATIC_SCRATCH_BYTES];

struct DeviceSlot {
    char *cached = nullptr;        // the kept block
    size_t cached_bytes = 0;
    char *copy = nullptr;          // the kept block for padded rows
    size_t copy_bytes = 0;
    bool busy = false;             // a call is using them
    char *static_ptr = nullptr;    // this device's copy of `scratch` (hipGetSymbolAddress, once per device)
    unsigned long long *counts = nullptr;   // pinned host memory, kept like the block: SEARCH_MAX_BLOCKS evaluation counts
};
static std::mutex g_ws_mu;
static DeviceSlot g_dev[RNND_MAX_DEVICES];
static int g_poison = 0;           // testing aid: every workspace is filled with 0xA5 bytes before it is cleared

enum WsSource { WS_NONE = 0, WS_CACHED, WS_FRESH, WS_STATIC };
struct WsLease {
    char *base = nullptr, *copy = nullptr;
    int dev = -1;
    WsSource src = WS_NONE;
};

__global__ void k_fill_u32(u32 *p, size_t n, u32 v)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

// No device holds a workspace of this size; asking for one is an allocation failure that needs no device to detect.
#define RNND_WS_HARD_LIMIT ((size_t)1 << 40)

static int ws_acquire(size_t bytes, bool static_only, hipStream_t st, WsLease *out)
{
    int rc = RNND_OK, dev = 0;
    if (!static_only && bytes > RNND_WS_HARD_LIMIT) return RNND_ERR_OOM;
    if (static_only && bytes > RNND_STATIC_SCRATCH_BYTES) return RNND_ERR_SCRATCH;
    HIPCHK(hipGetDevice(&dev));
    if (dev < 0 || dev >= RNND_MAX_DEVICES) {
        snprintf(g_last_hip_error, sizeof g_last_hip_error, "device index %d is beyond the %d this library tracks", dev,
                 RNND_MAX_DEVICES);
        return RNND_ERR_HIP;
    }
    {
        std::lock_guard<std::mutex> lock(g_ws_mu);
        DeviceSlot &d = g_dev[dev];
        if (static_only) {
            if (!d.static_ptr) {
                char *ptr = nullptr;
                HIPCHK(hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch)));
                d.static_ptr = ptr;
            }
            out->base = d.static_ptr;
            out->src = WS_STATIC;
        } else if (!d.busy) {
            if (d.cached && d.cached_bytes < bytes) {
                (void)hipFree(d.cached);
                d.cached = nullptr;
                d.cached_bytes = 0;
            }
            if (!d.cached) {
                if (d.copy && hipMalloc((void **)&d.cached, bytes) != hipSuccess) {
                    (void)hipGetLastError();
                    d.cached = nullptr;
                    (void)hipFree(d.copy);
                    d.copy = nullptr;
                    d.copy_bytes = 0;
                }
                if (!d.cached) HIPCHK(hipMalloc((void **)&d.cached, bytes));
                d.cached_bytes = bytes;
            }
            d.busy = true;
            out->base = d.cached;
            out->src = WS_CACHED;
        } else {
            HIPCHK(hipMalloc((void **)&out->base, bytes));
            out->src = WS_FRESH;
        }
        out->dev = dev;
    }
    if (g_poison) hipLaunchKernelGGL(k_fill_u32, dim3(2048), dim3(256), 0, st, (u32 *)out->base, bytes / 4, 0xA5A5A5A5u);
done:
    return rc;
}

// A block for padded rows next to the one the lease holds; false where there is no room for it.
static bool ws_acquire_copy(WsLease *l, size_t bytes, hipStream_t st)
{
    if (bytes > RNND_WS_HARD_LIMIT) return false;
    if (l->src == WS_CACHED) {
        std::lock_guard<std::mutex> lock(g_ws_mu);
        DeviceSlot &d = g_dev[l->dev];       // busy: no other call touches the slot's blocks
        if (d.copy_bytes < bytes) {
            if (d.copy) (void)hipFree(d.copy);
            d.copy = nullptr;
            d.copy_bytes = 0;
            if (hipMalloc((void **)&d.copy, bytes) != hipSuccess) d.copy = nullptr;
            else d.copy_bytes = bytes;
        }
        l->copy = d.copy;
    } else if (hipMalloc((void **)&l->copy, bytes) != hipSuccess) {
        l->copy = nullptr;
    }
    if (!l->copy) (void)hipGetLastError();      // not an error of the call
    else if (g_poison) hipLaunchKernelGGL(k_fill_u32, dim3(2048), dim3(256), 0, st, (u32 *)l->copy, bytes / 4, 0xA5A5A5A5u);
    return l->copy != nullptr;
}

// Lays out and acquires the workspace of a build or of UpdateNeighbors calls.  Where there is no room for the padded
// copy of X the plan does without it.  (The static array holds the copy as well, if it is large enough.)
static int ws_open(Workspace &w, WsLease *lease, ScanPlan &plan, const void *X, long long N, int R, int d, int dtype, int n_ctr,
                   bool own_graph, bool static_only, hipStream_t st)
{
    const bool apart = plan.extra() && !static_only;
    w.bytes = ws_layout(w, N, R, n_ctr, own_graph, apart ? 0 : plan.copy_bytes);
    int rc = ws_acquire(w.bytes, static_only, st, lease);
    bool no_copy = rc ? rc == RNND_ERR_SCRATCH && plan.extra() : apart && !ws_acquire_copy(lease, align_up(plan.copy_bytes) + plan.half_bytes, st);
    if (no_copy && !rc && plan.half_rb) {      // no room for the half-precision rows: do without these first
        plan.half_rb = 0;
        plan.half_bytes = 0;
        no_copy = plan.extra() && !ws_acquire_copy(lease, plan.copy_bytes, st);
    }
    if (no_copy) plan = scan_plan_for(X, N, d, dtype, false);
    if (no_copy && rc) {
        w.bytes = ws_layout(w, N, R, n_ctr, own_graph, plan.copy_bytes);
        rc = ws_acquire(w.bytes, static_only, st, lease);
    }
    if (rc) return rc;
    w.base = lease->base;
    ws_layout(w, N, R, n_ctr, own_graph, apart ? 0 : plan.copy_bytes);
    if (lease->copy) {
        w.xs = (int8_t *)lease->copy;
        w.half = lease->copy + align_up(plan.copy_bytes);
    }
    return RNND_OK;
}

static void ws_release(WsLease *l)
{
    if (l->src == WS_FRESH) {
        (void)hipFree(l->base);
        if (l->copy) (void)hipFree(l->copy);
    } else if (l->src == WS_CACHED) {
        std::lock_guard<std::mutex> lock(g_ws_mu);
        g_dev[l->dev].busy = false;
    }
    l->src = WS_NONE;
    l->base = l->copy = nullptr;
}

extern "C" int rnnd_release_workspace(void)
{
    int rc = RNND_OK, dev = 0;
    HIPCHK(hipGetDevice(&dev));
    if (dev >= 0 && dev < RNND_MAX_DEVICES) {
        std::lock_guard<std::mutex> lock(g_ws_mu);
        DeviceSlot &d = g_dev[dev];
        if (d.cached && !d.busy) {
            HIPCHK(hipFree(d.cached));
            d.cached = nullptr;
            d.cached_bytes = 0;
        }
        if (d.copy && !d.busy) {
            HIPCHK(hipFree(d.copy));
            d.copy = nullptr;
            d.copy_bytes = 0;
        }
        if (d.counts && !d.busy) {
            HIPCHK(hipHostFree(d.counts));
            d.counts = nullptr;
        }
    }
done:
    return rc;
}

// Where the blocks of a search put their evaluation counts: the kept buffer if the lease holds the kept block, else one
// of its own (freed by counts_release).
static int counts_acquire(const WsLease &l, unsigned long long **out)
{
    int rc = RNND_OK;
    if (l.src == WS_CACHED) {       // busy: no other call touches the slot's buffer
        DeviceSlot &d = g_dev[l.dev];
        if (!d.counts) HIPCHK(hipHostMalloc((void **)&d.counts, SEARCH_MAX_BLOCKS * sizeof(unsigned long long), hipHostMallocDefault));
        *out = d.counts;
    } else {
        HIPCHK(hipHostMalloc((void **)out, SEARCH_MAX_BLOCKS * sizeof(unsigned long long), hipHostMallocDefault));
    }
done:
    return rc;
}
static void counts_release(const WsLease &l, unsigned long long *p)
{
    if (p && l.src != WS_CACHED) (void)hipHostFree(p);
}

extern "C" int rnnd_set_workspace_poison(int on)
{
    g_poison = on ? 1 : 0;
    return RNND_OK;
}

extern "C" int rnnd_workspace_bytes(int64_t N, int32_t d, int dtype, int32_t R, int64_t rounds, size_t *bytes)
{
    if (!bytes) return RNND_ERR_NULL;
    if (dtype != RNND_U8 && dtype != RNND_F32 && dtype != RNND_F16 && dtype != RNND_BF16) return RNND_ERR_UNSUPPORTED;
    if (N < 2 || N > 2147483646LL || d < 1) return RNND_ERR_BAD_SHAPE;
    if (R < 1 || R > RNND_MAX_R || rounds < 1 || rounds > RNND_MAX_RUN_SLOTS) return RNND_ERR_BAD_PARAM;
    Workspace w;
    // what no call can do without: the int8 copy of uint8 rows of 32, 64 or 128 bytes, but no padded copy (see ScanPlan)
    *bytes = ws_layout(w, N, R, (int)rounds + 2, true,
                       (dtype == RNND_U8 && (d == 32 || d == 64 || d == 128)) ? (size_t)N * d : 0);
    return RNND_OK;
}

template <int DT>
static void launch_random_graph_dt(const void *X, long long N, int d, int vec_ok, int S, int R, u64 seed, u64 *keys,
                                   int *deg, int8_t *vcls, int use_classes, hipStream_t st)
{
    hipLaunchKernelGGL(k_random_graph<DT>, dim3(vertex_blocks(N)), dim3(BLOCK), 0, st, X, N, d, vec_ok, S, R, seed, keys,
                       deg, vcls, use_classes);
}

static void launch_random_graph(const void *X, long long N, int d, int dtype, int vec_ok, int S, int R, u64 seed,
                                u64 *keys, int *deg, int8_t *vcls, int use_classes, hipStream_t st)
{
    if (dtype == RNND_U8) launch_random_graph_dt<DT_U8>(X, N, d, vec_ok, S, R, seed, keys, deg, vcls, use_classes, st);
    else if (dtype == RNND_F16) launch_random_graph_dt<DT_F16>(X, N, d, vec_ok, S, R, seed, keys, deg, vcls, use_classes, st);
    else if (dtype == RNND_BF16) launch_random_graph_dt<DT_BF16>(X, N, d, vec_ok, S, R, seed, keys, deg, vcls, use_classes, st);
    else launch_random_graph_dt<DT_F32>(X, N, d, vec_ok, S, R, seed, keys, deg, vcls, use_classes, st);
}

// per-pass statistics of a block-sequential run: slot sums of the runs of each pass
static void fill_pass_stats(rnnd_stats *s, const RoundCtr *h, int passes, int per_pass)
{
    rnnd_stats one;
    s->rounds = passes;
    for (int p = 0; p < passes && p < RNND_MAX_ROUNDS; ++p) {
        for (int k = 0; k < per_pass; ++k) {
            memset(&one, 0, sizeof one);
            fill_round_stats(&one, h + (size_t)p * per_pass + k, 1);
            s->group_scans += one.group_scans;
            s->active[p] += one.active[0];
            s->algo_evals[p] += one.algo_evals[0];
            s->exec_evals[p] += one.exec_evals[0];
            s->gathered_rows[p] += one.gathered_rows[0];
            s->proposals[p] += one.proposals[0];
            s->dropped[p] += one.dropped[0];
        }
    }
}

// Alg. 6, every variant of the driver.
//   M       slots per row = the bound every UpdateNeighbors merge cuts a list to (M = R: rnnd_build;
//           M > R: rnnd_build_wide, where only AddReverseEdges cuts to R)
//   blocks  0: synchronous rounds; >= 1: block-sequential passes of that many runs (rnnd_build_blocks)
//   fixed   the workspace is the static scratch array: no allocation of any kind, hence no statistics
static int build_impl(const void *X, int64_t N, int32_t d, int dtype, int metric, int32_t S, int32_t R, int32_t M,
                      int32_t T1, int32_t T2, uint64_t seed, int64_t blocks, int32_t *graph_out,
                      int32_t *degree_out, uint64_t *keys_out, rnnd_stats *stats, void *stream, bool fixed)
{
    int rc = check_data_args(X, N, d, dtype, metric, M);
    if (rc) return rc;
    if (R < 1 || R > M) return RNND_ERR_BAD_PARAM;
    if (!graph_out || !degree_out) return RNND_ERR_NULL;
    if (S < 1 || S > R || (int64_t)S > N - 1 || T1 < 1 || T2 < 1) return RNND_ERR_BAD_PARAM;
    if ((int64_t)T1 * T2 > RNND_MAX_RUN_SLOTS || blocks < 0 || blocks > N) return RNND_ERR_BAD_PARAM;
    const long long per_pass = blocks ? runs_per_pass(N, blocks) : 1;
    if ((long long)T1 * T2 * per_pass > RNND_MAX_RUN_SLOTS) return RNND_ERR_BAD_PARAM;
    hipStream_t st = (hipStream_t)stream;
    const int rounds = T1 * T2, n_ctr = (int)(rounds * per_pass) + 2;
    // (padded float rows read a flag back: not in a call that may not allocate)
    ScanPlan plan = scan_plan_for(X, N, d, dtype, worth_padding(N, d, dtype, false) && (!fixed || dtype == RNND_U8), !fixed);
    // events (only when statistics are wanted): 0 start, 1 end of init, last: the end.  Per-round times come from the
    // device clock (RoundCtr::t_*), which costs nothing; with rnnd_set_event_timing(1), and for block-sequential
    // passes, from events as well: 2 + 3t .. 4 + 3t = scan start, scan stop, end of round t (block-sequential passes
    // record only the last), then the end of each reverse call
    const bool ev_rounds = stats && (g_event_timing || blocks);
    const int e_rev = 2 + 3 * rounds, e_end = e_rev + T1, n_ev = stats ? e_end + 1 : 0;
    Workspace w;
    WsLease lease;
    hipEvent_t *ev = nullptr;
    RoundCtr *hctr = nullptr;
    int n_ev_made = 0;
    rc = ws_open(w, &lease, plan, X, N, M, d, dtype, n_ctr, true, fixed, st);
    if (rc) return rc;
    if (stats) {
        ev = (hipEvent_t *)calloc(n_ev + 1, sizeof(hipEvent_t));
        hctr = (RoundCtr *)calloc(n_ctr, sizeof(RoundCtr));
        if (!ev || !hctr) { rc = RNND_ERR_OOM; goto done; }
        for (; n_ev_made < n_ev; ++n_ev_made)
            if (ev_rounds || n_ev_made < 2 || n_ev_made == e_end) HIPCHK(hipEventCreate(&ev[n_ev_made]));
    }
    {
        int t = 0;
        if (stats) HIPCHK(hipEventRecord(ev[0], st));
        ws_clear(w, st);
        RowsView rows;
        HIPCHK(prepare_rows(w, plan, X, N, d, dtype, st, false, nullptr, &rows));
        const int variant = plan.variant, use_classes = plan.classes();
        launch_random_graph(rows.X, N, rows.d, dtype, rows.vec_ok, S, M, (u64)seed, w.keys, w.deg, w.vcls, use_classes, st);
        if (!blocks) launch_compact_all(w, N, 0, st, stats ? ev[1] : nullptr);
        else if (stats) HIPCHK(hipEventRecord(ev[1], st));
        HIPCHK(hipGetLastError());
        for (int t1 = 0; t1 < T1; ++t1) {
            for (int t2 = 0; t2 < T2; ++t2, ++t) {
                if (blocks) {
                    int used = 0;
                    HIPCHK(launch_update_pass_blocks(w, rows, N, plan, dtype, M, w.keys, w.deg,
                                                     (int)(t * per_pass), blocks, st, &used));
                    if (stats) HIPCHK(hipEventRecord(ev[4 + 3 * t], st));
                    continue;
                }
                RoundEvents re;
                // a round ends where the next one starts; only the last round before a reverse call or
                // the export needs a mark of its own for that
                if (ev_rounds) {
                    re.scan_start = ev[2 + 3 * t];
                    re.scan_stop = ev[3 + 3 * t];
                    if (t2 == T2 - 1) re.round_stop = ev[4 + 3 * t];
                }
                HIPCHK(launch_update_round(w, rows, N, plan, dtype, M, w.keys, w.deg, t, st, re));
                if (stats && !ev_rounds && t2 == T2 - 1)
                    hipLaunchKernelGGL(k_stamp, dim3(1), dim3(64), 0, st, &w.ctr[t].t_round_stop);
            }
            if (t1 != T1 - 1) {
                HIPCHK(launch_reverse(w, N, R, use_classes, w.keys, w.deg, blocks ? -1 : t, st,
                                      ev_rounds ? ev[e_rev + t1] : nullptr, M));
            }
        }
        launch_export(N, M, w.keys, w.deg, graph_out, degree_out, st);
        HIPCHK(hipGetLastError());
        if (keys_out)
            HIPCHK(hipMemcpyAsync(keys_out, w.keys, (size_t)N * M * 8, hipMemcpyDeviceToDevice, st));
        if (stats) {
            HIPCHK(hipEventRecord(ev[e_end], st));
            HIPCHK(hipMemcpyAsync(hctr, w.ctr, (size_t)n_ctr * sizeof(RoundCtr), hipMemcpyDeviceToHost, st));
        }
        HIPCHK(hipStreamSynchronize(st));
        if (stats) {
            memset(stats, 0, sizeof *stats);
            if (blocks) fill_pass_stats(stats, hctr, rounds, (int)per_pass);
            else fill_round_stats(stats, hctr, rounds);
            stats->reverse_calls = T1 - 1;
            stats->init_evals = (int64_t)N * S;
            stats->kernel_variant = variant;
            float ms = 0;
            (void)hipEventElapsedTime(&ms, ev[0], ev[1]); stats->init_ms = ms;
            int tt = 0;
            // device clock: ticks per millisecond, and the time between two marks (0 where one is missing)
            int dev = 0, khz = 0;
            (void)hipGetDevice(&dev);
            (void)hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev);
            auto clk_ms = [khz](u64 a, u64 b) { return (a && b > a && khz > 0) ? (float)((double)(b - a) / (double)khz) : 0.f; };
            for (int t1 = 0; t1 < T1 && !ev_rounds; ++t1) {
                for (int t2 = 0; t2 < T2; ++t2, ++tt) {
                    if (tt >= RNND_MAX_ROUNDS) continue;
                    stats->scan_ms[tt] = clk_ms(hctr[tt].t_scan_start, hctr[tt].t_scan_stop);
                    stats->round_ms[tt] = clk_ms(hctr[tt].t_scan_start, t2 == T2 - 1 ? hctr[tt].t_round_stop : hctr[tt + 1].t_scan_start);
                }
                // an AddReverseEdges call ends where the next round's scan starts
                if (t1 != T1 - 1 && t1 < RNND_MAX_ROUNDS) stats->reverse_ms[t1] = clk_ms(hctr[tt - 1].t_round_stop, hctr[tt].t_scan_start);
            }
            for (int t1 = 0; t1 < T1 && ev_rounds; ++t1) {
                for (int t2 = 0; t2 < T2; ++t2, ++tt) {
                    if (tt >= RNND_MAX_ROUNDS) continue;
                    if (blocks) {
                        // a pass starts where the one before it, the init or the reverse call ended
                        hipEvent_t from = t2 > 0 ? ev[4 + 3 * (tt - 1)] : (t1 == 0 ? ev[1] : ev[e_rev + t1 - 1]);
                        (void)hipEventElapsedTime(&ms, from, ev[4 + 3 * tt]); stats->round_ms[tt] = ms;
                        continue;
                    }
                    (void)hipEventElapsedTime(&ms, ev[2 + 3 * tt], ev[3 + 3 * tt]); stats->scan_ms[tt] = ms;
                    (void)hipEventElapsedTime(&ms, ev[2 + 3 * tt], t2 == T2 - 1 ? ev[4 + 3 * tt] : ev[2 + 3 * (tt + 1)]);
                    stats->round_ms[tt] = ms;
                }
                if (t1 != T1 - 1 && t1 < RNND_MAX_ROUNDS) {
                    // from the end of the last round before the call to the end of the call
                    (void)hipEventElapsedTime(&ms, ev[4 + 3 * (tt - 1)], ev[e_rev + t1]);
                    stats->reverse_ms[t1] = ms;
                }
            }
            (void)hipEventElapsedTime(&ms, ev[0], ev[e_end]); stats->total_ms = ms;
        }
    }
done:
    if (rc == RNND_ERR_HIP || rc == RNND_ERR_OOM) (void)hipStreamSynchronize(st);   // nothing may still use the workspace
    for (int i = 0; i < n_ev_made; ++i)
        if (ev[i]) (void)hipEventDestroy(ev[i]);
    free(ev);
    free(hctr);
    ws_release(&lease);
    return rc;
}

extern "C" int rnnd_build_ex(const void *X, int64_t N, int32_t d, int dtype, int metric, int32_t S,
                             int32_t R, int32_t T1, int32_t T2, uint64_t seed, int32_t *graph_out,
                             int32_t *degree_out, uint64_t *keys_out, rnnd_stats *stats, void *stream)
{
    return build_impl(X, N, d, dtype, metric, S, R, R, T1, T2, seed, 0, graph_out, degree_out, keys_out, stats, stream, false);
}

extern "C" int rnnd_build_wide(const void *X, int64_t N, int32_t d, int dtype, int metric, int32_t S, int32_t R,
                               int32_t M, int32_t T1, int32_t T2, uint64_t seed, int32_t *graph_out,
                               int32_t *degree_out, uint64_t *keys_out, rnnd_stats *stats, void *stream)
{
    if (M < 1 || M > RNND_MAX_R) return X ? RNND_ERR_BAD_PARAM : RNND_ERR_NULL;
    return build_impl(X, N, d, dtype, metric, S, R, M, T1, T2, seed, 0, graph_out, degree_out, keys_out, stats, stream, false);
}

extern "C" int rnnd_build(const void *X, int64_t N, int32_t d, int dtype, int metric, int32_t S, int32_t R,
                          int32_t T1, int32_t T2, uint64_t seed, int32_t *graph_out, int32_t *degree_out,
                          void *stream)
{
    return build_impl(X, N, d, dtype, metric, S, R, R, T1, T2, seed, 0, graph_out, degree_out, nullptr, nullptr, stream, false);
}

extern "C" int rnnd_build_static(const void *X, int64_t N, int32_t d, int dtype, int metric, int32_t S, int32_t R,
                                 int32_t T1, int32_t T2, uint64_t seed, int32_t *graph_out, int32_t *degree_out,
                                 void *stream)
{
    return build_impl(X, N, d, dtype, metric, S, R, R, T1, T2, seed, 0, graph_out, degree_out, nullptr, nullptr, stream, true);
}

extern "C" int rnnd_build_blocks(const void *X, int64_t N, int32_t d, int dtype, int metric, int32_t S,
                                 int32_t R, int32_t T1, int32_t T2, uint64_t seed, int64_t blocks,
                                 int32_t *graph_out, int32_t *degree_out, uint64_t *keys_out, rnnd_stats *stats,
                                 void *stream)
{
    if (blocks < 1) return X ? RNND_ERR_BAD_PARAM : RNND_ERR_NULL;
    return build_impl(X, N, d, dtype, metric, S, R, R, T1, T2, seed, blocks, graph_out, degree_out, keys_out, stats, stream, false);
}

extern "C" int rnnd_random_graph(const void *X, int64_t N, int32_t d, int dtype, int metric, int32_t S,
                                 int32_t R, uint64_t seed, uint64_t *keys, int32_t *deg, void *stream)
{
    int rc = check_data_args(X, N, d, dtype, metric, R);
    if (rc) return rc;
    if (!keys || !deg) return RNND_ERR_NULL;
    if (S < 1 || S > R || (int64_t)S > N - 1) return RNND_ERR_BAD_PARAM;
    hipStream_t st = (hipStream_t)stream;
    launch_random_graph(X, N, d, dtype, vec_ok_for(X, d, dtype), S, R, (u64)seed, (u64 *)keys, deg, (int8_t *)nullptr, 0, st);
    HIPCHK(hipGetLastError());
    HIPCHK(hipStreamSynchronize(st));
done:
    return rc;
}

// UpdateNeighbors applied in place to a caller's snapshot: n_rounds synchronous rounds (blocks = 0) or
// block-sequential passes of `blocks` runs.
static int update_impl(const void *X, int64_t N, int32_t d, int dtype, int metric, int32_t R, uint64_t *keys,
                       int32_t *deg, int32_t n_rounds, int64_t blocks, rnnd_stats *stats, void *stream)
{
    int rc = check_data_args(X, N, d, dtype, metric, R);
    if (rc) return rc;
    if (!keys || !deg) return RNND_ERR_NULL;
    if (n_rounds < 1 || n_rounds > RNND_MAX_RUN_SLOTS || blocks < 0 || blocks > N) return RNND_ERR_BAD_PARAM;
    const long long per_pass = blocks ? runs_per_pass(N, blocks) : 1;
    if ((long long)n_rounds * per_pass > RNND_MAX_RUN_SLOTS) return RNND_ERR_BAD_PARAM;
    hipStream_t st = (hipStream_t)stream;
    const int n_ctr = (int)(n_rounds * per_pass) + 2;
    ScanPlan plan = scan_plan_for(X, N, d, dtype, worth_padding(N, d, dtype, true));
    Workspace w;
    WsLease lease;
    RoundCtr *hctr = nullptr;
    RowsView rows;
    const SnapshotRound round = {(const u64 *)keys, deg, R};
    bool listed = false;
    rc = ws_open(w, &lease, plan, X, N, R, d, dtype, n_ctr, false, false, st);
    if (rc) return rc;
    if (stats) {
        hctr = (RoundCtr *)calloc(n_ctr, sizeof(RoundCtr));
        if (!hctr) { rc = RNND_ERR_OOM; goto done; }
    }
    listed = (plan.copy == COPY_ROWS || plan.copy == COPY_ROWS_PERMUTED) && !blocks && n_rounds == 1 && N >= LISTED_MIN_N;
    ws_clear(w, st);
    // (the copy first, where it does not depend on the lists: it runs while the other launches are submitted)
    if (!listed) HIPCHK(prepare_rows(w, plan, X, N, d, dtype, st, true, nullptr, &rows));
    hipLaunchKernelGGL(k_classify, dim3(vertex_blocks(N)), dim3(BLOCK), 0, st, (long long)N, R, (const u64 *)keys,
                       deg, w.vcls, plan.classes());
    if (!blocks) launch_compact_all(w, N, 0, st);
    if (listed) HIPCHK(prepare_rows(w, plan, X, N, d, dtype, st, true, &round, &rows));
    for (int t = 0; t < n_rounds; ++t) {
        if (blocks) {
            int used = 0;
            HIPCHK(launch_update_pass_blocks(w, rows, N, plan, dtype, R, (u64 *)keys, deg,
                                             (int)(t * per_pass), blocks, st, &used));
        } else {
            HIPCHK(launch_update_round(w, rows, N, plan, dtype, R, (u64 *)keys, deg, t, st));
        }
    }
    if (stats) {
        if (!blocks) hipLaunchKernelGGL(k_stamp, dim3(1), dim3(64), 0, st, &w.ctr[n_rounds - 1].t_round_stop);
        HIPCHK(hipMemcpyAsync(hctr, w.ctr, (size_t)n_ctr * sizeof(RoundCtr), hipMemcpyDeviceToHost, st));
    }
    HIPCHK(hipStreamSynchronize(st));
    if (stats) {
        memset(stats, 0, sizeof *stats);
        if (blocks) fill_pass_stats(stats, hctr, n_rounds, (int)per_pass);
        else fill_round_stats(stats, hctr, n_rounds);
        stats->kernel_variant = plan.variant;
        if (!blocks) {      // per-round times from the device clock (see build_impl)
            int dev = 0, khz = 0;
            (void)hipGetDevice(&dev);
            (void)hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev);
            auto clk_ms = [khz](u64 a, u64 b) { return (a && b > a && khz > 0) ? (float)((double)(b - a) / (double)khz) : 0.f; };
            for (int t = 0; t < n_rounds && t < RNND_MAX_ROUNDS; ++t) {
                stats->scan_ms[t] = clk_ms(hctr[t].t_scan_start, hctr[t].t_scan_stop);
                stats->round_ms[t] = clk_ms(hctr[t].t_scan_start, t == n_rounds - 1 ? hctr[t].t_round_stop : hctr[t + 1].t_scan_start);
            }
        }
    }
done:
    if (rc == RNND_ERR_HIP || rc == RNND_ERR_OOM) (void)hipStreamSynchronize(st);
    free(hctr);
    ws_release(&lease);
    return rc;
}

extern "C" int rnnd_update_neighbors(const void *X, int64_t N, int32_t d, int dtype, int metric, int32_t R,
                                     uint64_t *keys, int32_t *deg, int32_t n_rounds, rnnd_stats *stats,
                                     void *stream)
{
    return update_impl(X, N, d, dtype, metric, R, keys, deg, n_rounds, 0, stats, stream);
}

extern "C" int rnnd_update_neighbors_blocks(const void *X, int64_t N, int32_t d, int dtype, int metric, int32_t R,
                                            uint64_t *keys, int32_t *deg, int32_t n_passes, int64_t blocks,
                                            rnnd_stats *stats, void *stream)
{
    if (blocks < 1) return X ? RNND_ERR_BAD_PARAM : RNND_ERR_NULL;
    return update_impl(X, N, d, dtype, metric, R, keys, deg, n_passes, blocks, stats, stream);
}

extern "C" int rnnd_add_reverse_edges_wide(int64_t N, int32_t R, int32_t M, uint64_t *keys, int32_t *deg,
                                           void *stream)
{
    int rc = RNND_OK;
    if (!keys || !deg) return RNND_ERR_NULL;
    if (N < 2 || N > 2147483646LL) return RNND_ERR_BAD_SHAPE;
    if (R < 1 || M < R || M > RNND_MAX_R) return RNND_ERR_BAD_PARAM;
    if ((unsigned long long)N * (unsigned long long)M > RNND_MAX_SLOTS) return RNND_ERR_BAD_SHAPE;
    hipStream_t st = (hipStream_t)stream;
    Workspace w;
    WsLease lease;
    w.bytes = ws_layout(w, N, M, 2, false, 0);
    rc = ws_acquire(w.bytes, false, st, &lease);
    if (rc) return rc;
    w.base = lease.base;
    ws_layout(w, N, M, 2, false, 0);
    ws_clear(w, st);      // launch_reverse expects fill[] == 0, cnt[] == 0 and zeroed counters
    HIPCHK(launch_reverse(w, N, R, 0, (u64 *)keys, deg, 0, st, nullptr, M));
    HIPCHK(hipStreamSynchronize(st));
done:
    if (rc == RNND_ERR_HIP || rc == RNND_ERR_OOM) (void)hipStreamSynchronize(st);
    ws_release(&lease);
    return rc;
}

extern "C" int rnnd_add_reverse_edges(int64_t N, int32_t R, uint64_t *keys, int32_t *deg, void *stream)
{
    return rnnd_add_reverse_edges_wide(N, R, R, keys, deg, stream);
}

extern "C" int rnnd_export_graph(int64_t N, int32_t R, const uint64_t *keys, const int32_t *deg,
                                 int32_t *graph_out, int32_t *degree_out, void *stream)
{
    int rc = RNND_OK;
    if (!keys || !deg || !graph_out || !degree_out) return RNND_ERR_NULL;
    if (N < 1 || N > 2147483646LL) return RNND_ERR_BAD_SHAPE;
    if (R < 1 || R > RNND_MAX_R) return RNND_ERR_BAD_PARAM;
    hipStream_t st = (hipStream_t)stream;
    launch_export(N, R, (const u64 *)keys, deg, graph_out, degree_out, st);
    HIPCHK(hipGetLastError());
    HIPCHK(hipStreamSynchronize(st));
done:
    return rc;
}

extern "C" int rnnd_search(const void *X, int64_t N, int32_t d, int dtype, int metric, const int32_t *graph,
                           const int32_t *degree, int32_t row_stride, const void *Q, int64_t nq, int32_t L,
                           int32_t K, int32_t k, uint64_t seed, int32_t *out_ids, uint32_t *out_dist_bits,
                           int64_t *dist_evals, void *stream)
{
    int rc = check_data_args(X, N, d, dtype, metric, 1);
    if (rc) return rc;
    if (nq < 0 || nq > 2147483646LL) return RNND_ERR_BAD_SHAPE;
    if (row_stride < 1 || L < 1 || L > SEARCH_MAX_L || K < 1 || k < 1 || k > L) return RNND_ERR_BAD_PARAM;
    if (!graph || !degree || ((!out_ids || !Q) && nq > 0)) return RNND_ERR_NULL;
    hipStream_t st = (hipStream_t)stream;
    if (dist_evals) *dist_evals = 0;
    if (nq == 0) return RNND_OK;
    const size_t rowbytes = (size_t)d * dt_size(dtype);
    const int vec_ok = (rowbytes % 16 == 0) && (((uintptr_t)X) % 16 == 0) && (((uintptr_t)Q) % 16 == 0);
    // few queries: a team of four wavefronts for each (rows of up to 128 bytes: one, which evaluates while the table answers),
    // and the LDS is free for larger tables (fewer collisions)
    const bool few = nq <= 4ll * cu_count();
    // The table of evaluated vertices takes LDS that wavefronts need, holds 7/8 of its slots - 64 vertices (384, 832, 1,728,
    // 3,520; see SeenSet) and costs most when it overflows: then the bitmap has to be cleared all the same.  A query evaluates
    // about 300 vertices + 12 per place of its candidate list, 15 with wide rows (K > 40); on rows of up to 128 bytes 20 and 28 (100,000
    // to 1M vertices, eight kinds of rows).  Few queries have the LDS for 4,096 slots, alone for 8,192.  The others:
    //   rounds of queries   the smallest table that holds what is expected: 10,000 queries on 1M x 128 uint8, K = 32, bitmap
    //     follow each other / 1,024 / 2,048 / 4,096 slots: L = 16 (571 evaluated) 728 / 314 / 333 / 408 us, L = 24 (717) 841 /
    //                       490 / 408 / 477, L = 64 (1,348) 1,313 / 1,845 / 887 / 993, L = 90 (1,711) 1,629 / 2,148 / 1,516 / 1,404, L = 128
    //                       (2,196) 2,029 / 2,603 / 2,526 / 1,914; beyond 1,728 expected the bitmap alone, as 4,096 slots are
    //                       twice as slow on rows of 384 bytes (300,000 x 96 float32, L = 90: 1,345 / 1,623 / 1,027 / 2,249).  Rows of
    //                       more than 128 bytes have fewer wavefronts per CU anyway: 2,048 slots at least (L = 32: 656 / 472 / 437).
    //                       Short rows of a small index, whose bitmaps stay in cache: 200,000 x 128 uint8, L = 16 296 / 253 / 283,
    //                       L = 64 (1,049) 763 / 946 / 778, L = 90 961 / 1,278 / 1,144: bitmap beyond 1,024 slots
    //   all at once         as many slots, up to 4,096, as leave all queries resident: 1,500 queries, 1M x 128, L = 64 bitmap / 2,048
    //                       / 4,096: 322 / 370 / 266 us, L = 128 523 / 716 / 471; 1M x 32 uint8, L = 90 (2,225) 320 / 467 / 311, L = 128
    //                       (3,003) 414 / 683 / 435; 4,000 queries, 1M x 128, L = 16 349 / 171 / 221 (1,024 slots 224)
    const bool short_rows = vec_ok && rowbytes <= 128;
    const u32 expect = 300u + (u32)L * (short_rows ? (K > 40 ? 28u : 20u) : (K > 40 ? 15u : 12u));
    const size_t q_bytes = ((dtype == RNND_U8 ? rowbytes : (size_t)d * 8) + 15) / 16 * 16;
    auto all_resident = [&](u32 sl) { return (size_t)((nq + cu_count() - 1) / cu_count()) * (sl * 4 + q_bytes + sizeof(SearchSmem)) <= (160u << 10); };
    u32 slots;
    if (few) slots = short_rows && expect > 2000u ? SEARCH_MAX_SLOTS : SEARCH_MAX_SLOTS / 2u;
    else if (expect <= 2400u && all_resident(4096u)) slots = 4096u;
    else if (expect <= 1728u && all_resident(2048u)) slots = 2048u;
    else if ((short_rows || !vec_ok) && expect <= 700u) slots = 1024u;
    else if (short_rows && N <= 262144) slots = 0;
    else slots = expect <= 1728u ? 2048u : 0u;
    const bool q_lds = (size_t)slots * 4 + q_bytes <= SEARCH_MAX_DYN_LDS;
    const EvalShape shape = !q_lds ? (vec_ok ? EVAL_LONG_GLOBAL : EVAL_SINGLE_GLOBAL)
                                   : !vec_ok ? EVAL_SINGLE : rowbytes <= 128 ? EVAL_SHORT : rowbytes <= 512 ? EVAL_MID : EVAL_LONG;
    const size_t dyn_lds = (size_t)slots * 4 + (q_lds ? q_bytes : 0);
    // queries in flight: what the LDS of a CU holds, at most 8 wavefronts per SIMD; one bitmap of N bits each (for queries
    // that outgrow the table), at most 1 GiB of them
    const size_t bitmap_words = (((size_t)N + 31) / 32 + 63) / 64 * 64;
    long long per_cu = (long long)((160u << 10) / (dyn_lds + sizeof(SearchSmem)));
    if (per_cu > (few ? 8 : 32)) per_cu = few ? 8 : 32;
    long long waves = (long long)cu_count() * per_cu;
    const long long by_mem = (long long)((1ull << 30) / (bitmap_words * 4));
    if (waves > by_mem) waves = by_mem;
    if (waves > nq) waves = nq;
    if (waves > SEARCH_MAX_BLOCKS) waves = SEARCH_MAX_BLOCKS;
    if (waves < 1) waves = 1;
    const unsigned blocks = (unsigned)waves;
    const size_t bm_bytes = (size_t)blocks * bitmap_words * 4;
    unsigned long long *counts = nullptr;
    WsLease lease;
    rc = ws_acquire(bm_bytes, false, st, &lease);      // the block kept between calls, like the builds' workspace
    if (rc) return rc;
    rc = counts_acquire(lease, &counts);
    if (rc) {
        ws_release(&lease);
        return rc;
    }
    {
        // (the bitmaps are cleared by the queries that need them)
        u32 *bitmaps = (u32 *)lease.base;
        const SearchLaunch sl = {X, Q, graph, degree, (long long)N, (long long)nq, d, dtype, row_stride, L, K, k, (u64)seed, bitmaps, bitmap_words, slots,
                                 out_ids, out_dist_bits, counts, (unsigned)blocks, (unsigned)dyn_lds, shape, few, st};
        launch_search(sl);
        HIPCHK(hipGetLastError());
        HIPCHK(hipStreamSynchronize(st));
        int64_t sum = 0;
        for (unsigned b = 0; b < blocks; ++b) sum += (int64_t)counts[b];
        if (dist_evals) *dist_evals = sum;
    }
done:
    if (rc == RNND_ERR_HIP || rc == RNND_ERR_OOM) (void)hipStreamSynchronize(st);
    counts_release(lease, counts);
    ws_release(&lease);
    return rc;
}

template <int LPR>
static void launch_probe_gather(const void *X, u32 n_rows, u32 pieces, u64 trips, u64 seed, u32 *sink, int blocks,
                                hipStream_t st)
{
    hipLaunchKernelGGL(k_probe_gather<LPR>, dim3(blocks), dim3(256), 0, st, (const uint4 *)X, n_rows, pieces, trips,
                       seed, sink);
}

template <int LPR>
static void launch_probe_gather_map(int ppl, const void *X, u32 n_rows, u64 trips, u64 seed, u32 *sink, int blocks,
                                    hipStream_t st)
{
    const uint4 *x = (const uint4 *)X;
    if (ppl == 1) hipLaunchKernelGGL((k_probe_gather_map<LPR, 1>), dim3(blocks), dim3(256), 0, st, x, n_rows, trips, seed, sink);
    else if (ppl == 2) hipLaunchKernelGGL((k_probe_gather_map<LPR, 2>), dim3(blocks), dim3(256), 0, st, x, n_rows, trips, seed, sink);
    else if (ppl == 4) hipLaunchKernelGGL((k_probe_gather_map<LPR, 4>), dim3(blocks), dim3(256), 0, st, x, n_rows, trips, seed, sink);
    else hipLaunchKernelGGL((k_probe_gather_map<LPR, 8>), dim3(blocks), dim3(256), 0, st, x, n_rows, trips, seed, sink);
}

// lanes_per_row 0: the probe of the benchmark line (the largest power of two that divides the number of 16-byte
// pieces, at most 8 lanes per row; four rows per lane in flight, any row length); otherwise the map probe
static int probe_gather_impl(const void *X, int64_t n_rows, int64_t row_bytes, int64_t n_gather, int lanes_per_row,
                             uint64_t seed, double *gbytes_per_s, void *stream)
{
    int rc = RNND_OK;
    if (!X || !gbytes_per_s) return RNND_ERR_NULL;
    if (n_rows < 1 || n_rows > 2147483646LL || n_gather < 1) return RNND_ERR_BAD_SHAPE;
    if (row_bytes < 16 || row_bytes % 16 != 0 || row_bytes > (1 << 20) || ((uintptr_t)X & 15) != 0)
        return RNND_ERR_BAD_PARAM;
    hipStream_t st = (hipStream_t)stream;
    const u32 pieces = (u32)(row_bytes / 16);
    int ppl = 0;        // pieces per lane of the map probe
    if (lanes_per_row != 0) {
        if (lanes_per_row != 1 && lanes_per_row != 2 && lanes_per_row != 4 && lanes_per_row != 8) return RNND_ERR_BAD_PARAM;
        if (pieces % (u32)lanes_per_row != 0) return RNND_ERR_BAD_PARAM;
        ppl = (int)(pieces / (u32)lanes_per_row);
        if (ppl != 1 && ppl != 2 && ppl != 4 && ppl != 8) return RNND_ERR_BAD_PARAM;
    }
    const int lpr = lanes_per_row ? lanes_per_row : pieces % 8 == 0 ? 8 : pieces % 4 == 0 ? 4 : pieces % 2 == 0 ? 2 : 1;
    const int rows_per_trip = ppl ? (8 / ppl) * (64 / lpr) : 4 * (64 / lpr);
    const u64 trips = ((u64)n_gather + rows_per_trip - 1) / rows_per_trip;
    const int blocks = persistent_blocks();
    u32 *sink = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    float ms = 0;
    HIPCHK(hipMalloc((void **)&sink, (size_t)blocks * 256 * 4));
    HIPCHK(hipEventCreate(&e0));
    HIPCHK(hipEventCreate(&e1));
    for (int rep = 0; rep < 2; ++rep) {     // the second pass is the one that is timed
        HIPCHK(hipEventRecord(e0, st));
        if (ppl) {
            if (lpr == 8) launch_probe_gather_map<8>(ppl, X, (u32)n_rows, trips, seed + rep, sink, blocks, st);
            else if (lpr == 4) launch_probe_gather_map<4>(ppl, X, (u32)n_rows, trips, seed + rep, sink, blocks, st);
            else if (lpr == 2) launch_probe_gather_map<2>(ppl, X, (u32)n_rows, trips, seed + rep, sink, blocks, st);
            else launch_probe_gather_map<1>(ppl, X, (u32)n_rows, trips, seed + rep, sink, blocks, st);
        } else if (lpr == 8) launch_probe_gather<8>(X, (u32)n_rows, pieces, trips, seed + rep, sink, blocks, st);
        else if (lpr == 4) launch_probe_gather<4>(X, (u32)n_rows, pieces, trips, seed + rep, sink, blocks, st);
        else if (lpr == 2) launch_probe_gather<2>(X, (u32)n_rows, pieces, trips, seed + rep, sink, blocks, st);
        else launch_probe_gather<1>(X, (u32)n_rows, pieces, trips, seed + rep, sink, blocks, st);
        HIPCHK(hipGetLastError());
        HIPCHK(hipEventRecord(e1, st));
        HIPCHK(hipStreamSynchronize(st));
    }
    HIPCHK(hipEventElapsedTime(&ms, e0, e1));
    *gbytes_per_s = ms > 0 ? (double)trips * rows_per_trip * (double)row_bytes / (ms * 1e-3) / 1e9 : 0.0;
done:
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (sink) (void)hipFree(sink);
    return rc;
}

extern "C" int rnnd_probe_gather(const void *X, int64_t n_rows, int64_t row_bytes, int64_t n_gather, uint64_t seed,
                                 double *gbytes_per_s, void *stream)
{
    return probe_gather_impl(X, n_rows, row_bytes, n_gather, 0, seed, gbytes_per_s, stream);
}

extern "C" int rnnd_probe_gather_map(const void *X, int64_t n_rows, int64_t row_bytes, int64_t n_gather,
                                     int lanes_per_row, uint64_t seed, double *gbytes_per_s, void *stream)
{
    if (lanes_per_row == 0) return RNND_ERR_BAD_PARAM;
    return probe_gather_impl(X, n_rows, row_bytes, n_gather, lanes_per_row, seed, gbytes_per_s, stream);
}

// 0: automatic; 1: generic scan for every input; 2: automatic, but the float matrix-core scan runs in
// double precision only (no single-precision first pass)
extern "C" int rnnd_set_kernel_variant(int variant)
{
    if (variant < 0 || variant > 2) return RNND_ERR_BAD_PARAM;
    g_kernel_variant = variant;
    return RNND_OK;
}

extern "C" int rnnd_set_scan_launches(int mode)
{
    if (mode < 0 || mode > 3) return RNND_ERR_BAD_PARAM;
    g_scan_launches = mode;
    return RNND_OK;
}

extern "C" int rnnd_set_event_timing(int on)
{
    g_event_timing = on ? 1 : 0;
    return RNND_OK;
}

extern "C" int rnnd_set_transpose_path(int path)
{
    if (path < 0 || path > 2) return RNND_ERR_BAD_PARAM;
    g_transpose_path = path;
    return RNND_OK;
}

extern "C" const char *rnnd_strerror(int status)
{
    switch (status) {
    case RNND_OK: return "ok";
    case RNND_ERR_NULL: return "a required pointer is NULL";
    case RNND_ERR_BAD_SHAPE: return "bad shape (N < 2, N too large, d < 1, or uint8 d > 33025)";
    case RNND_ERR_BAD_PARAM: return "bad parameter (S, R, T1 or T2 out of range)";
    case RNND_ERR_UNSUPPORTED: return "unsupported dtype or metric";
    case RNND_ERR_OOM: return "out of device memory";
    case RNND_ERR_SCRATCH: return "the workspace for these sizes does not fit the static scratch array (rnnd_build_static)";
    case RNND_ERR_HIP: return g_last_hip_error[0] ? g_last_hip_error : "HIP error";
    default: return "unknown status";
    }
}

extern "C" int rnnd_version(void) { return 200; }
