// Graph search (Alg. 1) with the out-degree cap K of Eq. 4, one wavefront per query.
//
// The candidate list C (at most L <= 128 points, ascending by (delta, id)) lives in registers, one or
// two keys per lane: key = (delta bits << 32) | (id << 1) | unvisited.  One step of the loop:
//   select     first unvisited member u of C (ballot), marked visited;
//   expand     its first min(deg(u), K) neighbours (rows are nearest-first), 64 per pass;
//   visited?   a neighbour already evaluated for this query is skipped (SeenSet);
//   evaluate   delta(q, v) for the rest, 8 lanes per vertex, as many vertices at a time as their rows allow;
//   insert     C <- the L smallest of C and the new points: the new keys are sorted, reversed, and merged
//              into C by a bitonic merge whose upper half is never formed; keys not below C's last one
//              are dropped first when C is full, and the merge is skipped when none is left.
// The loop ends when C holds no unvisited point (the loop's exit).  InitializeCandidates is
// min(L, N) distinct seeded random vertices from the same counter-based generator as RandomGraph,
// keyed by the query index.  Inserting the new points one by one, as the algorithm is written, and
// merging them at once give the same C, because each keeps the L smallest of what has been seen.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include "dist.h"
#include "wave_prims.h"

#define SEARCH_MAX_L 128

// S distinct ids != u in [0, n) from draw(seed, u, j), j = 0, 1, ...: draws are examined 64 at a time; a
// draw is accepted iff its id differs from every earlier draw's id, which is the same set, in the same
// order, as accepting one by one.  ids[] is LDS private to the wavefront (at least S entries).
__device__ __forceinline__ u64 splitmix_finish(u64 z)
{
    z ^= z >> 30; z *= 0xBF58476D1CE4E5B9ull;
    z ^= z >> 27; z *= 0x94D049BB133111EBull;
    z ^= z >> 31;
    return z;
}

// Does `id` equal the value some rotation R in [FIRST, END) of `src` within rows of 16 lanes brings to this lane,
// counting only rotations R <= limit (rotation R brings lane (l - R) mod 16: with limit = l the earlier lanes of the row)?
template <int R, int END>
__device__ __forceinline__ bool rotations_match(int id, int src, int limit)
{
    if constexpr (R >= END) {
        return false;
    } else {
        int o = src;
        if constexpr (R > 0) o = __builtin_amdgcn_update_dpp(0, src, 0x120 + R, 0xF, 0xF, true);      // row_ror:R
        // no short-circuit: every lane must take part in every rotation
        const bool here = (o == id) & (R <= limit);
        const bool rest = rotations_match<R + 1, END>(id, src, limit);
        return here | rest;
    }
}

__device__ __forceinline__ void wave_random_ids(u64 seed, long long n, long long u, int S, int *ids, int lane)
{
    const u64 G = 0x9E3779B97F4A7C15ull;
    const u64 hu = splitmix_finish(seed + G * (u64)(u + 1));
    const u64 jmax = 64ull * (u64)S + 1024ull;
    int cnt = 0;
    for (u64 j0 = 0; j0 < jmax && cnt < S;) {
        // examine the next W draws (a few more than still needed; any W gives the same result)
        const int W = (S - cnt) + 12 < 64 ? (S - cnt) + 12 : 64;
        const u64 j = j0 + lane;
        const u64 z = splitmix_finish(hu + G * (j + 1));
        const u64 c = ((z >> 32) * (u64)(n - 1)) >> 32;
        const int id = (int)(c + (c >= (u64)u ? 1 : 0));
        bool ok = lane < W && j < jmax;
        for (int k = 0; k < cnt; ++k) ok = ok && (ids[k] != id);
        if (W <= 32) {
            // the draws under examination sit in lanes 0 .. 31: every lane meets the other 15 of its row of 16 through
            // row rotations (rotation r brings the id of lane (l - r) mod 16, an earlier lane iff r <= l), and the
            // second row meets the whole first one through its copy swapped across rows
            const int l16 = lane & 15;
            const int x = __builtin_amdgcn_ds_swizzle(id, 0x401F);                              // lane xor 16
            const bool in_row = rotations_match<1, 16>(id, id, l16), in_other = rotations_match<0, 16>(id, x, 16);
            const bool dupe = in_row | (((lane & 16) != 0) & in_other);
            ok = ok && !dupe;
        } else {
            for (int l = 0; l < W - 1; ++l) {   // l is the same for the whole wavefront: a scalar read of lane l
                const int o = __builtin_amdgcn_readlane(id, l);
                if (l < lane && o == id) ok = false;
            }
        }
        const u64 m = __builtin_amdgcn_ballot_w64(ok);
        const int pos = cnt + __popcll(m & lanes_below(lane));
        if (ok && pos < S) ids[pos] = id;
        cnt += __popcll(m);
        if (cnt > S) cnt = S;
        j0 += W;
        wave_sync();
    }
    if (cnt < S) {   // fallback, practically unreachable: smallest unused ids
        for (long long id = 0; id < n && cnt < S; ++id) {
            if (id == u) continue;
            bool dup = false;
            for (int k = 0; k < cnt; ++k) dup = dup || (ids[k] == (int)id);
            if (!dup) {
                if (lane == 0) ids[cnt] = (int)id;
                ++cnt;
                wave_sync();
            }
        }
    }
}

struct SearchSmem {
    int id[SEARCH_MAX_L];      // vertices to evaluate
    u32 dist[SEARCH_MAX_L];    // their delta(q, .) bits
    int todo;                  // how many of them there are (0: the query is done)
    int pad[3];
};

// Where a query's coordinates come from.  QueryRaw: as they lie in memory.  QueryDouble (float and 16-bit rows): already
// converted, in LDS, which takes a quarter of the arithmetic out of every distance.
template <int DT> struct EvalAcc { typedef double type; };
template <> struct EvalAcc<DT_U8> { typedef int type; };

template <int DT>
__device__ __forceinline__ double coord_of_piece(const uint4 &x, int t)     // coordinate t of a 16-byte piece of a float or 16-bit row
{
    if constexpr (DT == DT_F32) {
        return (double)__uint_as_float(t == 0 ? x.x : t == 1 ? x.y : t == 2 ? x.z : x.w);
    } else {
        const u32 w = (t >> 1) == 0 ? x.x : (t >> 1) == 1 ? x.y : (t >> 1) == 2 ? x.z : x.w;
        return (double)coord16_to_float<DT>((unsigned short)(w >> (16 * (t & 1))));
    }
}
template <int DT> struct PieceCoords { static constexpr int n = DT == DT_F32 ? 4 : DT == DT_U8 ? 16 : 8; };

struct QueryRaw { const void *q; };
struct QueryDouble { const double *q; };

// One 16-byte piece of a row, and the same piece of the query, into a distance: the arithmetic and the order of
// group8_dist_bits (the sign of a difference does not matter to its square).
template <int DT>
__device__ __forceinline__ void add_piece(typename EvalAcc<DT>::type &acc, const uint4 &a, const uint4 &b)
{
    if constexpr (DT == DT_U8) {
        acc = sqdiff_piece_u8(a, b, acc);
    } else {
#pragma unroll
        for (int i = 0; i < PieceCoords<DT>::n; ++i) {
            const double t = coord_of_piece<DT>(a, i) - coord_of_piece<DT>(b, i);
            acc = fma(t, t, acc);
        }
    }
}
template <int DT, int RB>
__device__ __forceinline__ void add_pieces(typename EvalAcc<DT>::type (&acc)[RB], const uint4 (&v)[RB], QueryRaw q, int c)
{
    const uint4 vq = ((const uint4 *)q.q)[c];
#pragma unroll
    for (int j = 0; j < RB; ++j) add_piece<DT>(acc[j], v[j], vq);
}
template <int DT, int RB>
__device__ __forceinline__ void add_pieces(typename EvalAcc<DT>::type (&acc)[RB], const uint4 (&v)[RB], QueryDouble q, int c)
{
    constexpr int V = PieceCoords<DT>::n;
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const double b = q.q[V * c + i];
#pragma unroll
        for (int j = 0; j < RB; ++j) {
            const double t = coord_of_piece<DT>(v[j], i) - b;
            acc[j] = fma(t, t, acc[j]);
        }
    }
}
// (in the first four lanes of a group)
__device__ __forceinline__ u32 eval_bits(int acc) { return (u32)group8_sum_low(acc); }
__device__ __forceinline__ u32 eval_bits(double acc) { return __float_as_uint((float)group8_sum_low(acc)); }

// UF pieces per lane, from piece c0 on, of RB rows.  The loads are unconditional (a lane past the end of the row reads
// its last piece and drops the outcome): a branch around each would make the wavefront wait for one load after the other.
template <int DT, int RB, int UF, typename QUERY>
__device__ __forceinline__ void eval_pieces(const uint4 *const (&row)[RB], QUERY q, int npiece, int c0, int sub,
                                            typename EvalAcc<DT>::type (&acc)[RB])
{
    uint4 v[UF][RB];
#pragma unroll
    for (int k = 0; k < UF; ++k) {
        const int c = c0 + 8 * k + sub, cc = c < npiece ? c : npiece - 1;
#pragma unroll
        for (int j = 0; j < RB; ++j) v[k][j] = row[j][cc];
    }
#pragma unroll
    for (int k = 0; k < UF; ++k) {
        const int c = c0 + 8 * k + sub, cc = c < npiece ? c : npiece - 1;
        typename EvalAcc<DT>::type next[RB];
#pragma unroll
        for (int j = 0; j < RB; ++j) next[j] = acc[j];
        add_pieces<DT, RB>(next, v[k], q, cc);
#pragma unroll
        for (int j = 0; j < RB; ++j) acc[j] = c < npiece ? next[j] : acc[j];
    }
}

// delta(q, ids[b .. b + 8 RB)) -> dist: 8 lanes per vertex, RB vertices per 8-lane group, up to UF pieces per lane of each
// in flight together.  A search waits for its dependent trips to memory, so what counts is how few there are.
template <int DT, int RB, int UF, typename QUERY>
__device__ __forceinline__ void eval_rows(const void *X, QUERY q, int npiece, size_t rowbytes, SearchSmem &sm, int b, int cnt, int lane)
{
    const int sub = lane & 7, grp = lane >> 3;
    const uint4 *row[RB];
    typename EvalAcc<DT>::type acc[RB];
#pragma unroll
    for (int j = 0; j < RB; ++j) {
        const int p = b + 8 * j + grp;
        row[j] = (const uint4 *)((const char *)X + (size_t)sm.id[p < cnt ? p : cnt - 1] * rowbytes);
        acc[j] = 0;
    }
    for (int c0 = 0; c0 < npiece;) {
        const int left = (npiece - c0 + 7) / 8;
        if (UF >= 16 && left > 8) {
            eval_pieces<DT, RB, UF>(row, q, npiece, c0, sub, acc);
            c0 += 8 * UF;
        } else if (UF >= 8 && left > 4) {
            eval_pieces<DT, RB, (UF >= 8 ? 8 : UF)>(row, q, npiece, c0, sub, acc);
            c0 += 64;
        } else if (UF >= 4 && left > 3) {
            eval_pieces<DT, RB, (UF >= 4 ? 4 : UF)>(row, q, npiece, c0, sub, acc);
            c0 += 32;
        } else {
            eval_pieces<DT, RB, (UF >= 4 ? 3 : UF)>(row, q, npiece, c0, sub, acc);
            c0 += 8 * (UF >= 4 ? 3 : UF);
        }
    }
#pragma unroll
    for (int j = 0; j < RB; ++j) {
        const u32 bits = eval_bits(acc[j]);
        const int p = b + 8 * j + grp;
        if (p < cnt && sub == 0) sm.dist[p] = bits;
    }
}

// The same for rows that cannot be read in 16-byte pieces: lane s of 8 takes coordinates s, s + 8, ...
template <int DT, int RB, int UF, typename QUERY>
__device__ __forceinline__ void eval_rows_single(const void *X, QUERY qs, int d, SearchSmem &sm, int b, int cnt, int lane)
{
    typedef typename std::conditional<DT == DT_U8, uint8_t, typename std::conditional<DT == DT_F32, float, unsigned short>::type>::type T;
    constexpr bool ready = std::is_same<QUERY, QueryDouble>::value;
    const int sub = lane & 7, grp = lane >> 3;
    const T *row[RB];
    typename EvalAcc<DT>::type acc[RB];
    auto widen = [](T x) -> double {
        if constexpr (DT == DT_F32) return (double)x;
        else if constexpr (DT == DT_U8) return 0.0;
        else return (double)coord16_to_float<DT>(x);
    };
#pragma unroll
    for (int j = 0; j < RB; ++j) {
        const int p = b + 8 * j + grp;
        row[j] = (const T *)X + (size_t)sm.id[p < cnt ? p : cnt - 1] * (size_t)d;
        acc[j] = 0;
    }
    for (int c0 = 0; c0 < d; c0 += 8 * UF) {
        T v[RB][UF], vq[UF];
#pragma unroll
        for (int k = 0; k < UF; ++k) {
            const int c = c0 + 8 * k + sub, cc = c < d ? c : d - 1;
            if constexpr (!ready) vq[k] = ((const T *)qs.q)[cc];
#pragma unroll
            for (int j = 0; j < RB; ++j) v[j][k] = row[j][cc];
        }
#pragma unroll
        for (int k = 0; k < UF; ++k) {
            if (c0 + 8 * k >= d) break;     // wave-uniform
            const int c = c0 + 8 * k + sub, cc = c < d ? c : d - 1;
            if constexpr (DT == DT_U8) {
#pragma unroll
                for (int j = 0; j < RB; ++j) {
                    const int t = (int)v[j][k] - (int)vq[k];
                    acc[j] += c < d ? t * t : 0;
                }
            } else {
                double b64;
                if constexpr (ready) b64 = qs.q[cc];
                else b64 = widen(vq[k]);
#pragma unroll
                for (int j = 0; j < RB; ++j) {
                    const double t = widen(v[j][k]) - b64;
                    const double next = fma(t, t, acc[j]);
                    acc[j] = c < d ? next : acc[j];
                }
            }
        }
    }
#pragma unroll
    for (int j = 0; j < RB; ++j) {
        const u32 bits = eval_bits(acc[j]);
        const int p = b + 8 * j + grp;
        if (p < cnt && sub == 0) sm.dist[p] = bits;
    }
}

// How many vertices and pieces travel together follows from the row length, which also decides how many registers the
// search needs, so each shape is a kernel of its own:
//   EVAL_SHORT   rows of up to 128 bytes: one piece per lane, 32 vertices at a time
//   EVAL_MID     up to 512 bytes: up to four pieces per lane
//   EVAL_LONG    longer: 16 pieces in flight per lane
//   EVAL_SINGLE  rows that cannot be read in 16-byte pieces
// and the last two with a query too long for LDS (float and 16-bit rows only)
enum EvalShape { EVAL_SHORT = 0, EVAL_MID, EVAL_LONG, EVAL_SINGLE, EVAL_LONG_GLOBAL, EVAL_SINGLE_GLOBAL };
#define SEARCH_MAX_DYN_LDS (60u << 10)      // table and query; with SearchSmem below the 64 KB a launch may ask for without more ado
#define SEARCH_MAX_SLOTS 8192u              // of the table: alone; 4,096 for rows of more than 128 bytes
static_assert(SEARCH_MAX_SLOTS * 4u + 128u * 8u <= SEARCH_MAX_DYN_LDS && SEARCH_MAX_SLOTS / 2u * 4u + 256u * 8u <= SEARCH_MAX_DYN_LDS,
              "queries of up to 128 bytes (128 doubles), and of up to 512 (256), always lie in LDS");
static_assert(SEARCH_MAX_SLOTS / 2u * 4u + 33040u <= SEARCH_MAX_DYN_LDS, "uint8 queries (d <= 33025) always do");

// delta(q, ids[first .. cnt)) -> dist, the part of wavefront `wave` of a team of TEAM: eight vertices at a time each, or
// (alone) as many as there are, so that no lane works on vertices that are not there.
template <int DT, int SHAPE, int TEAM, typename QUERY>
__device__ __forceinline__ void eval_all(const void *X, QUERY q, int d, int npiece, size_t rowbytes, SearchSmem &sm, int cnt, int lane, int wave)
{
    if constexpr (TEAM > 1) {
        for (int b = 8 * wave; b < cnt; b += 8 * TEAM) {
            if constexpr (SHAPE == EVAL_MID) eval_rows<DT, 1, 4>(X, q, npiece, rowbytes, sm, b, cnt, lane);
            else if constexpr (SHAPE == EVAL_LONG) eval_rows<DT, 1, 16>(X, q, npiece, rowbytes, sm, b, cnt, lane);
            else eval_rows_single<DT, 1, 16>(X, q, d, sm, b, cnt, lane);
        }
    } else if constexpr (SHAPE == EVAL_MID) {
        for (int b = 0; b < cnt;) {
            if (cnt - b <= 8) { eval_rows<DT, 1, 4>(X, q, npiece, rowbytes, sm, b, cnt, lane); b += 8; }
            else { eval_rows<DT, 2, 4>(X, q, npiece, rowbytes, sm, b, cnt, lane); b += 16; }
        }
    } else if constexpr (SHAPE == EVAL_LONG) {
        for (int b = 0; b < cnt;) {
            if (cnt - b <= 8) { eval_rows<DT, 1, 16>(X, q, npiece, rowbytes, sm, b, cnt, lane); b += 8; }
            else { eval_rows<DT, 2, 8>(X, q, npiece, rowbytes, sm, b, cnt, lane); b += 16; }
        }
    } else {
        for (int b = 0; b < cnt;) {
            if (cnt - b <= 8) { eval_rows_single<DT, 1, 16>(X, q, d, sm, b, cnt, lane); b += 8; }
            else { eval_rows_single<DT, 2, 16>(X, q, d, sm, b, cnt, lane); b += 16; }
        }
    }
}

// The same with the query in global memory, 8 vertices at a time for long rows (RandomGraph: every wavefront has a
// vertex of its own and the chip is full, so fewer registers count for more than fewer trips).
template <int DT>
__device__ __forceinline__ void search_eval(const void *X, const void *qv, int d, int vec_ok, size_t rowbytes,
                                            SearchSmem &sm, int cnt, int lane)
{
    const int sub = lane & 7, grp = lane >> 3;
    if (DT == DT_U8 && vec_ok && d <= 128) {
        for (int b = 0; b < cnt; b += 32) eval_rows<DT, 4, 1>(X, QueryRaw{qv}, d >> 4, rowbytes, sm, b, cnt, lane);
        return;
    }
    for (int b = 0; b < cnt; b += 8) {
        const int p = b + grp;
        const int id = sm.id[p < cnt ? p : cnt - 1];
        const u32 db = group8_dist_bits<DT>(qv, (const char *)X + (size_t)id * rowbytes, d, vec_ok, sub);
        if (p < cnt && sub == 0) sm.dist[p] = db;
    }
}

// C (E registers, ascending, KEY_PAD past its end) <- the 64 E smallest of C and the sorted-ascending
// register kn.  Bitonic merge: against the reversed kn, the element-wise minima are exactly the
// smallest keys and form a bitonic sequence, which strides 64 E / 2 ... 1 then sort.
template <int E>
__device__ __forceinline__ void merge_into_candidates(u64 (&C)[E], u64 kn, int lane)
{
    const u64 rev = shfl_u64(kn, 63 - lane);     // descending
    u64 &top = C[E - 1];
    top = top < rev ? top : rev;
    if (E == 2) {
        const u64 a = C[0], b = C[1];
        C[0] = a < b ? a : b;
        C[1] = a < b ? b : a;
    }
#pragma unroll
    for (int r = 0; r < E; ++r) merge_ascending<32>(C[r]);
}

__device__ __forceinline__ u64 read_lane_u64(u64 v, int src)      // src the same in every lane
{
    const u32 lo = (u32)__builtin_amdgcn_readlane((int)(u32)v, src), hi = (u32)__builtin_amdgcn_readlane((int)(u32)(v >> 32), src);
    return ((u64)hi << 32) | lo;
}
// the vertex in place i (the same in every lane) of the candidate list
template <int E>
__device__ __forceinline__ int member_id(const u64 (&C)[E], int i)
{
    const u32 w = (u32)(E == 2 && i >= 64 ? C[E - 1] : C[0]);
    return (int)key_id((u64)(u32)__builtin_amdgcn_readlane((int)w, i & 63));
}

// The vertices a query has evaluated: an open-addressed table of `slots` ids in LDS (double hashing: the step is odd, so
// it visits every slot).  Membership was a bit per vertex in global memory before: one device-scope atomic per
// neighbour, a trip to memory in every step of the loop, and N bits to clear per query.  A table seven eighths full takes
// no more; what comes after goes to the wavefront's bitmap in global memory, which is cleared only then.
#define SEEN_EMPTY 0xFFFFFFFFu
struct SeenSet {
    u32 *tab;
    u32 slots, count, limit;
    u32 *bitmap;
    size_t bitmap_words;

    __device__ __forceinline__ void clear_bitmap(int lane)
    {
        for (size_t w4 = (size_t)lane * 4; w4 < bitmap_words; w4 += 256) *(uint4 *)(bitmap + w4) = make_uint4(0u, 0u, 0u, 0u);
    }
    __device__ __forceinline__ void clear(int lane)
    {
        if (slots == 0) {       // no table at all
            clear_bitmap(lane);
            count = 1, limit = 0;
            return;
        }
        for (u32 i = 4u * (u32)lane; i < slots; i += 256u) *(uint4 *)(tab + i) = make_uint4(SEEN_EMPTY, SEEN_EMPTY, SEEN_EMPTY, SEEN_EMPTY);
        count = 0;
    }
    // true for one lane of those that hold a vertex v (want) nobody held before
    __device__ __forceinline__ bool add(int v, bool want, int lane)
    {
        const u32 h = (u32)v * 0x9E3779B1u, step = ((u32)v * 0x85EBCA6Bu >> 7) | 1u;
        u32 at = (h >> 8) & (slots - 1u);
        bool fresh = false, open = want;
        if (count <= limit) {
            while (__builtin_amdgcn_ballot_w64(open)) {      // a free slot exists: at most limit + 64 are taken
                if (open) {
                    const u32 old = atomicCAS(&tab[at], SEEN_EMPTY, (u32)v);
                    fresh = old == SEEN_EMPTY;
                    open = old != SEEN_EMPTY && old != (u32)v;
                    at = (at + step) & (slots - 1u);
                }
            }
            count += (u32)__popcll(__builtin_amdgcn_ballot_w64(fresh));
            if (count > limit) {      // from now on the bitmap takes what is new
                clear_bitmap(lane);
                __threadfence();
            }
            return fresh;
        }
        bool in_table = false;
        while (slots && __builtin_amdgcn_ballot_w64(open)) {
            if (open) {
                const u32 old = tab[at];
                in_table = old == (u32)v;
                open = old != SEEN_EMPTY && !in_table;
                at = (at + step) & (slots - 1u);
            }
        }
        if (want && !in_table) {
            const u32 bit = 1u << (v & 31);
            fresh = (atomicOr(&bitmap[v >> 5], bit) & bit) == 0u;
        }
        return fresh;
    }
};

// A block is a query: one wavefront, or (TEAM > 1, where there are fewer queries than the chip has room for) a team of
// which the first wavefront searches and all evaluate, eight vertices each.  Dynamic LDS: the seen table, then the query,
// as doubles where its coordinates are floats.  evals: one count per block, in host memory (a counter on the device would
// have to be cleared before and copied after: two more trips for a call that may take 100 us).  Every phase stands in the loop once: a lone wavefront pays about five
// cycles per instruction, and fetches the code of a second copy anew.
template <int DT, int E, int SHAPE_, int TEAM>
__global__ __launch_bounds__(64 * TEAM, 4) void k_search(const void *X, long long N, int d,
                                                      const int *graph, const int *degree, int W, const void *Q,
                                                      long long nq, int L, int K, int k, u64 seed, u32 *bitmaps,
                                                      size_t bitmap_words, u32 slots, int *out_ids, u32 *out_dist,
                                                      unsigned long long *evals)
{
    constexpr bool in_lds = SHAPE_ < EVAL_LONG_GLOBAL;
    constexpr int SHAPE = SHAPE_ == EVAL_LONG_GLOBAL ? EVAL_LONG : SHAPE_ == EVAL_SINGLE_GLOBAL ? EVAL_SINGLE : SHAPE_;
    static_assert(SHAPE != EVAL_SHORT || TEAM == 1, "short rows are evaluated by the searching wavefront itself");
    constexpr bool AT_ONCE = SHAPE == EVAL_SHORT;      // neighbours are evaluated before the table has answered
    extern __shared__ uint4 s_dyn[];
    __shared__ SearchSmem sm;
    const int lane = threadIdx.x & 63, wave = TEAM > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
    const long long gw = blockIdx.x, nw = gridDim.x;
    SeenSet seen;
    seen.tab = (u32 *)s_dyn;
    seen.slots = slots;
    seen.limit = slots - slots / 8u - 64u;
    seen.count = 0;
    seen.bitmap = bitmaps + (size_t)gw * bitmap_words;
    seen.bitmap_words = bitmap_words;
    uint4 *sq = s_dyn + slots / 4u;
    const size_t rowbytes = (size_t)d * dt_size(DT);
    const int npiece = (int)(rowbytes / 16u);
    const int L0 = (long long)L < N ? L : (int)N;
    unsigned long long ev = 0;
    for (long long q = gw; q < nq; q += nw) {
        const void *qv = (const char *)Q + (size_t)q * rowbytes;
        u64 C[E];
#pragma unroll
        for (int r = 0; r < E; ++r) C[r] = KEY_PAD;
        int m = 0;                          // members of C
        int at0 = 0, left = 0;              // InitializeCandidates: the start vertices sm.id[at0 .. at0 + left) wait for their turn
        int u = 0, v0 = -1, du = 0, t0 = 0;     // the vertex being expanded, the first 64 entries of its row, its degree, entries done
        int pf_u = -1, pf_v = -1, pf_d = 0;     // a row of the graph asked for while the one before it is still being expanded
        if (wave == 0) {
            wave_sync();
            // ---- nothing has been evaluated for this query yet
            seen.clear(lane);
            if constexpr (in_lds) {
                if constexpr (DT == DT_U8) {
                    for (int c = lane; c < d; c += 64) ((uint8_t *)sq)[c] = ((const uint8_t *)qv)[c];
                } else if constexpr (DT == DT_F32) {
                    for (int c = lane; c < d; c += 64) ((double *)sq)[c] = (double)((const float *)qv)[c];
                } else {
                    for (int c = lane; c < d; c += 64) ((double *)sq)[c] = (double)coord16_to_float<DT>(((const unsigned short *)qv)[c]);
                }
            }
            // ---- InitializeCandidates
            if ((long long)L0 == N) {
                for (int t = lane; t < L0; t += 64) sm.id[t] = t;
            } else {
                wave_random_ids(seed + 0x9E3779B97F4A7C15ull * (u64)q, N + 1, N, L0, sm.id, lane);
            }
            wave_sync();
            left = L0;
        }
        for (;;) {
            int nf = 0;       // vertices to evaluate, in sm.id[0 .. nf)
            int span = 0;     // the new keys sit in lanes 0 .. span - 1
            u64 kn = KEY_PAD;
            if (wave == 0) {
                do {
                    int v = -1;
                    if (left > 0) {
                        const int n = left < 64 ? left : 64;
                        if (lane < n) v = sm.id[at0 + lane];
                        at0 += n;
                        left -= n;
                    } else {
                        if (t0 >= du) {
                            // select: the first unvisited member of C, and the one after it
                            int iu = -1, in = -1;
#pragma unroll
                            for (int r = E - 1; r >= 0; --r) {
                                const u64 b = __builtin_amdgcn_ballot_w64(64 * r + lane < m && (C[r] & 1ull));
                                if (b) {
                                    const u64 rest = b & (b - 1ull);
                                    in = rest ? 64 * r + (int)__builtin_ctzll(rest) : iu;
                                    iu = 64 * r + (int)__builtin_ctzll(b);
                                }
                            }
                            if (iu < 0) break;
                            u = member_id<E>(C, iu);
#pragma unroll
                            for (int r = 0; r < E; ++r)
                                if (64 * r + lane == iu) C[r] &= ~1ull;
                            v0 = pf_v;
                            du = pf_d;
                            if (u != pf_u) {
                                // the first 64 entries of u's row are read without waiting for its degree (rows are W wide)
                                v0 = -1;
                                if (lane < W && lane < K) v0 = graph[(size_t)u * W + lane];
                                du = degree[u];
                            }
                            pf_u = -1;
                            if (in >= 0) {      // next, unless this expansion finds something nearer
                                pf_u = member_id<E>(C, in);
                                pf_v = -1;
                                if (lane < W && lane < K) pf_v = graph[(size_t)pf_u * W + lane];
                                pf_d = degree[pf_u];
                            }
                            if (du > K) du = K;     // Eq. 4: rows are nearest-first
                            if (du > W) du = W;
                            t0 = 0;
                            if (du <= 0) continue;     // (nf is 0: the next vertex)
                        }
                        // expand
                        const int t = t0 + lane;
                        if (t < du) v = t0 == 0 ? v0 : graph[(size_t)u * W + t];
                        t0 += 64;
                    }
                    // what was evaluated before is skipped; what is not a vertex is ignored
                    const bool isv = v >= 0 && (long long)v < N;
                    if constexpr (AT_ONCE) {
                        // short rows cost less to read than to wait for: all neighbours are evaluated, the loads of the
                        // first 32 travel while the table answers which of them are new
                        const int sub = lane & 7, grp = lane >> 3, piece = sub < npiece ? sub : npiece - 1;
                        const u64 any = __builtin_amdgcn_ballot_w64(isv);
                        span = any ? 64 - (int)__builtin_clzll(any) : 0;
                        const int vid = isv ? v : 0;
                        uint4 x[4];
                        auto fetch = [&](int b) __attribute__((always_inline)) {
#pragma unroll
                            for (int j = 0; j < 4; ++j)
                                x[j] = ((const uint4 *)((const char *)X + (size_t)__shfl(vid, (b + 8 * j + grp) & 63) * rowbytes))[piece];
                        };
                        auto distances = [&](int b) __attribute__((always_inline)) {
#pragma unroll
                            for (int j = 0; j < 4; ++j) {
                                typename EvalAcc<DT>::type acc[1] = {0};
                                const uint4 xj[1] = {x[j]};
                                if constexpr (DT == DT_U8) add_pieces<DT, 1>(acc, xj, QueryRaw{sq}, piece);
                                else add_pieces<DT, 1>(acc, xj, QueryDouble{(const double *)sq}, piece);
                                if (sub >= npiece) acc[0] = 0;
                                const u32 bits = eval_bits(acc[0]);
                                if (sub == 0) sm.dist[b + 8 * j + grp] = bits;
                            }
                        };
                        fetch(0);
                        const bool fresh = seen.add(v, isv, lane);
                        nf = __popcll(__builtin_amdgcn_ballot_w64(fresh));
                        if (nf == 0) continue;
                        wave_sync();
                        distances(0);
                        if (span > 32) {
                            fetch(32);
                            distances(32);
                        }
                        wave_sync();
                        if (fresh) kn = make_key(sm.dist[lane], (u32)v, 1u);
                    } else {
                        const bool fresh = seen.add(v, isv, lane);
                        const u64 fm = __builtin_amdgcn_ballot_w64(fresh);
                        nf = __popcll(fm);
                        wave_sync();
                        if (fresh) sm.id[__popcll(fm & lanes_below(lane))] = v;
                    }
                } while (nf == 0);
            }
            // ---- evaluate
            if (TEAM > 1) {
                if (threadIdx.x == 0) sm.todo = nf;
                __syncthreads();
                nf = sm.todo;
            }
            if (nf == 0) break;
            if constexpr (!AT_ONCE) {
                wave_sync();
                if constexpr (!in_lds) eval_all<DT, SHAPE, TEAM>(X, QueryRaw{qv}, d, npiece, rowbytes, sm, nf, lane, wave);
                else if constexpr (DT == DT_U8) eval_all<DT, SHAPE, TEAM>(X, QueryRaw{sq}, d, npiece, rowbytes, sm, nf, lane, wave);
                else eval_all<DT, SHAPE, TEAM>(X, QueryDouble{(const double *)sq}, d, npiece, rowbytes, sm, nf, lane, wave);
                if (TEAM > 1) __syncthreads();
                else wave_sync();
                if (wave > 0) continue;
                if (lane < nf) kn = make_key(sm.dist[lane], (u32)sm.id[lane], 1u);
                span = nf;
            }
            // ---- insert
            ev += (unsigned long long)nf;
            if (m == L) {
                const u64 last = E == 2 && L > 64 ? read_lane_u64(C[E - 1], L - 65) : read_lane_u64(C[0], L - 1);
                if ((kn >> 1) >= (last >> 1)) kn = KEY_PAD;
            }
            const int na = __popcll(__builtin_amdgcn_ballot_w64(kn != KEY_PAD));
            if (na == 0) continue;
            // a group of lanes without a new key has nothing to sort
            if (span <= 16) kn = group_sort<16>(kn);
            else if (span <= 32) kn = group_sort<32>(kn);
            else kn = group_sort<64>(kn);
            merge_into_candidates<E>(C, kn, lane);
            m = m + na < L ? m + na : L;
            // the registers hold 64 E keys; C is its first L
#pragma unroll
            for (int r = 0; r < E; ++r)
                if (64 * r + lane >= m) C[r] = KEY_PAD;
        }
        // ---- output: the k nearest members of C
        if (wave == 0) {
#pragma unroll
            for (int r = 0; r < E; ++r) {
                const int t = 64 * r + lane;
                if (t < k) {
                    out_ids[(size_t)q * k + t] = t < m ? (int)key_id(C[r]) : -1;
                    if (out_dist) out_dist[(size_t)q * k + t] = t < m ? key_dist(C[r]) : 0xFFFFFFFFu;
                }
            }
        }
        if (TEAM > 1) __syncthreads();      // the team has seen the end of this query
    }
    if (threadIdx.x == 0) evals[blockIdx.x] = ev;
}
