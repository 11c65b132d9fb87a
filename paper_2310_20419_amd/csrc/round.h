// What the kernels of a round share: the counters, the clock marks, the record of a redirected edge.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "wave_prims.h"

#define NDEG 8   // degree classes of the active lists (see degree_class)
#define NMRG 4   // merge classes of the touched lists: kept + received at most 16, 32, 64, more

// Per-round device counters.  Round t reads ctr[t].n_active[] and fills the rest; its compact step
// writes ctr[t+1].n_active[].  Zeroed once per call, never reset, so they double as statistics.
#define STAT_SLOTS 64
struct RoundCtr {
    u32 n_active[NDEG];   // lengths of this round's active lists
    u32 groups;           // float scan: this round (or run) takes groups of 16 rows instead of tiles (see group_form)
    u32 sample_pairs, sample_open;      // float scan, first round: pairs of a sample of the lists, and those the tiles would leave open
    u32 n_open;           // float scan by tiles: pairs left to the exact distance, by a sample of the wavefronts
    u32 n_touched[NMRG];  // distinct targets of the redirected edges, by size of the merge they need
    u32 nonfinite;        // slot 0: k_prepare_rows met a coordinate that is NaN or infinite
    u32 n_redo;           // float scan: vertices the first form leaves to another launch (the double-precision form; R > 96: lists
                          // of more than 96 entries, the pair-at-a-time kernel)
    u32 pad[2];
    // ticks of the device's constant-rate clock (0 = not taken): the round's first scan launch starts, the launch after
    // its scans starts (= they have ended: launches of one stream run back to back), the round's last kernel has ended
    // (taken by k_stamp after the last round before an AddReverseEdges call or the export, only where statistics
    // ask for it; every other round, and an AddReverseEdges call, ends where the next round's scan starts)
    u64 t_scan_start, t_scan_stop, t_round_stop;
    // statistics, spread over STAT_SLOTS addresses so that the adds of many blocks do not queue up
    // on one: [slot][0..4] = algorithmic evals, executed evals, rows gathered, edges redirected, entries a merge
    // dropped because the list was full
    u64 stat[STAT_SLOTS][5];
};

// One add per wavefront into the slot of its block.
__device__ __forceinline__ void add_round_stats(RoundCtr *ctr, u64 algo, u64 exec, u64 rows, u64 props)
{
    u64 *s = ctr->stat[blockIdx.x & (STAT_SLOTS - 1)];
    atomicAdd(&s[0], algo);
    atomicAdd(&s[1], exec);
    atomicAdd(&s[2], rows);
    atomicAdd(&s[3], props);
}

// Statistics take the scan time of a round from the device's own clock instead of events attached to the launches:
// an event costs 4-7 microseconds of idle queue after its kernel, three per round used to add 1 ms to a 27 ms build.
__device__ __forceinline__ void stamp_scan_start(RoundCtr *ctr)
{   // the first scan launch of a round that comes by fills the field (the clock is read before the field is, which takes a microsecond)
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
        const u64 now = wall_clock64();
        if (ctr->t_scan_start == 0ull) ctr->t_scan_start = now;
    }
}
__device__ __forceinline__ void stamp_scan_stop(RoundCtr *ctr)
{
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) ctr->t_scan_stop = wall_clock64();
}

// Whether a float scan takes its lists in groups of 16 rows, by scan_mfma_f32.h, instead of tiles of 32 on the 16-bit matrix cores: float32
// rows whole and in single precision, 16-bit rows under the narrower error bound of that form.  Where clusters are tight next to the
// distances between them, rows differ in size by orders of magnitude, or 16-bit rows lie far from the origin, the tiles leave most
// pairs to the exact distance.  So once a round has left more than GROUP_OPEN per active vertex (0.3 on the average, 1.1 at most in the
// builds of this repository's float workloads), the following ones take the other form (block-sequential passes: the following runs).
// A round decides this only if it has `enough` active vertices: below, the sample is not one (a few lists lie in wavefronts that are all
// sampled, or none), and the last rounds before an AddReverseEdges call, of a handful of vertices, say nothing about
// the rounds after it.  The launch after the scan decides (the scatter or, where the scan has scattered, the merge: end_scan), so that the scan, whose first loads
// everything waits for, has none more.
// The first round of a call has none before it; it takes groups if more than a GROUP_SHARE-th of the pairs of a sample of its lists
// (k_float_sample) lie within the tiles' tolerance.
#define OPEN_SAMPLE 32u
#define GROUP_OPEN 6u
#define GROUP_SHARE 12u
#define SAMPLE_MIN_PAIRS 256u
__device__ __forceinline__ void decide_next_form(RoundCtr *ctr, u32 active, u32 enough)
{
    if (ctr->groups != 0u || (active >= enough && (u64)ctr->n_open * OPEN_SAMPLE > (u64)GROUP_OPEN * active)) ctr[1].groups = 1u;
}
__device__ __forceinline__ bool group_form(RoundCtr *ctr)
{
    // (loaded next to the lists' lengths, before the kernel's first store: a trip to memory more costs 2 us in each block, 7 % of a scan of
    // lists of up to 32 entries at 120,000 x 96)
    const u32 was = ctr->groups, pairs = ctr->sample_pairs, open = ctr->sample_open;
    const bool on = (was != 0u) | ((pairs >= SAMPLE_MIN_PAIRS) & (open * GROUP_SHARE > pairs));
    if (on && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) ctr->groups = 1u;
    return on;
}

struct Prop {          // one redirected edge (Alg. 4, the edge update): `key` enters `tgt`'s list
    u64 key;
    u32 tgt;
    u32 next;          // set by whoever scatters, for edges past the inbox: the edge (its place in props) that was on tgt's list before
};

// A key whose distance is still to be computed (by the merge, see close_keys): these bits in place of the distance.  A NaN can
// have them too; computing it once more gives the same bits.
#define OPEN_DIST 0xFFFFFFFFu
#define INFINITE_DIST 0x7F800000u     // float rows: greater bits are a NaN's

// The edge update of Alg. 4: (w, v) enters E.  Recorded in the scanning vertex's own slot.
__device__ __forceinline__ void emit_redirect(u64 key, u32 tgt, Prop *slot)
{
    Prop pr;
    pr.key = key;
    pr.tgt = tgt;
    pr.next = 0;
    *slot = pr;
}
