// Host side of the launches: grid sizes, and the float scans' entry points (scan_float.hip, scan_f32.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include "half_rows.h"
#include "round.h"
#include "scatter.h"

static inline int cu_count()
{
    static int cus = 0;
    if (!cus) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
            cus = 256;
    }
    return cus;
}

static inline int persistent_blocks() { return cu_count() * 8; }   // 32 wavefronts per CU

// A grid that walks a list of at most N vertices, one or more per wavefront of a 4-wavefront block, needs no more
// than N / 4 blocks: small inputs get small grids (a launch costs by its workgroups even when they find no work).
static inline unsigned capped(long long blocks, long long N)
{
    const long long need = (N + 3) / 4;
    return (unsigned)(blocks < need ? blocks : (need < 1 ? 1 : need));
}

// Blocks of `kernel` (256 threads, static LDS only) that one CU keeps resident; the persistent
// scans launch exactly that many per CU so that every wavefront starts at once.
template <typename K>
static int resident_blocks_per_cu(K kernel, int fallback)
{
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, 256, 0) != hipSuccess || nb < 1) {
        (void)hipGetLastError();
        nb = fallback;
    }
    return nb;
}

// A round's active lists and where its scan leaves its results.
struct ScanLaunch {
    const void *X;              // rows of d coordinates
    int d, R;
    u64 *keys;
    int *deg;
    long long N;
    const int *lists;           // [NDEG * N], by degree class
    EdgeSink sink;
    RoundCtr *c;
    int *redo;                  // [2 * N] vertices that a first form leaves to another
    hipStream_t st;
    hipEvent_t e_start, e_stop;
    int round;                  // 0: no round before it in this call's counters
    long long vertices;         // of the round or run
    u32 enough;                 // active vertices from which a round decides about the form of the next
};

// float32 rows by degree classes 0 .. 6, single precision
void launch_f32_scan(const ScanLaunch &l);
// the double-precision form: l.redo[0 .. c->n_redo), or every class (R <= 96: e_stop after the last)
void launch_f64_redo(const ScanLaunch &l, int dtype);
void launch_f64_classes(const ScanLaunch &l, int dtype);
// 16-bit rows, or the half-precision copy of float32 rows, by degree classes 0 .. 5
void launch_float_scan(const ScanLaunch &l, int dtype, const void *rows, u32 rowbytes, const HalfPar *par);

// A search as rnnd_search has planned it (search.hip): shape is an EvalShape, few = a team of wavefronts per query.
struct SearchLaunch {
    const void *X, *Q;
    const int *graph, *degree;
    long long N, nq;
    int d, dtype, row_stride, L, K, k;
    u64 seed;
    u32 *bitmaps;
    size_t bitmap_words;
    u32 slots;
    int *out_ids;
    u32 *out_dist;
    unsigned long long *counts;
    unsigned blocks, dyn_lds;
    int shape;
    bool few;
    hipStream_t st;
};
void launch_search(const SearchLaunch &l);
