// Launches of the float scans on the 16-bit matrix cores.
#include "launch.h"
#include "scan_float.h"

// Up to here one launch for all classes (lists of up to 96 slots), above and on wider rows, where that launch has the registers of
// one block per CU, the short lists' launch and one for the longer classes.  60-round builds, two launches / one, ms:
//   R = 96   float32 x 96     20,000 3.51 / 3.15 (R = 64)   40,000 5.05 / 4.83   70,000 7.43 / 7.64   100,000 10.1 / 10.5   200,000 21.3 / 22.2
//            float32 x 304    70,000 13.8 / 13.5            float32 x 960 5,000 4.22 / 3.62, 20,000 10.3 / 9.5
//            bfloat16 x 128   50,000 5.72 / 5.44            x 768 20,000 7.01 / 6.44, 70,000 22.3 / 21.8, 300,000 103.0 / 108.7
//   R = 128  float32 x 96     20,000 3.73 / 3.82            200,000 22.2 / 29.1     float16 x 320 20,000 4.98 / 5.10
#define FLOAT_SHARED_MAX_N 65536

// Up to here the vertices that a scan of lists of 33 .. 96 entries leaves are finished by the wavefronts that left them, above by a launch of
// their own, which has the registers for it (at two wavefronts per SIMD that form spills 200).  float32 200,000 x 100, R = 96, 8
// rounds, in the scan / in a launch, ms: rows 100 times each 17.7 / 15.4, clusters of radius 0.003 14.5 / 13.4, two places 10^4 apart
// 24.8 / 24.1; an empty launch is 4.5 us, 3 % of a round at 70,000 x 96.
#define FINISH_MAX_N 131072

// From how many vertices on the first round of a call looks at a sample of its lists first (about 10 us; without it a first round that
// the tiles do not suit, 20,000 x 96, R = 96: norms over 12 binades 473 us instead of 130, two places 10^4 apart 727 instead of 230).
#define SAMPLE_MIN_N 8192

template <int DT>
static void launch(const ScanLaunch &l, FloatRows fr, const void *rows, u32 rowbytes)
{
    const int8_t *G = (const int8_t *)rows;
    if (l.round == 0 && l.vertices >= SAMPLE_MIN_N)
        hipLaunchKernelGGL((k_float_sample<DT>), dim3(SAMPLE_BLOCKS), dim3(256), 0, l.st, (const char *)rows, rowbytes, fr, l.R, l.keys, l.deg, l.lists, l.enough, l.c);
    const hipEvent_t e_stop = l.R <= 96 ? l.e_stop : (hipEvent_t) nullptr;      // (else the pair-at-a-time kernel follows)
    auto blocks = [&](int per_cu) {
        const unsigned gx = capped((long long)cu_count() * per_cu, l.N);
        return dim3(gx < 8 ? 8 : gx);      // a block at least for every class
    };
    if (l.R > 32 && l.R <= 96 && l.N <= FLOAT_SHARED_MAX_N) {
        static const int per_cu = resident_blocks_per_cu(k_scan_float_all<DT, 5, 0, true>, 2);
        hipExtLaunchKernelGGL((k_scan_float_all<DT, 5, 0, true>), blocks(per_cu), dim3(256), 0, l.st, l.e_start, e_stop, 0, G, rowbytes, fr, l.R, l.keys, l.deg,
                              l.lists, l.sink, l.c);
        return;
    }
    static const int per_s = resident_blocks_per_cu(k_scan_float_small<DT>, 4);
    const int ny = 1 + (l.R > 8) + (l.R > 16);
    // Half the blocks that a vertex per wavefront would take, for each of three classes, where a round waits for its launches more than for its rows.  R = 32, a vertex per wavefront / half, ms: rows of 192
    // bytes 300 0.749 / 0.678, 4,000 1.235 / 1.197; 256 bytes 1,000 0.866 / 0.870, 6,000 1.568 / 1.507; 768 bytes 1,000 1.046 / 1.054, 2,000 1.319 / 1.337, 4,000 1.707 / 1.683; 1,920 bytes 2,000 2.02 / 2.11,
    // 4,000 2.48 / 2.52, 8,000 3.544 / 3.526; 4,000 bytes 2,000 3.35 / 3.55, 6,000 5.54 / 5.58.
    const bool halve = rowbytes <= 256u || l.N >= 4ll * rowbytes;
    hipExtLaunchKernelGGL((k_scan_float_small<DT>), dim3(capped(cu_count() * per_s, halve ? l.N / 2 : l.N), ny), dim3(256), 0, l.st, l.e_start, l.R <= 32 ? e_stop : (hipEvent_t) nullptr, 0, G, rowbytes, fr,
                          l.R, l.keys, l.deg, l.lists, l.sink, l.c);
    if (l.R <= 32) return;
    if (l.R > 96) {
        static const int per_cu = resident_blocks_per_cu(k_scan_float_all<DT, 6, 3, true>, 1);
        hipExtLaunchKernelGGL((k_scan_float_all<DT, 6, 3, true>), blocks(per_cu), dim3(256), 0, l.st, nullptr, e_stop, 0, G, rowbytes, fr, l.R, l.keys, l.deg, l.lists,
                              l.sink, l.c);
    } else if (l.N <= FINISH_MAX_N) {
        static const int per_cu = resident_blocks_per_cu(k_scan_float_all<DT, 5, 3, true>, 2);
        hipExtLaunchKernelGGL((k_scan_float_all<DT, 5, 3, true>), blocks(per_cu), dim3(256), 0, l.st, nullptr, e_stop, 0, G, rowbytes, fr, l.R, l.keys, l.deg, l.lists,
                              l.sink, l.c);
    } else {
        static const int per_cu = resident_blocks_per_cu(k_scan_float_all<DT, 5, 3, false>, 2);
        fr.left = nullptr;
        hipExtLaunchKernelGGL((k_scan_float_all<DT, 5, 3, false>), blocks(per_cu), dim3(256), 0, l.st, nullptr, nullptr, 0, G, rowbytes, fr, l.R, l.keys, l.deg, l.lists,
                              l.sink, l.c);
        launch_f64_redo(l, DT);
    }
}

void launch_float_scan(const ScanLaunch &l, int dtype, const void *rows, u32 rowbytes, const HalfPar *par)
{
    const FloatRows fr = {(const char *)l.X, l.d, par, l.redo + l.N, l.redo, &l.c->n_redo, l.N};
    if (dtype == DT_F16) launch<DT_F16>(l, fr, rows, rowbytes);
    else if (dtype == DT_BF16) launch<DT_BF16>(l, fr, rows, rowbytes);
    else launch<DT_F32>(l, fr, rows, rowbytes);
}
