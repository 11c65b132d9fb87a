// Launches of the float scans that read whole float32 rows: single precision, and double precision for what the first forms leave.
#include "launch.h"
#include "scan_mfma_f32.h"

// (The times of the launch rules here are of builds that worked by these kernels throughout: float32 builds, and 16-bit ones, before they had the
// tiles of scan_float.h.  Static builds and step-wise calls on float32 rows still do.)
// Float scan: up to here one launch for all classes, which costs the shorter lists their occupancy; above, a launch for each of
// lists of up to 32, 64 and 96 entries.  Whole builds, S = 20, 60 rounds, three launches / one, ms:
//   R = 96          20,000        32,000        50,000         70,000         100,000         200,000
//   float32   96    4.05 / 3.83   5.33 / 5.49   7.61 / 8.11    9.97 / 11.0    13.7 / 16.1     27.4 / 34.4
//   float32  304    6.63 / 6.28   9.62 / 9.41   14.7 / 14.8    20.3 / 21.0    29.3 / 31.4     61.4 / 69.4
//   float16  320    5.12 / 4.80   6.99 / 6.91   9.90 / 10.3    13.1 / 14.2    18.1 / 20.4     35.8 / 42.5
//   bfloat16 128    3.87 / 3.62   5.04 / 5.01   7.08 / 7.28    9.16 / 9.75    12.6 / 14.0     24.1 / 29.1
//   bfloat16 768    9.83 / 7.88   12.4 / 11.1   17.0 / 16.2    22.2 / 22.1    30.5 / 31.2     60.9 / 67.5
//   R = 64
//   float32   96    3.85 / 3.55   5.07 / 4.88   7.08 / 7.01    9.36 / 9.42    12.8 / 13.2     25.2 / 26.4
//   float32  304    6.27 / 5.72   9.18 / 8.55   13.8 / 13.0    19.1 / 18.3    27.3 / 26.4     55.6 / 53.9
//   float16  320    4.89 / 4.42   6.64 / 6.22   9.36 / 9.06    12.4 / 12.3    17.0 / 17.2     32.6 / 34.0
//   bfloat16 128    3.71 / 3.38   4.76 / 4.51   6.63 / 6.34    8.63 / 8.39    11.7 / 11.6     22.0 / 22.6
//   bfloat16 768    6.76 / 5.94   8.89 / 8.11   12.5 / 11.8    16.9 / 16.2    23.4 / 22.8     46.9 / 47.1
// The lines suit rows of up to about 1 KB; longer ones would gain up to 5 % from later lines.
#define SMALL_FLOAT_MAX_N_64 65536      // R <= 64
#define SMALL_FLOAT_MAX_N_96 32768      // R > 64
// Lists of up to 32 entries of long float32 rows: two launches (up to 16, 17 .. 32).  Two / one: 60-round builds of 96 coordinates 70,000
// vertices 10.5 / 10.0 ms, 200,000 27.5 / 26.8, 1M 144.3 / 143.2, of 304 1M 312.5 / 310.6; of 960 150,000 113.0 / 112.0, 500,000 423.2 /
// 424.9, 1M 917.4 / 924.1.  (16-bit rows always take one.)
#define SPLIT_SHORT_LISTS_MIN_N 262144
#define SPLIT_SHORT_LISTS_MIN_D 512

// The single-precision form takes the active lists; vertices it leaves alone (ties in bulk) go to one redo list for all classes.
template <int NRCMAX, int C0, int CH>
static void launch_classes(const ScanLaunch &l, hipEvent_t e_start)
{
    static const int per_cu = resident_blocks_per_cu(k_update_scan_mfma_f32_all<NRCMAX, C0, CH>, 2);
    unsigned gx = capped((long long)cu_count() * per_cu, l.N);
    if (gx < 8) gx = 8;      // a block at least for every class
    hipExtLaunchKernelGGL((k_update_scan_mfma_f32_all<NRCMAX, C0, CH>), dim3(gx), dim3(256), 0, l.st, e_start, nullptr, 0,
                          (const char *)l.X, l.d, l.R, l.keys, l.deg, l.lists, l.N, l.sink.props, l.sink.nprop, l.c, l.redo, &l.c->n_redo);
}

void launch_f32_scan(const ScanLaunch &l)
{
    const int R = l.R;
    const long long N = l.N;
    const bool wide = l.d % 32 == 0;     // two 64-byte chunks per iteration
    if (R > 32 && N <= (R <= 64 ? SMALL_FLOAT_MAX_N_64 : SMALL_FLOAT_MAX_N_96)) {
        if (R <= 64) {
            if (wide) launch_classes<4, 0, 2>(l, l.e_start);
            else launch_classes<4, 0, 1>(l, l.e_start);
        } else {
            if (wide) launch_classes<6, 0, 2>(l, l.e_start);
            else launch_classes<6, 0, 1>(l, l.e_start);
        }
        return;
    }
    if (N > SPLIT_SHORT_LISTS_MIN_N && l.d > SPLIT_SHORT_LISTS_MIN_D) {
        if (wide) launch_classes<1, 0, 2>(l, l.e_start);
        else launch_classes<1, 0, 1>(l, l.e_start);
        if (R > 16) {
            if (wide) launch_classes<2, 2, 2>(l, nullptr);
            else launch_classes<2, 2, 1>(l, nullptr);
        }
    } else {
        if (wide) launch_classes<2, 0, 2>(l, l.e_start);
        else launch_classes<2, 0, 1>(l, l.e_start);
    }
    if (R > 32) launch_classes<4, 3, 1>(l, nullptr);
    if (R > 64) launch_classes<6, 5, 1>(l, nullptr);
}

template <int NG, int CH, int NRC, int DT, bool SCATTER = false>
static void launch_f64(const ScanLaunch &l, const int *list, const u32 *n_list, hipEvent_t e_start, hipEvent_t e_stop)
{
    // wavefronts that fit per SIMD: about 4 for NG = 1, 2 for NG = 2, 1 for NG = 3 (21 accumulator tiles)
    static const int per_cu = resident_blocks_per_cu(k_update_scan_f64<NG, CH, NRC, DT, SCATTER>, NG == 1 ? 4 : NG == 2 ? 2 : 1);
    hipExtLaunchKernelGGL((k_update_scan_f64<NG, CH, NRC, DT, SCATTER>), dim3(capped(cu_count() * per_cu, l.N)), dim3(256), 0,
                          l.st, e_start, e_stop, 0, (const char *)l.X, l.d, l.R, l.keys, l.deg, list, n_list, l.sink, l.c);
}

void launch_f64_redo(const ScanLaunch &l, int dtype)
{
    const u32 *n = &l.c->n_redo;
    if (l.sink.count) {      // the scan before it has scattered
        if (dtype == DT_F16) launch_f64<3, 1, 6, DT_F16, true>(l, l.redo, n, nullptr, l.e_stop);
        else if (dtype == DT_BF16) launch_f64<3, 1, 6, DT_BF16, true>(l, l.redo, n, nullptr, l.e_stop);
        else launch_f64<3, 1, 6, DT_F32, true>(l, l.redo, n, nullptr, l.e_stop);
        return;
    }
    if (dtype == DT_F16) launch_f64<3, 1, 6, DT_F16>(l, l.redo, n, nullptr, l.e_stop);
    else if (dtype == DT_BF16) launch_f64<3, 1, 6, DT_BF16>(l, l.redo, n, nullptr, l.e_stop);
    else launch_f64<3, 1, 6, DT_F32>(l, l.redo, n, nullptr, l.e_stop);
}

// Kernel variant 2: the double-precision form on the active lists.
template <int DT>
static void launch_f64_all(const ScanLaunch &l)
{
    const int R = l.R;
    const int last = (R > 8) + (R > 16) + (R > 32) + (R > 48) + (R > 64) + (R > 80);
    int k = 0;
    auto go = [&](auto launch, int cls) {
        launch(l, l.lists + (size_t)cls * l.N, &l.c->n_active[cls], k == 0 ? l.e_start : (hipEvent_t) nullptr, k == last ? l.e_stop : (hipEvent_t) nullptr);
        ++k;
    };
    go(launch_f64<1, 1, 1, DT>, 0);
    if (R > 8) go(launch_f64<1, 1, 1, DT>, 1);
    if (R > 16) go(launch_f64<1, 1, 2, DT>, 2);
    if (R > 32) go(launch_f64<2, 1, 4, DT>, 3);
    if (R > 48) go(launch_f64<2, 1, 4, DT>, 4);
    if (R > 64) go(launch_f64<3, 1, 5, DT>, 5);
    if (R > 80) go(launch_f64<3, 1, 6, DT>, 6);
}

void launch_f64_classes(const ScanLaunch &l, int dtype)
{
    if (dtype == DT_F16) launch_f64_all<DT_F16>(l);
    else if (dtype == DT_BF16) launch_f64_all<DT_BF16>(l);
    else launch_f64_all<DT_F32>(l);
}
