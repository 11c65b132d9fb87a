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

template <int DT>
static void launch(const ScanLaunch &l, const FloatRows &fr, const void *rows, u32 rowbytes)
{
    const int8_t *G = (const int8_t *)rows;
    const hipEvent_t e_stop = l.last ? l.e_stop : (hipEvent_t) nullptr;
    auto blocks = [&](int per_cu) {
        const unsigned gx = capped((long long)cu_count() * per_cu, l.N);
        return dim3(gx < 8 ? 8 : gx);      // a block at least for every class
    };
    if (l.R > 32 && l.R <= 96 && l.N <= FLOAT_SHARED_MAX_N) {
        static const int per_cu = resident_blocks_per_cu(k_scan_float_all<DT, 5, 0>, 2);
        hipExtLaunchKernelGGL((k_scan_float_all<DT, 5, 0>), blocks(per_cu), dim3(256), 0, l.st, l.e_start, e_stop, 0, G, rowbytes, fr, l.R, l.keys, l.deg,
                              l.lists, l.props, l.nprop, l.c, l.round);
        return;
    }
    static const int per_s = resident_blocks_per_cu(k_scan_float_small<DT>, 4);
    const int ny = 1 + (l.R > 8) + (l.R > 16);
    hipExtLaunchKernelGGL((k_scan_float_small<DT>), dim3(capped(cu_count() * per_s, l.N), ny), dim3(256), 0, l.st, l.e_start, l.R <= 32 ? e_stop : (hipEvent_t) nullptr, 0, G, rowbytes, fr,
                          l.R, l.keys, l.deg, l.lists, l.props, l.nprop, l.c, l.round);
    if (l.R <= 32) return;
    static const int per5 = resident_blocks_per_cu(k_scan_float_all<DT, 5, 3>, 2), per6 = resident_blocks_per_cu(k_scan_float_all<DT, 6, 3>, 1);
    if (l.R <= 96)
        hipExtLaunchKernelGGL((k_scan_float_all<DT, 5, 3>), blocks(per5), dim3(256), 0, l.st, nullptr, e_stop, 0, G, rowbytes, fr, l.R, l.keys, l.deg, l.lists,
                              l.props, l.nprop, l.c, l.round);
    else
        hipExtLaunchKernelGGL((k_scan_float_all<DT, 6, 3>), blocks(per6), dim3(256), 0, l.st, nullptr, e_stop, 0, G, rowbytes, fr, l.R, l.keys, l.deg, l.lists,
                              l.props, l.nprop, l.c, l.round);
}

// A round of fewer active vertices than this does not decide which form the next one takes: 32 sampled wavefronts, or a sixteenth
// of the vertices.
#define DECIDE_MIN_ACTIVE 1024
void launch_float_scan(const ScanLaunch &l, int dtype, const void *rows, u32 rowbytes, const HalfPar *par)
{
    const u32 share = (u32)(l.vertices / 16);
    const FloatRows fr = {(const char *)l.X, l.d, par, l.redo, &l.c->n_redo[0], l.N, share > DECIDE_MIN_ACTIVE ? share : DECIDE_MIN_ACTIVE};
    if (dtype == DT_F16) launch<DT_F16>(l, fr, rows, rowbytes);
    else if (dtype == DT_BF16) launch<DT_BF16>(l, fr, rows, rowbytes);
    else launch<DT_F32>(l, fr, rows, rowbytes);
}
