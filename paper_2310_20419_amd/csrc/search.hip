// Launches of the graph search.  (A source of its own: next to the build's kernels the compiler makes the search's loop 45
// instructions longer, 2 % of a single query.)
#include "launch.h"
#include "search.h"

#define RNND_SEARCH_TEAM(DT, E, SHAPE, TEAM)                                                                          \
    hipLaunchKernelGGL((k_search<DT, E, SHAPE, TEAM>), dim3(l.blocks), dim3(64 * TEAM), l.dyn_lds, l.st, l.X, l.N, l.d, l.graph, \
                       l.degree, l.row_stride, l.Q, l.nq, l.L, l.K, l.k, l.seed, l.bitmaps, l.bitmap_words, l.slots,        \
                       l.out_ids, l.out_dist, l.counts)
#define RNND_SEARCH_ALONE(DT, E, SHAPE) RNND_SEARCH_TEAM(DT, E, SHAPE, 1)
#define RNND_SEARCH_LAUNCH(DT, E, SHAPE)          \
    if (l.few) RNND_SEARCH_TEAM(DT, E, SHAPE, 4);   \
    else RNND_SEARCH_TEAM(DT, E, SHAPE, 1)
#define RNND_SEARCH_E(DT, E)                                            \
    if (l.shape == EVAL_SHORT) { RNND_SEARCH_ALONE(DT, E, EVAL_SHORT); }  \
    else if (l.shape == EVAL_MID) { RNND_SEARCH_LAUNCH(DT, E, EVAL_MID); } \
    else if (l.shape == EVAL_LONG) { RNND_SEARCH_LAUNCH(DT, E, EVAL_LONG); } \
    else if (l.shape == EVAL_SINGLE) { RNND_SEARCH_LAUNCH(DT, E, EVAL_SINGLE); }
#define RNND_SEARCH_FLOAT_E(DT, E)                                      \
    RNND_SEARCH_E(DT, E)                                                \
    else if (l.shape == EVAL_LONG_GLOBAL) { RNND_SEARCH_LAUNCH(DT, E, EVAL_LONG_GLOBAL); } \
    else { RNND_SEARCH_LAUNCH(DT, E, EVAL_SINGLE_GLOBAL); }
#define RNND_SEARCH_FLOAT(DT)                   \
    if (l.L <= 64) { RNND_SEARCH_FLOAT_E(DT, 1) } \
    else { RNND_SEARCH_FLOAT_E(DT, 2) }

void launch_search(const SearchLaunch &l)
{
    if (l.dtype == DT_U8 && l.L <= 64) { RNND_SEARCH_E(DT_U8, 1) }
    else if (l.dtype == DT_U8) { RNND_SEARCH_E(DT_U8, 2) }
    else if (l.dtype == DT_F16) { RNND_SEARCH_FLOAT(DT_F16) }
    else if (l.dtype == DT_BF16) { RNND_SEARCH_FLOAT(DT_BF16) }
    else { RNND_SEARCH_FLOAT(DT_F32) }
}
