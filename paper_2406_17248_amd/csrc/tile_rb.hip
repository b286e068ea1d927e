// One instantiation of the register-blocked passes: QSV_RB_REAL (float or double), QSV_RB_ADJ
// (true: reverse sweep) and QSV_RB_MULTI (1: many circuits in one launch) are given on the
// command line, so the instantiations compile in parallel.
#include "tile_rb.h"

namespace qsv {
#if QSV_RB_MULTI
template hipError_t rb_multi_dispatch<QSV_RB_REAL, QSV_RB_ADJ>(int, const PassArgs*, const uint32_t*, int, uint32_t,
                                                               int, int, hipStream_t);
#else
template hipError_t rb_dispatch<QSV_RB_REAL, QSV_RB_ADJ>(int, int, const PassArgs&, uint64_t, int, hipStream_t);
#endif
}  // namespace qsv
