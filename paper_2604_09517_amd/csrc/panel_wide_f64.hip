// The PFACT leaf's wide form for FP64 panels (a source of its own: it compiles
// beside the other precision).
#include "panel_wide.h"

namespace mxlu {
template int panel_leaf_wide<double>(int64_t, int, double *, int64_t, int64_t, int32_t *, int,
                                  const PanelExchange &, int *, hipStream_t);
template int panel_leaf_swap<double>(double *, int64_t, int64_t, int64_t, int64_t, int, int,
                                   const int32_t *, int64_t, hipStream_t);
}  // namespace mxlu
