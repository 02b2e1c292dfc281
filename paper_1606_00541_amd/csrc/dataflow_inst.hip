// Instances of the dataflow kernels for one value type, one or several
// right-hand sides, with or without the per-step clocks (HEC_DF_T, HEC_DF_R1,
// HEC_DF_TRACE), or of the two-triangle kernel (HEC_DF_LU); HEC_DF_NAME is the
// selector.  Compiled once per combination.
#include "dataflow.h"

namespace hec {

namespace {

#if !HEC_DF_LU
template <bool UNIT, bool TAIL> OwnerKernel by_width(int w)
{
    switch (w) {
#define HEC_DF_CASE(W) \
    case W: return k_dataflow<HEC_DF_T, W, UNIT, TAIL, HEC_DF_R1, HEC_DF_TRACE>;
        HEC_DF_CASE(1)
        HEC_DF_CASE(2)
        HEC_DF_CASE(3)
        HEC_DF_CASE(4)
        HEC_DF_CASE(5)
        HEC_DF_CASE(6)
        HEC_DF_CASE(7)
        HEC_DF_CASE(8)
        HEC_DF_CASE(10)
        HEC_DF_CASE(12)
        HEC_DF_CASE(16)
#undef HEC_DF_CASE
    default: return nullptr;
    }
}
#endif

#if HEC_DF_LU
LuKernel lu_by_width(int w)
{
    switch (w) {
#define HEC_DF_CASE(W) \
    case W: return k_dataflow_lu<HEC_DF_T, W, HEC_DF_R1>;
        HEC_DF_CASE(1)
        HEC_DF_CASE(2)
        HEC_DF_CASE(3)
        HEC_DF_CASE(4)
        HEC_DF_CASE(5)
        HEC_DF_CASE(6)
        HEC_DF_CASE(7)
        HEC_DF_CASE(8)
        HEC_DF_CASE(10)
        HEC_DF_CASE(12)
        HEC_DF_CASE(16)
#undef HEC_DF_CASE
    default: return nullptr;
    }
}
#endif

}  // namespace

#if HEC_DF_LU
LuKernel HEC_DF_NAME(int w) { return lu_by_width(w); }
#else
OwnerKernel HEC_DF_NAME(int w, bool unit, bool tail)
{
    if (unit) return tail ? by_width<true, true>(w) : by_width<true, false>(w);
    return tail ? by_width<false, true>(w) : by_width<false, false>(w);
}
#endif

}  // namespace hec
