// Instances of the pipelined system queue for one value type (HEC_SQ_T),
// columns of a thread (HEC_SQ_C) and output (HEC_SQ_MODE; HEC_SQ_F64: 1 if the type is FP64); HEC_SQ_NAME is
// the selector.  Compiled once per
// combination.
#include "sysq.h"

namespace hec {

namespace {

template <typename TIn, int M, int FORM> SysqKernel by_width(int w)
{
    switch (w) {
#define HEC_SQ_CASE(W) \
    case W: return k_sysq_pipe<HEC_SQ_T, TIn, W, HEC_SQ_C, M, HEC_SQ_MODE, FORM>;
        HEC_SQ_CASE(2)
        HEC_SQ_CASE(3)
        HEC_SQ_CASE(4)
        HEC_SQ_CASE(6)
        HEC_SQ_CASE(8)
#undef HEC_SQ_CASE
    default: return nullptr;
    }
}
// four values beyond the ring: rows of three entries or more, one row a thread
// (two, or four columns in FP64, would spill most of their registers)
template <typename TIn> SysqKernel by_width_far4(int w)
{
#if HEC_SQ_C == 1 || !HEC_SQ_F64
    switch (w) {
#define HEC_SQ_CASE(W) \
    case W: return k_sysq_pipe<HEC_SQ_T, TIn, W, HEC_SQ_C, 1, HEC_SQ_MODE, 4>;
        HEC_SQ_CASE(3)
        HEC_SQ_CASE(4)
        HEC_SQ_CASE(6)
        HEC_SQ_CASE(8)
#undef HEC_SQ_CASE
    default: break;
    }
#endif
    return nullptr;
}

template <typename TIn> SysqKernel by_form(int w, int rows, int form)
{
    switch (form) {
    case 0: return rows == 1 ? by_width<TIn, 1, 0>(w) : by_width<TIn, 2, 0>(w);
    case kSysqShared: return rows == 1 ? by_width<TIn, 1, kSysqShared>(w) : by_width<TIn, 2, kSysqShared>(w);
    case 2: return rows == 1 ? by_width<TIn, 1, 2>(w) : by_width<TIn, 2, 2>(w);
    default: return by_width_far4<TIn>(w);
    }
}

}  // namespace

SysqKernel HEC_SQ_NAME(int w, bool in_f64, int rows, int form)
{
    return in_f64 ? by_form<double>(w, rows, form) : by_form<float>(w, rows, form);
}

}  // namespace hec
