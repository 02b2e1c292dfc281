// Instances of the pipelined system queue for one value type (HEC_SQ_T),
// columns of an item (HEC_SQ_C) and output (HEC_SQ_MODE); HEC_SQ_NAME is the selector.  Compiled once per
// combination.
#include "sysq.h"

namespace hec {

namespace {

template <typename TIn, int M, bool FAR> SysqKernel by_width(int w)
{
    switch (w) {
#define HEC_SQ_CASE(W) \
    case W: return k_sysq_pipe<HEC_SQ_T, TIn, W, HEC_SQ_C, M, HEC_SQ_MODE, FAR>;
        HEC_SQ_CASE(2)
        HEC_SQ_CASE(3)
        HEC_SQ_CASE(4)
        HEC_SQ_CASE(6)
        HEC_SQ_CASE(8)
#undef HEC_SQ_CASE
    default: return nullptr;
    }
}

template <typename TIn> SysqKernel by_rows(int w, int rows, bool far)
{
    if (rows == 1) return far ? by_width<TIn, 1, true>(w) : by_width<TIn, 1, false>(w);
    return far ? by_width<TIn, 2, true>(w) : by_width<TIn, 2, false>(w);
}

}  // namespace

SysqKernel HEC_SQ_NAME(int w, bool in_f64, int rows, bool far)
{
    return in_f64 ? by_rows<double>(w, rows, far) : by_rows<float>(w, rows, far);
}

}  // namespace hec
