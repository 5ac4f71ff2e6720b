// The decision function of few query rows (predict.hip).
#pragma once

#include "common.hpp"

namespace msvm {

// Floats of kernel values that the two-kernel path for few query rows keeps
// between its kernels, or 0 where the one-kernel path is faster.
int64_t predict_few_floats(int64_t nsv, int64_t m, int64_t ldp);

// Length of the one-kernel path's chain of support tiles, in units of about
// half a microsecond.
int64_t predict_chain(int64_t nsv, int64_t ldp);

// launch_predict for such a call: kbuf holds predict_few_floats floats (a.part
// is not used).  The same bits as launch_predict.
void launch_predict_few(const PredictArgs& a, float* kbuf, hipStream_t s);

}  // namespace msvm
