// Arguments and launches of the loop that runs many outer iterations to a
// launch (resident.hip).
#pragma once

#include "common.hpp"

namespace msvm {

// Many outer iterations per launch for problems whose whole kernel matrix is
// in HBM (k_resident, q <= 16): a problem's rows are dealt to R blocks, at
// most kResUnits units of two rows each.
constexpr int kResUnits = kSelThreads - 64;
constexpr int kResRows = 2 * kResUnits;
constexpr int kResBlocks = 32;  // of one problem, at most
struct ResidentProblem {
    const float* K;       // n rows of ldc floats: K(x_s, .), and one of zeros
    double* F;
    double* alpha;
    uint8_t* st;
    const float* z;       // labels (C-SVC) or targets (eps-SVR)
    WorkingSet* ws;
    int32_t* seen;        // n: -1 until the sample has been used
    uint64_t* xch;        // R > 1: resident_xch_words(R), zero before a solve
    double C, eps, tol, inner_ratio;
    int64_t max_iter;
    int32_t max_inner;
};
struct ResidentArgs {
    const ResidentProblem* p;  // one per R blocks of the grid
    uint32_t* hs;         // R > 1: two words a problem, zero before a launch
    int64_t n, ldc;
    int32_t R, half;
    int32_t iters;        // outer iterations of this launch, at most
    uint64_t wait;        // R > 1: for the blocks to start, 100 MHz ticks
    uint64_t lag;         // R > 1: how long each problem's last block waits
                          // between taking the other blocks' candidates and
                          // using them (tests; 0: not at all)
};

// every K(x_i, x_j): K[i * ldc + j], the values of the row kernel bit for bit,
// and row n: zeros
void launch_gram(const float* X, const float* sq, int64_t n, int64_t ldp,
                 const KernelFn& kf, float* K, int64_t ldc, hipStream_t s);
size_t resident_xch_words(int R);
void launch_resident(const ResidentArgs& a, int problems, bool svr,
                     hipStream_t s);

}  // namespace msvm
