// The L^T pass of the transposed solve.
#pragma once

#include "common.hpp"
#include "launch_rules.hpp"

namespace bandlu {

struct LtParams {
    const double *AB;
    const int32_t *ipiv;
    double *B;
    int64_t ldab, strideAB, strideP, ldb, strideB;
    int n, kl, kv, nrhs, R;
};

constexpr int kLtMfmaMaxKl = 1024;

// kl <= kLtMfmaMaxKl, n >= 2
int launch_getrs_lt(LtParams P, int64_t systems, hipStream_t s);

}  // namespace bandlu
