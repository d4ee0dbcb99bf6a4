// Band Cholesky in 16 x 16 tiles (where chol_tile_fits()).
#pragma once

#include "common.hpp"
#include "launch_rules.hpp"

namespace bandlu {

struct CholParams {
    double *AB;
    int32_t *info;
    int64_t ldab, strideAB;
    int n, kd;
};

// batch <= max_groups(kCholTileThreads)
int launch_pbtrf_tile(const CholParams &P, int64_t batch, hipStream_t s);

}  // namespace bandlu
