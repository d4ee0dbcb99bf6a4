// Band Cholesky in 16 x 16 tiles (kd <= kCholTileMaxKd).
#pragma once

#include "common.hpp"

namespace bandlu {

struct CholParams {
    double *AB;
    int32_t *info;
    int64_t ldab, strideAB;
    int n, kd;
};

// the window's tiles fill LDS at 12 tile rows
constexpr int kCholTileMaxKd = 144;

int launch_pbtrf_tile(const CholParams &P, int64_t batch, hipStream_t s);

}  // namespace bandlu
