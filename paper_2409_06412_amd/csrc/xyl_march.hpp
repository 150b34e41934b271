// Three steps per pass of large FP32 lattices (xyl_march.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "xyl_internal.hpp"

namespace xyl {

constexpr int kMarchSteps = 3;
struct MarchBuffers {        // in and out are different arrays
    const float* th_in;
    const float* u_in;
    float* th_out;
    float* u_out;
};
struct MarchPlan {
    int ntx = 0, strips = 0;  // column tiles of at most 248 sites, strips of rows
    double us = 0.0;          // modelled time per step
};
// For widths that are multiples of 4 and at least 3 rows.
MarchPlan march_plan(int Lx, int Ly, int cus);
// Loads this file's kernels on the current device.
void load_march_kernels();
// Steps k .. k + 2 of a lattice with the factored kick.
void launch_march(const Lat<float>& v, const MarchBuffers& b, const MarchPlan& p, uint64_t k, hipStream_t s);

}  // namespace xyl
