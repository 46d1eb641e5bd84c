// The operator on canonical spinors (fs_op.hip).
#pragma once

#include "fs_kernels.h"

namespace fs {

struct OpPlan {
    int T[3], nt[3];  // tile extents in x, y, z and tiles per axis
    int tc;           // t-slices per workgroup
    int lanes;        // threads per workgroup
    int n_rhs;
    int two_rows;     // FP32: rows 0-1 of the links, row 2 rebuilt
    long long n_wg;
};
OpPlan op_plan(int prec, const int* L, int n_rhs, bool two_rows);
// out = (D + sigma) in for n_rhs spinors of 12 V complex128 each, diag = 4 + m0 +
// sigma, spinors and links rounded to prec (not FP16); 16-byte aligned, in and out
// disjoint.
void launch_op(int prec, const OpPlan& p, const LatDesc& ld, double diag, const double* in, double* out,
               hipStream_t s);

}  // namespace fs
