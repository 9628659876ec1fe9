// One row of the near-field CSR operator (FP64) by a group of lanes.
#pragma once

#include "bem_internal.h"

namespace bem {

// Lanes per vertex of the kernels that add the near field: a row has about 19
// entries of four blocks, so one lane per row is a chain of about 19 dependent
// gathers (20-38 us at any mesh size up to 10 242 vertices); 16 lanes make it
// two (5-7 us).
constexpr int NEAR_LANES = 16;

// Adds row i of the four blocks times x = [psi; phi] to this lane's share of
// (y1, y2); near_sum adds the shares of the group's lanes.
__device__ __forceinline__ void near_row(int lane, int64_t i, const int32_t *__restrict__ rowptr,
                                         const int32_t *__restrict__ col,
                                         const double2 *__restrict__ nf, int64_t nnz,
                                         const double2 *__restrict__ x, int64_t N, double2 &y1,
                                         double2 &y2) {
    const double2 *C11 = nf, *C12 = nf + nnz, *C21 = nf + 2 * nnz, *C22 = nf + 3 * nnz;
    const int e1 = rowptr[i + 1];
    for (int e = rowptr[i] + lane; e < e1; e += NEAR_LANES) {
        const int j = col[e];
        const double2 p = x[j], f = x[N + j];
        const double2 a = C11[e], b = C12[e], c = C21[e], d = C22[e];
        y1.x += a.x * p.x - a.y * p.y + b.x * f.x - b.y * f.y;
        y1.y += a.x * p.y + a.y * p.x + b.x * f.y + b.y * f.x;
        y2.x += c.x * p.x - c.y * p.y + d.x * f.x - d.y * f.y;
        y2.y += c.x * p.y + c.y * p.x + d.x * f.y + d.y * f.x;
    }
}

// Sum over the group's lanes, fixed butterfly order (all 16 lanes active).
__device__ __forceinline__ double near_sum(double v) {
    for (int o = NEAR_LANES / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, NEAR_LANES);
    return v;
}

}   // namespace bem
