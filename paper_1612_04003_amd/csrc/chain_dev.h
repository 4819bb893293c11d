// Device code shared by the kernels of the outer-step chain (chain.hip) and the
// CSR updates that finish a chain step: the geometry of the block-triangular
// inverse and the coordinate update x[idx] += delta.
#pragma once

#include "internal.h"

namespace cabcd {
namespace cdev {

// Link word of row p of an outer step: bit 16 set when no earlier row has the
// same index; bit 17 when a block of its superblock is not positive definite; low 16
// bits: 1 + the next row with the same index (0: none).
constexpr int kLinkFirst = 1 << 16, kLinkBad = 1 << 17;

// x[idx] += delta for one step by one workgroup of T threads, a single writer
// per coordinate: the first row of an index adds that index's rows in row order.
// What the inversions ahead found in the step's blocks is reported here, as a run
// may stop before a step whose Gram was computed ahead.
template <int T>
__device__ __forceinline__ void scatter_delta(const int32_t* __restrict__ idx,
                                              const int* __restrict__ link, const double* delta,
                                              int m, double* __restrict__ x, int* status) {
  for (int p = threadIdx.x; p < m; p += T) {
    int l = link[p];
    if ((l & kLinkBad) != 0) raise_status(status, DEV_NOTSPD);
    if ((l & kLinkFirst) == 0) continue;
    const int i = idx[p];
    double v = x[i] + delta[p];
    for (int q = (l & 0xFFFF) - 1; q >= 0; q = (link[q] & 0xFFFF) - 1) v += delta[q];
    x[i] = v;
  }
}

// Right-hand side of a row of an outer step from its Y u (mode 0 primal, 1 dual).
__device__ __forceinline__ double rhs_of(int mode, double lambda, double n, double yu, double xi,
                                         double yi) {
  return mode == 0 ? (-lambda * xi - yu / n) : ((yu - xi - yi) / n);
}

// T^-1 of a step: superblock (i, j) of 256 doubles, and the place of item i of a lane in
// one (row 4 i + lane / 16, column lane % 16).
__host__ __device__ constexpr int tri_block(int i, int j) { return i * (i + 1) / 2 + j; }
__host__ __device__ constexpr int tri_at(int i, int lane) {
  return (i >> 1) * 128 + 2 * lane + (i & 1);
}

}  // namespace cdev
}  // namespace cabcd
