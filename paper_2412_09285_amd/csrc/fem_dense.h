// Dense-W MaxCut step (fem_dense.hip): launcher and tile layouts.  Not part
// of the public ABI.
#pragma once

#include "fem_internal.h"

namespace fem {

// W and the int8 digit planes are zero-padded to a multiple of this many
// rows and columns (the contraction of four waves' operands)
constexpr int DENSE_LD_ALIGN = 128;

// replicas of each int8 digit plane of the marginal copy
inline int dense_rows_padded(int R) { return (R + 31) / 32 * 32; }

// byte of (row, k) in the int8 image of W and in each digit plane (row: node
// or replica; rows of ld bytes): blocks of 32 rows x 32 k, the 16 bytes of
// k / 16 and a row together
inline __host__ __device__ size_t dense_i8_at(int row, int k, int ld)
{
    return ((size_t)(row >> 5) * (ld >> 5) + (k >> 5)) * 1024 + ((k >> 4) & 1) * 512 + (row & 31) * 16 + (k & 15);
}

// rows and replicas of a workgroup's block; a dense problem's tiles are the
// row blocks
struct DenseShape {
    int rows, cols;
};
// the block for R replicas of a dense problem
DenseShape dense_shape(const Problem& p, int R);

// One explicit-gradient MaxCut step with phi = W m formed by matrix-core
// products: exact int32 products of int8 weights and the four int8 digit
// planes of the fixed-point marginals when the problem holds dense_w8 (W
// integral, |W| <= 127), FP64 products of the float32 W and marginals
// otherwise.  Float32 marginal type only.  n_tiles: ceil(n / shape.rows).
hipError_t launch_dense_step(const Problem& p, const DenseShape& shape, int dtype, bool en, bool nt, int n_tiles,
                             const StepArgs& a, hipStream_t st);
// the digit planes of the marginals of a.h into a.marg_nxt (int8 path); src:
// new fields on the device, set with cleared moments in the same pass, or null
hipError_t launch_dense_i8_init(const Problem& p, const StepArgs& a, const float* src, hipStream_t st);

}  // namespace fem
