// Read-out of one-logit problems on bit words, and the best replica on the
// device (fem_readout.hip).
#pragma once

#include "fem_internal.h"

namespace fem {

// 32-bit words per row of read-out bits: replica r is bit r % 32 of word r / 32
inline int bit_words(int R) { return (R + 31) / 32; }
// words of a row that the lanes of a workgroup take, parts of its entries, each
// with lanes of its own, and rows per workgroup
inline int bit_lanes(int R) { return pow2ceil(bit_words(R) < 64 ? bit_words(R) : 64); }
int bit_parts(const Problem& p, int R);
int bit_tile_rows(const Problem& p, int R);
// whether the problem is evaluated on bit words
bool bit_evaluation(const Problem& p);

// bits[i][w] of the fields, and zeros into count[0, n_inst R)
hipError_t launch_pack_bits(int32_t n, int32_t R, const float* h, int64_t srow, uint32_t* bits, int32_t* count,
                            size_t n_count, hipStream_t st);
// adds to count[inst][R] the ordered cut of +-1 weights or the unsatisfied
// clauses of the rows of tiles [0, n_tiles) (tiles of bit_tile_rows rows)
hipError_t launch_eval_bits(const Problem& p, int32_t R, const Tile* tiles, int n_tiles, const uint32_t* bits,
                            int32_t* count, hipStream_t st);
// v = count as double, and with best not null the anytime best (scores, lower
// is better: -cut, unsatisfied clauses)
hipError_t launch_count_finish(int kind, size_t n_count, const int32_t* count, double* v, double* best,
                               hipStream_t st);
// per instance the replica of the lowest score (ties to the lowest index) and
// its v; the scores are those of best_update_kernel
hipError_t launch_pick(int kind, int R, int n_inst, int q, double lam, const double* v, const long long* sizes,
                       const double* v2, double* value, int32_t* replica, hipStream_t st);
// state of every node in its instance's replica, from the fields
hipError_t launch_config(int kind, int32_t n, int32_t q, const float* h, int64_t srow, int n_inst,
                         const int32_t* inst_off, const int32_t* replica, uint8_t* out, hipStream_t st);

}  // namespace fem
