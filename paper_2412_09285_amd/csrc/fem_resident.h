// Resident anneals: small one-logit instances whose replicas stay on one
// compute unit for a whole range of steps (fem_resident.hip).
#pragma once

#include "fem_internal.h"

namespace fem {

// Rows per instance at most: eight per thread of a 1024-thread workgroup, less
// the two constant slots, so that 16-bit byte offsets reach two planes of
// values; Max-k-SAT four per thread and 15 bits.
constexpr int RES_MAX_ROWS = 8 * 1024 - 2;
constexpr int RES_MAX_ROWS_SAT = 4 * 1024 - 8;
// Entries (of 8 bytes) that may be streamed from L2 instead of lying in LDS.
constexpr int64_t RES_MAX_STREAM = 1 << 16;
// LDS for the energy terms of the waves, in front of the values
constexpr int RES_PART_BYTES = 2 * 16 * 2 * 8;

// Longest schedule whose per-step scalars are kept as a device table (about
// 150 bytes a step).
constexpr int RES_MAX_STEPS = 1 << 20;

// Scalars of one annealing step, as the device reads them.
struct ResStep {
    StepScalars sc;
    double beta;
};

// One resident instance.  Its rows take positions 0..npos-1 by falling degree
// (ties by index), so that the 64 rows of a wave have nearly equal degrees;
// position p belongs to thread p % threads.  Entries are stored per slice of
// 64 positions, 8 bytes per lane and round, lanes side by side.
struct ResInst {
    int32_t inst, row0, n, npos;
    int32_t pos0;      // first entry of perm
    int32_t slice0;    // first entry of slice
    int64_t adj0;      // first entry of adj (and of wgt)
    int32_t n_adj;     // entries of adj
    int32_t pad;
};

// The instances of one launch: same workgroup size and rows per thread.
struct ResClass {
    int threads = 0, rpt = 0;
    int n_inst = 0;
    int first = 0;         // offset into ResData::inst
    bool adj_lds = false;  // every instance's entries fit in LDS beside the marginals
    size_t lds = 0;        // dynamic LDS of the launch
};

struct ResData {
    std::vector<ResClass> classes;
    bool all = false;             // the problem's instances are resident
    bool pm1 = false;             // graphs: weights +-1, carried in the entries
    size_t dev_lds = 0;           // LDS a workgroup may use
    int planes = 1;               // values per position that neighbours read
    int min_steps = 1;            // shorter ranges are faster on the row-tiled kernels
    void* block = nullptr;        // device: the one allocation behind the tables
    ResInst* inst = nullptr;
    int32_t* perm = nullptr;      // position -> global row, -1 for padding
    int2* slice = nullptr;        // {first round, rounds} of each slice
    uint2* adj = nullptr;
    float4* wgt = nullptr;        // graphs with other weights: four per lane and round
    ResStep* steps = nullptr;     // [T + 1]
};

struct ResArgs {
    const ResInst* inst;
    const int32_t* perm;
    const int2* slice;
    const uint2* adj;
    const float4* wgt;
    const ResStep* steps;
    const double* nrm;            // manipulated gradients
    const double* wtot;
    float* h;
    float* m1;
    float* m2;
    int64_t srow;
    float* grad;                  // of the last step, or null
    double* eout;                 // [record][inst][3][R]
    int64_t erecord;              // stride between records (0: one slot)
    int32_t energy_every;         // 0: no energies
    int32_t R;
    int32_t t0, t1;
    int32_t bf16;                 // the values neighbours read are rounded to bfloat16
    int32_t kind;
    int32_t planes;
};

// Says whether a solver's instances are resident (the rule and its
// measurements stand at the definition) and starts r.
bool resident_choose(const Problem& p, int R, bool manip, int eval_every, ResData& r);
// Builds the device structure; steps: host table of T + 1 entries.
hipError_t resident_build(const Problem& p, const std::vector<ResStep>& steps, ResData& r);
void resident_free(ResData& r);
// Enqueues steps [a.t0, a.t1) of the instances of class cls.
hipError_t resident_launch(const Problem& p, const ResData& r, int cls, bool manip, ResArgs a, hipStream_t st);

}  // namespace fem
