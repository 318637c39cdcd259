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
// Entries (of 8 bytes, and 16 of weights where they are not +-1) that may be
// streamed from L2 instead of lying in LDS, at most.
constexpr int64_t RES_MAX_STREAM = 1 << 16;
// LDS for the energy terms of the waves, in front of the values
constexpr int RES_PART_BYTES = 2 * 16 * 2 * 8;

// Longest schedule whose per-step scalars are kept as a device table (104 bytes
// a step).
constexpr int RES_MAX_STEPS = 1 << 20;

// Scalars of one annealing step, as the device reads them.
struct ResStep {
    StepScalars sc;
    double beta;
};
static_assert(sizeof(ResStep) == 104, "the size stated above and in fem.h");

// One resident instance.  Its rows take positions 0..npos-1 by falling degree
// (ties by index), so that the 64 rows of a wave have nearly equal degrees;
// position p belongs to thread p % threads.  Entries are stored per slice of
// 64 positions, 8 bytes per lane and round, lanes side by side.
struct ResInst {
    int32_t inst, n, npos;
    int32_t pos0;      // first entry of perm
    int32_t slice0;    // first entry of slice
    int32_t n_adj;     // entries of adj
    int64_t adj0;      // first entry of adj (and of wgt)
};

// The instances of one launch: same workgroup size and rows per thread.
struct ResClass {
    int threads = 0, rpt = 0;
    int rows = 0;          // most rows of an instance
    int n_inst = 0;
    int first = 0;         // offset into ResTables::inst
    bool adj_lds = false;  // every instance's entries fit in LDS beside the marginals
    int64_t stream = 0;    // else the most entries of one instance
    size_t lds = 0;        // dynamic LDS of the launch
};

// What a problem's solvers share: built by the first that is resident, under
// fem_problem::lock, and released with the problem.
struct ResTables {
    bool planned = false;
    bool fits = false;            // every instance can be resident
    std::vector<ResClass> classes;
    uint64_t threads = 0;         // of one replica of every instance
    bool pm1 = false;             // graphs: weights +-1, carried in the entries
    int planes = 1;               // values per position that neighbours read
    int dev_lds = 0;              // LDS a workgroup may use
    std::vector<ResInst> h_inst;  // the plan, until the tables are on the device
    std::vector<int32_t> h_perm;
    void* block = nullptr;        // device: the one allocation behind the tables
    ResInst* inst = nullptr;
    int32_t* perm = nullptr;      // position -> global row, -1 for padding
    int2* slice = nullptr;        // {first round, rounds} of each slice
    uint2* adj = nullptr;
    float4* wgt = nullptr;        // graphs with other weights: four per lane and round
};

// A solver's part.
struct ResData {
    bool all = false;             // its instances are resident
    int min_steps = 1;            // shorter ranges are faster on the row-tiled kernels
    const ResTables* t = nullptr;
    ResStep* steps = nullptr;     // [T + 1], in the solver's memory
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
// measurements stand at the definition) and starts r; the tables of fp are
// built if they are not there.
hipError_t resident_choose(fem_problem& fp, int R, bool manip, int eval_every, ResData& r);
// Enqueues steps [a.t0, a.t1) of the instances of class cls.
hipError_t resident_launch(const Problem& p, const ResData& r, int cls, bool manip, ResArgs a, hipStream_t st);

}  // namespace fem
