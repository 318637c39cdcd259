// Internal declarations of the FEM library (host structures, kernel launch
// parameters).  Not part of the public ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <string>
#include <vector>

namespace fem {

struct ResTables;   // fem_resident.h
void resident_release(ResTables* t);

enum Kind { KIND_MAXCUT = 0, KIND_BMINCUT = 1, KIND_MAXSAT = 2 };

// One tile = a contiguous row range of a single instance; one workgroup per
// tile (times the replica segments along grid.y).
struct Tile {
    int32_t inst, row_begin, row_end, slot;   // slot: index of the tile's partial sums
};

// Device-resident problem.
struct Problem {
    int device = 0;
    int kind = KIND_MAXCUT;
    int32_t n = 0;         // total rows (nodes / variables) over all instances
    int32_t q = 2;         // states (2 for one-logit kinds)
    int64_t nnz = 0;       // adjacency entries or literal incidences
    int32_t n_inst = 1;
    int32_t sat_width = 2; // Max-k-SAT: other literals stored per incidence (2 or 3)
    int32_t sat_k = 2;     // Max-k-SAT: most literals of a clause (2 to 4)
    int64_t n_clauses = 0;
    bool integral = true;  // all weights integral (exact integer cut values)
    std::vector<int32_t> inst_off;   // host [n_inst+1] node offsets
    std::vector<double> inst_wtot;   // host [n_inst] sum of undirected weights
    // device arrays
    int64_t* row_off = nullptr;      // [n+1]
    int2* adj = nullptr;             // graphs: {col, float bits of w}
    int32_t* adj_pm1 = nullptr;      // MaxCut with every weight +-1: col | (w < 0) << 31 (4 B per entry)
    int2* inc2 = nullptr;            // Max-k-SAT, <= 2 other literals per incidence
    int4* inc4 = nullptr;            // Max-k-SAT, <= 3 other literals per incidence
    float* wdeg = nullptr;           // bMinCut: sum_j W_ij per node
    double* nrm = nullptr;           // graphs: sum_j |W_ij| per node (normalisers of the manipulated gradients)
    int32_t* nw = nullptr;           // bMinCut node weights V_i (null: all 1)
    double* v2 = nullptr;            // bMinCut: [n_inst] sum_i V_i^2 per instance
    int32_t* inst_off_d = nullptr;   // [n_inst+1] node offsets of the instances
    // dense MaxCut: W as a zero-padded row-major float matrix [dense_ld][dense_ld]
    // (the CSR above is still built, for read-out and evaluation)
    float* dense_w = nullptr;
    int32_t dense_ld = 0;
    int8_t* dense_w8 = nullptr;      // the same as int8 when W is integral with |W| <= 127
    // host copies kept for batching and validation
    std::vector<int64_t> h_row_off;
    std::vector<int2> h_adj;
    std::vector<int2> h_inc2;
    std::vector<int4> h_inc4;
    std::vector<float> h_wdeg;
    std::vector<double> h_nrm;
    std::vector<int32_t> h_nw;       // empty: unit node weights
    std::vector<double> inst_v2;     // host [n_inst] sum_i V_i^2 (the node count for unit weights)
};

// Marginal-copy literal packing for Max-k-SAT incidence records:
//   bit 31: literal is positive; bits 0..29: variable; the value
//   SAT_NONE in bits 0..29 marks an unused slot (treated as a false literal
//   with probability 1, i.e. a neutral factor).
constexpr uint32_t SAT_VAR_MASK = 0x3FFFFFFFu;
constexpr uint32_t SAT_NONE = 0x3FFFFFFFu;
constexpr uint32_t SAT_POS = 0x80000000u;
// flag bits carried in bit 30 of the first / second slot
constexpr uint32_t SAT_FLAG = 0x40000000u;   // slot0: own literal positive; slot1: owner incidence

// Largest workgroup of a step kernel: register-heavy instantiations (8 values
// per lane; Potts with q >= 8) get a smaller bound so that the compiler may use
// up to 256 (512 threads) or 512 (256 threads) VGPRs without spilling.
__host__ __device__ constexpr int step_max_threads(int kind, int per_lane)
{
    return kind == KIND_BMINCUT ? (per_lane >= 16 ? 256 : (per_lane >= 8 ? 512 : 1024))
                                : (per_lane >= 8 ? 512 : 1024);
}

// bMinCut step kernel: per-lane running sums in LDS up to q = 16 (q + 3
// doubles per thread); the block reduction reuses that space
__host__ __device__ constexpr bool potts_lds_acc(int q) { return q <= 16; }
inline size_t potts_step_lds(int threads, int lanes, int q)
{
    const size_t red = (size_t)(threads / 64) * lanes * (q > 3 ? q : 3) * 8;
    const size_t acc = potts_lds_acc(q) ? (size_t)threads * (q + 3) * 8 : 0;
    return red > acc ? red : acc;
}

struct TileShape {
    int vec = 1, waves = 4, rows = 4;
    int nt = 0;      // non-temporal access to h, m1, m2
    int lanes = 0;   // cap on lanes per team (power of two <= 64; 0 = 64)
};

// Per-step scalars, computed on the host in double and passed as float.
struct StepScalars {
    double inv_beta_d;   // 1/beta and lambda in double for the gradient combination
    double lam_d;
    double gamma_d;      // gamma_grad (manipulated gradients and Max-k-SAT; 1 otherwise)
    float inv_beta;
    float lam;
    float step_size;   // lr / (1 - b1^n)
    float bc2_sqrt;    // sqrt(1 - b2^n)
    float inv_bc2_sqrt;   // 1 / sqrt(1 - b2^n)
    float b1, one_m_b1, b2, one_m_b2, eps, wd;
    int opt;            // 0 Adam, 1 RMSprop, 2 SGD
    int first;          // SGD: first step (the momentum buffer starts as g)
    float mom, damp, rms_alpha, one_m_rms, lr;
};

struct LaunchGeom {
    int lanes;        // lanes per team (power of two, <= 64)
    int nseg;         // replica segments
    int teams_per_block;
    int n_tiles;
    int seg_major;    // grid (nseg, n_tiles) instead of (n_tiles, nseg)
};

inline int pow2ceil(int x)
{
    int p = 1;
    while (p < x) p <<= 1;
    return p;
}

// Teams of lanes covering R replicas at per_lane values per lane, at most
// max_lanes lanes (0 or 64: a full wave), and the replica segments left over.
inline LaunchGeom make_geom(int per_lane, int R, int waves, int max_lanes = 64)
{
    LaunchGeom g{};
    const int need = (R + per_lane - 1) / per_lane;
    const int cap = max_lanes > 0 ? max_lanes : 64;
    const int p2 = pow2ceil(need);
    g.lanes = cap < p2 ? cap : p2;
    g.nseg = (need + g.lanes - 1) / g.lanes;
    g.teams_per_block = waves * (64 / g.lanes);
    return g;
}

// Launch shape of the integer evaluation (fem_eval_int and its allocation-free
// form, whose scratch limit counts on these tiles): four waves, four rows per
// team, as many replicas per lane as keep a team's row within one wave.
inline TileShape eval_shape(int kind, int R)
{
    TileShape t;
    if (kind == KIND_BMINCUT) return t;
    if (R % 4 == 0 && R >= 128) t.vec = 4;
    else if (R % 2 == 0 && R >= 64) t.vec = 2;
    return t;
}

// Default launch shape before tuning: values per lane, waves, rows per team,
// lanes per team and non-temporal state access by size, from sweeps of 500 ..
// 300000 rows and R = 16 .. 512 on an MI355X (microseconds per step, the other
// choice first).
//  * One row per team while that leaves few workgroups, up to four beyond
//    (`blocks` workgroups for the next doubling): 9000 rows at R = 16 with four
//    rows 19.7, with one 13.3.
//  * As many values per lane as still fill the chip: MaxCut 50000 rows, R = 32,
//    one value 36, two 26; 11361 rows, R = 20, 14.5 / 13.5; 300000 rows, one 119,
//    four 89.  Max-k-SAT stays at
//    two (rounds of four incidences): 20000 variables, R = 64, 44 / 34; and
//    where one would take a second segment: 8000, k = 3, R = 76, 31 / 26.  Four
//    where they leave no more lanes idle: at two literals a clause (70000, R =
//    200: two 190, four 160; R = 288, half the lanes of a second segment idle: 264
//    / 286), at three from 30000 variables on in idle lanes (36000, R = 160:
//    126 / 120; 20000, ratio 8, R = 200: 122 / 131; 36000, R = 256: 153 / 166), at
//    four in idle lanes (36000, R = 160: 371 / 316; R = 256: 442 / 480).  In bf16
//    only at four literals (36000, R = 256: 309 / 275; three, R = 200: 120 / 172).  It
//    also stays at two rows (100000 variables, R = 64: four 198, two 182; 12000,
//    R = 200: 61 / 55), one row for longer in a single segment of two values
//    (12000, ratio 8, R = 76: two 49, one 45; in two segments, 5000, R = 200: one
//    30, two 28).
//  * MaxCut in float32 at R >= 256: up to eight replica segments, one per XCD,
//    while a segment of the marginals fits its 4 MB L2 (30000 rows, R = 256: 81
//    / 72; R = 512, 7.7 MB: 142 / 149) and segments are whole cache lines
//    (24000 rows, degree 40, R = 256: 142 / 106, 288: 202 / 173, but 200: 114 /
//    203, 300: 224 / 244).  Six and seven segments do not pin theirs to an
//    XCD (R = 192: 102 / 91, of degree 6 39 / 41; 224: 121 / 136, 45 / 50).
//  * Manipulated gradients (short rows of bits): two waves and one row up to
//    larger grids, 30000 rows of degree 20, R = 100: 38 / 31; several segments
//    of single values four waves and two rows (7861 rows, R = 225: 35.0 / 34.0).
//  * bMinCut: 32 lanes where that leaves a quarter fewer idle (R = 66, 8000
//    nodes, q = 16: 160 / 120), at q < 16 also where it leaves some fewer and 32
//    replicas of the marginals fit an XCD's L2 (R = 130, 2500 nodes, q = 4: 55 / 43;
//    but 30000 nodes, q = 2, 7.7 MB: 116 / 130, and R = 200, seven segments, 8000
//    nodes, q = 4: 135 / 162).  At q >= 16 a lane's states alone are a cache
//    line: up to 6500 nodes down to eight lanes (R = 100, 2400 nodes, q = 16: 86 / 56;
//    5000, q = 32, R = 66: 501 / 301), but not for q = 16 at about two waves (3500
//    nodes, R = 150: 217 / 258; R = 200: 316 / 281); from there to 10000 the gathers
//    of so many segments cost more than the idle lanes (8000, q = 32, R = 50:
//    338 / 399; q = 16, R = 33: 68 / 88); above, more than a wave of replicas takes
//    down to sixteen where each halving leaves some fewer idle (30000, q = 16, R =
//    100: 694 / 628, R = 66 with 32 451, with 16 432), and for q = 32 from 20000 on
//    less than a wave down to eight (30000, R = 24: 672 / 603; but 12000, R = 50:
//    507 / 580).  Rows of q = 32 are long: larger tiles from fewer blocks on (8000
//    nodes, R = 20, two rows 176, four 163).
//  * State past the Infinity Cache is not found there again: non-temporal
//    from 256 MB of state and marginals on (bMinCut 200000 nodes, q = 8, R = 16:
//    404 / 334; at exactly 256 MB, MaxCut 50000 rows, R = 256: 111 / 111).  With
//    manipulated gradients the copy is the read-out, a bit or a byte per (node,
//    replica): MaxCut 60000 rows, cached and non-temporal, R = 332 (244 MB) 146 /
//    172, R = 364 (267 MB) 176 / 175, R = 416 193 / 175.
inline TileShape default_shape(int kind, bool manip, int64_t n, int R, int q, int sat_k, int marg_bytes)
{
    TileShape t;
    const double vals = (double)n * R * (kind == KIND_BMINCUT ? q : 1);
    t.waves = 4;
    const double copy_bytes = !manip ? marg_bytes : kind == KIND_BMINCUT ? 1.0 / q : 0.125;   // per value
    t.nt = vals * (12 + 2 * copy_bytes) > 256e6 && !(kind == KIND_BMINCUT && q >= 16) ? 1 : 0;
    int cap = 4;
    double blocks = 1024;
    // share of the lanes of R's segments that hold a replica
    const auto used = [&](int l, int vec = 1) {
        const LaunchGeom g = make_geom(vec, R, t.waves, l);
        return (double)R / ((double)g.nseg * g.lanes * vec);
    };
    if (kind == KIND_BMINCUT) {
        blocks = q == 32 && n > 6500 ? 180 : 448;
        t.lanes = 64;
        const bool two_waves = q == 16 && n >= 2000 && R > 128 && R < 192;
        if (q >= 16 && (n <= 6500 ? !two_waves : n > 20000 && q == 32 && R <= 64)) {
            for (int l = 32; l >= 8; l >>= 1)
                if (used(l) > 1.05 * used(t.lanes)) t.lanes = l;
        } else if (q >= 16 && n > 10000 && R > 64 && !manip) {
            for (int l = 32; l >= 16; l >>= 1)
                if (used(l) >= 1.12 * used(t.lanes)) t.lanes = l;
        } else if (used(32) >= 1.3 * used(64) ||
                   (q < 16 && used(32) >= 1.15 * used(64) && (double)n * 32 * q * copy_bytes <= 2.6e6)) {
            t.lanes = 32;
        }
    } else if (kind == KIND_MAXSAT) {
        t.vec = R % 2 == 0 && (R > 64 || (R == 64 && vals >= 1e6)) ? 2 : 1;
        cap = 2;
        const double used4 = used(64, 4);
        if (R % 4 == 0 && R > 128 && used4 >= used(64, 2) &&
            (marg_bytes == 2 ? sat_k == 4 : sat_k == 2 || (used4 < 0.8 && (sat_k == 4 || n >= 30000))))
            t.vec = 4;
        if (t.vec == 4 || (t.vec == 2 && R <= 128)) blocks = 2048;
    } else if (manip) {
        t.vec = R % 4 == 0 && vals >= 4e5 ? 4 : R % 2 == 0 && vals >= 1e5 ? 2 : 1;
        const bool single = t.vec == 1 && R > 64;
        t.waves = single ? 4 : 2;
        blocks = single ? 2048 : 8192;
        cap = 2;
    } else {
        t.vec = R % 4 == 0 && (vals >= 4e6 || R >= 128) ? 4 : R % 2 == 0 && vals >= 2e5 ? 2 : 1;
        if (R >= 256 && R % 32 == 0 && marg_bytes == 4 && vals * 4 / 8 <= 4e6) {
            const int l = pow2ceil((R / t.vec + 7) / 8);
            t.lanes = l < 64 ? l : 64;
        }
    }
    const LaunchGeom g = make_geom(t.vec, R, t.waves, t.lanes);
    t.rows = 1;
    while (t.rows < cap && (double)n * g.nseg >= blocks * g.teams_per_block * 2 * t.rows) t.rows <<= 1;
    return t;
}

// Arguments shared by the step kernels.
struct StepArgs {
    const int64_t* row_off;
    const int2* adj;
    const int32_t* adj_pm1;       // the same entries in 4 bytes when every weight is +-1, else null
    const int2* inc2;
    const int4* inc4;
    const float* wdeg;
    const double* nrm;            // per-node sum_j |W_ij| (manipulated gradients)
    const int32_t* nw;            // bMinCut node weights (null: all 1)
    const Tile* tiles;
    const void* marg_cur;
    void* marg_nxt;
    float* h;                     // rows of h, m1, m2 are srow floats apart
    float* m1;
    float* m2;
    int64_t srow;
    float* grad;                  // may be null; [n][R(q)]
    double* epart;                // [n_tiles][NE][R] or null (no energies this step)
    const double* ctil;           // bMinCut: centred column sums C~ [inst][R][q]
    long long* cpart;             // bMinCut: column-sum partials of the new P [n_tiles][R][q]
    int32_t n;
    int32_t R;
    int32_t q;
    int32_t rw;                   // MaxCut manipulated: 32-bit words per row of the sign bits
    int32_t lanes_log2;
    int32_t seg_major;            // block -> (tile, segment) mapping of the grid
    StepScalars sc;
};

// record the text of a failure for fem_last_error() (fem_host.hip); returns st
int set_error(int st, const char* msg);

// host-side kernel launchers (fem_kernels.hip)
hipError_t launch_step(int kind, int dtype, int vec, bool nt, const LaunchGeom& g, int waves,
                       const StepArgs& a, hipStream_t st);
// marginal copy of a.h into a.marg_nxt; for bMinCut also the column-sum
// partials a.cpart.  src (dense [n][R] or [n][R][q] on the device, or null): new
// fields, which a.h is set to, with a.m1 and a.m2 cleared
hipError_t launch_init_marginals(int kind, int dtype, const LaunchGeom& g, int waves,
                                 const StepArgs& a, const float* src, hipStream_t st);
hipError_t launch_fill(size_t count, double x, double* out, hipStream_t st);
// out[inst][c] = sum over the instance's tiles of part[tile][c] (two fixed-order stages)
template <typename T>
hipError_t launch_seg_reduce(const T* part, int cols, const int32_t* chunk_off, int n_chunks,
                             const int32_t* inst_chunk_off, int n_inst, T* tmp, T* out,
                             hipStream_t st);
// What follows a step (energies, bMinCut column sums), from the per-tile
// partials of every instance.
struct FinishArgs {
    const double* epart;          // [tile or chunk][NE][R]
    const long long* cpart;       // [tile or chunk][R][q]
    const int32_t* inst_chunk_off;   // chunks of instance b: [inst_chunk_off[b], inst_chunk_off[b + 1])
    const int32_t* chunk_off;     // not null: the arrays are per tile, chunk c has [chunk_off[c], chunk_off[c + 1])
    const double* wtot;
    double* csum;                 // [inst][R][q]: cpart summed, times scale
    double* ctil;                 // csum minus its mean over the states
    double* eout;                 // [inst][3][R]: U, S, F of the step, with the csum before it
    double lam, beta;
    double scale;                 // 2^-40 for fixed-point marginal sums, 1 for state counts
    int32_t kind, R, q;
    uint32_t first;               // first workgroup of this launch (of every instance's replica groups)
};
// epart and cpart (cols 0: absent) summed per chunk of tiles
hipError_t launch_chunks(const double* epart, int ecols, const long long* cpart, int ccols, const int32_t* chunk_off,
                         int n_chunks, double* esum, long long* csum, hipStream_t st);
// max_tiles: most tiles (or chunks) of one instance
hipError_t launch_finish(FinishArgs a, int n_inst, int max_tiles, bool energies, bool columns, hipStream_t st);
// manipulated gradients (fem_manip.hip): the step kernel, and the read-out copy
// of a.h (sign bits or argmax states, with per-tile state counts for bMinCut)
hipError_t launch_manip_step(int kind, int vec, bool nt, const LaunchGeom& g, int waves, const StepArgs& a,
                             hipStream_t st);
hipError_t launch_manip_init(int kind, const LaunchGeom& g, int waves, const StepArgs& a, hipStream_t st);
hipError_t launch_round(int kind, int32_t n, int32_t R, int32_t q, const float* h, int64_t srow, uint8_t* sigma,
                        hipStream_t st);
// n rows of w floats: dst[i ds + c] = src[i ss + c] (src not null), and zeros
// into z1[i ds + c] and z2[i ds + c] (where not null)
hipError_t launch_rows(int32_t n, int64_t w, float* dst, int64_t ds, const float* src, int64_t ss, float* z1,
                       float* z2, hipStream_t st);
hipError_t launch_transpose_sigma(int32_t n, int32_t R, const int32_t* sig_rn, uint8_t* sig_nr,
                                  hipStream_t st);
hipError_t launch_eval(const Problem& p, const LaunchGeom& g, int waves, const Tile* tiles,
                       int32_t R, const uint8_t* sigma, double* vpart, int* spart,
                       hipStream_t st);
hipError_t launch_sizes_widen(size_t count, const int* in, long long* out, hipStream_t st);
// v2: bMinCut per-instance sum_i V_i^2 (the constant that makes the balance
// penalty vanish on a perfect split of unit weights)
hipError_t launch_best_update(int kind, int R, int n_inst, int q, double lam, const double* vout,
                              const long long* sout, const double* v2, double* best, hipStream_t st);

}  // namespace fem

// Problems are reference counted: every solver holds one reference, so a
// problem released by its owner stays alive until its last solver is gone.
struct fem_problem {
    fem::Problem p;
    std::mutex lock;   // of what follows: solvers may be made and destroyed by several threads
    int refs = 0;
    bool released = false;
    fem::ResTables* res = nullptr;
    ~fem_problem() { fem::resident_release(res); }
};
