// Resident anneals for small instances of the one-logit problems (MaxCut with
// explicit or manipulated gradients, Max-k-SAT).
//
// Replicas never exchange anything, so one workgroup can carry one replica of
// one instance through a whole range of steps: h and the moments stay in its
// registers, the values neighbours read in its LDS, and the adjacency in LDS
// too where it fits (else it streams from L2).  What bounds a step of a small
// instance on the row-tiled kernels is latency: a launch, a chain of dependent
// loads (row bounds, entries, neighbour rows) and one to four reduction
// launches, for microseconds of arithmetic.  Here a step is the arithmetic and
// the LDS reads of n rows on one compute unit, which is what bounds it: a
// gather is one add, one LDS read, one conversion and one double add.
//
// Rows are taken by falling degree, one lane per row, entries in slices of 64
// rows (lanes side by side, padded to the slice's longest row): a wave's
// lanes finish together, and entry loads are contiguous.  Every row sums its
// neighbours in CSR order in double, and the update is the tiled kernels', so
// the fields are bit-identical to theirs.
//
// Measured per step with energies in a long range (MI355X; resident / best of
// seven row-tiled shapes), MaxCut +-1 at R = 16 and R = 512:
//   n =  200, degree  20:  1.13 /  6.9 us    1.37 /  7.3 us
//   n =  800, degree  48:  3.00 /  8.5 us    5.85 / 13.6 us
//   n = 2000, degree  20:  3.31 /  8.2 us    6.38 / 15.9 us
//   n = 8000, degree   3:  6.38 /  8.9 us   12.8  / 32.6 us
// Max-3-SAT, 200 variables, 1200 clauses: 1.96 / 8.5 us and 2.36 / 9.7 us.
#include "fem_resident.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <numeric>
#include <utility>

#include "fem_device.h"
#include "fem_readout.h"

namespace fem {

// Values per plane (see ResCtx): the positions and two constant slots, which
// take the last two positions where the offsets end there.
__host__ __device__ constexpr int res_zero_slot(int npos) { return npos < RES_MAX_ROWS ? npos : RES_MAX_ROWS; }
__host__ __device__ constexpr int res_values(int npos) { return (res_zero_slot(npos) + 2 + 3) & ~3; }
// Up to four rows per thread the values are double-buffered (one barrier per
// step); beyond, LDS is kept for the entries and a step takes two barriers.
__host__ __device__ constexpr int res_buffers(int rpt) { return rpt <= 4 ? 2 : 1; }

// Element i of a table that no kernel writes, i uniform: through the constant
// address space, so that it is a scalar load whatever the kernel stores.
template <typename T>
__device__ __forceinline__ T uniform_at(const T* p, int i)
{
    constexpr int N = sizeof(T) / 4;
    struct Words {
        uint32_t w[N];
    } v;
    const auto* q = (const __attribute__((address_space(4))) uint32_t*)(p + i);
#pragma unroll
    for (int k = 0; k < N; ++k) v.w[k] = q[k];
    return __builtin_bit_cast(T, v);
}

// The parts of a resident kernel that do not depend on the problem kind.
//
// What neighbours read lies in planes of one float per position, chosen by
// the entry's own offset, so that a gather is an add, a load and the sum:
// MaxCut m and -m (the second only where a weight is -1), Max-k-SAT the
// probability that a negative and that a positive literal is false.
struct ResCtx {
    ResInst in;
    int r, T, tid, lane, wave, nwaves;
    char* m;              // [buffers][planes][values]
    int plane, buf;       // bytes per plane and per buffer
    double* part;         // [2][16][2] energy terms per wave
    uint2* adj;           // LDS copy of the entries
    float4* wgt;          // ... and of the weights
};

// One workgroup = one (instance, replica).  Consecutive workgroups go to the
// eight XCDs in turn, so an XCD gets a contiguous range of an instance's
// replicas: neighbours in the state rows share cache lines.
template <int RPT>
__device__ __forceinline__ void res_ctx(const ResArgs& a, char* lds, ResCtx& c)
{
    const int ii = blockIdx.x / a.R, k = blockIdx.x % a.R, x = k & 7;
    c.in = uniform_at(a.inst, ii);
    c.r = x * (a.R >> 3) + min(x, a.R & 7) + (k >> 3);
    c.T = blockDim.x;
    c.tid = threadIdx.x;
    c.lane = threadIdx.x & 63;
    c.wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    c.nwaves = blockDim.x >> 6;
    c.plane = res_values(c.in.npos) * 4;
    c.buf = c.plane * a.planes;
    c.part = reinterpret_cast<double*>(lds);
    c.m = lds + RES_PART_BYTES;
    c.adj = reinterpret_cast<uint2*>(c.m + res_buffers(RPT) * c.buf);
    c.wgt = reinterpret_cast<float4*>(c.adj + c.in.n_adj);
}

// x plus x of the lane that a row rotation by N lanes brings here
template <int N>
__device__ __forceinline__ double add_ror(double x)
{
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x120 + N, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x120 + N, 0xf, 0xf, true);
    return x + __longlong_as_double(((long long)hi << 32) | (uint32_t)lo);
}
__device__ __forceinline__ double row16_sum(double x) { return add_ror<1>(add_ror<2>(add_ror<4>(add_ror<8>(x)))); }

// The wave's sums of the two energy terms, in double and in a fixed order, to
// its slots of part: the lower half-wave sums the first term, the upper the
// second.
template <typename T>
__device__ __forceinline__ void res_partial(const ResCtx& c, int t, T e0, T e1)
{
    const bool up = c.lane >= 32;
    const T other = __shfl_xor(up ? e0 : e1, 32, 64);
    double x = row16_sum((double)(up ? e1 : e0) + (double)other);
    x += __shfl_xor(x, 16, 64);
    if ((c.lane & 31) == 0) c.part[((t & 1) * 16 + c.wave) * 2 + (up ? 1 : 0)] = x;
}

// Energies of step t from the waves' partial sums, after the step's barrier:
// formed by the last wave (the one with the fewest neighbours) while the
// others go on.
__device__ __forceinline__ void res_energy(const ResArgs& a, const ResCtx& c, int t)
{
    const int w = c.lane & 31;
    double x = w < c.nwaves ? c.part[((t & 1) * 16 + w) * 2 + (c.lane >> 5)] : 0.0;
    x = row16_sum(x);   // at most 16 waves: one row of lanes per term
    const long long b = __double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)b, 32);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), 32);
    const double S = __longlong_as_double(((long long)hi << 32) | lo);
    if (c.lane == 0) {
        const double U = a.kind == KIND_MAXCUT ? -a.wtot[c.in.inst] + 0.5 * x : x;
        double* o = a.eout + (t / a.energy_every) * a.erecord + (size_t)c.in.inst * 3 * a.R + c.r;
        o[0] = U;
        o[a.R] = S;
        o[2 * a.R] = U - S / uniform_at(a.steps, t).beta;
    }
}

__device__ __forceinline__ float lds_val(const char* m, uint32_t off) { return *reinterpret_cast<const float*>(m + off); }

// The gather of one row: sum_j W_ij m_j, four entries per round, CSR order.
// first: the first two rounds, already loaded (entries beyond a slice belong
// to the next one, or to the padding at the end of the array: never used).
template <bool UNIT>
struct ResRound {
    uint2 e;
    float4 w;   // weights, where they are not +-1
};
template <bool UNIT, typename AP, typename WP>
__device__ __forceinline__ ResRound<UNIT> res_round_at(AP ap, WP wp, int at)
{
    ResRound<UNIT> q;
    q.e = ap[at];
    if constexpr (!UNIT) q.w = wp[at];
    return q;
}
template <bool UNIT>
__device__ __forceinline__ double res_add(const char* m, const ResRound<UNIT>& q, double acc)
{
    const float v[4] = {lds_val(m, q.e.x & 0xffffu), lds_val(m, q.e.x >> 16), lds_val(m, q.e.y & 0xffffu),
                        lds_val(m, q.e.y >> 16)};
    if constexpr (UNIT) {
#pragma unroll
        for (int u = 0; u < 4; ++u) acc += (double)v[u];
    } else {
        acc = fma((double)q.w.x, (double)v[0], acc);
        acc = fma((double)q.w.y, (double)v[1], acc);
        acc = fma((double)q.w.z, (double)v[2], acc);
        acc = fma((double)q.w.w, (double)v[3], acc);
    }
    return acc;
}

__device__ __forceinline__ float res_bf16(float x, int bf16) { return bf16 ? bf16_to_f32(f32_to_bf16(x)) : x; }

// MaxCut: phi = sum_j W_ij m_j, g = P(1-P) [2 phi + h/beta] (maxcut_step_kernel),
// or with MANIP m_j = +-1 the read-out, g = gamma P(1-P) [c phi + h/beta]
// (maxcut_manip_kernel).  UNIT: weights +-1, the sign in the entry's plane.
template <int RPT, bool MANIP, bool UNIT, bool ALDS>
__global__ void __launch_bounds__(1024) res_maxcut_kernel(ResArgs a)
{
    extern __shared__ __align__(16) char lds[];
    constexpr bool TWO = res_buffers(RPT) == 2;
    ResCtx c;
    res_ctx<RPT>(a, lds, c);
    // per row: the state, e = exp(-|h|) and 1/(1 + e), the normaliser
    float h[RPT], m1[RPT], m2[RPT], ex[RPT], rc[RPT];
    double cn[MANIP ? RPT : 1];
    int row[RPT];
    int2 sl[RPT];
    const bool signs = a.planes == 2;
    // the value neighbours read of row k, into the buffer at m
    auto publish = [&](char* m, int k) {
        float v;
        if constexpr (MANIP) {
            v = h[k] > 0.0f ? 1.0f : -1.0f;
        } else {
            v = res_bf16(tanh_half(h[k], ex[k], rc[k]), a.bf16);
        }
        float* p = reinterpret_cast<float*>(m) + k * c.T + c.tid;
        *p = v;
        if (signs) *reinterpret_cast<float*>(reinterpret_cast<char*>(p) + c.plane) = -v;
    };
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        row[k] = a.perm[c.in.pos0 + k * c.T + c.tid];
        sl[k] = uniform_at(a.slice, c.in.slice0 + k * c.nwaves + c.wave);
        h[k] = m1[k] = m2[k] = ex[k] = rc[k] = 0.0f;
        if constexpr (MANIP) cn[k] = 0.0;
        if (row[k] >= 0) {
            const size_t s = (size_t)row[k] * a.srow + c.r;
            h[k] = a.h[s];
            m1[k] = a.m1[s];
            m2[k] = a.m2[s];
            if constexpr (MANIP) {
                const double l1 = a.nrm[row[k]];
                cn[k] = l1 > 0.0 ? 1.0 / l1 : 0.0;
            }
            publish(c.m + (TWO ? (a.t0 & 1) * c.buf : 0), k);
        }
    }
    if (c.tid < res_buffers(RPT))
        reinterpret_cast<float*>(c.m + c.tid * c.buf)[res_zero_slot(c.in.npos)] = 0.0f;
    if constexpr (ALDS) {
        for (int k = c.tid; k < c.in.n_adj; k += c.T) {
            c.adj[k] = a.adj[c.in.adj0 + k];
            if constexpr (!UNIT) c.wgt[k] = a.wgt[c.in.adj0 + k];
        }
    }
    __syncthreads();
    StepScalars sc = uniform_at(a.steps, a.t0).sc;
    for (int t = a.t0; t < a.t1; ++t) {
        const bool en = !MANIP && a.energy_every > 0 && t % a.energy_every == 0;
        const bool last = t + 1 == a.t1;
        const char* mc = c.m + (TWO ? (t & 1) * c.buf : 0);
        char* mn = c.m + (TWO ? ((t & 1) ^ 1) * c.buf : 0);
        float e0 = 0.0f, e1 = 0.0f;
        auto field = [&](int k, const ResRound<UNIT>& q0, const ResRound<UNIT>& q1) -> double {
            double acc = 0.0;
            const int rounds = sl[k].y;
            if constexpr (ALDS) {
                const uint2* ap = c.adj + sl[k].x * 64 + c.lane;
                const float4* wp = c.wgt + sl[k].x * 64 + c.lane;
#pragma unroll 4
                for (int g = 0; g < rounds; ++g) acc = res_add<UNIT>(mc, res_round_at<UNIT>(ap, wp, g * 64), acc);
            } else if constexpr (!UNIT) {
                const uint2* ap = a.adj + c.in.adj0 + sl[k].x * 64 + c.lane;
                const float4* wp = a.wgt + c.in.adj0 + sl[k].x * 64 + c.lane;
#pragma unroll 2
                for (int g = 0; g < rounds; ++g) acc = res_add<UNIT>(mc, res_round_at<UNIT>(ap, wp, g * 64), acc);
            } else {
                // entries from L2: two rounds ahead
                const uint2* ap = a.adj + c.in.adj0 + sl[k].x * 64 + c.lane;
                const float4* wp = nullptr;
                ResRound<UNIT> x0 = q0, x1 = q1;
                for (int g = 0; g < rounds; g += 2) {
                    const ResRound<UNIT> n0 = res_round_at<UNIT>(ap, wp, (g + 2) * 64);
                    const ResRound<UNIT> n1 = res_round_at<UNIT>(ap, wp, (g + 3) * 64);
                    acc = res_add<UNIT>(mc, x0, acc);
                    if (g + 1 < rounds) acc = res_add<UNIT>(mc, x1, acc);
                    x0 = n0;
                    x1 = n1;
                }
            }
            return acc;
        };
        auto first = [&](int k, int g) -> ResRound<UNIT> {
            ResRound<UNIT> q{};
            q.e = a.adj[c.in.adj0 + (sl[k].x + g) * 64 + c.lane];
            return q;
        };
        // the update of row k from its field
        auto update = [&](int k, double acc) {
            const float x = h[k], e = MANIP ? exp_neg(fabsf(x)) : ex[k];
            const float r = MANIP ? rcp_f(1.0f + e) : rc[k];
            const float pmin = e * r;   // min(P, 1 - P)
            const float pq = pmin * r;  // P (1 - P)
            float g;
            if constexpr (MANIP) g = (float)(sc.gamma_d * ((double)pq * (cn[k] * acc + (double)x * sc.inv_beta_d)));
            else g = (float)((double)pq * fma((double)x, sc.inv_beta_d, 2.0 * acc));
            if (en && row[k] >= 0) {
                const float m_own = copysignf((1.0f - e) * r, x);
                e0 += (float)((double)m_own * acc);
                e1 += log1p_f(e) + fabsf(x) * pmin;
            }
            h[k] = adam_update(x, g, m1[k], m2[k], sc);
            if (row[k] >= 0) {
                publish(mn, k);
                if (last && a.grad) a.grad[(size_t)row[k] * a.R + c.r] = g;
            }
        };
        ResRound<UNIT> q0{}, q1{};
        if constexpr (!ALDS && UNIT) {
            q0 = first(0, 0);
            q1 = first(0, 1);
        }
        double acc[RPT];
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            if ((k * c.nwaves + c.wave) * 64 >= c.in.n) continue;   // no rows in this slice
            ResRound<UNIT> n0{}, n1{};
            if constexpr (!ALDS && UNIT) {
                const int kn = k + 1 < RPT ? k + 1 : k;   // the next row's first rounds
                n0 = first(kn, 0);
                n1 = first(kn, 1);
            }
            acc[k] = field(k, q0, q1);
            q0 = n0;
            q1 = n1;
            if constexpr (TWO) update(k, acc[k]);
        }
        if constexpr (TWO) {
            if (en) res_partial(c, t, e0, e1);
        } else {
            __syncthreads();   // every gather has read the old values
            // at most four float32 terms to a sum, as on the row-tiled kernels
            double f0 = 0.0, f1 = 0.0;
#pragma unroll
            for (int k = 0; k < RPT; ++k) {
                if ((k * c.nwaves + c.wave) * 64 < c.in.n) update(k, acc[k]);
                if (k % 4 == 3) {
                    f0 += (double)e0;
                    f1 += (double)e1;
                    e0 = e1 = 0.0f;
                }
            }
            if (en) res_partial(c, t, f0, f1);
        }
        sc = uniform_at(a.steps, t + 1).sc;   // the table has an entry beyond the last step
        __syncthreads();
        if (en && c.wave == c.nwaves - 1) res_energy(a, c, t);
    }
#pragma unroll
    for (int k = 0; k < RPT; ++k)
        if (row[k] >= 0) {
            const size_t s = (size_t)row[k] * a.srow + c.r;
            a.h[s] = h[k];
            a.m1[s] = m1[k];
            a.m2[s] = m2[k];
        }
}

// Max-k-SAT (sat_step_kernel): W other literals per incidence; 8 bytes hold
// two incidences of two literals or one of three.  Bit 31 of the first word
// of an incidence is its own literal's sign, bit 15 marks the clause's owner.
template <int RPT, int W, bool ALDS>
__global__ void __launch_bounds__(1024) res_sat_kernel(ResArgs a)
{
    extern __shared__ __align__(16) char lds[];
    ResCtx c;
    res_ctx<RPT>(a, lds, c);
    float h[RPT], m1[RPT], m2[RPT], ex[RPT], rc[RPT];
    int row[RPT];
    int2 sl[RPT];
    // the probabilities that a negative and a positive literal of row k are
    // false, from the stored form of its marginal
    auto publish = [&](char* m, int k) {
        ex[k] = exp_neg(fabsf(h[k]));
        rc[k] = rcp_f(1.0f + ex[k]);
        const float small = ex[k] * rc[k];   // sat_encode
        const float s = res_bf16(h[k] > 0.0f ? -small : small, a.bf16);
        float* p = reinterpret_cast<float*>(m) + k * c.T + c.tid;
        *p = sat_u_bits(s, 0u);
        *reinterpret_cast<float*>(reinterpret_cast<char*>(p) + c.plane) = sat_u_bits(s, SAT_POS);
    };
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        row[k] = a.perm[c.in.pos0 + k * c.T + c.tid];
        sl[k] = uniform_at(a.slice, c.in.slice0 + k * c.nwaves + c.wave);
        h[k] = m1[k] = m2[k] = ex[k] = rc[k] = 0.0f;
        if (row[k] >= 0) {
            const size_t s = (size_t)row[k] * a.srow + c.r;
            h[k] = a.h[s];
            m1[k] = a.m1[s];
            m2[k] = a.m2[s];
            publish(c.m + (a.t0 & 1) * c.buf, k);
        }
    }
    // a padding record has a literal that is false with probability 0, an
    // unused literal slot the factor 1
    if (c.tid < 2) {
        float* z = reinterpret_cast<float*>(c.m + c.tid * c.buf) + res_zero_slot(c.in.npos);
        z[0] = 0.0f;
        z[1] = 1.0f;
    }
    if constexpr (ALDS)
        for (int k = c.tid; k < c.in.n_adj; k += c.T) c.adj[k] = a.adj[c.in.adj0 + k];
    __syncthreads();
    StepScalars sc = uniform_at(a.steps, a.t0).sc;
    for (int t = a.t0; t < a.t1; ++t) {
        const bool en = a.energy_every > 0 && t % a.energy_every == 0;
        const bool last = t + 1 == a.t1;
        const char* mc = c.m + (t & 1) * c.buf;
        char* mn = c.m + ((t & 1) ^ 1) * c.buf;
        float e0 = 0.0f, e1 = 0.0f;
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            if ((k * c.nwaves + c.wave) * 64 >= c.in.n) continue;   // no rows in this slice
            const int base = sl[k].x * 64 + c.lane;
            const float x = h[k];
            const float pmin = ex[k] * rc[k];   // min(P, 1 - P)
            const float pq = pmin * rc[k];      // P (1 - P)
            // own literal false, by its sign
            const float u_neg = x > 0.0f ? 1.0f - pmin : pmin, u_pos = x > 0.0f ? pmin : 1.0f - pmin;
            double d = 0.0;
            auto add = [&](float cv, uint32_t e) {
                d += (double)__uint_as_float(__float_as_uint(cv) ^ (e & 0x80000000u));
                if (en) {
                    const float uo = (int)e < 0 ? u_pos : u_neg;
                    e0 += (e & 0x8000u) ? uo * cv : 0.0f;
                }
            };
            const uint2* ap = ALDS ? c.adj + base : a.adj + c.in.adj0 + base;
#pragma unroll 4
            for (int g = 0; g < sl[k].y; ++g) {
                const uint2 q = ap[g * 64];
                const uint32_t p = q.x & 0x7fff7fffu, o = q.y & 0x7fff7fffu;
                if constexpr (W == 2) {
                    add(lds_val(mc, p & 0xffffu) * lds_val(mc, p >> 16), q.x);
                    add(lds_val(mc, o & 0xffffu) * lds_val(mc, o >> 16), q.y);
                } else {
                    float cv = lds_val(mc, p & 0xffffu) * lds_val(mc, p >> 16);
                    cv *= lds_val(mc, o & 0xffffu);
                    add(cv, q.x);
                }
            }
            const float g = (float)(sc.gamma_d * ((double)pq * fma((double)x, sc.inv_beta_d, d)));
            if (en && row[k] >= 0) e1 += log1p_f(ex[k]) + fabsf(x) * pmin;
            h[k] = adam_update(x, g, m1[k], m2[k], sc);
            if (row[k] >= 0) {
                publish(mn, k);
                if (last && a.grad) a.grad[(size_t)row[k] * a.R + c.r] = g;
            }
        }
        if (en) res_partial(c, t, e0, e1);
        sc = uniform_at(a.steps, t + 1).sc;   // the table has an entry beyond the last step
        __syncthreads();
        if (en && c.wave == c.nwaves - 1) res_energy(a, c, t);
    }
#pragma unroll
    for (int k = 0; k < RPT; ++k)
        if (row[k] >= 0) {
            const size_t s = (size_t)row[k] * a.srow + c.r;
            a.h[s] = h[k];
            a.m1[s] = m1[k];
            a.m2[s] = m2[k];
        }
}

// ------------------------------------------------------------------- host --
// Workgroup, entries and LDS of an instance.
struct ResPlan {
    int threads = 64, rpt = 1;
    int64_t n_adj = 0;       // entries of 8 bytes, padding included
    size_t lds = 0;          // energy terms, values and (adj_lds) entries
    bool adj_lds = false;
    bool ok = false;
};

// per: incidences or adjacency entries in 8 bytes
static int res_per(const Problem& p) { return p.kind != KIND_MAXSAT ? 4 : p.sat_width == 2 ? 2 : 1; }

// The plan of instance b; its rows by falling degree (ties by index) are
// appended to perm, padded to the positions.
static ResPlan res_plan(const Problem& p, int b, int planes, bool unit, size_t dev_lds, std::vector<int32_t>& count,
                        std::vector<int32_t>& perm)
{
    ResPlan r;
    const bool sat = p.kind == KIND_MAXSAT;
    const int32_t row0 = p.inst_off[(size_t)b];
    const int64_t n = p.inst_off[(size_t)b + 1] - row0;
    if (p.kind == KIND_BMINCUT || n > (sat ? RES_MAX_ROWS_SAT : RES_MAX_ROWS)) return r;
    while (r.threads < n && r.threads < 1024) r.threads <<= 1;
    while ((int64_t)r.rpt * r.threads < n) r.rpt <<= 1;
    const int64_t* ro = p.h_row_off.data() + row0;
    const int per = res_per(p);
    if (ro[n] - ro[0] > RES_MAX_STREAM * per) return r;   // no arrangement of so many is accepted
    // by counting: degrees are few, and the rows keep their order
    int64_t most = 0;
    for (int64_t i = 0; i < n; ++i) most = std::max(most, ro[i + 1] - ro[i]);
    count.assign((size_t)most + 2, 0);
    for (int64_t i = 0; i < n; ++i) ++count[(size_t)(most - (ro[i + 1] - ro[i]) + 1)];
    for (int64_t d = 0; d <= most; ++d) count[(size_t)d + 1] += count[(size_t)d];
    const size_t base = perm.size();
    perm.resize(base + (size_t)r.threads * r.rpt, -1);
    for (int64_t i = 0; i < n; ++i)
        perm[base + (size_t)count[(size_t)(most - (ro[i + 1] - ro[i]))]++] = row0 + (int32_t)i;
    for (int64_t s = 0; s < n; s += 64) {
        const int64_t i = perm[base + (size_t)s] - row0;
        r.n_adj += (ro[i + 1] - ro[i] + per - 1) / per * 64;
    }
    r.lds = RES_PART_BYTES + (size_t)res_buffers(r.rpt) * planes * res_values(r.threads * r.rpt) * 4;
    const size_t with = r.lds + (size_t)r.n_adj * (unit ? 8 : 24);
    r.adj_lds = with <= dev_lds;
    if (r.adj_lds) r.lds = with;
    r.ok = r.lds <= dev_lds && (r.rpt <= 4 || (unit && r.adj_lds));
    if (!r.adj_lds && r.n_adj > RES_MAX_STREAM) r.ok = false;
    return r;
}

// The plan of all instances, larger ones first: the longest workgroups start
// first.
static void res_plan_all(const Problem& p, ResTables& t)
{
    t.planned = true;
    const bool sat = p.kind == KIND_MAXSAT;
    if (p.kind == KIND_BMINCUT || p.dense_w ||
        hipDeviceGetAttribute(&t.dev_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, p.device) != hipSuccess)
        return;
    auto rows_of = [&](int b) { return (int)(p.inst_off[(size_t)b + 1] - p.inst_off[(size_t)b]); };
    std::vector<int> ids((size_t)p.n_inst);
    std::iota(ids.begin(), ids.end(), 0);
    std::stable_sort(ids.begin(), ids.end(), [&](int x, int y) { return rows_of(x) > rows_of(y); });
    if (rows_of(ids[0]) > (sat ? RES_MAX_ROWS_SAT : RES_MAX_ROWS)) return;
    t.pm1 = !sat && p.adj_pm1 != nullptr;
    t.planes = sat ? 2 : 1;
    for (size_t k = 0; t.pm1 && t.planes == 1 && k < p.h_adj.size(); ++k)
        if ((uint32_t)p.h_adj[k].y & 0x80000000u) t.planes = 2;
    std::vector<int32_t> count;
    int64_t adj0 = 0;
    int32_t slice0 = 0;
    t.fits = true;
    for (int b : ids) {
        ResInst in{};
        in.pos0 = (int32_t)t.h_perm.size();
        const ResPlan plan = res_plan(p, b, t.planes, t.pm1 || sat, (size_t)t.dev_lds, count, t.h_perm);
        if (!plan.ok || t.h_perm.size() > (size_t)INT32_MAX) {   // positions are 32-bit
            t = ResTables{};
            t.planned = true;
            return;
        }
        if (t.classes.empty() || t.classes.back().threads != plan.threads || t.classes.back().rpt != plan.rpt ||
            t.classes.back().adj_lds != plan.adj_lds) {
            ResClass c;
            c.threads = plan.threads;
            c.rpt = plan.rpt;
            c.first = (int)t.h_inst.size();
            c.adj_lds = plan.adj_lds;
            t.classes.push_back(c);
        }
        t.classes.back().n_inst++;
        t.classes.back().rows = std::max(t.classes.back().rows, rows_of(b));
        t.classes.back().lds = std::max(t.classes.back().lds, plan.lds);
        if (!plan.adj_lds) t.classes.back().stream = std::max(t.classes.back().stream, plan.n_adj);
        t.threads += (uint64_t)plan.threads;
        in.inst = b;
        in.n = rows_of(b);
        in.npos = plan.threads * plan.rpt;
        in.slice0 = slice0;
        in.n_adj = (int32_t)plan.n_adj;
        in.adj0 = adj0;
        slice0 += in.npos / 64;
        adj0 += plan.n_adj;
        t.h_inst.push_back(in);
    }
}

void resident_release(ResTables* t)
{
    if (t && t->block) (void)hipFree(t->block);
    delete t;
}

// The tables of a plan: per row its entries, as the kernels read them.
static hipError_t res_build(const Problem& p, ResTables& t)
{
    const bool sat = p.kind == KIND_MAXSAT, unit = sat || t.pm1;
    const int per = res_per(p);
    const ResInst& end = t.h_inst.back();
    const size_t n_slice = (size_t)end.slice0 + end.npos / 64;
    // entries are read two rounds ahead
    const size_t n_adj = (size_t)end.adj0 + end.n_adj + 4 * 64;
    size_t bytes = 0;
    auto take = [&](size_t b) {
        const size_t at = bytes;
        bytes = (bytes + b + 255) & ~(size_t)255;
        return at;
    };
    const size_t o_inst = take(t.h_inst.size() * sizeof(ResInst)), o_perm = take(t.h_perm.size() * 4),
                 o_slice = take(n_slice * sizeof(int2)), o_adj = take(n_adj * sizeof(uint2)),
                 o_wgt = take(unit ? 0 : n_adj * sizeof(float4));
    std::vector<char> host(bytes);
    std::memcpy(host.data() + o_inst, t.h_inst.data(), t.h_inst.size() * sizeof(ResInst));
    std::memcpy(host.data() + o_perm, t.h_perm.data(), t.h_perm.size() * 4);
    int2* slice = reinterpret_cast<int2*>(host.data() + o_slice);
    uint2* adj = reinterpret_cast<uint2*>(host.data() + o_adj);
    float4* wgt = unit ? nullptr : reinterpret_cast<float4*>(host.data() + o_wgt);
    std::vector<uint32_t> pos;   // byte offset of a row's value
    for (const ResInst& in : t.h_inst) {
        const int32_t row0 = p.inst_off[(size_t)in.inst];
        const int32_t* perm = t.h_perm.data() + in.pos0;
        const int64_t* ro = p.h_row_off.data();
        pos.resize((size_t)in.n);
        for (int k = 0; k < in.n; ++k) pos[(size_t)(perm[k] - row0)] = (uint32_t)k << 2;
        auto at = [&](uint32_t row) { return pos[(size_t)row - (size_t)row0]; };
        const uint32_t zero = (uint32_t)res_zero_slot(in.npos) << 2, one = zero + 4;
        const uint32_t plane = (uint32_t)res_values(in.npos) << 2;
        auto lit = [&](uint32_t l) {   // a literal slot of an incidence record
            const uint32_t var = l & SAT_VAR_MASK;
            if (var == SAT_NONE) return one;
            return at(var) + ((l & SAT_POS) ? plane : 0u);
        };
        auto sat_word = [&](uint32_t s0, uint32_t s1, bool own_pos, bool owner) {
            return lit(s0) | (lit(s1) << 16) | (owner ? 0x8000u : 0u) | (own_pos ? 0x80000000u : 0u);
        };
        // entry g of the row [q, q1), 8 bytes
        auto pack = [&](int64_t q, int64_t q1, float* wf) {
            if (!sat) {
                uint32_t w[4];
                for (int u = 0; u < 4; ++u, ++q) {
                    w[u] = zero;
                    if (q < q1) {
                        const int2 ad = p.h_adj[(size_t)q];
                        w[u] = at((uint32_t)ad.x) + (t.pm1 && ad.y < 0 ? plane : 0u);
                        if (wf) std::memcpy(&wf[u], &ad.y, 4);
                    }
                }
                return make_uint2(w[0] | w[1] << 16, w[2] | w[3] << 16);
            }
            if (p.sat_width == 2) {
                uint32_t w[2];
                for (int u = 0; u < 2; ++u, ++q) {
                    w[u] = zero | (one << 16);
                    if (q < q1) {
                        const uint32_t x = (uint32_t)p.h_inc2[(size_t)q].x, y = (uint32_t)p.h_inc2[(size_t)q].y;
                        w[u] = sat_word(x & ~SAT_FLAG, y & ~SAT_FLAG, x & SAT_FLAG, y & SAT_FLAG);
                    }
                }
                return make_uint2(w[0], w[1]);
            }
            if (q >= q1) return make_uint2(zero | (one << 16), one);
            const int4 rec = p.h_inc4[(size_t)q];
            return make_uint2(sat_word((uint32_t)rec.x, (uint32_t)rec.y, rec.w & 1, rec.w & 2), lit((uint32_t)rec.z));
        };
        int first = 0;   // round of the instance
        for (int s = 0; s < in.npos / 64; ++s) {
            const int64_t i = perm[s * 64];   // the slice's longest row
            const int rounds = i < 0 ? 0 : (int)((ro[i + 1] - ro[i] + per - 1) / per);
            slice[in.slice0 + s] = make_int2(first, rounds);
            uint2* a = adj + in.adj0 + (size_t)first * 64;
            for (int l = 0; l < 64 && rounds > 0; ++l) {
                const int32_t row = perm[s * 64 + l];
                const int64_t q0 = row < 0 ? 0 : ro[row], q1 = row < 0 ? 0 : ro[row + 1];
                for (int g = 0; g < rounds; ++g) {
                    const size_t e = (size_t)g * 64 + l;
                    a[e] = pack(q0 + (int64_t)g * per, q1, wgt ? &wgt[in.adj0 + first * 64 + (int64_t)e].x : nullptr);
                }
            }
            first += rounds;
        }
    }
    char* d = nullptr;
    hipError_t e = hipMalloc(reinterpret_cast<void**>(&d), bytes);
    if (e != hipSuccess) return e;
    if ((e = hipMemcpy(d, host.data(), bytes, hipMemcpyHostToDevice)) != hipSuccess) {
        (void)hipFree(d);
        return e;
    }
    t.block = d;
    t.inst = reinterpret_cast<ResInst*>(d + o_inst);
    t.perm = reinterpret_cast<int32_t*>(d + o_perm);
    t.slice = reinterpret_cast<int2*>(d + o_slice);
    t.adj = reinterpret_cast<uint2*>(d + o_adj);
    t.wgt = reinterpret_cast<float4*>(d + o_wgt);
    std::vector<ResInst>().swap(t.h_inst);
    std::vector<int32_t>().swap(t.h_perm);
    return hipSuccess;
}

// The rule: an instance is resident if its rows fit the registers of one
// workgroup (RES_MAX_ROWS) and its entries fit LDS beside the values, or
// number at most RES_MAX_STREAM and stream from L2.  A batch is resident if
// each of its instances is: beside row-tiled instances a resident one saves no
// launch (R = 20, bfloat16, 2000 and 11361 nodes: 457 us for 24 steps, both
// row-tiled 368; sixty-four of 1000 .. 50000 nodes at R = 32: 4035 and 3869 for
// 25).
// In LDS it won at every size measured (the table above).  Streaming, one
// compute unit reads all entries while the row-tiled kernels read them from the
// whole chip, which pays as long as few replicas leave most of it idle: the more
// rows, the fewer entries.  us a step, resident / row-tiled, R = 16 and R = 64:
//                                     explicit            manipulated
//   n = 1000, +-1,    62 k entries   12.3/14.6 12.4/15.1  11.8/18.7 12.0/19.7
//   n = 2000, +-1,    50 k           11.0/10.9 11.1/13.7  10.4/10.4 10.7/13.2
//   n = 4000, +-1,    32 k            8.5/9.3   8.7/15.6   7.8/6.5   8.0/8.2
//   n = 4000, +-1,    48 k           11.4/9.8  11.6/17.4  10.7/7.5  11.0/9.5
//   n = 1000, others, 62 k           16.9/15.0 17.0/15.5  16.4/18.9 16.6/19.7
//   n = 2000, others, 30 k            8.8/9.8   8.9/12.6   8.4/7.9   8.6/9.7
//   n = 2000, others, 50 k           13.5/11.3 13.7/14.6  13.2/10.6 13.6/13.2
//   n = 4000, others, 24 k            7.9/9.1   8.2/14.0   7.2/5.7   7.5/7.1
//   n = 4000, others, 48 k           13.7/9.8  13.8/17.1  13.0/7.6  13.4/9.4
//   n = 4000, 3-SAT,  45 k           13.4/11.5 13.7/17.4
// (R = 128, n = 4000, 48 k: 12.1/20.7 and 11.3/12.1; R = 24 and 40, +-1 11.6/12.1
// 11.6/15.2, others 13.3/12.9 13.3/15.9; n = 4000, others, 25 k, R = 16 8.1/9.7, 29 k
// 9.8/9.7).  So RES_MAX_STREAM entries of one row per thread, three quarters of
// two, half of four (a quarter with manipulated gradients, three fifths for
// Max-k-SAT), times three quarters for other weights (nine tenths of four rows with
// explicit gradients), and more the more of the chip the row-tiled kernels need: a
// quarter more from R = 24, twice from 40 (manipulated from 64), four times from
// 128 on.  Eight rows per thread are instantiated only where they fit the
// registers: +-1 weights, entries in LDS.
// A launch has a workgroup per (instance, replica), and HIP takes fewer than
// 2^32 threads.
//
// Every launch loads the state (a cache line for each float of it) and the
// entries again, so short ranges, of the caller or between read-outs, stay
// row-tiled.  us a step of ranges of 1, 2, 4, 8 and 16 steps, resident, and
// row-tiled at any of them:
//   n =  200, degree 20, R =  64:   5.8   3.8   2.6   1.9   1.7    8.3
//   n =  800, degree 48, R = 512:  24.2  15.1  10.5   8.4   7.3   14.8
//   n = 2000, degree 20, R =  16:  16.0   9.9   6.8   5.1   4.3    9.0
//   n = 2000, degree 20, R = 512:  41.3  24.1  15.4  11.2   9.1   16.3
//   n = 4000, degree  6, R =  16:  25.6  14.9   9.4   6.7   5.3    9.5
//   n = 4000, 16800 clauses, 16:   29.6  19.3  14.3  11.5  10.1   10.8
//   n = 8000, degree  3, R =  16:  46.6  26.9  16.6  11.7   9.1   10.5
//   n = 8000, degree  3, R = 256:  69.6  38.3  22.7  14.8  11.0   22.6
// so one step where the workgroup is not the largest, else by the rows: 1.5 steps
// for each 1024, 0.75 where the replicas fill the chip and are not more than it
// holds (n = 4000, degree 6, R = 64: 27.7 15.7 10.2 7.0 5.4, row-tiled 12.6), one for
// a single replica, whose lines of state are shared by rows, less half a step (n =
// 3000, R = 1: 11.9 7.6 5.5 4.2 3.7, row-tiled 7.9; 1200: 6.8 4.3 3.1, 8.1).  Twice
// as many with manipulated gradients, whose row-tiled kernels gather bits (n =
// 2000, R = 16: 16.6 9.7 6.4 4.7 3.9, row-tiled 5.7) and fill the chip later; with
// eight rows per thread and few replicas they are the faster ones at any length
// (n = 8000, degree 4, R = 16, 32 steps 6.3, row-tiled 5.0).
// Several classes are several launches, in turn until a solver has side streams
// (make_side_streams).  us a step of 8, 16 and 48 steps in turn, of 96 side by
// side, and row-tiled:
//   2 sizes, 1100 and 2500, R =   8:  8.1  6.1  4.7   2.9    9.1 .. 10
//   5 sizes, 100 .. 3000,   R =   8:       10.6  8.6   5.4    9.2
//                           R =  50:       11.2  8.7   4.4   12
//                           R = 200: 16.8 12.1  9.0   8.4   20
//   8 sizes, 40 .. 6000,    R =   8:       21.5 17.9   8.8    9.3
//                           R =  50:       22.5 17.9  14.5   16
//                           R = 200:       24.2 18.4  15.1   29
// A read-out by bytes is five launches, which a graph of row-tiled steps replays
// faster (67 nodes, real weights, R = 1, every step: 19.4 / 13).
hipError_t resident_choose(fem_problem& fp, int R, bool manip, int eval_every, ResData& r)
{
    const Problem& p = fp.p;
    std::lock_guard<std::mutex> lock(fp.lock);
    if (!fp.res) fp.res = new ResTables;
    ResTables& t = *fp.res;
    if (!t.planned) {
        ResTables plan;   // whole or, where host memory runs out, not at all
        res_plan_all(p, plan);
        t = std::move(plan);
    }
    if (!t.fits || t.threads * (uint64_t)R > UINT32_MAX) return hipSuccess;
    const size_t classes = t.classes.size();
    int steps = classes == 1 ? 1 : classes <= 3 || (classes <= 5 && R >= 128) ? 8 : R >= 128 ? 16 : classes <= 5 ? 24 : 48;
    const ResClass& big = t.classes.front();
    if (big.threads == 1024) {
        const double f = R == 1 ? 1.0 : R > 256 || R < (manip ? 128 : 64) ? 1.5 : 0.75;
        const double rows = big.rows / 1024.0 - (R == 1 ? 0.5 : 0.0);
        steps = std::max(steps, (int)std::ceil(f * (manip ? 2 : 1) * rows));
    }
    if ((manip && big.rpt == 8 && R < 64) || (classes > 5 && R < 32)) return hipSuccess;
    if (eval_every > 0 && eval_every < std::max(steps, bit_evaluation(p) ? 1 : 4)) return hipSuccess;
    for (const ResClass& c : t.classes) {
        const bool sat = p.kind == KIND_MAXSAT;
        const double rows = c.rpt == 1 ? 1.0 : c.rpt == 2 ? 0.75 : sat ? 0.6 : manip ? 0.25 : 0.5;
        const double weights = t.pm1 || sat ? 1.0 : c.rpt == 4 && !manip ? 0.9 : 0.75;
        const double fill = R >= 128 ? 4.0 : R >= (manip ? 64 : 40) ? 2.0 : R >= 24 && !manip ? 1.25 : 1.0;
        const double limit = rows * weights * fill;
        if ((double)c.stream > limit * (double)RES_MAX_STREAM) return hipSuccess;
    }
    if (!t.block) {
        const hipError_t e = res_build(p, t);
        if (e != hipSuccess) return e;
    }
    r.t = &t;
    r.min_steps = steps;
    r.all = true;
    return hipSuccess;
}

typedef void (*ResKernel)(ResArgs);

template <bool MANIP, bool PM1, bool ALDS>
static ResKernel maxcut_kernel(int rpt)
{
    switch (rpt) {
    case 1: return res_maxcut_kernel<1, MANIP, PM1, ALDS>;
    case 2: return res_maxcut_kernel<2, MANIP, PM1, ALDS>;
    case 4: return res_maxcut_kernel<4, MANIP, PM1, ALDS>;
    case 8:
        if constexpr (PM1 && ALDS) return res_maxcut_kernel<8, MANIP, PM1, ALDS>;
        return nullptr;
    default: return nullptr;
    }
}

template <int W, bool ALDS>
static ResKernel sat_kernel(int rpt)
{
    switch (rpt) {
    case 1: return res_sat_kernel<1, W, ALDS>;
    case 2: return res_sat_kernel<2, W, ALDS>;
    case 4: return res_sat_kernel<4, W, ALDS>;
    default: return nullptr;
    }
}

template <bool ALDS>
static ResKernel pick(const Problem& p, bool pm1, bool manip, int rpt)
{
    if (p.kind == KIND_MAXSAT) return p.sat_width == 2 ? sat_kernel<2, ALDS>(rpt) : sat_kernel<3, ALDS>(rpt);
    if (manip) return pm1 ? maxcut_kernel<true, true, ALDS>(rpt) : maxcut_kernel<true, false, ALDS>(rpt);
    return pm1 ? maxcut_kernel<false, true, ALDS>(rpt) : maxcut_kernel<false, false, ALDS>(rpt);
}

hipError_t resident_launch(const Problem& p, const ResData& r, int cls, bool manip, ResArgs a, hipStream_t st)
{
    (void)hipGetLastError();   // drop stale errors of earlier calls
    const ResTables& t = *r.t;
    const ResClass& c = t.classes[(size_t)cls];
    a.inst = t.inst + c.first;
    a.perm = t.perm;
    a.slice = t.slice;
    a.adj = t.adj;
    a.wgt = t.wgt;
    a.steps = r.steps;
    a.nrm = p.nrm;
    a.kind = p.kind;
    a.planes = t.planes;
    ResKernel k = c.adj_lds ? pick<true>(p, t.pm1, manip, c.rpt) : pick<false>(p, t.pm1, manip, c.rpt);
    if (!k) return hipErrorInvalidValue;
    if (c.lds > 64 * 1024) {
        // the attribute is the kernel's, for all threads: one value, so that
        // another solver does not lower it between this call and the launch
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, t.dev_lds);
        if (e != hipSuccess) return e;
    }
    k<<<dim3((unsigned)c.n_inst * (unsigned)a.R), dim3(c.threads), c.lds, st>>>(a);
    return hipGetLastError();
}

}  // namespace fem
