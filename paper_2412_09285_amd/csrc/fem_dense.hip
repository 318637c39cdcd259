// Dense-W MaxCut step for complete or near-complete graphs on gfx950 matrix
// cores.
//
// On a complete graph the field product phi = W m (m = tanh(h/2)) is a dense
// matrix product n x n x R, so it runs on MFMA instead of the gather of the
// sparse kernel.  Two kernels, both as exact as the sparse kernel's FP64
// accumulation: for integral weights (|W| <= 127) int8 products of the
// fixed-point marginals' digit planes (maxcut_dense_i8_step_kernel, second
// half of this file); for any other W the FP64 kernel below.
//
// Both give a workgroup of four waves a small block of phi and each wave a
// quarter of the contraction, straight from memory to the matrix cores: the
// operands of a wave are whole lines that no other wave of the workgroup
// reads, so LDS would only pass them on.  The partial blocks meet in LDS
// once, and every thread then steps a few nodes of one replica.  Blocks of
// 64 x 64 staged through LDS, each wave the whole contraction for a quarter,
// left most of the chip idle up to some hundred replicas, and all phases of a
// step (state in, products, update, state out) in step with one another above
// that.
//
// The epilogue is the explicit-gradient MaxCut step of the sparse kernel
// (one-logit reduction, supplementary "Simplification of FEM for solving the
// MaxCut problem"): g_i = P_i (1 - P_i) [2 phi_i + h_i / beta], the optimiser
// update, the new marginal, and per-replica energy partials [sum m phi,
// sum H2(P)] for the block's rows; the gradient terms are combined in double
// as there.
#include "fem_device.h"
#include "fem_dense.h"

#include <algorithm>
#include <type_traits>

namespace fem {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

// h, m1, m2 of (node i, replica r).  The kernels load every entry of the
// thread before the K loop, so that these loads are in flight while the
// matrix cores run (issued after the first store they would wait for it:
// the state arrays may alias as far as the compiler knows).
template <bool NT>
__device__ __forceinline__ void dense_load(const StepArgs& a, int i, int r, float& x, float& m1v, float& m2v)
{
    const size_t sbase = (size_t)i * a.srow + r;
    if constexpr (NT) {
        x = __builtin_nontemporal_load(a.h + sbase);
        m1v = __builtin_nontemporal_load(a.m1 + sbase);
        m2v = __builtin_nontemporal_load(a.m2 + sbase);
    } else {
        x = a.h[sbase];
        m1v = a.m1[sbase];
        m2v = a.m2[sbase];
    }
}

// The step of one (node i, replica r) given its field phi and loaded state:
// gradient, the optimiser update of h, m1, m2, energy terms; returns the new
// marginal and stores the gradient when it is kept.
template <bool EN, bool NT>
__device__ __forceinline__ float dense_update(const StepArgs& a, const StepScalars& sc, int i, int r, double phi,
                                              float x, float m1v, float m2v, double& e_mphi, double& e_h2)
{
    const size_t sbase = (size_t)i * a.srow + r;
    const float ax = fabsf(x);
    const float e = exp_neg(ax);
    const float rr = rcp_f(1.0f + e);
    const float pmin = e * rr;          // min(P, 1 - P)
    const float pq = pmin * rr;         // P(1-P) without cancellation
    const float g = (float)((double)pq * fma((double)x, sc.inv_beta_d, 2.0 * phi));
    if constexpr (EN) {
        // own marginal sign(h) (1 - e) / (1 + e): its cancellation near h = 0
        // leaves an absolute error of about 1e-7, far below the scale of U
        e_mphi += (double)copysignf((1.0f - e) * rr, x) * phi;
        e_h2 += (double)(log1p_f(e) + ax * pmin);
    }
    const float nh = adam_update(x, g, m1v, m2v, sc);
    if constexpr (NT) {
        __builtin_nontemporal_store(nh, a.h + sbase);
        __builtin_nontemporal_store(m1v, a.m1 + sbase);
        __builtin_nontemporal_store(m2v, a.m2 + sbase);
    } else {
        a.h[sbase] = nh;
        a.m1[sbase] = m1v;
        a.m2[sbase] = m2v;
    }
    if (a.grad) a.grad[(size_t)i * a.R + r] = g;
    return tanh_half(nh);
}

// The block (row block x, replica block y) of a workgroup of a grid of nx ny.
// Workgroup b runs on XCD b % 8; each XCD takes a contiguous eighth of an
// order that walks panels of an eighth of the replicas, row block by row
// block: its slice of the marginals stays in the XCD's L2 while W passes
// through once.
__device__ __forceinline__ void dense_block(int nx, int ny, int& x, int& y)
{
    const unsigned b = blockIdx.x, nb = gridDim.x, c = b & 7;
    const unsigned at = c * (nb >> 3) + min(c, nb & 7) + (b >> 3);
    const unsigned pw = ((unsigned)ny + 7) >> 3, panel = at / ((unsigned)nx * pw);
    const unsigned in = at - panel * (unsigned)nx * pw, w = min(pw, (unsigned)ny - panel * pw);
    x = __builtin_amdgcn_readfirstlane((int)(in / w));
    y = __builtin_amdgcn_readfirstlane((int)(panel * pw + in % w));
}

// Energy partials of a workgroup whose threads t hold replica t % C: lanes of
// the same replica by butterflies, then the four waves in order.
template <int C>
__device__ __forceinline__ void dense_energy(const StepArgs& a, int slot, int r0, double e_mphi, double e_h2,
                                             double (*sE)[2][C])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = C; k < 64; k <<= 1) {
        e_mphi += __shfl_xor(e_mphi, k, 64);
        e_h2 += __shfl_xor(e_h2, k, 64);
    }
    if (lane < C) {
        sE[wave][0][lane] = e_mphi;
        sE[wave][1][lane] = e_h2;
    }
    __syncthreads();
    const int r = r0 + (int)threadIdx.x % C, term = (int)threadIdx.x / C;
    if (term < 2 && r < a.R)
        a.epart[((size_t)slot * 2 + term) * a.R + r] =
            ((sE[0][term][threadIdx.x % C] + sE[1][term][threadIdx.x % C]) + sE[2][term][threadIdx.x % C]) +
            sE[3][term][threadIdx.x % C];
}

// FP64 kernel.  The products and sums are formed in double, as the sparse
// kernel accumulates: near equilibrium the gradient 2 phi + h / beta is a
// small difference, and float32 accumulation over ~10^3 neighbours leaves
// errors of order 1e-5 of the gradient there (a float32 matrix-core variant
// measured 1.0e-5 on a 300-node complete graph).  The marginal copy is float,
// node-major [n][R].  A workgroup owns a 16 B x 16 B block of phi; wave w
// multiplies the rows j = 16 s + 4 w + (0..3), s = 0, 1, ..., and thread t
// picks up B B outputs of replica t % (16 B).
//
// Bound by the FP64 matrix rate once the chip is full (n = 2000: 156 us a
// step at R = 1000, 53 of 79 TFLOP/s; 64 x 64 blocks through LDS 200), by the
// chain of one workgroup before (n = 2000, R = 50: 24 us, was 146; n = 500,
// R = 100: 8.4, was 45).  Two products of a wave in flight suffice with four
// waves a SIMD; eight, with two waves, measured 161 us.
template <bool EN, bool NT, int B>
__global__ void __launch_bounds__(256, 4) maxcut_dense_step_kernel(StepArgs a, const float* __restrict__ W, int32_t ld)
{
    constexpr int BM = B, BN = B;
    constexpr int DM = 16 * BM, DN = 16 * BN;
    constexpr int U = B == 1 ? 4 : 2;   // four-row products of a wave per group
    constexpr int KG = 16 * U;          // rows of a group
    constexpr int RS = 256 / DN;        // rows between a thread's outputs
    constexpr int NO = BM * BN;         // outputs of a thread
    static_assert(DENSE_LD_ALIGN % (2 * KG) == 0, "the K loop takes two groups at a time");
    int bx, by;
    dense_block((a.n + DM - 1) / DM, (a.R + DN - 1) / DN, bx, by);
    const int i0 = bx * DM, r0 = by * DN;
    const int R = a.R, n = a.n;
    const float* __restrict__ mc = static_cast<const float*>(a.marg_cur);
    float* __restrict__ mn = static_cast<float*>(a.marg_nxt);
    __shared__ double sP[4][DM][DN];
    __shared__ double sE[4][2][DN];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int kq = lane >> 4, c16 = lane & 15;   // MFMA lane: k index, row / column
    const int oc = threadIdx.x % DN, orow = threadIdx.x / DN;
    const int r = r0 + oc;
    // the state of this thread's outputs, in flight during the products
    float xs[NO], m1s[NO], m2s[NO];
#pragma unroll
    for (int q = 0; q < NO; ++q) {
        const int i = i0 + orow + RS * q;
        xs[q] = m1s[q] = m2s[q] = 0.0f;
        if (r < R && i < a.n) dense_load<NT>(a, i, r, xs[q], m1s[q], m2s[q]);
    }
    // operands: A(lane) = W[j + kq][i0 + 16 bm + c16] (W is symmetric), B(lane) =
    // m[j + kq][r0 + 16 bn + c16].  Rows j >= n of W are zero and meet row
    // n - 1 of m; replicas past R meet replica R - 1 and are dropped.
    const float* __restrict__ wp = W + i0 + c16;
    int cb[BN];
#pragma unroll
    for (int bn = 0; bn < BN; ++bn) cb[bn] = min(r0 + 16 * bn + c16, R - 1);
    float ra[2][U][BM], rb[2][U][BN];
    auto gload = [&](int g, int buf) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = KG * g + 16 * u + 4 * wave + kq;   // < ld
            const float* __restrict__ wj = wp + (size_t)j * ld;
            const float* __restrict__ mj = mc + (size_t)min(j, n - 1) * R;
#pragma unroll
            for (int bm = 0; bm < BM; ++bm) ra[buf][u][bm] = wj[16 * bm];
#pragma unroll
            for (int bn = 0; bn < BN; ++bn) rb[buf][u][bn] = mj[cb[bn]];
        }
    };
    f64x4 acc[BM][BN];
#pragma unroll
    for (int bm = 0; bm < BM; ++bm)
#pragma unroll
        for (int bn = 0; bn < BN; ++bn)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[bm][bn][v] = 0.0;
    auto products = [&](int buf) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int bm = 0; bm < BM; ++bm)
#pragma unroll
                for (int bn = 0; bn < BN; ++bn)
                    acc[bm][bn] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)ra[buf][u][bm], (double)rb[buf][u][bn],
                                                                       acc[bm][bn], 0, 0, 0);
    };
    const int ng = ld / KG;
    gload(0, 0);
    // the barriers keep the compiler from moving loads down to their use
    for (int g = 0; g < ng; g += 2) {
        gload(g + 1, 1);
        __builtin_amdgcn_sched_barrier(0);
        products(0);
        gload(min(g + 2, ng - 1), 0);   // past the end: loaded again, not used
        __builtin_amdgcn_sched_barrier(0);
        products(1);
    }
    // output layout of the f64 16x16x4 MFMA: lane group kq holds rows kq,
    // kq + 4, kq + 8, kq + 12 of column c16
#pragma unroll
    for (int bm = 0; bm < BM; ++bm)
#pragma unroll
        for (int bn = 0; bn < BN; ++bn)
#pragma unroll
            for (int v = 0; v < 4; ++v) sP[wave][16 * bm + kq + 4 * v][16 * bn + c16] = acc[bm][bn][v];
    __syncthreads();
    const StepScalars sc = a.sc;
    double e_mphi = 0.0, e_h2 = 0.0;
#pragma unroll
    for (int q = 0; q < NO; ++q) {
        const int il = orow + RS * q, i = i0 + il;
        if (r >= R || i >= a.n) continue;
        const double phi = ((sP[0][il][oc] + sP[1][il][oc]) + sP[2][il][oc]) + sP[3][il][oc];
        mn[(size_t)i * R + r] = dense_update<EN, NT>(a, sc, i, r, phi, xs[q], m1s[q], m2s[q], e_mphi, e_h2);
    }
    if constexpr (EN) dense_energy<DN>(a, bx, r0, e_mphi, e_h2, sE);
}

// ------------------------------------------------ integer weights: int8 ---
// For integral W with |W_ij| <= 127 the marginal copy is kept in fixed point,
// m_fx = rint(m 2^30) (|m| <= 1, so |m_fx| <= 2^30), written as four signed
// base-256 digits m_fx = d0 + 2^8 d1 + 2^16 d2 + 2^24 d3 (d0..d2 in
// [-128, 127], |d3| <= 65).  Each digit plane is an int8 matrix, and
// S_d = W d_d is an exact int32 product on the int8 matrix cores
// (v_mfma_i32_32x32x32_i8; |S_d| <= 127 * 128 * n < 2^31 for n <= 32768), so
// phi = 2^-30 sum_d 2^(8d) S_d is the field of the fixed-point marginals
// without any rounding (all terms are integers below 2^53).  Against the
// float32 copy the only difference is the quantisation of m to 2^-30.
// W and the planes (Rp replicas, R rounded up to 32; nodes j >= n and
// replicas r >= R hold zeros) are stored as the operands of the MFMA: the 32
// rows x 32 k of one operand are 1024 contiguous bytes, 16 of each lane (see
// dense_i8_at), so a wave's load is eight whole lines.
constexpr int QB = 1024;   // bytes of an operand

__device__ __forceinline__ void to_digits(float m, int (&d)[4])
{
    int x = (int)rintf(m * 1073741824.0f);   // exact scaling by 2^30
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        d[k] = ((x & 0xff) ^ 0x80) - 0x80;   // low byte as a signed digit
        x = (x - d[k]) >> 8;                  // exact: x - d[k] is a multiple of 256
    }
    d[3] = x;
}

// byte u of the words w[d] = the digits of m
__device__ __forceinline__ void add_digits(float m, int u, uint32_t (&w)[4])
{
    int dg[4];
    to_digits(m, dg);
#pragma unroll
    for (int d = 0; d < 4; ++d) w[d] |= (uint32_t)(dg[d] & 0xff) << (8 * u);
}

// byte of (row, k), both below 32, in an operand: lane (k / 16, row) holds the
// 16 bytes k % 16
__device__ __forceinline__ int dense_i8_lane(int row, int k)
{
    return (k >> 4) * 512 + row * 16 + (k & 15);
}

// A workgroup owns 32 BM x 32 outputs; wave w takes operands w, w + 4, ... of
// each of its row blocks.
//
// Bound by the chain of a workgroup (state loads, a quarter of the contraction,
// LDS, the step, stores) with few of them at once: n = 2000, R = 1000 is 1024
// workgroups of 64 x 32 outputs, two rounds of the 512 that fit at two waves a
// SIMD, whose phases coincide.  No unit is full in its 37 us: 112 MB past L2, 3
// TB/s; 4.1 M requests to the L2, 44% of one a cycle and channel, 78% hits;
// vector units 25 k and matrix cores 16 k of the 72 k cycles that the shaders are
// busy.  32 x 32 blocks, 660 MB of operands from the L2 instead of 403, took 3%
// longer.  With operands that lay row by row (32 bytes of each line per load)
// 32 x 32 blocks took 100 us instead of 45 (n = 2000, R = 1000) and 19 instead
// of 12 (R = 50).  Three K blocks of operands in flight leave these three waves
// a SIMD: two, or four with fewer waves, measured 3 to 10% slower.
template <bool EN, bool NT, int BM>
__global__ void __launch_bounds__(256, BM == 1 ? 3 : 2) maxcut_dense_i8_step_kernel(StepArgs a,
                                                                                    const int8_t* __restrict__ W8,
                                                                                    int32_t ld, int32_t Rp)
{
    constexpr int D = 32, DM = D * BM;
    constexpr int PF = 3;                // K blocks in flight
    constexpr int QK = DENSE_LD_ALIGN;   // K block: an operand of each wave
    int bx, by;
    dense_block((a.n + DM - 1) / DM, (a.R + D - 1) / D, bx, by);
    const int i0 = bx * DM, r0 = by * D;
    const int R = a.R;
    const size_t plane = (size_t)Rp * ld;
    const int8_t* __restrict__ qc = static_cast<const int8_t*>(a.marg_cur);
    int8_t* __restrict__ qn = static_cast<int8_t*>(a.marg_nxt);
    __shared__ double sP[4][D][D];
    __shared__ __attribute__((aligned(16))) int8_t sT[4][QB];
    __shared__ double sE[4][2][D];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kh = lane >> 5, c32 = lane & 31;
    const int orow = (tid >> 5) * 4;   // outputs of a thread: four rows of each 32, replica c32
    const int r = r0 + c32;
    float xs[BM][4], m1s[BM][4], m2s[BM][4];
#pragma unroll
    for (int bm = 0; bm < BM; ++bm)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = i0 + D * bm + orow + q;
            xs[bm][q] = m1s[bm][q] = m2s[bm][q] = 0.0f;
            if (r < R && i < a.n) dense_load<NT>(a, i, r, xs[bm][q], m1s[bm][q], m2s[bm][q]);
        }
    const size_t band = (size_t)ld * 32;
    const int8_t* __restrict__ ap = W8 + (i0 / D) * band + wave * QB + 16 * lane;
    const int8_t* __restrict__ bp = qc + (r0 / D) * band + wave * QB + 16 * lane;
    i32x4 ra[PF][BM], rb[PF][4];
    const int nk = ld / QK;
    auto gload = [&](int kb, int s) {
#pragma unroll
        for (int bm = 0; bm < BM; ++bm)
            ra[s][bm] = *reinterpret_cast<const i32x4*>(ap + bm * band + (size_t)kb * (4 * QB));
#pragma unroll
        for (int d = 0; d < 4; ++d)
            rb[s][d] = *reinterpret_cast<const i32x4*>(bp + d * plane + (size_t)kb * (4 * QB));
    };
    i32x16 acc[BM][4];
#pragma unroll
    for (int bm = 0; bm < BM; ++bm)
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[bm][d][v] = 0;
    auto products = [&](int s) {
#pragma unroll
        for (int bm = 0; bm < BM; ++bm)
#pragma unroll
            for (int d = 0; d < 4; ++d)
                acc[bm][d] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ra[s][bm], rb[s][d], acc[bm][d], 0, 0, 0);
    };
#pragma unroll
    for (int s = 0; s < PF; ++s) gload(min(s, nk - 1), s);
    int kb = 0;
    for (; kb + PF <= nk; kb += PF)
#pragma unroll
        for (int s = 0; s < PF; ++s) {
            products(s);
            gload(min(kb + s + PF, nk - 1), s);   // past the end: loaded again, not used
        }
#pragma unroll
    for (int s = 0; s < PF - 1; ++s)
        if (kb + s < nk) products(s);
    const StepScalars sc = a.sc;
    double e_mphi = 0.0, e_h2 = 0.0;
#pragma unroll
    for (int bm = 0; bm < BM; ++bm) {
        // register v of lane (kh, c32): row 8 (v / 4) + 4 kh + v % 4, replica c32
#pragma unroll
        for (int v = 0; v < 16; ++v)
            sP[wave][8 * (v >> 2) + 4 * kh + (v & 3)][c32] =
                fma((double)acc[bm][3][v], 16777216.0,
                    fma((double)acc[bm][2][v], 65536.0, fma((double)acc[bm][1][v], 256.0, (double)acc[bm][0][v])));
        __syncthreads();
        uint32_t dw[4] = {0, 0, 0, 0};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int il = orow + q, i = i0 + D * bm + il;
            float mnew = 0.0f;   // rows past n and replicas past R keep zero digits
            if (r < R && i < a.n) {
                const double phi =
                    (((sP[0][il][c32] + sP[1][il][c32]) + sP[2][il][c32]) + sP[3][il][c32]) * (1.0 / 1073741824.0);
                mnew = dense_update<EN, NT>(a, sc, i, r, phi, xs[bm][q], m1s[bm][q], m2s[bm][q], e_mphi, e_h2);
            }
            add_digits(mnew, q, dw);
        }
        // the digits as the operand they are next
#pragma unroll
        for (int d = 0; d < 4; ++d) *reinterpret_cast<uint32_t*>(&sT[d][dense_i8_lane(c32, orow)]) = dw[d];
        __syncthreads();
        *reinterpret_cast<i32x4*>(qn + wave * plane + (r0 / D) * band + (size_t)(i0 / D + bm) * QB + 16 * lane) =
            *reinterpret_cast<const i32x4*>(&sT[wave][16 * lane]);
    }
    if constexpr (EN) dense_energy<D>(a, bx, r0, e_mphi, e_h2, sE);
}

// digit planes of the marginals of h (rows j < n, replicas r < R); src: new
// fields [n][R] to set with cleared moments on the way, or null.  A thread
// takes 16 nodes of a replica: rows are read, and operands written, by whole
// lines (n = 2000, R = 1000: one node a thread, nodes first, 15 us).
__global__ void __launch_bounds__(256) dense_i8_init_kernel(StepArgs a, const float* __restrict__ src, int32_t ld,
                                                            int32_t Rp)
{
    const size_t k = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int r = (int)(k % Rp), j0 = (int)(k / Rp) * 16;
    if (r >= a.R || j0 >= a.n) return;
    int8_t* __restrict__ q = static_cast<int8_t*>(a.marg_nxt);
    const size_t plane = (size_t)Rp * ld, at = dense_i8_at(r, j0, ld);
    float x[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int j = min(j0 + u, a.n - 1);
        x[u] = src ? src[(size_t)j * a.R + r] : a.h[(size_t)j * a.srow + r];
    }
    i32x4 out[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        uint32_t dw[4] = {0, 0, 0, 0};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = j0 + 4 * v + u;
            add_digits(j < a.n ? tanh_half(x[4 * v + u]) : 0.0f, u, dw);
            if (src && j < a.n) {
                const size_t s = (size_t)j * a.srow + r;
                a.h[s] = x[4 * v + u];
                a.m1[s] = 0.0f;
                a.m2[s] = 0.0f;
            }
        }
#pragma unroll
        for (int d = 0; d < 4; ++d) out[d][v] = (int)dw[d];
    }
#pragma unroll
    for (int d = 0; d < 4; ++d) *reinterpret_cast<i32x4*>(q + d * plane + at) = out[d];
}

hipError_t launch_dense_i8_init(const Problem& p, const StepArgs& a, const float* src, hipStream_t st)
{
    (void)hipGetLastError();   // drop stale errors of earlier calls
    if (!p.dense_w8 || p.dense_ld % DENSE_LD_ALIGN != 0) return hipErrorInvalidValue;
    const int Rp = dense_rows_padded(a.R);
    const size_t blocks = ((size_t)Rp * ((a.n + 15) / 16) + 255) / 256;
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    dense_i8_init_kernel<<<(unsigned)blocks, 256, 0, st>>>(a, src, p.dense_ld, Rp);
    return hipGetLastError();
}

// int8: 64 x 32 blocks halve the traffic of W but hold the chip with two
// waves a SIMD instead of three; they pay once the 32 x 32 blocks are more
// than the two rounds of 768 that the chip holds (n = 2000, R = 600: 1197
// blocks, 28.7 against 30.3 us; R = 1000: 2016, 40.9 against 39.7; n = 4000,
// R = 1000: 4000, 115 against 95).  FP64: 32 x 32 blocks read half of what
// four 16 x 16 ones do, which spread a small product over the chip (n = 200,
// R = 600: 133 blocks of 32 x 32, 9.5 against 8.2 us; n = 1400, R = 100: 176,
// 22.8 against 25.2).
DenseShape dense_shape(const Problem& p, int R)
{
    const size_t blocks = (size_t)((p.n + 31) / 32) * ((R + 31) / 32);
    if (p.dense_w8) return DenseShape{blocks > 1536 ? 64 : 32, 32};
    return blocks >= 160 ? DenseShape{32, 32} : DenseShape{16, 16};
}

hipError_t launch_dense_step(const Problem& p, const DenseShape& shape, int dtype, bool en, bool nt, int n_tiles,
                             const StepArgs& a, hipStream_t st)
{
    (void)hipGetLastError();   // drop stale errors of earlier calls
    if (!p.dense_w || p.kind != KIND_MAXCUT || dtype != 0 || p.dense_ld % DENSE_LD_ALIGN != 0)
        return hipErrorInvalidValue;
    const size_t blocks = (size_t)n_tiles * ((a.R + shape.cols - 1) / shape.cols);
    if (n_tiles != (a.n + shape.rows - 1) / shape.rows || blocks > INT32_MAX) return hipErrorInvalidValue;
    const dim3 g((unsigned)blocks), b(256);
    auto run = [&](auto en_c, auto nt_c) {
        constexpr bool EN = decltype(en_c)::value, NT = decltype(nt_c)::value;
        const int Rp = dense_rows_padded(a.R);
        if (p.dense_w8 && shape.rows == 64)
            maxcut_dense_i8_step_kernel<EN, NT, 2><<<g, b, 0, st>>>(a, p.dense_w8, p.dense_ld, Rp);
        else if (p.dense_w8)
            maxcut_dense_i8_step_kernel<EN, NT, 1><<<g, b, 0, st>>>(a, p.dense_w8, p.dense_ld, Rp);
        else if (shape.rows == 32)
            maxcut_dense_step_kernel<EN, NT, 2><<<g, b, 0, st>>>(a, p.dense_w, p.dense_ld);
        else
            maxcut_dense_step_kernel<EN, NT, 1><<<g, b, 0, st>>>(a, p.dense_w, p.dense_ld);
    };
    if (en) {
        if (nt) run(std::true_type{}, std::true_type{});
        else run(std::true_type{}, std::false_type{});
    } else {
        if (nt) run(std::false_type{}, std::true_type{});
        else run(std::false_type{}, std::false_type{});
    }
    return hipGetLastError();
}

}  // namespace fem
