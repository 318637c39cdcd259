// Learned warm start for MaxCut FEM: a two-layer message-passing network of
// width 64 that maps the state of one replica part-way through an anneal to a
// proposal for that replica's final read-out (one logit per node); the anneal
// then continues from h = alpha * z with a shorter, colder schedule.  Node
// features: bias, ln(1+deg), mean incident weight, tanh(s/2) and
// clamp(s/4, -2, 2) of the replica's fields s, and three uniform random
// features from a counter-based generator.  Training uses FEM's own runs (the
// state at the early step and the final read-out of the same replica), a
// binary cross-entropy, the analytic backward pass and Adam; every kernel here
// is hand-written HIP.  The paper has no such network: this is an addition on
// top of the method.
//
// Network (per draw d, node i; a(v)_i = (1/max(deg_i,1)) sum_j W_ij v_j):
//   pre1 = x A1 + a(x) B1 + b1,    H1 = relu(pre1)
//   pre2 = H1 A2 + a(H1) B2 + b2,  H2 = relu(pre2)
//   z    = H2 c + d
// Weights are used as bfloat16 (round to nearest even) with float32
// arithmetic; the float32 master copy and the Adam moments stay float32.
//
// Random features: Philox4x32-10 (Salmon et al., SC 2011) with counter
// (i, draw, block, 0) and key (seed mod 2^32, seed div 2^32); a uniform in
// [-1, 1) is the top 24 bits of a word times 2^-23, minus one (exact).
//
// Determinism: every sum runs in a fixed order (neighbour order of the CSR,
// the matrix-core steps of layer 2 in a fixed sequence, butterflies within a
// wave, rows in order within a workgroup, workgroups in order in the final
// reduction).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "../../include/fem.h"
#include "fem_internal.h"

using namespace fem;

namespace {

constexpr int D_IN = 8, HID = 64;
constexpr int OFF_A1 = 0, OFF_B1 = 512, OFF_b1 = 1024, OFF_A2 = 1088, OFF_B2 = 5184, OFF_b2 = 9280, OFF_c = 9344,
              OFF_d = 9408;
constexpr int NP = 9409;
constexpr int WG_BLOCKS = 512;   // workgroups of the weight-gradient reduction

typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

__device__ __forceinline__ uint16_t to_bf16(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

struct U4 {
    uint32_t x, y, z, w;
};

// Philox4x32 with 10 rounds
__device__ __forceinline__ U4 philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1)
{
    for (int r = 0; r < 10; ++r) {
        if (r) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
        const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
        const uint32_t n0 = hi1 ^ c1 ^ k0, n1 = lo1, n2 = hi0 ^ c3 ^ k1, n3 = lo0;
        c0 = n0; c1 = n1; c2 = n2; c3 = n3;
    }
    return U4{c0, c1, c2, c3};
}

__device__ __forceinline__ float upm1(uint32_t w) { return (float)(w >> 8) * 0x1p-23f - 1.0f; }

// ------------------------------------------------------------- forward ----
// features of node i from the replica's fields state[i * stride]
__global__ void feat_kernel(int32_t n, const int64_t* __restrict__ row_off, const int2* __restrict__ adj,
                            const float* __restrict__ state, int64_t stride, uint32_t k0, uint32_t k1, uint32_t draw,
                            float* __restrict__ X, float* __restrict__ inv_deg, int with_graph)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        float* x = X + (size_t)i * D_IN;
        if (with_graph) {   // inputs 0..2 and 1 / deg depend on the graph only
            const int64_t b = row_off[i], e = row_off[i + 1];
            float ws = 0.0f;
            for (int64_t k = b; k < e; ++k) ws += __int_as_float(adj[k].y);
            const float deg = (float)(e - b);
            x[0] = 1.0f;
            x[1] = log1pf(deg);
            x[2] = e > b ? ws / deg : 0.0f;
            inv_deg[i] = 1.0f / fmaxf(deg, 1.0f);
        }
        const float sv = state[(size_t)i * stride];
        const U4 r0 = philox((uint32_t)i, draw, 0u, 0u, k0, k1);
        x[3] = tanhf(0.5f * sv);
        x[4] = fminf(fmaxf(0.25f * sv, -2.0f), 2.0f);
        x[5] = upm1(r0.x);
        x[6] = upm1(r0.y);
        x[7] = upm1(r0.z);
    }
}

// A wave takes L1_NB = 8 nodes at a time.  Gather: lane 8q + c aggregates
// feature c of node q (four neighbour rows in flight); the nodes' [x | a(x)]
// are staged in the wave's LDS slice.  Dense part (skipped when pre1 is
// null): lane j owns hidden unit j (its 16 weights in registers) and reads the
// staged inputs as broadcasts; layer 2 gathers the pre1 rows.
constexpr int L1_NB = 8;
__global__ void __launch_bounds__(256) layer1_kernel(int32_t n, const int64_t* __restrict__ row_off,
                                                     const int2* __restrict__ adj, const float* __restrict__ X,
                                                     const float* __restrict__ inv_deg, const uint16_t* __restrict__ w,
                                                     float* __restrict__ A1agg, float* __restrict__ pre1)
{
    __shared__ float4 sxa[4][L1_NB][2 * D_IN / 4];   // per wave: L1_NB nodes x [x | a(x)]
    const int lane = threadIdx.x & 63;
    const int wl = threadIdx.x >> 6;
    const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int nw = (gridDim.x * blockDim.x) >> 6;
    float colA[D_IN], colB[D_IN];
#pragma unroll
    for (int k = 0; k < D_IN; ++k) {
        colA[k] = bf(w[OFF_A1 + k * HID + lane]);
        colB[k] = bf(w[OFF_B1 + k * HID + lane]);
    }
    const float bias = bf(w[OFF_b1 + lane]);
    float* sf = reinterpret_cast<float*>(&sxa[wl][0][0]);
    const int q = lane >> 3, c = lane & 7;
    for (int i0 = wave * L1_NB; i0 < n; i0 += nw * L1_NB) {
        const int i = i0 + q;
        if (i < n) {
            float a = 0.0f;
            int64_t k = row_off[i];
            const int64_t kend = row_off[i + 1];
            for (; k + 4 <= kend; k += 4) {
                const int2 e0 = adj[k], e1 = adj[k + 1], e2 = adj[k + 2], e3 = adj[k + 3];
                const float v0 = X[(size_t)e0.x * D_IN + c], v1 = X[(size_t)e1.x * D_IN + c];
                const float v2 = X[(size_t)e2.x * D_IN + c], v3 = X[(size_t)e3.x * D_IN + c];
                a = fmaf(__int_as_float(e0.y), v0, a);
                a = fmaf(__int_as_float(e1.y), v1, a);
                a = fmaf(__int_as_float(e2.y), v2, a);
                a = fmaf(__int_as_float(e3.y), v3, a);
            }
            for (; k < kend; ++k) {
                const int2 e = adj[k];
                a = fmaf(__int_as_float(e.y), X[(size_t)e.x * D_IN + c], a);
            }
            a *= inv_deg[i];
            sf[q * 2 * D_IN + c] = X[(size_t)i * D_IN + c];
            sf[q * 2 * D_IN + D_IN + c] = a;
            A1agg[(size_t)i * D_IN + c] = a;
        }
        __builtin_amdgcn_wave_barrier();
        const int cnt = (n - i0) < L1_NB ? (n - i0) : L1_NB;
        for (int qq = 0; pre1 && qq < cnt; ++qq) {
            const float4 x0 = sxa[wl][qq][0], x1 = sxa[wl][qq][1], a0 = sxa[wl][qq][2], a1 = sxa[wl][qq][3];
            float acc = bias;
            acc = fmaf(x0.x, colA[0], acc); acc = fmaf(x0.y, colA[1], acc);
            acc = fmaf(x0.z, colA[2], acc); acc = fmaf(x0.w, colA[3], acc);
            acc = fmaf(x1.x, colA[4], acc); acc = fmaf(x1.y, colA[5], acc);
            acc = fmaf(x1.z, colA[6], acc); acc = fmaf(x1.w, colA[7], acc);
            acc = fmaf(a0.x, colB[0], acc); acc = fmaf(a0.y, colB[1], acc);
            acc = fmaf(a0.z, colB[2], acc); acc = fmaf(a0.w, colB[3], acc);
            acc = fmaf(a1.x, colB[4], acc); acc = fmaf(a1.y, colB[5], acc);
            acc = fmaf(a1.z, colB[6], acc); acc = fmaf(a1.w, colB[7], acc);
            pre1[(size_t)(i0 + qq) * HID + lane] = acc;
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Layer 2 on the matrix cores, sixteen nodes per wave at a time.
// Gather: lane l = 16 g + i takes node i0 + i and hidden units 16 g .. 16 g +
// 15 of its own and its neighbours' layer-1 pre-activation rows (four float4
// of a 256-byte row, ReLU applied on load, two neighbours in flight); every
// a(H1) sum runs in CSR order, as in a single-node evaluation.
// (Units 16 c + 4 g .. + 3, 64 contiguous bytes at a time for the four lanes of
// a node, took 77 instead of 97 us on 135 k nodes of mean degree 6.5, but add
// the products in another order: a pre-activation within a rounding of zero
// then changes sides, and with it the gradient, by up to 5e-6 of its norm.)
// Dense: pre2 for the 16 nodes is four 16 x 16 output tiles (16 units each),
// each 32 steps of v_mfma_f32_16x16x4_f32 (A: nodes x 4 inputs, B: 4 inputs x
// units).  Step s of the H1 half takes the inputs 16 g' + s (g' = 0..3), so a
// lane supplies its own s-th gathered value as its A element and nothing is
// staged; the a(H1) half follows.  [A2; B2] (128 x 64, float) sits in LDS
// with rows padded to L2_LD = 65 floats, which puts the four input rows of a
// step in distinct banks.  Output element (node 4 g + v, unit 16 t + i) is
// register v of lane l in tile t.  Each output depends on its own node's
// inputs only, in a fixed order.
constexpr int L2_NB = 16;
constexpr int L2_LD = 65;
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) layer2_kernel(int32_t n, const int64_t* __restrict__ row_off,
                                                     const int2* __restrict__ adj, const float* __restrict__ inv_deg,
                                                     const uint16_t* __restrict__ w, const float* __restrict__ pre1,
                                                     float* __restrict__ a2out, float* __restrict__ pre2out,
                                                     float* __restrict__ z)
{
    __shared__ float sW[2 * HID * L2_LD];   // row k < 64: A2[k][:], row 64 + k: B2[k][:]
    for (int t = threadIdx.x; t < HID * HID; t += blockDim.x) {
        const int k = t / HID, j = t % HID;
        sW[k * L2_LD + j] = bf(w[OFF_A2 + t]);
        sW[(HID + k) * L2_LD + j] = bf(w[OFF_B2 + t]);
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int g = lane >> 4, li = lane & 15;
    const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int nw = (gridDim.x * blockDim.x) >> 6;
    float bias[4], cl[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        bias[t] = bf(w[OFF_b2 + 16 * t + li]);
        cl[t] = bf(w[OFF_c + 16 * t + li]);
    }
    const float dd = bf(w[OFF_d]);
    auto relu = [](float x) { return fmaxf(x, 0.0f); };
    for (int i0 = wave * L2_NB; i0 < n; i0 += nw * L2_NB) {
        const int i = i0 + li;
        float hs[16], ag[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            hs[u] = 0.0f;
            ag[u] = 0.0f;
        }
        if (i < n) {
            const float4* hp = reinterpret_cast<const float4*>(pre1 + (size_t)i * HID + 16 * g);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float4 v = hp[c];
                hs[4 * c] = relu(v.x); hs[4 * c + 1] = relu(v.y); hs[4 * c + 2] = relu(v.z); hs[4 * c + 3] = relu(v.w);
            }
            int64_t k = row_off[i];
            const int64_t kend = row_off[i + 1];
            for (; k + 2 <= kend; k += 2) {
                const int2 e0 = adj[k], e1 = adj[k + 1];
                const float4* p0 = reinterpret_cast<const float4*>(pre1 + (size_t)e0.x * HID + 16 * g);
                const float4* p1 = reinterpret_cast<const float4*>(pre1 + (size_t)e1.x * HID + 16 * g);
                float4 v0[4], v1[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    v0[c] = p0[c];
                    v1[c] = p1[c];
                }
                const float w0 = __int_as_float(e0.y), w1 = __int_as_float(e1.y);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    ag[4 * c] = fmaf(w0, relu(v0[c].x), ag[4 * c]);
                    ag[4 * c + 1] = fmaf(w0, relu(v0[c].y), ag[4 * c + 1]);
                    ag[4 * c + 2] = fmaf(w0, relu(v0[c].z), ag[4 * c + 2]);
                    ag[4 * c + 3] = fmaf(w0, relu(v0[c].w), ag[4 * c + 3]);
                    ag[4 * c] = fmaf(w1, relu(v1[c].x), ag[4 * c]);
                    ag[4 * c + 1] = fmaf(w1, relu(v1[c].y), ag[4 * c + 1]);
                    ag[4 * c + 2] = fmaf(w1, relu(v1[c].z), ag[4 * c + 2]);
                    ag[4 * c + 3] = fmaf(w1, relu(v1[c].w), ag[4 * c + 3]);
                }
            }
            if (k < kend) {
                const int2 e0 = adj[k];
                const float4* p0 = reinterpret_cast<const float4*>(pre1 + (size_t)e0.x * HID + 16 * g);
                const float w0 = __int_as_float(e0.y);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float4 v = p0[c];
                    ag[4 * c] = fmaf(w0, relu(v.x), ag[4 * c]);
                    ag[4 * c + 1] = fmaf(w0, relu(v.y), ag[4 * c + 1]);
                    ag[4 * c + 2] = fmaf(w0, relu(v.z), ag[4 * c + 2]);
                    ag[4 * c + 3] = fmaf(w0, relu(v.w), ag[4 * c + 3]);
                }
            }
            const float id = inv_deg[i];
#pragma unroll
            for (int u = 0; u < 16; ++u) ag[u] *= id;
            if (a2out) {
                float4* ap = reinterpret_cast<float4*>(a2out + (size_t)i * HID + 16 * g);
#pragma unroll
                for (int c = 0; c < 4; ++c) ap[c] = make_float4(ag[4 * c], ag[4 * c + 1], ag[4 * c + 2], ag[4 * c + 3]);
            }
        }
        // dense part, the whole wave
        v4f acc[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = v4f{bias[t], bias[t], bias[t], bias[t]};
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            // one step's weight loads at a time (hoisting all 128 of them
            // would cost the occupancy)
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 4; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(hs[s], sW[(16 * g + s) * L2_LD + 16 * t + li], acc[t],
                                                              0, 0, 0);
        }
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 4; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                    ag[s], sW[(HID + 16 * g + s) * L2_LD + 16 * t + li], acc[t], 0, 0, 0);
        }
        // z = relu(pre2) . c + d: per lane over its 4 tiles, then over the 16
        // lanes of its row group (fixed butterfly)
        float zp[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            zp[v] = 0.0f;
#pragma unroll
            for (int t = 0; t < 4; ++t) zp[v] = fmaf(relu(acc[t][v]), cl[t], zp[v]);
#pragma unroll
            for (int off = 1; off < 16; off <<= 1) zp[v] += __shfl_xor(zp[v], off, 64);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int node = i0 + 4 * g + v;
            if (node < n) {
                if (li == 0) z[node] = zp[v] + dd;
                if (pre2out) {
#pragma unroll
                    for (int t = 0; t < 4; ++t) pre2out[(size_t)node * HID + 16 * t + li] = acc[t][v];
                }
            }
        }
    }
}

// ------------------------------------------------- batched inference ----
// Inference of all R replicas in one pass.  The per-replica forward above
// gathers the 256-byte layer-1 rows of every neighbour, once per replica;
// here the work is shared across the replicas of a node:
//  * graph inputs (ln(1+deg), mean weight, 1/max(deg,1)) and their
//    aggregates, once per call;
//  * replica inputs r_f (tanh(s/2), clamp(s/4), three uniforms) and their
//    aggregates a(r_f), stored feature-major [n][5][R];
//  * layer 2 recomputes each neighbour's layer-1 activations from its 16
//    inputs on the matrix cores instead of storing and gathering them.
// A wave owns one node and 32 replicas (the N dimension of a 32 x 32 tile of
// v_mfma_f32_32x32x16_bf16).  Operands: A = weights (bfloat16, exact), B =
// activations split into three bfloat16 parts whose sum is the float value
// exactly (each product is then exact and the tile sums in float32, so the
// arithmetic is that of float32 up to summation order).  Lane l = 32 g + c
// holds replica c; in a K block of 16 it supplies inputs 8 g .. 8 g + 7, and
// of a 32 x 32 output tile t it holds units 32 t + 8 (v/4) + 4 g + v%4,
// v = 0..15 (so the next layer's K order is permuted to match, and its
// weights are laid out in that order: nothing is transposed).
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
constexpr int NRF = 5;   // replica inputs per node

__device__ __forceinline__ int out_unit(int t, int v, int g) { return 32 * t + 8 * (v >> 2) + 4 * g + (v & 3); }

// x = hi + mid + lo exactly: truncation to 8 significant bits twice, the
// rest (at most 8 significant bits) is a bfloat16 value; the three parts are
// the upper halves of x, r = x - hi and lo
__device__ __forceinline__ void split3(float x, uint32_t& xh, uint32_t& rm, uint32_t& lo)
{
    const float r = x - __uint_as_float(__float_as_uint(x) & 0xffff0000u);
    xh = __float_as_uint(x);
    rm = __float_as_uint(r);
    lo = __float_as_uint(r - __uint_as_float(rm & 0xffff0000u));
}

// the upper halves of a (low) and b (high) in one word
__device__ __forceinline__ uint32_t pack_hi(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

// the three bfloat16 operands of eight float values
__device__ __forceinline__ void split_operands(const float (&v)[8], bf16x8& bh, bf16x8& bm, bf16x8& bl)
{
    u32x4v H, M, L;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        uint32_t h0, m0, l0, h1, m1, l1;
        split3(v[2 * q], h0, m0, l0);
        split3(v[2 * q + 1], h1, m1, l1);
        H[q] = pack_hi(h0, h1);
        M[q] = pack_hi(m0, m1);
        L[q] = pack_hi(l0, l1);
    }
    bh = __builtin_bit_cast(bf16x8, H);
    bm = __builtin_bit_cast(bf16x8, M);
    bl = __builtin_bit_cast(bf16x8, L);
}

// max(x, 0) for finite x as one integer maximum (a negative float is a
// negative integer); -0 gives +0
__device__ __forceinline__ float relu_f(float x) { return __int_as_float(max(__float_as_int(x), 0)); }

// The constant input 1 of the layer-1 products as stored: its three bfloat16
// parts are 1, 2^-8 and 0, so the product of the middle parts can carry the
// bias (weights 256 b1 times 2^-8, exact) and no operand needs patching.
constexpr float ONE_B1 = 1.00390625f;

// graph inputs gf[i] = {ONE_B1, ln(1+deg), mean incident weight (0 if
// isolated), 1/max(deg,1)}, as the per-replica forward forms them; slot x is
// the constant input 1 of lane group 0 in the layer-1 products, stored as
// 1 + 2^-8 (see inf_layer2_kernel)
__global__ void inf_graph_kernel(int32_t n, const int64_t* __restrict__ row_off, const int2* __restrict__ adj,
                                 float4* __restrict__ gf)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const int64_t b = row_off[i], e = row_off[i + 1];
        float ws = 0.0f;
        for (int64_t k = b; k < e; ++k) ws += __int_as_float(adj[k].y);
        const float deg = (float)(e - b);
        gf[i] = make_float4(ONE_B1, log1pf(deg), e > b ? ws / deg : 0.0f, 1.0f / fmaxf(deg, 1.0f));
    }
}

// their aggregates ga[i] = {a(1), a(ln(1+deg)), a(mean weight), 0}, each sum
// in CSR order, then scaled by 1/max(deg,1)
__global__ void inf_graph_agg_kernel(int32_t n, const int64_t* __restrict__ row_off, const int2* __restrict__ adj,
                                     const float4* __restrict__ gf, float4* __restrict__ ga)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f;
        const int64_t kend = row_off[i + 1];
        // rounds of up to four neighbours in flight, summed in CSR order
        for (int64_t k = row_off[i]; k < kend; k += 4) {
            const int nb = (int)min((int64_t)4, kend - k);
            int2 e[4];
            float4 q[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (u < nb) e[u] = adj[k + u];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (u < nb) q[u] = gf[e[u].x];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (u < nb) {
                    const float w = __int_as_float(e[u].y);
                    a0 = fmaf(w, 1.0f, a0);
                    a1 = fmaf(w, q[u].y, a1);
                    a2 = fmaf(w, q[u].z, a2);
                }
        }
        const float id = gf[i].w;
        ga[i] = make_float4(a0 * id, a1 * id, a2 * id, 0.0f);
    }
}

// replica inputs Xr[i][f][r] of the fields state[i][r] (draw r)
__global__ void inf_feat_kernel(int32_t n, int32_t R, const float* __restrict__ state, uint32_t k0, uint32_t k1,
                                float* __restrict__ Xr)
{
    const size_t count = (size_t)n * R;
    for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < count; k += (size_t)gridDim.x * blockDim.x) {
        const int i = (int)(k / R), r = (int)(k % R);
        const float sv = state[k];
        const U4 w = philox((uint32_t)i, (uint32_t)r, 0u, 0u, k0, k1);
        float* x = Xr + (size_t)i * NRF * R + r;
        x[0] = tanhf(0.5f * sv);
        x[R] = fminf(fmaxf(0.25f * sv, -2.0f), 2.0f);
        x[2 * R] = upm1(w.x);
        x[3 * R] = upm1(w.y);
        x[4 * R] = upm1(w.z);
    }
}

// their aggregates AXr[i][f][r], each sum in CSR order, then scaled
__global__ void inf_agg_kernel(int32_t n, int32_t R, const int64_t* __restrict__ row_off, const int2* __restrict__ adj,
                               const float4* __restrict__ gf, const float* __restrict__ Xr, float* __restrict__ AXr)
{
    const size_t count = (size_t)n * R;
    for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < count; k += (size_t)gridDim.x * blockDim.x) {
        const int i = (int)(k / R), r = (int)(k % R);
        float a[NRF] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        int64_t q = row_off[i];
        const int64_t qend = row_off[i + 1];
        // rounds of up to four neighbours in flight, summed in CSR order
        for (; q < qend; q += 4) {
            const int nb = (int)min((int64_t)4, qend - q);
            int2 e[4];
            float xv[4][NRF];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (u < nb) e[u] = adj[q + u];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (u < nb) {
                    const float* x = Xr + (size_t)e[u].x * NRF * R + r;
#pragma unroll
                    for (int f = 0; f < NRF; ++f) xv[u][f] = x[(size_t)f * R];
                }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (u < nb) {
                    const float w = __int_as_float(e[u].y);
#pragma unroll
                    for (int f = 0; f < NRF; ++f) a[f] = fmaf(w, xv[u][f], a[f]);
                }
        }
        const float id = gf[i].w;
        float* o = AXr + (size_t)i * NRF * R + r;
#pragma unroll
        for (int f = 0; f < NRF; ++f) o[(size_t)f * R] = a[f] * id;
    }
}

#ifndef INF_NBUF
#define INF_NBUF 4
#endif

// Layer 1 (recomputed per neighbour), layer 2 and the output, one wave per
// (node, block of 32 replicas); h_out[i][r] = alpha z_i^r.
// Blocks go to the 8 XCDs in turn (block b to XCD b mod 8); the items are
// cut into 8 contiguous ranges of about equal work, and XCD x's blocks take
// range x, so that the neighbours one XCD gathers (nodes of the same
// instances) stay in its own L2.
constexpr int N_XCD = 8;
struct XcdRanges {
    int64_t b[N_XCD + 1];
};

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3)))
inf_layer2_kernel(int32_t n, int32_t R, const int64_t* __restrict__ row_off, const int2* __restrict__ adj,
                  const float4* __restrict__ gf, const float4* __restrict__ ga, const float* __restrict__ Xr,
                  const float* __restrict__ AXr, const uint16_t* __restrict__ w,
                  float alpha, XcdRanges xr,
                  float* __restrict__ h_out)
{
    // A operands of the output layer: [k block][output tile][lane], eight
    // bfloat16 weights each; k block kb = 4 src + 2 tt + half takes, in lane
    // group g, slot q, input unit out_unit(tt, 8 half + q, g) of H1 (src 0,
    // weights A2) or of a(H1) (src 1, weights B2)
    __shared__ u32x4v sW2[8][2][64];
    __shared__ float sB2[2][64][16], sC[2][64][16];   // b2 and c in the output layout of each lane
    for (int t = threadIdx.x; t < 8 * 2 * 64; t += blockDim.x) {
        const int kb = t >> 7, ot = (t >> 6) & 1, ln = t & 63;
        const int src = kb >> 2, tt = (kb >> 1) & 1, half = kb & 1, gg = ln >> 5, m = 32 * ot + (ln & 31);
        u32x4v v;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int u0 = out_unit(tt, 8 * half + 2 * q, gg), u1 = out_unit(tt, 8 * half + 2 * q + 1, gg);
            const int off = src ? OFF_B2 : OFF_A2;
            v[q] = (uint32_t)w[off + u0 * HID + m] | ((uint32_t)w[off + u1 * HID + m] << 16);
        }
        sW2[kb][ot][ln] = v;
    }
    for (int t = threadIdx.x; t < 2 * 64 * 16; t += blockDim.x) {
        const int ot = t >> 10, ln = (t >> 4) & 63, v = t & 15;
        const int u = out_unit(ot, v, ln >> 5);
        sB2[ot][ln][v] = bf(w[OFF_b2 + u]);
        sC[ot][ln][v] = bf(w[OFF_c + u]);
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, c = lane & 31, g = lane >> 5;
    // layer-1 A operands (tile t: units 32 t + c; inputs 8 g .. 8 g + 7, which
    // are x for g = 0 and a(x) for g = 1) and the biases b1 in the output layout
    // The bias enters through the product of the middle parts: input 0 of
    // lane group 0 is the constant 1, stored as ONE_B1 = 1 + 2^-8, whose parts
    // are 1, 2^-8 and 0; that product takes the weights 256 b1 in place of
    // A1[0] (b1 is a bfloat16 value, so 256 b1 is one too and the product
    // 256 b1 2^-8 = b1 is exact), so the accumulator needs no bias registers.
    bf16x8 aW1[2], aW1m[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        u32x4v v;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int off = g ? OFF_B1 : OFF_A1;
            v[q] = (uint32_t)w[off + (2 * q) * HID + 32 * t + c] | ((uint32_t)w[off + (2 * q + 1) * HID + 32 * t + c] << 16);
        }
        aW1[t] = __builtin_bit_cast(bf16x8, v);
        if (g == 0) {
            const uint32_t b256 = __float_as_uint(bf(w[OFF_b1 + 32 * t + c]) * 256.0f) >> 16;
            v[0] = b256 | (v[0] & 0xffff0000u);
        }
        aW1m[t] = __builtin_bit_cast(bf16x8, v);
    }
    const float dd = bf(w[OFF_d]);
    const float4* gp = g ? ga : gf;
    const float* xp = g ? AXr : Xr;
    const int nrb = (R + 31) / 32;
    // this XCD's range and the wave's place among the XCD's waves, stated
    // uniform so that node and neighbour indices live in scalar registers
    // and the branches on them are scalar
    const int x = (int)(blockIdx.x % N_XCD);
    const int wpb = (int)(blockDim.x >> 6);
    const int64_t wave = __builtin_amdgcn_readfirstlane((int)((blockIdx.x / N_XCD) * wpb + (threadIdx.x >> 6)));
    const int64_t nw = (int64_t)((gridDim.x - x + N_XCD - 1) / N_XCD) * wpb;
    const int64_t it_end = xr.b[x + 1];
    for (int64_t it = xr.b[x] + wave; it < it_end; it += nw) {
        // the output layer's weights, b2 and c are read from LDS where they
        // are used, not held in registers across the loop (they would cost
        // 128 registers per lane and the occupancy)
        asm volatile("" ::: "memory");
        const int i = (int)(it / nrb);
        const int r = (int)(it % nrb) * 32 + c;
        const bool ract = r < R;
        // the 8 inputs this lane supplies for node j, and the layer-1
        // pre-activations (bias included) from them
        // The raw loads of node j's inputs for this lane (a lane past R reads
        // replica 0); assemble() forms the 8 operand values where they are
        // used, so that no instruction needs a load's result early and the
        // loads of later neighbours stay in flight.
        struct In {
            float4 q;
            float x[NRF];
        };
        const int rl = ract ? r : 0;
        auto inputs = [&](int j, In& in) {
            in.q = gp[j];
            const float* x = xp + (size_t)j * NRF * R + rl;
#pragma unroll
            for (int f = 0; f < NRF; ++f) in.x[f] = x[(size_t)f * R];
        };
        // (lanes past R compute a column of their own from replica 0's
        // inputs and store nothing)
        auto assemble = [&](const In& in, float (&v)[8]) {
            v[0] = in.q.x;
            v[1] = in.q.y;
            v[2] = in.q.z;
#pragma unroll
            for (int f = 0; f < NRF; ++f) v[3 + f] = in.x[f];
        };
        auto pre1 = [&](const float (&v)[8], f32x16 (&acc)[2]) {
            bf16x8 bh, bm, bl;
            split_operands(v, bh, bm, bl);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aW1[t], bh, f32x16{}, 0, 0, 0);
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aW1m[t], bm, acc[t], 0, 0, 0);
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aW1[t], bl, acc[t], 0, 0, 0);
            }
        };
        f32x16 ag[2];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v2 = 0; v2 < 16; ++v2) ag[t][v2] = 0.0f;
        // Neighbours in CSR order, in chunks of up to 64: one load gives the
        // chunk's entries (one per lane) and readlane hands them out, so no
        // load waits on another.  NBUF input buffers in a fixed rotation (the
        // loop is unrolled by NBUF, so no register is copied): while
        // neighbour u's products run, the inputs of the next NBUF - 1
        // neighbours are in flight.  Reads past the chunk's end repeat its
        // last entry (in bounds, and skipped by a uniform branch).
        constexpr int NBUF = INF_NBUF;
        const int64_t kb = row_off[i], ke = row_off[i + 1];
        for (int64_t c0 = kb; c0 < ke; c0 += 64) {
            const int cnt = (int)min((int64_t)64, ke - c0);
            const int2 me = adj[c0 + min(lane, cnt - 1)];
            auto col = [&](int u) { return __builtin_amdgcn_readlane(me.x, min(u, cnt - 1)); };
            auto wgt = [&](int u) { return __int_as_float(__builtin_amdgcn_readlane(me.y, u)); };
            auto accumulate = [&](const In& in, float wij) {
                float v[8];
                assemble(in, v);
                f32x16 hj[2];
                pre1(v, hj);
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int v2 = 0; v2 < 16; ++v2) ag[t][v2] = fmaf(wij, relu_f(hj[t][v2]), ag[t][v2]);
            };
            In buf[NBUF];
            // issued in the order the loop consumes them (the barriers keep
            // the scheduler from reordering), so each use waits only on the
            // oldest loads
#pragma unroll
            for (int b = 0; b < NBUF; ++b) {
                inputs(col(b), buf[b]);
                asm volatile("" ::: "memory");
            }
            // full groups of NBUF neighbours in one block with no branch
            // between neighbours (2% faster than a uniform skip per
            // neighbour), then the last cnt mod NBUF
            int u = 0;
            for (; u + NBUF <= cnt; u += NBUF) {
#pragma unroll
                for (int b = 0; b < NBUF; ++b) {
                    accumulate(buf[b], wgt(u + b));
                    inputs(col(u + NBUF + b), buf[b]);
                }
                // keeps the compiler from turning the loads carried into the
                // next iteration into loads at its top (which would wait on
                // them at once)
                asm volatile("" ::: "memory");
            }
#pragma unroll
            for (int b = 0; b < NBUF - 1; ++b)
                if (u + b < cnt) accumulate(buf[b], wgt(u + b));
        }
        const float id = gf[i].w;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v2 = 0; v2 < 16; ++v2) ag[t][v2] *= id;
        // the node's own layer-1 activations, formed after the loop so that
        // they do not hold registers during it
        f32x16 h1[2];
        {
            In in;
            inputs(i, in);
            float v[8];
            assemble(in, v);
            pre1(v, h1);
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v2 = 0; v2 < 16; ++v2) h1[t][v2] = relu_f(h1[t][v2]);
        // output layer: pre2 = [H1 | a(H1)] [A2; B2] + b2
        f32x16 o[2];
#pragma unroll
        for (int ot = 0; ot < 2; ++ot)
#pragma unroll
            for (int v2 = 0; v2 < 16; ++v2) o[ot][v2] = sB2[ot][lane][v2];
#pragma unroll
        for (int kb = 0; kb < 8; ++kb) {
            const int src = kb >> 2, tt = (kb >> 1) & 1, half = kb & 1;
            float v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = src ? ag[tt][8 * half + q] : h1[tt][8 * half + q];
            bf16x8 bh, bm, bl;
            split_operands(v, bh, bm, bl);
#pragma unroll
            for (int ot = 0; ot < 2; ++ot) {
                const bf16x8 aw = __builtin_bit_cast(bf16x8, sW2[kb][ot][lane]);
                o[ot] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aw, bh, o[ot], 0, 0, 0);
                o[ot] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aw, bm, o[ot], 0, 0, 0);
                o[ot] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aw, bl, o[ot], 0, 0, 0);
            }
        }
        // z = relu(pre2) c + d: this lane's 32 units, then its partner's
        float zp = 0.0f;
#pragma unroll
        for (int ot = 0; ot < 2; ++ot)
#pragma unroll
            for (int v2 = 0; v2 < 16; ++v2) zp = fmaf(relu_f(o[ot][v2]), sC[ot][lane][v2], zp);
        zp += __shfl_xor(zp, 32, 64);
        if (g == 0 && ract) h_out[(size_t)i * R + r] = alpha * (zp + dd);
    }
}

// ------------------------------------------------------------ training ----
__device__ __forceinline__ float softplusf(float x) { return fmaxf(x, 0.0f) + log1pf(expf(-fabsf(x))); }

// per instance (one workgroup at a time): L = mean softplus(z) - y z, and
// dz_i = (sigmoid(z_i) - y_i) / (N_b B)
__global__ void __launch_bounds__(1024) loss_kernel(const int32_t* __restrict__ inst_off, int32_t B,
                                                    const float* __restrict__ z, const int32_t* __restrict__ y,
                                                    float* __restrict__ dz, double* __restrict__ L)
{
    __shared__ double s0[1024];
    for (int b = blockIdx.x; b < B; b += gridDim.x) {
        const int i0 = inst_off[b], i1 = inst_off[b + 1];
        const float nb = (float)(i1 - i0);
        double a0 = 0.0;
        for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
            const float zi = z[i], yi = (float)y[i];
            a0 += (double)(softplusf(zi) - yi * zi);
            const float sg = 1.0f / (1.0f + expf(-zi));
            dz[i] = (sg - yi) / (nb * (float)B);
        }
        s0[threadIdx.x] = a0;
        __syncthreads();
        for (int s = 512; s > 0; s >>= 1) {
            if ((int)threadIdx.x < s) s0[threadIdx.x] += s0[threadIdx.x + s];
            __syncthreads();
        }
        if (threadIdx.x == 0) L[b] = s0[0] / (double)(i1 > i0 ? i1 - i0 : 1);
        __syncthreads();   // s0 is the next instance's
    }
}

// Units of lane group g in step s: four float4 of a row, 64 contiguous bytes at
// a time for the four lanes of a node; rows of the weights four apart in
// distinct banks at a pitch of W2_LD floats.
constexpr int W2_LD = 68;
__device__ __forceinline__ int unit_of(int g, int s) { return 16 * (s >> 2) + 4 * g + (s & 3); }

// dpre2 = dz c [pre2 > 0] (formed where it is needed, not stored);
// dH1 (own term) = dpre2 A2^T, da2s = (dpre2 B2^T) / max(deg, 1), on the matrix
// cores, sixteen nodes per wave as layer 2 (the transposed weights in LDS).  Bound
// by its three 256-byte rows per node: 135 k nodes take 42 us (2.5 TB/s);
// with a broadcast and two multiply-adds per (unit, unit) it took 114 us.
__global__ void __launch_bounds__(256) back2_kernel(int32_t n, const float* __restrict__ inv_deg,
                                                    const uint16_t* __restrict__ w, const float* __restrict__ dz,
                                                    const float* __restrict__ pre2, float* __restrict__ dh1s,
                                                    float* __restrict__ da2s)
{
    __shared__ float sW[2 * HID * W2_LD];   // row j < 64: A2[:][j], row 64 + j: B2[:][j]
    for (int t = threadIdx.x; t < HID * HID; t += blockDim.x) {
        const int k = t / HID, j = t % HID;
        sW[j * W2_LD + k] = bf(w[OFF_A2 + t]);
        sW[(HID + j) * W2_LD + k] = bf(w[OFF_B2 + t]);
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, g = lane >> 4, li = lane & 15;
    const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int nw = (gridDim.x * blockDim.x) >> 6;
    float cl[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) cl[s] = bf(w[OFF_c + unit_of(g, s)]);
    for (int i0 = wave * L2_NB; i0 < n; i0 += nw * L2_NB) {
        const int i = i0 + li;
        float dp[16];
#pragma unroll
        for (int s = 0; s < 16; ++s) dp[s] = 0.0f;
        if (i < n) {
            const float dzi = dz[i];
            const float4* pp = reinterpret_cast<const float4*>(pre2 + (size_t)i * HID) + g;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float4 v = pp[4 * c];
                dp[4 * c] = v.x > 0.0f ? dzi * cl[4 * c] : 0.0f;
                dp[4 * c + 1] = v.y > 0.0f ? dzi * cl[4 * c + 1] : 0.0f;
                dp[4 * c + 2] = v.z > 0.0f ? dzi * cl[4 * c + 2] : 0.0f;
                dp[4 * c + 3] = v.w > 0.0f ? dzi * cl[4 * c + 3] : 0.0f;
            }
        }
        v4f ha[4], hb[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) ha[t] = hb[t] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            __builtin_amdgcn_sched_barrier(0);   // one step's weight loads at a time
            const int row = unit_of(g, s) * W2_LD + li;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                ha[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(dp[s], sW[row + 16 * t], ha[t], 0, 0, 0);
                hb[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(dp[s], sW[HID * W2_LD + row + 16 * t], hb[t], 0, 0, 0);
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int node = i0 + 4 * g + v;
            if (node < n) {
                const float id = inv_deg[node];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    dh1s[(size_t)node * HID + 16 * t + li] = ha[t][v];
                    da2s[(size_t)node * HID + 16 * t + li] = hb[t][v] * id;
                }
            }
        }
    }
}

// dpre1_j = [pre1_j > 0] (dH1s_j + sum_{i in N(j)} W_ij da2s_i): four nodes per
// wave, sixteen lanes and one float4 each per row, so that a load brings four
// neighbour rows.
__global__ void __launch_bounds__(256) back1_kernel(int32_t n, const int64_t* __restrict__ row_off,
                                                    const int2* __restrict__ adj, const float* __restrict__ pre1,
                                                    const float* __restrict__ dh1s, const float* __restrict__ da2s,
                                                    float* __restrict__ dpre1)
{
    const int li = threadIdx.x & 15;
    const int team = (blockIdx.x * blockDim.x + threadIdx.x) >> 4, teams = (gridDim.x * blockDim.x) >> 4;
    const float4* own = reinterpret_cast<const float4*>(dh1s) + li;
    const float4* rows = reinterpret_cast<const float4*>(da2s) + li;
    const float4* act = reinterpret_cast<const float4*>(pre1) + li;
    float4* out = reinterpret_cast<float4*>(dpre1) + li;
    for (int j = team; j < n; j += teams) {
        const size_t at = (size_t)j * (HID / 4);
        float4 g = own[at];
        const float4 p = act[at];
        auto add = [&](const int2& e, const float4& v) {
            const float wij = __int_as_float(e.y);
            g.x = fmaf(wij, v.x, g.x);
            g.y = fmaf(wij, v.y, g.y);
            g.z = fmaf(wij, v.z, g.z);
            g.w = fmaf(wij, v.w, g.w);
        };
        int64_t k = row_off[j];
        const int64_t kend = row_off[j + 1];
        for (; k + 4 <= kend; k += 4) {
            int2 e[4];
            float4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) e[u] = adj[k + u];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = rows[(size_t)e[u].x * (HID / 4)];
#pragma unroll
            for (int u = 0; u < 4; ++u) add(e[u], v[u]);
        }
        for (; k < kend; ++k) {
            const int2 e = adj[k];
            add(e, rows[(size_t)e.x * (HID / 4)]);
        }
        out[at] = make_float4(p.x > 0.0f ? g.x : 0.0f, p.y > 0.0f ? g.y : 0.0f, p.z > 0.0f ? g.z : 0.0f,
                              p.w > 0.0f ? g.w : 0.0f);
    }
}

// Weight gradients as sums of outer products over the rows, on the matrix
// cores: [H1 | a(H1)]^T dpre2 is 4 x 4 tiles of 16 x 16 for either half and
// [x | a(x)]^T dpre1 four tiles, four rows per v_mfma_f32_16x16x4_f32.  Lane
// 16 g + i holds, of row 4 s + g, the units 4 i .. 4 i + 3 of every array (one
// float4 each, a wave reads four whole rows per load), so tile (a, b) pairs
// the units 4 m + a with 4 c + b.  Wave v of the launch owns the contiguous
// rows [v n / V, (v + 1) n / V); a workgroup adds its four waves in order and
// writes one partial vector.  Bound by its four 256-byte rows per node: 135 k
// nodes take 54 us (2.6 TB/s), 128 us with one multiply-add per lane and
// product out of LDS.
struct WgradArgs {
    int32_t n;
    const float *X, *A1agg, *pre1, *a2, *pre2, *dz, *dpre1;
    const uint16_t* w;
    float* part;   // [G][NP]
};

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) wgrad_kernel(WgradArgs a)
{
    __shared__ float sum[NP];
    const int lane = threadIdx.x & 63, g = lane >> 4, li = lane & 15;
    const int wl = threadIdx.x >> 6;
    const int64_t V = (int64_t)gridDim.x * 4, wave = (int64_t)blockIdx.x * 4 + wl;
    const int64_t r0 = a.n * wave / V, r1 = a.n * (wave + 1) / V;
    v4f gA[4][4], gB[4][4], gX[4];
    float gb2[4], gc[4], cl[4], gd = 0.0f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
#pragma unroll
        for (int v = 0; v < 4; ++v) gA[u][v] = gB[u][v] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        gX[u] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        gb2[u] = gc[u] = 0.0f;
        cl[u] = bf(a.w[OFF_c + 4 * li + u]);
    }
    struct Rows {
        float4 p1, a2, p2, d1;
        float x, dz;
    };
    auto load = [&](int64_t r) {   // row r + g; zeros past the range contribute nothing
        Rows q{};
        if (r + g < r1) {
            const size_t at = (size_t)(r + g) * (HID / 4) + li;
            q.p1 = reinterpret_cast<const float4*>(a.pre1)[at];
            q.a2 = reinterpret_cast<const float4*>(a.a2)[at];
            q.p2 = reinterpret_cast<const float4*>(a.pre2)[at];
            q.d1 = reinterpret_cast<const float4*>(a.dpre1)[at];
            q.x = li < D_IN ? a.X[(size_t)(r + g) * D_IN + li] : a.A1agg[(size_t)(r + g) * D_IN + li - D_IN];
            q.dz = a.dz[r + g];
        }
        return q;
    };
    Rows q = load(r0);
    for (int64_t r = r0; r < r1; r += 4) {
        const Rows nx = load(r + 4);   // in flight during this round's products
        const float h1[4] = {fmaxf(q.p1.x, 0.0f), fmaxf(q.p1.y, 0.0f), fmaxf(q.p1.z, 0.0f), fmaxf(q.p1.w, 0.0f)};
        const float av[4] = {q.a2.x, q.a2.y, q.a2.z, q.a2.w};
        const float p2[4] = {q.p2.x, q.p2.y, q.p2.z, q.p2.w};
        const float d1[4] = {q.d1.x, q.d1.y, q.d1.z, q.d1.w};
        float dp[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            dp[u] = p2[u] > 0.0f ? q.dz * cl[u] : 0.0f;
            gb2[u] += dp[u];
            gc[u] = fmaf(q.dz, fmaxf(p2[u], 0.0f), gc[u]);
        }
        gd += q.dz;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                gA[u][v] = __builtin_amdgcn_mfma_f32_16x16x4f32(h1[u], dp[v], gA[u][v], 0, 0, 0);
                gB[u][v] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u], dp[v], gB[u][v], 0, 0, 0);
            }
            gX[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(q.x, d1[u], gX[u], 0, 0, 0);
        }
        q = nx;
    }
    // the four row groups of the vectors, in a fixed butterfly
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        gb2[u] += __shfl_xor(gb2[u], 16, 64);
        gb2[u] += __shfl_xor(gb2[u], 32, 64);
        gc[u] += __shfl_xor(gc[u], 16, 64);
        gc[u] += __shfl_xor(gc[u], 32, 64);
    }
    gd += __shfl_xor(gd, 16, 64);
    gd += __shfl_xor(gd, 32, 64);
    for (int turn = 0; turn < 4; ++turn) {
        if (wl == turn) {
            auto put = [&](int at, float x) { sum[at] = turn ? sum[at] + x : x; };
            // tile register v of lane 16 g + i: row index 4 g + v, column i
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = 4 * g + v;
#pragma unroll
                for (int ub = 0; ub < 4; ++ub) {
                    const int j = 4 * li + ub;
#pragma unroll
                    for (int ua = 0; ua < 4; ++ua) {
                        put(OFF_A2 + (4 * m + ua) * HID + j, gA[ua][ub][v]);
                        put(OFF_B2 + (4 * m + ua) * HID + j, gB[ua][ub][v]);
                    }
                    put((m < D_IN ? OFF_A1 + m * HID : OFF_B1 + (m - D_IN) * HID) + j, gX[ub][v]);
                    if (m == 0) put(OFF_b1 + j, gX[ub][v]);   // input 0 is the constant 1
                }
            }
            if (g == 0) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    put(OFF_b2 + 4 * li + u, gb2[u]);
                    put(OFF_c + 4 * li + u, gc[u]);
                }
            }
            if (lane == 0) put(OFF_d, gd);
        }
        __syncthreads();
    }
    float* p = a.part + (size_t)blockIdx.x * NP;
    for (int k = threadIdx.x; k < NP; k += 256) p[k] = sum[k];
}

// Sums the partial vectors in double (thread (s, p): partials s, s + 8, ...,
// then the eight in order), and applies Adam to the master weights: 32
// parameters per workgroup.  A chain of 512 dependent-latency loads per
// parameter took 127 us; this takes 8.
__global__ void __launch_bounds__(256) grad_adam_kernel(int G, const float* __restrict__ part, float* __restrict__ grad,
                                                        float* __restrict__ theta, float* __restrict__ m1,
                                                        float* __restrict__ m2, uint16_t* __restrict__ wbf,
                                                        float step_size, float bc2_sqrt, float b1, float b2, float eps)
{
    __shared__ double lds[256];
    const int p = blockIdx.x * 32 + (threadIdx.x & 31), sub = threadIdx.x >> 5;
    double s = 0.0;
    if (p < NP)
#pragma unroll 16
        for (int b = sub; b < G; b += 8) s += (double)part[(size_t)b * NP + p];
    lds[threadIdx.x] = s;
    __syncthreads();
    if (sub != 0 || p >= NP) return;
    for (int k = 1; k < 8; ++k) s += lds[k * 32 + threadIdx.x];
    const float gg = (float)s;
    grad[p] = gg;
    const float a = b1 * m1[p] + (1.0f - b1) * gg;
    const float v = b2 * m2[p] + (1.0f - b2) * (gg * gg);
    m1[p] = a;
    m2[p] = v;
    const float th = theta[p] - step_size * (a / (sqrtf(v) / bc2_sqrt + eps));
    theta[p] = th;
    wbf[p] = to_bf16(th);
}

// new master weights: their bfloat16 form, and cleared Adam moments
__global__ void round_weights_kernel(const float* __restrict__ theta, uint16_t* __restrict__ wbf,
                                     float* __restrict__ m1, float* __restrict__ m2)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < NP) {
        wbf[p] = to_bf16(theta[p]);
        m1[p] = 0.0f;
        m2[p] = 0.0f;
    }
}

}  // namespace

// ================================================================ host ====
static fem_status mfail(fem_status st, const char* what, hipError_t e = hipSuccess)
{
    std::string msg = what;
    if (e != hipSuccess) {
        msg += ": ";
        msg += hipGetErrorString(e);
    }
    return (fem_status)fem::set_error(st, msg.c_str());
}

#define MCHK(expr)                                                                                 \
    do {                                                                                           \
        hipError_t e_ = (expr);                                                                    \
        if (e_ != hipSuccess)                                                                      \
            return mfail(e_ == hipErrorOutOfMemory ? FEM_E_NOMEM : FEM_E_HIP, #expr, e_);          \
    } while (0)

struct fem_mpnn {
    int device = 0;
    float* theta = nullptr;
    uint16_t* wbf = nullptr;
    float* m1 = nullptr;
    float* m2 = nullptr;
    float* grad = nullptr;
    float* part = nullptr;
    int64_t adam_t = 0;
    size_t cap = 0;      // rows the work buffers hold
    size_t cap_inst = 0;
    float *X = nullptr, *A1agg = nullptr, *inv_deg = nullptr, *pre1 = nullptr, *a2 = nullptr, *pre2 = nullptr,
          *z = nullptr, *dz = nullptr, *dh1s = nullptr, *da2s = nullptr, *dpre1 = nullptr;
    float* state = nullptr;   // one replica's fields (training input)
    int32_t* y = nullptr;
    double* L = nullptr;      // instance losses, with the gradient behind them
    float* tbuf = nullptr;   // inference: graph and replica inputs with their aggregates
    size_t tcap = 0;         // floats tbuf holds
};

template <typename T>
static void mfree(T*& p)
{
    if (p) (void)hipFree(p);
    p = nullptr;
}

static void free_work(fem_mpnn* m)
{
    mfree(m->X); mfree(m->A1agg); mfree(m->inv_deg); mfree(m->pre1); mfree(m->a2); mfree(m->pre2);
    mfree(m->z); mfree(m->dz); mfree(m->dh1s); mfree(m->da2s); mfree(m->dpre1);
    mfree(m->state); mfree(m->y); mfree(m->L);
    m->grad = nullptr;
    m->cap = 0;
    m->cap_inst = 0;
}

static fem_status ensure_work(fem_mpnn* m, size_t n, size_t n_inst)
{
    if (n <= m->cap && n_inst <= m->cap_inst) return FEM_OK;
    free_work(m);
    const size_t c = n + 1, ci = n_inst + 1;
    MCHK(hipMalloc(&m->X, c * D_IN * 4));
    MCHK(hipMalloc(&m->A1agg, c * D_IN * 4));
    MCHK(hipMalloc(&m->inv_deg, c * 4));
    MCHK(hipMalloc(&m->pre1, c * HID * 4));
    MCHK(hipMalloc(&m->a2, c * HID * 4));
    MCHK(hipMalloc(&m->pre2, c * HID * 4));
    MCHK(hipMalloc(&m->z, c * 4));
    MCHK(hipMalloc(&m->dz, c * 4));
    MCHK(hipMalloc(&m->dh1s, c * HID * 4));
    MCHK(hipMalloc(&m->da2s, c * HID * 4));
    MCHK(hipMalloc(&m->dpre1, c * HID * 4));
    MCHK(hipMalloc(&m->state, c * 4));
    MCHK(hipMalloc(&m->y, c * 4));
    MCHK(hipMalloc(&m->L, ci * 8 + NP * 4));
    m->grad = reinterpret_cast<float*>(m->L + ci);
    m->cap = n;
    m->cap_inst = n_inst;
    return FEM_OK;
}

static int grid_rows(int32_t n, int waves_per_block)
{
    const int64_t w = (int64_t)n;   // one wave per row, capped
    int64_t blocks = (w + waves_per_block - 1) / waves_per_block;
    if (blocks > 8192) blocks = 8192;
    return (int)(blocks > 0 ? blocks : 1);
}

// forward for one replica state (device, state[i * stride]) and draw: z (and,
// with train, the activations kept for backward).  graph_ready: the graph-only
// inputs of this problem are already in the work buffers (a previous forward
// of the same call).
static fem_status forward(fem_mpnn* m, const Problem& p, const float* state, int64_t stride, uint64_t seed,
                          int32_t draw, bool train, hipStream_t st, bool graph_ready = false)
{
    const int32_t n = p.n;
    const uint32_t k0 = (uint32_t)(seed & 0xffffffffu), k1 = (uint32_t)(seed >> 32);
    (void)hipGetLastError();
    feat_kernel<<<(n + 255) / 256, 256, 0, st>>>(n, p.row_off, p.adj, state, stride, k0, k1, (uint32_t)draw, m->X,
                                                 m->inv_deg, graph_ready ? 0 : 1);
    layer1_kernel<<<grid_rows((n + L1_NB - 1) / L1_NB, 4), 256, 0, st>>>(n, p.row_off, p.adj, m->X, m->inv_deg, m->wbf,
                                                                         m->A1agg, m->pre1);
    layer2_kernel<<<grid_rows((n + L2_NB - 1) / L2_NB, 4), 256, 0, st>>>(
        n, p.row_off, p.adj, m->inv_deg, m->wbf, m->pre1, train ? m->a2 : nullptr, train ? m->pre2 : nullptr, m->z);
    MCHK(hipGetLastError());
    return FEM_OK;
}

extern "C" {

fem_status fem_mpnn_create(int device, const float* theta0, int32_t n_params, fem_mpnn** out)
{
    if (!out || !theta0) return mfail(FEM_E_INVAL, "NULL argument");
    *out = nullptr;
    if (n_params != NP) return mfail(FEM_E_INVAL, "the network has 9409 parameters");
    auto* m = new (std::nothrow) fem_mpnn;
    if (!m) return mfail(FEM_E_NOMEM, "host allocation failed");
    m->device = device;
    auto bail = [&](fem_status s) {
        fem_mpnn_destroy(m);
        return s;
    };
    hipError_t e = hipSetDevice(device);
    if (e != hipSuccess) return bail(mfail(FEM_E_HIP, "hipSetDevice", e));
    if ((e = hipMalloc(&m->theta, NP * 4)) != hipSuccess || (e = hipMalloc(&m->wbf, NP * 2)) != hipSuccess ||
        (e = hipMalloc(&m->m1, NP * 4)) != hipSuccess || (e = hipMalloc(&m->m2, NP * 4)) != hipSuccess ||
        (e = hipMalloc(&m->part, (size_t)WG_BLOCKS * NP * 4)) != hipSuccess)
        return bail(mfail(FEM_E_NOMEM, "device allocation", e));
    if ((e = hipMemcpy(m->theta, theta0, NP * 4, hipMemcpyHostToDevice)) != hipSuccess)
        return bail(mfail(FEM_E_HIP, "upload of the parameters", e));
    (void)hipGetLastError();
    round_weights_kernel<<<(NP + 255) / 256, 256>>>(m->theta, m->wbf, m->m1, m->m2);
    if ((e = hipDeviceSynchronize()) != hipSuccess) return bail(mfail(FEM_E_HIP, "round_weights_kernel", e));
    *out = m;
    return FEM_OK;
}

void fem_mpnn_destroy(fem_mpnn* m)
{
    if (!m) return;
    (void)hipSetDevice(m->device);
    free_work(m);
    mfree(m->tbuf);
    mfree(m->theta); mfree(m->wbf); mfree(m->m1); mfree(m->m2); mfree(m->part);
    delete m;
}

fem_status fem_mpnn_get_params(fem_mpnn* m, float* theta)
{
    if (!m || !theta) return mfail(FEM_E_INVAL, "NULL argument");
    MCHK(hipSetDevice(m->device));
    MCHK(hipMemcpy(theta, m->theta, NP * 4, hipMemcpyDeviceToHost));
    return FEM_OK;
}

fem_status fem_mpnn_set_params(fem_mpnn* m, const float* theta)
{
    if (!m || !theta) return mfail(FEM_E_INVAL, "NULL argument");
    MCHK(hipSetDevice(m->device));
    MCHK(hipMemcpy(m->theta, theta, NP * 4, hipMemcpyHostToDevice));
    m->adam_t = 0;
    (void)hipGetLastError();
    round_weights_kernel<<<(NP + 255) / 256, 256>>>(m->theta, m->wbf, m->m1, m->m2);
    MCHK(hipDeviceSynchronize());
    return FEM_OK;
}

fem_status fem_mpnn_forward(fem_mpnn* m, const fem_problem* fp, const float* state, uint64_t seed, int32_t draw,
                            float* z, int on_device)
{
    if (!m || !fp || !state || !z) return mfail(FEM_E_INVAL, "NULL argument");
    const Problem& p = fp->p;
    if (p.kind != KIND_MAXCUT) return mfail(FEM_E_UNSUPPORTED, "the warm-start network is for MaxCut problems");
    if (draw < 0) return mfail(FEM_E_INVAL, "draw must be >= 0");
    MCHK(hipSetDevice(m->device));
    fem_status s = ensure_work(m, (size_t)p.n, (size_t)p.n_inst);
    if (s != FEM_OK) return s;
    const float* st = state;
    if (!on_device) {
        MCHK(hipMemcpy(m->state, state, (size_t)p.n * 4, hipMemcpyHostToDevice));
        st = m->state;
    }
    s = forward(m, p, st, 1, seed, draw, false, nullptr);
    if (s != FEM_OK) return s;
    MCHK(hipMemcpy(z, m->z, (size_t)p.n * 4, on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost));
    return FEM_OK;
}

fem_status fem_mpnn_train_step(fem_mpnn* m, const fem_problem* fp, const float* state, const int32_t* labels,
                               uint64_t seed, int32_t draw0, double lr, double* loss, float* grad_out)
{
    if (!m || !fp || !state || !labels) return mfail(FEM_E_INVAL, "NULL argument");
    const Problem& p = fp->p;
    if (p.kind != KIND_MAXCUT) return mfail(FEM_E_UNSUPPORTED, "the warm-start network is for MaxCut problems");
    if (!(lr > 0.0) || draw0 < 0) return mfail(FEM_E_INVAL, "need lr > 0 and draw0 >= 0");
    int32_t other = 0;   // bits that a label of 0 or 1 does not have
    for (int32_t i = 0; i < p.n; ++i) other |= labels[i] & ~1;
    if (other) return mfail(FEM_E_INVAL, "labels must be 0 or 1");
    MCHK(hipSetDevice(m->device));
    const int32_t n = p.n, B = p.n_inst;
    fem_status s = ensure_work(m, (size_t)n, (size_t)B);
    if (s != FEM_OK) return s;
    MCHK(hipMemcpy(m->state, state, (size_t)n * 4, hipMemcpyHostToDevice));
    MCHK(hipMemcpy(m->y, labels, (size_t)n * 4, hipMemcpyHostToDevice));
    // one forward over the union: the random features are keyed by the node's
    // index in the batch and the draw
    s = forward(m, p, m->state, 1, seed, draw0, true, nullptr);
    if (s != FEM_OK) return s;
    (void)hipGetLastError();
    loss_kernel<<<std::min(B, 1 << 16), 1024>>>(p.inst_off_d, B, m->z, m->y, m->dz, m->L);
    back2_kernel<<<grid_rows((n + L2_NB - 1) / L2_NB, 4), 256>>>(n, m->inv_deg, m->wbf, m->dz, m->pre2, m->dh1s,
                                                                m->da2s);
    back1_kernel<<<grid_rows((n + 3) / 4, 4), 256>>>(n, p.row_off, p.adj, m->pre1, m->dh1s, m->da2s, m->dpre1);
    WgradArgs wa{n, m->X, m->A1agg, m->pre1, m->a2, m->pre2, m->dz, m->dpre1, m->wbf, m->part};
    // at least sixteen rows a wave: a partial vector costs as much to write
    // and read as 37 rows
    const int G = (int)std::min<int64_t>(WG_BLOCKS, ((int64_t)n + 63) / 64);
    wgrad_kernel<<<G, 256>>>(wa);
    // Adam on the master weights (torch.optim.Adam defaults 0.9 / 0.999 / 1e-8)
    const int64_t t = m->adam_t + 1;
    const double b1 = 0.9, b2 = 0.999;
    const float step = (float)(lr / (1.0 - std::pow(b1, (double)t)));
    const float bc2s = (float)std::sqrt(1.0 - std::pow(b2, (double)t));
    grad_adam_kernel<<<(NP + 31) / 32, 256>>>(G, m->part, m->grad, m->theta, m->m1, m->m2, m->wbf, step, bc2s, (float)b1,
                                              (float)b2, 1e-8f);
    MCHK(hipGetLastError());
    m->adam_t = t;
    // the per-instance losses and the gradient in one copy, which also waits
    // for the step; the loss is their mean
    const size_t g0 = (size_t)((char*)m->grad - (char*)m->L);
    std::vector<char> out(grad_out ? g0 + NP * 4 : (size_t)B * 8);
    MCHK(hipMemcpy(out.data(), m->L, out.size(), hipMemcpyDeviceToHost));
    double tot = 0.0;
    for (int32_t b = 0; b < B; ++b) {
        double Lb;
        std::memcpy(&Lb, out.data() + (size_t)b * 8, 8);
        tot += Lb / B;
    }
    if (loss) *loss = tot;
    if (grad_out) std::memcpy(grad_out, out.data() + g0, NP * 4);
    return FEM_OK;
}

// The inference kernels for device state src and proposal dst, enqueued on
// st (the work buffer grows first if it has to; hipFree waits for the device).
static fem_status infer_enqueue(fem_mpnn* m, const Problem& p, int32_t R, const float* src, uint64_t seed,
                                float alpha, float* dst, hipStream_t st)
{
    const size_t n = (size_t)p.n, nR = n * (size_t)R;
    // work: graph inputs and their aggregates (float4 per node each), replica
    // inputs and their aggregates (NRF x R floats per node each)
    const size_t need = 8 * (n + 1) + 2 * NRF * nR;
    if (m->tcap < need) {
        mfree(m->tbuf);
        m->tcap = 0;
        hipError_t ea = hipMalloc(&m->tbuf, need * 4);
        if (ea != hipSuccess) {
            m->tbuf = nullptr;
            return mfail(FEM_E_NOMEM, "device allocation of the inference buffers", ea);
        }
        m->tcap = need;
    }
    if (n == 0) return FEM_OK;
    float4* gf = reinterpret_cast<float4*>(m->tbuf);
    float4* ga = gf + (n + 1);
    float* Xr = m->tbuf + 8 * (n + 1);
    float* AXr = Xr + NRF * nR;
    const uint32_t k0 = (uint32_t)(seed & 0xffffffffu), k1 = (uint32_t)(seed >> 32);
    const unsigned gn = (unsigned)std::min<size_t>((n + 255) / 256, 65536);
    const unsigned gnr = (unsigned)std::min<size_t>((nR + 255) / 256, 65536);
    (void)hipGetLastError();
    inf_graph_kernel<<<gn, 256, 0, st>>>(p.n, p.row_off, p.adj, gf);
    inf_graph_agg_kernel<<<gn, 256, 0, st>>>(p.n, p.row_off, p.adj, gf, ga);
    inf_feat_kernel<<<gnr, 256, 0, st>>>(p.n, R, src, k0, k1, Xr);
    inf_agg_kernel<<<gnr, 256, 0, st>>>(p.n, R, p.row_off, p.adj, gf, Xr, AXr);
    // XCD ranges of about equal work: a node costs about as much as
    // NODE_COST neighbours (its output layer)
    const int nrb = (R + 31) / 32;
    const int64_t items = (int64_t)n * nrb;
    constexpr int64_t NODE_COST = 5;
    const int64_t total = p.h_row_off[n] + NODE_COST * (int64_t)n;
    XcdRanges xr;
    xr.b[0] = 0;
    int32_t lo = 0;
    for (int x = 1; x < N_XCD; ++x) {
        const int64_t want = total * x / N_XCD;
        while ((size_t)lo < n && p.h_row_off[lo] + NODE_COST * (int64_t)lo < want) ++lo;
        xr.b[x] = (int64_t)lo * nrb;
    }
    xr.b[N_XCD] = items;
    const unsigned gl = (unsigned)std::min<int64_t>(((items + 3) / 4 + N_XCD - 1) / N_XCD * N_XCD, 8192);
    inf_layer2_kernel<<<gl, 256, 0, st>>>(p.n, R, p.row_off, p.adj, gf, ga, Xr, AXr, m->wbf, alpha, xr, dst);
    hipError_t el = hipGetLastError();
    if (el != hipSuccess) return mfail(FEM_E_HIP, "inference kernels", el);
    return FEM_OK;
}

static fem_status infer_check(fem_mpnn* m, const fem_problem* fp, int32_t R)
{
    if (fp->p.kind != KIND_MAXCUT) return mfail(FEM_E_UNSUPPORTED, "the warm-start network is for MaxCut problems");
    if (R < 1) return mfail(FEM_E_INVAL, "need R >= 1");
    MCHK(hipSetDevice(m->device));
    return FEM_OK;
}

fem_status fem_mpnn_infer(fem_mpnn* m, const fem_problem* fp, int32_t R, const float* state, uint64_t seed,
                          float alpha, float* h_out, int on_device)
{
    if (!m || !fp || !state || !h_out) return mfail(FEM_E_INVAL, "NULL argument");
    fem_status s = infer_check(m, fp, R);
    if (s != FEM_OK) return s;
    const size_t nR = (size_t)fp->p.n * (size_t)R;
    const size_t bytes = nR * 4;
    const float* src = state;
    float* dst = h_out;
    float* tmp = nullptr;
    if (!on_device) {
        MCHK(hipMalloc(&tmp, 2 * bytes));
        hipError_t e = hipMemcpy(tmp, state, bytes, hipMemcpyHostToDevice);
        if (e != hipSuccess) {
            (void)hipFree(tmp);
            return mfail(FEM_E_HIP, "copy of the state", e);
        }
        src = tmp;
        dst = tmp + nR;
    }
    s = infer_enqueue(m, fp->p, R, src, seed, alpha, dst, nullptr);
    hipError_t e = hipDeviceSynchronize();
    if (s == FEM_OK && e != hipSuccess) s = mfail(FEM_E_HIP, "fem_mpnn_infer", e);
    if (tmp) {
        if (s == FEM_OK) {
            e = hipMemcpy(h_out, dst, bytes, hipMemcpyDeviceToHost);
            if (e != hipSuccess) s = mfail(FEM_E_HIP, "copy of the proposal", e);
        }
        (void)hipFree(tmp);
    }
    return s;
}

fem_status fem_mpnn_infer_async(fem_mpnn* m, const fem_problem* fp, int32_t R, const float* state, uint64_t seed,
                                float alpha, float* h_out, void* stream)
{
    if (!m || !fp || !state || !h_out) return mfail(FEM_E_INVAL, "NULL argument");
    fem_status s = infer_check(m, fp, R);
    if (s != FEM_OK) return s;
    return infer_enqueue(m, fp->p, R, state, seed, alpha, h_out, static_cast<hipStream_t>(stream));
}

fem_status fem_mpnn_save(fem_mpnn* m, const char* path)
{
    if (!m || !path) return mfail(FEM_E_INVAL, "NULL argument");
    std::vector<float> th(NP);
    fem_status s = fem_mpnn_get_params(m, th.data());
    if (s != FEM_OK) return s;
    FILE* f = std::fopen(path, "wb");
    if (!f) return mfail(FEM_E_INVAL, "cannot open the file for writing");
    const char magic[8] = {'F', 'E', 'M', 'M', 'P', 'N', 'N', '1'};
    const int32_t np = NP;
    const bool ok = std::fwrite(magic, 1, 8, f) == 8 && std::fwrite(&np, 4, 1, f) == 1 &&
                    std::fwrite(th.data(), 4, NP, f) == (size_t)NP;
    std::fclose(f);
    return ok ? FEM_OK : mfail(FEM_E_INVAL, "short write");
}

fem_status fem_mpnn_load(fem_mpnn* m, const char* path)
{
    if (!m || !path) return mfail(FEM_E_INVAL, "NULL argument");
    FILE* f = std::fopen(path, "rb");
    if (!f) return mfail(FEM_E_INVAL, "cannot open the file");
    char magic[8];
    int32_t np = 0;
    std::vector<float> th(NP);
    const bool ok = std::fread(magic, 1, 8, f) == 8 && std::memcmp(magic, "FEMMPNN1", 8) == 0 &&
                    std::fread(&np, 4, 1, f) == 1 && np == NP && std::fread(th.data(), 4, NP, f) == (size_t)NP;
    std::fclose(f);
    if (!ok) return mfail(FEM_E_INVAL, "not a network parameter file");
    return fem_mpnn_set_params(m, th.data());
}

}  // extern "C"
