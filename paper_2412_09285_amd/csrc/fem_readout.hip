// Read-out and integer evaluation of one-logit problems on bit words, and the
// selection of the best replica on the device.
//
// A configuration is one bit per (node, replica), so a word carries 32
// replicas through the neighbour gather, and the numbers counted per replica
// (differing neighbours, unsatisfied clauses) are kept bit-sliced: plane k of
// a lane holds bit k of 32 counters, and full adders take four words at a
// time.  Sums are integers and exact in any order.  The byte form that the
// general evaluation reads costs a byte of gather and several instructions
// per (neighbour, replica); here both shrink by the word's width, and what is
// left is reading the fields once (4 of the 12 bytes a row's state holds).
//
// Read-out of 10^5 nodes, 6 10^5 +-1 entries, R = 256 (MI355X): rounding 41,
// evaluation 64 and reduction 12 us in the byte form; packing 32 us (3.2 TB/s
// of the fields), evaluation 29 and counts 5 us here.  fem_best of the same
// solver: 2.08 ms when every configuration was copied to the host to pick one
// from, 0.13 ms with the selection below.
#include "fem_readout.h"

#include "fem_device.h"

namespace fem {

constexpr int PLANES = 8;    // counters hold up to 255 between flushes

// ------------------------------------------------------------ bits of h > 0
// Each half-wave forms words from 32 coalesced loads and a ballot, four words
// in flight.
__global__ void __launch_bounds__(256) pack_bits_kernel(int32_t n, int32_t R, int32_t rw, const float* __restrict__ h,
                                                        int64_t srow, uint32_t* __restrict__ bits,
                                                        int32_t* __restrict__ count, size_t n_count)
{
    for (size_t k = (size_t)blockIdx.x * 256 + threadIdx.x; k < n_count; k += (size_t)gridDim.x * 256) count[k] = 0;
    const int lane = threadIdx.x & 63, b = lane & 31;
    const uint32_t half = (blockIdx.x * 256 + threadIdx.x) >> 5, halves = gridDim.x * 8;
    // word (i, w) advances by `halves` words per turn
    int64_t i = half / (uint32_t)rw;
    uint32_t w = half % (uint32_t)rw;
    const uint32_t di = halves / (uint32_t)rw, dw = halves % (uint32_t)rw;
    constexpr int U = 4;
    // both halves of a wave take the same number of turns
    const size_t words = (size_t)n * rw;
    for (size_t k = half & ~1u; k < words; k += (size_t)U * halves) {
        float x[U];
        int64_t at[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = 32 * (int)w + b;
            at[u] = i < n ? i * rw + w : -1;
            x[u] = i < n && r < R ? h[i * srow + r] : 0.0f;
            i += di;
            w += dw;
            if (w >= (uint32_t)rw) {
                w -= (uint32_t)rw;
                ++i;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t m = __ballot(x[u] > 0.0f);
            if (b == 0 && at[u] >= 0) bits[at[u]] = lane ? (uint32_t)(m >> 32) : (uint32_t)m;
        }
    }
}

// ------------------------------------------------- bit-sliced counter sums --
__device__ __forceinline__ uint32_t maj3(uint32_t a, uint32_t b, uint32_t c) { return (a & b) | (c & (a | b)); }

struct BitCounter {
    uint32_t p[PLANES];
    int used;   // words added since the planes were empty
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int k = 0; k < PLANES; ++k) p[k] = 0;
        used = 0;
    }
    __device__ __forceinline__ void add4(const uint32_t (&x)[4])
    {
        const uint32_t c0 = maj3(p[0], x[0], x[1]);
        p[0] ^= x[0] ^ x[1];
        const uint32_t c1 = maj3(p[0], x[2], x[3]);
        p[0] ^= x[2] ^ x[3];
        uint32_t c = maj3(p[1], c0, c1);
        p[1] ^= c0 ^ c1;
#pragma unroll
        for (int k = 2; k < PLANES; ++k) {
            const uint32_t t = p[k] & c;
            p[k] ^= c;
            c = t;
        }
        used += 4;
    }
    // adds the 32 counters, less `off` each, to sum[0..31]; every lane starts
    // at another counter, so that lanes of the same word do not collide
    __device__ __forceinline__ void flush(int* sum, int off, int start)
    {
        for (int j = 0; j < 32; ++j) {
            const int b = (start + j) & 31;
            int v = -off;
#pragma unroll
            for (int k = 0; k < PLANES; ++k) v += (int)((p[k] >> b) & 1u) << k;
            atomicAdd(sum + b, v);
        }
        clear();
    }
};

struct BitArgs {
    const int64_t* row_off;
    const int32_t* adj_pm1;
    const int2* inc2;
    const int4* inc4;
    const Tile* tiles;
    const uint32_t* bits;
    int32_t* count;
    int32_t R, rw, lanes_log2, parts_log2;
};

// KIND 0: ordered cut of +-1 weights.  A weight -1 contributes -d = (1 - d) - 1:
// its complement is counted and the number of such entries taken off.
// KIND 2 / 3: unsatisfied clauses at owner incidences with two / three other
// literals.
template <int KIND>
__global__ void __launch_bounds__(256) eval_bits_kernel(BitArgs a)
{
    extern __shared__ int sums[];   // [words of this segment][32]
    const Tile tile = a.tiles[blockIdx.x];
    const int L = 1 << a.lanes_log2, tl = threadIdx.x & (L - 1);
    const int parts = 1 << a.parts_log2, part = (threadIdx.x >> a.lanes_log2) & (parts - 1);
    const int team = threadIdx.x >> (a.lanes_log2 + a.parts_log2), teams = 256 >> (a.lanes_log2 + a.parts_log2);
    const int w0 = blockIdx.y * L, w = w0 + tl;
    const int words = min(L, a.rw - w0);
    for (int k = threadIdx.x; k < words * 32; k += 256) sums[k] = 0;
    __syncthreads();
    if (w < a.rw) {
        BitCounter c;
        c.clear();
        int off = 0;
        const uint32_t* __restrict__ bits = a.bits + w;
        const int rw = a.rw;
        auto room = [&]() {
            if (c.used + 4 > (1 << PLANES) - 1) {
                c.flush(sums + tl * 32, off, threadIdx.x);
                off = 0;
            }
        };
        for (int i = tile.row_begin + team; i < tile.row_end; i += teams) {
            const uint32_t own = bits[(size_t)i * rw];
            const int64_t kend = a.row_off[i + 1];
            for (int64_t k = a.row_off[i] + 4 * part; k < kend; k += 4 * parts) {
                room();
                uint32_t x[4];
                if constexpr (KIND == 0) {
                    int32_t e[4];
                    uint32_t y[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) e[u] = k + u < kend ? a.adj_pm1[k + u] : i;   // row i itself: no difference
#pragma unroll
                    for (int u = 0; u < 4; ++u) y[u] = bits[(size_t)(e[u] & 0x7fffffff) * rw];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int s = e[u] >> 31;
                        x[u] = own ^ y[u] ^ (uint32_t)s;
                        off -= s;
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        x[u] = 0;
                        if (k + u >= kend) continue;
                        uint32_t lit[3];
                        bool own_pos, owner;
                        if constexpr (KIND == 2) {
                            const int2 rec = a.inc2[k + u];
                            lit[0] = (uint32_t)rec.x;
                            lit[1] = (uint32_t)rec.y;
                            lit[2] = SAT_NONE;
                            own_pos = (lit[0] & SAT_FLAG) != 0;
                            owner = (lit[1] & SAT_FLAG) != 0;
                        } else {
                            const int4 rec = a.inc4[k + u];
                            lit[0] = (uint32_t)rec.x;
                            lit[1] = (uint32_t)rec.y;
                            lit[2] = (uint32_t)rec.z;
                            own_pos = (rec.w & 1) != 0;
                            owner = (rec.w & 2) != 0;
                        }
                        if (!owner) continue;
                        x[u] = own_pos ? ~own : own;
#pragma unroll
                        for (int s = 0; s < KIND; ++s) {
                            const uint32_t var = lit[s] & SAT_VAR_MASK;
                            if (var != SAT_NONE) {
                                const uint32_t y = bits[(size_t)var * rw];
                                x[u] &= (lit[s] & SAT_POS) ? ~y : y;
                            }
                        }
                    }
                }
                c.add4(x);
            }
        }
        c.flush(sums + tl * 32, off, threadIdx.x);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < words * 32; k += 256) {
        const int r = w0 * 32 + k;
        if (r < a.R && sums[k] != 0) atomicAdd(a.count + (size_t)tile.inst * a.R + r, sums[k]);
    }
}

__global__ void count_finish_kernel(int kind, size_t n_count, const int32_t* __restrict__ count,
                                    double* __restrict__ v, double* __restrict__ best)
{
    const size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n_count) return;
    const double x = (double)count[k];
    v[k] = x;
    if (best) {
        const double score = kind == KIND_MAXCUT ? -0.5 * x : x;
        if (score < best[k]) best[k] = score;
    }
}

// ---------------------------------------------------------- best replica ---
// One workgroup per instance; the scores of fem_best: -(ordered cut),
// unsatisfied clauses, or 2 cut + lam (sum_s W_s^2 - sum_i V_i^2).
__global__ void __launch_bounds__(256) pick_kernel(int kind, int R, int q, double lam, const double* __restrict__ v,
                                                   const long long* __restrict__ sizes,
                                                   const double* __restrict__ v2, double* __restrict__ value,
                                                   int32_t* __restrict__ replica)
{
    __shared__ double ls[256];
    __shared__ int lr[256];
    const int inst = blockIdx.x;
    double bs = __builtin_inf();
    int br = 0x7fffffff;
    for (int r = threadIdx.x; r < R; r += 256) {
        const size_t k = (size_t)inst * R + r;
        double score;
        if (kind == KIND_MAXCUT) {
            score = -v[k];
        } else if (kind == KIND_MAXSAT) {
            score = v[k];
        } else {
            double pen = -v2[inst];
            for (int s = 0; s < q; ++s) {
                const double x = (double)sizes[k * q + s];
                pen += x * x;
            }
            score = v[k] + lam * pen;
        }
        if (score < bs) {
            bs = score;
            br = r;
        }
    }
    ls[threadIdx.x] = bs;
    lr[threadIdx.x] = br;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < (unsigned)o) {
            const double s = ls[threadIdx.x + o];
            const int r = lr[threadIdx.x + o];
            if (s < ls[threadIdx.x] || (s == ls[threadIdx.x] && r < lr[threadIdx.x])) {
                ls[threadIdx.x] = s;
                lr[threadIdx.x] = r;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const int r = lr[0] == 0x7fffffff ? 0 : lr[0];   // no comparable score: the first replica
        replica[inst] = r;
        value[inst] = v[(size_t)inst * R + r];
    }
}

__global__ void __launch_bounds__(256) config_kernel(int kind, int32_t n, int32_t q, const float* __restrict__ h,
                                                     int64_t srow, int n_inst, const int32_t* __restrict__ inst_off,
                                                     const int32_t* __restrict__ replica, uint8_t* __restrict__ out)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        int lo = 0, hi = n_inst;   // inst_off[lo] <= i < inst_off[hi]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (inst_off[mid] <= i) lo = mid;
            else hi = mid;
        }
        const float* x = h + i * srow + (size_t)replica[lo] * (kind == KIND_BMINCUT ? q : 1);
        int best = 0;
        if (kind != KIND_BMINCUT) {
            best = x[0] > 0.0f ? 1 : 0;
        } else {
            float bv = x[0];
            for (int s = 1; s < q; ++s)
                if (x[s] > bv) {
                    bv = x[s];
                    best = s;
                }
        }
        out[i] = (uint8_t)best;
    }
}

// -------------------------------------------------------------- launchers --
bool bit_evaluation(const Problem& p)
{
    // counts per instance stay below 2^31 in every partial sum
    return p.nnz <= INT32_MAX && (p.kind == KIND_MAXSAT || (p.kind == KIND_MAXCUT && p.adj_pm1 != nullptr));
}

// Long rows of few words are shared by several lanes while a lane keeps 32
// entries and more and the chip has lanes to spare: alone, a lane of a complete
// graph walks its row through as many dependent rounds as it has entries / 4
// (a read-out of n = 2500, R = 8: 705 us, by bytes 549, in 64 parts 27).
int bit_parts(const Problem& p, int R)
{
    int parts = 1;
    while (bit_lanes(R) * parts < 64 && p.nnz / p.n >= 64 * parts && (int64_t)p.n * bit_lanes(R) * parts < 1 << 18)
        parts <<= 1;
    return parts;
}

// A lane's 32 counters are flushed at the end of its rows (some 700
// instructions): up to eight rows a lane, fewer while that would leave less
// than 512 workgroups.
int bit_tile_rows(const Problem& p, int R)
{
    const int teams = 256 / (bit_lanes(R) * bit_parts(p, R));
    const int64_t rows = p.n / ((int64_t)teams * 512);
    return teams * (int)(rows < 1 ? 1 : rows > 8 ? 8 : rows);
}

hipError_t launch_pack_bits(int32_t n, int32_t R, const float* h, int64_t srow, uint32_t* bits, int32_t* count,
                            size_t n_count, hipStream_t st)
{
    (void)hipGetLastError();   // drop stale errors of earlier calls
    const size_t words = (size_t)n * bit_words(R);
    const size_t blocks = (words + 31) / 32;   // four words per half-wave
    pack_bits_kernel<<<(unsigned)(blocks < 4096 ? blocks : 4096), 256, 0, st>>>(n, R, bit_words(R), h, srow, bits,
                                                                               count, n_count);
    return hipGetLastError();
}

hipError_t launch_eval_bits(const Problem& p, int32_t R, const Tile* tiles, int n_tiles, const uint32_t* bits,
                            int32_t* count, hipStream_t st)
{
    (void)hipGetLastError();   // drop stale errors of earlier calls
    if (n_tiles == 0) return hipSuccess;
    BitArgs a{};
    a.row_off = p.row_off;
    a.adj_pm1 = p.adj_pm1;
    a.inc2 = p.inc2;
    a.inc4 = p.inc4;
    a.tiles = tiles;
    a.bits = bits;
    a.count = count;
    a.R = R;
    a.rw = bit_words(R);
    const int L = bit_lanes(R);
    while ((1 << a.lanes_log2) < L) ++a.lanes_log2;
    while ((1 << a.parts_log2) < bit_parts(p, R)) ++a.parts_log2;
    const dim3 g(n_tiles, (a.rw + L - 1) / L);
    const size_t lds = (size_t)L * 32 * sizeof(int);
    if (p.kind == KIND_MAXCUT) eval_bits_kernel<0><<<g, 256, lds, st>>>(a);
    else if (p.sat_width == 2) eval_bits_kernel<2><<<g, 256, lds, st>>>(a);
    else eval_bits_kernel<3><<<g, 256, lds, st>>>(a);
    return hipGetLastError();
}

hipError_t launch_count_finish(int kind, size_t n_count, const int32_t* count, double* v, double* best,
                               hipStream_t st)
{
    (void)hipGetLastError();   // drop stale errors of earlier calls
    count_finish_kernel<<<(unsigned)((n_count + 255) / 256), 256, 0, st>>>(kind, n_count, count, v, best);
    return hipGetLastError();
}

hipError_t launch_pick(int kind, int R, int n_inst, int q, double lam, const double* v, const long long* sizes,
                       const double* v2, double* value, int32_t* replica, hipStream_t st)
{
    (void)hipGetLastError();   // drop stale errors of earlier calls
    if (kind == KIND_BMINCUT && (!v2 || !sizes)) return hipErrorInvalidValue;
    pick_kernel<<<n_inst, 256, 0, st>>>(kind, R, q, lam, v, sizes, v2, value, replica);
    return hipGetLastError();
}

hipError_t launch_config(int kind, int32_t n, int32_t q, const float* h, int64_t srow, int n_inst,
                         const int32_t* inst_off, const int32_t* replica, uint8_t* out, hipStream_t st)
{
    (void)hipGetLastError();   // drop stale errors of earlier calls
    const int blocks = (n + 255) / 256;
    config_kernel<<<blocks < 4096 ? blocks : 4096, 256, 0, st>>>(kind, n, q, h, srow, n_inst, inst_off, replica, out);
    return hipGetLastError();
}

}  // namespace fem
