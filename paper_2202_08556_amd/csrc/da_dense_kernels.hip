// Dense products of a graph-convolution layer on the fp32 matrix cores (v_mfma_f32_16x16x4f32): a tall
// matrix of node features against a small weight matrix.  Both shapes are bound by reading the tall
// operands once (100 000 x 96 and 100 000 x 64 floats: 64 MB, 13 us at copy rate; the arithmetic takes
// 8 us), which the general GEMM library does not reach when one side of the product is small: it took
// 310 us for the weight gradient and 36 to 45 us for the other two.
//
// Operand layout of the instruction: lane l holds A[l % 16][l / 16], B[l / 16][l % 16] and, in register r,
// D[4 * (l / 16) + r][l % 16].
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace daspmm {

typedef float mfma_acc __attribute__((ext_vector_type(4)));

__device__ __forceinline__ mfma_acc mfma16(float a, float b, mfma_acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// ------------------------------------------------------------------------------------------
// dW = X^T . G:  X rows x fin, G rows x fout, both row-major.
//
// The long dimension is the sum: a block owns a range of rows and a 64 x 64 tile of dW, its four waves
// take 16 rows at a time in turn and keep the whole tile in registers (16 accumulators).  Element t of a
// lane's 16-byte load of a row belongs to accumulator t, so tile row 4 i + t is lane i's element t: any
// assignment of columns to lanes gives the same sums, and this one needs no shuffling or LDS between
// memory and the matrix cores.  The waves' tiles are added in LDS, the blocks' by weight_grad_sum_kernel,
// in a fixed order, so the result does not depend on the schedule.
// Lanes past the last column repeat the last four columns (fin, fout >= 4) and write the same results.
// ------------------------------------------------------------------------------------------
constexpr int kWgTile = 64;
constexpr int kWgBlock = 256;
constexpr int kWgPart = kWgTile * kWgTile;                // floats of a block's partial result

__device__ __forceinline__ float4 load4(const float* __restrict__ p) {
    typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
    const f4 x = *reinterpret_cast<const f4*>(p);
    return make_float4(x.x, x.y, x.z, x.w);
}

__global__ __launch_bounds__(kWgBlock) void weight_grad_kernel(
    int rows, int fin, int fout, const float* __restrict__ X, long ldx, const float* __restrict__ G, long ldg,
    int rows_per_block, float* __restrict__ part)
{
    constexpr int U = 4;                                   // groups of 4 rows a wave takes at once
    __shared__ float tile[3][kWgTile * kWgTile];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = lane & 15, kk = lane >> 4;
    const int tiles_n = (fout + kWgTile - 1) / kWgTile;
    const int tm = blockIdx.y / tiles_n, tn = blockIdx.y % tiles_n;
    const int cx = min(tm * kWgTile + 4 * i, fin - 4), cg = min(tn * kWgTile + 4 * i, fout - 4);
    const int r0 = blockIdx.x * rows_per_block, r1 = min(r0 + rows_per_block, rows);
    mfma_acc acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = mfma_acc{0.f, 0.f, 0.f, 0.f};
    auto step = [&](const float4& x, const float4& g) {
        const float xa[4] = {x.x, x.y, x.z, x.w}, gb[4] = {g.x, g.y, g.z, g.w};
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[a][b] = mfma16(xa[a], gb[b], acc[a][b]);
    };
    int r = r0 + wave * 4 * U;
    for (; r + 4 * U <= r1; r += 4 * 4 * U) {
        float4 x[U], g[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long row = r + 4 * u + kk;
            x[u] = load4(X + row * ldx + cx);
            g[u] = load4(G + row * ldg + cg);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) step(x[u], g[u]);
    }
    for (int u = 0; u < U; ++u) {                          // the last rows of the range, at most one wave's turn
        if (r + 4 * u >= r1) break;
        const long row = r + 4 * u + kk;
        float4 x = make_float4(0.f, 0.f, 0.f, 0.f), g = x;
        if (row < r1) { x = load4(X + row * ldx + cx); g = load4(G + row * ldg + cg); }
        step(x, g);
    }
    // accumulator (a, b), register q: tile row 4 * (4 kk + q) + a, tile column 4 i + b
    if (wave > 0) {
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<float4*>(&tile[wave - 1][(4 * (4 * kk + q) + a) * kWgTile + 4 * i]) =
                    make_float4(acc[a][0][q], acc[a][1][q], acc[a][2][q], acc[a][3][q]);
    }
    __syncthreads();
    float* __restrict__ out = part + ((long)blockIdx.y * gridDim.x + blockIdx.x) * kWgPart;
    if (wave == 0) {
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int at = (4 * (4 * kk + q) + a) * kWgTile + 4 * i;
                float4 s = make_float4(acc[a][0][q], acc[a][1][q], acc[a][2][q], acc[a][3][q]);
#pragma unroll
                for (int w = 0; w < 3; ++w) {
                    const float4 o = *reinterpret_cast<const float4*>(&tile[w][at]);
                    s.x += o.x; s.y += o.y; s.z += o.z; s.w += o.w;
                }
                *reinterpret_cast<float4*>(&out[at]) = s;
            }
    }
}

// Sum of nblocks values `stride` floats apart, cut into 16 stretches, one per wave of a block of 1024; the
// result is the first wave's.
__device__ __forceinline__ float sum_over_blocks(const float* __restrict__ p, int nblocks, long stride) {
    constexpr int U = 8;
    __shared__ float sh[16][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int per = (nblocks + 15) / 16;
    const int b0 = min(wave * per, nblocks), b1 = min(b0 + per, nblocks);
    float s = 0.f;
    for (int b = b0; b < b1; b += U) {
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = p[(long)min(b + u, b1 - 1) * stride];
#pragma unroll
        for (int u = 0; u < U; ++u) s += b + u < b1 ? v[u] : 0.f;
    }
    sh[wave][lane] = s;
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int w = 1; w < 16; ++w) s += sh[w][lane];
    }
    return s;
}

// Adds the blocks' partial results; a block owns one row of one tile.
__global__ __launch_bounds__(1024) void weight_grad_sum_kernel(const float* __restrict__ part, int nblocks, int fin, int fout,
                                                               float* __restrict__ dW)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int tiles_n = (fout + kWgTile - 1) / kWgTile;
    const int tm = blockIdx.y / tiles_n, tn = blockIdx.y % tiles_n;
    const float s = sum_over_blocks(part + (long)blockIdx.y * nblocks * kWgPart + blockIdx.x * 64 + lane, nblocks, kWgPart);
    if (wave == 0) {
        // a tile's columns and rows 4 i + t stand for min(4 i, last four) + t of the matrix
        const int col = min(tn * kWgTile + (lane & ~3), fout - 4) + (lane & 3);
        const int row = min(tm * kWgTile + ((int)blockIdx.x & ~3), fin - 4) + ((int)blockIdx.x & 3);
        dW[(long)row * fout + col] = s;
    }
}

// ------------------------------------------------------------------------------------------
// Column sums of a tall row-major matrix (the gradient of a layer's bias).  A thread owns one column and
// every (256 / L)-th row of its block's range, L = columns rounded up to a power of two; 8 rows in flight.
// (The framework's reduction took 1.3 ms on 262 144 x 41, where the matrix is read in 10 us.)
// ------------------------------------------------------------------------------------------
constexpr int kCsBlock = 256;

__global__ __launch_bounds__(kCsBlock) void column_sums_kernel(int rows, int n, int lanes, const float* __restrict__ G, long ldg,
                                                               int rows_per_block, float* __restrict__ part)
{
    constexpr int U = 8;
    __shared__ float sh[kCsBlock];
    const int c = threadIdx.x & (lanes - 1), rl = threadIdx.x / lanes, step = kCsBlock / lanes;
    const int col = blockIdx.y * lanes + c;
    const int r0 = blockIdx.x * rows_per_block, r1 = min(r0 + rows_per_block, rows);
    float s[U];
#pragma unroll
    for (int u = 0; u < U; ++u) s[u] = 0.f;
    if (col < n) {
        const float* __restrict__ g = G + col;
        int r = r0 + rl;
        for (; r + (U - 1) * step < r1; r += U * step) {
#pragma unroll
            for (int u = 0; u < U; ++u) s[u] += g[(long)(r + u * step) * ldg];
        }
        for (; r < r1; r += step) s[0] += g[(long)r * ldg];
    }
#pragma unroll
    for (int d = U / 2; d >= 1; d >>= 1)
#pragma unroll
        for (int u = 0; u < d; ++u) s[u] += s[u + d];
    sh[threadIdx.x] = s[0];
    for (int d = kCsBlock / 2; d >= lanes; d >>= 1) {
        __syncthreads();
        if ((int)threadIdx.x < d) sh[threadIdx.x] += sh[threadIdx.x + d];
    }
    if (rl == 0 && col < n) part[(long)blockIdx.x * n + col] = sh[c];
}

__global__ __launch_bounds__(1024) void column_sums_sum_kernel(const float* __restrict__ part, int nblocks, int n,
                                                               float* __restrict__ out)
{
    const int col = blockIdx.x * 64 + (threadIdx.x & 63);
    const float s = sum_over_blocks(part + min(col, n - 1), nblocks, n);
    if (threadIdx.x < 64 && col < n) out[col] = s;
}

// ------------------------------------------------------------------------------------------
// Z = relu(Z + bias), either part optional, in place: one pass over Z instead of one per operation.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void bias_relu_kernel(long rows, int n, float* __restrict__ Z, const float* __restrict__ bias,
                                                        int relu)
{
    typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
    const long total = rows * n, vecs = total / 4;
    const long stride = (long)gridDim.x * 256;
    auto put = [&](float z, long at) {
        if (bias) z += bias[at % n];
        return relu ? (z > 0.f || z != z ? z : 0.f) : z;   // NaN stays NaN
    };
    const long first = (long)blockIdx.x * 256 + threadIdx.x;
    int at = (int)((4 * first) % n);                       // column of the vector's first element
    const int advance = (int)((4 * stride) % n);
    for (long v = first; v < vecs; v += stride) {
        f4 z = *reinterpret_cast<f4*>(Z + 4 * v);
        int c = at;
        at += advance;
        if (at >= n) at -= n;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float x = z[q];
            if (bias) x += bias[c];
            z[q] = relu ? (x > 0.f || x != x ? x : 0.f) : x;
            c = c + 1 == n ? 0 : c + 1;
        }
        *reinterpret_cast<f4*>(Z + 4 * v) = z;
    }
    if (blockIdx.x == 0 && threadIdx.x < total - 4 * vecs) {
        const long at = 4 * vecs + threadIdx.x;
        Z[at] = put(Z[at], at);
    }
}

// ------------------------------------------------------------------------------------------
// C = A . W:  A rows x k row-major, W k x n with element (p, q) at W[p*wk + q*wn] (so that the same kernel
// multiplies by a weight matrix and by its transpose), C rows x n row-major.
//
// A block keeps its NT * 16 columns of W in LDS, column by column so that a lane takes four consecutive k
// with one 16-byte read, and its waves walk over the rows of A, 16 at a time, with A straight from memory:
// 16 bytes (the same four k) per lane.  A register that a matrix instruction has consumed is requested
// again for the wave's next 16 rows at once, so memory is busy while the matrix cores are.  Column tiles
// stand as the first operand of the instruction, so that the four registers of an accumulator are four
// neighbouring columns of one row of C and leave in one 16-byte store.
// Memory bounds it: 100 003 x 96 times 96 x 64 is 64 MB, 13 us at copy rate, 8 us of arithmetic.  (Staging
// W in pieces of 64 rows for one set of rows per wave took 33 us, the library 31 to 45 us and, at any
// size, 18 us of host time.)
// ------------------------------------------------------------------------------------------
constexpr int kDpBlock = 256;

__host__ __device__ constexpr int dense_pitch(int k) { return (k + 15) / 16 * 16 + 4; }   // 8 neighbouring columns: 8 bank groups
template <int NT> constexpr size_t dense_lds(int k) { return (size_t)NT * 16 * dense_pitch(k) * sizeof(float); }

template <int NT, int KS>
__global__ __launch_bounds__(kDpBlock) void dense_product_kernel(
    int rows, int n, int k, const float* __restrict__ A, long lda, const float* __restrict__ W, long wk, long wn,
    float* __restrict__ C, long ldc)
{
    extern __shared__ __align__(16) float ws[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = lane & 15, kk = lane >> 4;
    const int n0 = blockIdx.y * NT * 16;
    const int ks = (k + 15) >> 4, pitch = dense_pitch(k);
    const int tiles = (rows + 15) >> 4;
    float4 x[KS];
    auto fetch = [&](int tile, int s) {
        const float* p = A + (long)min(tile * 16 + i, rows - 1) * lda + 16 * s + 4 * kk;
        const int left = k - 16 * s - 4 * kk;
        if (16 * s + 16 <= k) {                            // uniform
            x[s] = load4(p);
        } else {                                           // past the end: zeros, whatever lies there in memory
            x[s].x = left > 0 ? p[0] : 0.f;
            x[s].y = left > 1 ? p[1] : 0.f;
            x[s].z = left > 2 ? p[2] : 0.f;
            x[s].w = left > 3 ? p[3] : 0.f;
        }
    };
    int tile = blockIdx.x * 4 + wave;
    if (tile < tiles) {
#pragma unroll
        for (int s = 0; s < KS; ++s) if (s < ks) fetch(tile, s);
    }
    // Stage W, four elements a request along its unit stride and four requests of a thread in flight (element
    // by element it took longer than everything else on a few thousand rows).
    const int kpad = ks * 16;
    const bool by_column = wn == 1;
    const int inner = by_column ? NT * 16 : kpad;          // extent along the unit stride
    const int groups = NT * 16 * kpad / 4, per_line = inner / 4;
    const bool unit = by_column || wk == 1;
    for (int e0 = threadIdx.x; e0 < groups; e0 += 4 * kDpBlock) {
        float v[4][4];
        int at[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = min(e0 + u * kDpBlock, groups - 1);
            const int line = e / per_line, in4 = (e - line * per_line) * 4;
            const int p = by_column ? line : in4, q = by_column ? in4 : line;
            const float* w = W + (long)p * wk + (long)(n0 + q) * wn;
            const int left = by_column ? (p < k ? n - n0 - q : 0) : (n0 + q < n ? k - p : 0);
            at[u] = q * pitch + p;
            if (unit && left >= 4) {
                const float4 x4 = load4(w);
                v[u][0] = x4.x; v[u][1] = x4.y; v[u][2] = x4.z; v[u][3] = x4.w;
            } else {
                const long stride = by_column ? wn : wk;
#pragma unroll
                for (int c = 0; c < 4; ++c) v[u][c] = c < left ? w[c * stride] : 0.f;
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (e0 + u * kDpBlock < groups) {
#pragma unroll
                for (int c = 0; c < 4; ++c) ws[at[u] + (by_column ? c * pitch : c)] = v[u][c];
            }
        }
    }
    __syncthreads();
    typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
    const float* wl = ws + i * pitch + 4 * kk;
    for (; tile < tiles; tile += gridDim.x * 4) {
        const int next = tile + gridDim.x * 4;
        mfma_acc acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = mfma_acc{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            if (s < ks) {
                float4 w[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t) w[t] = *reinterpret_cast<const float4*>(wl + 16 * t * pitch + 16 * s);
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] = mfma16(w[t].x, x[s].x, acc[t]);
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] = mfma16(w[t].y, x[s].y, acc[t]);
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] = mfma16(w[t].z, x[s].z, acc[t]);
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] = mfma16(w[t].w, x[s].w, acc[t]);
                if (next < tiles) fetch(next, s);
            }
        }
        const long row = (long)tile * 16 + i;
        if (row < rows) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int col = n0 + 16 * t + 4 * kk;
                float* __restrict__ c = C + row * ldc + col;
                if (col + 4 <= n) {
                    *reinterpret_cast<f4*>(c) = f4{acc[t][0], acc[t][1], acc[t][2], acc[t][3]};
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) if (col + q < n) c[q] = acc[t][q];
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------------------
// The same product with every fp32 number taken as the exact sum of three bf16 numbers (rounded to nearest one
// after another: 8 + 8 + 8 significant bits) and six of the nine products of the pieces on the bf16 matrix cores
// (v_mfma_f32_16x16x32_bf16, fp32 accumulation); the three left out are below 2^-24 of the product.  The leading
// product has accumulators of its own, to which the sum of the other five is added once at the end.
//
// dense_split_weights_kernel lays the pieces of W out in the order in which lanes read them, 32 inner positions a
// step.  A block of dense_split_kernel is 4 waves of 32 rows of A each and up to 128 columns.  A wave reads its
// rows itself, whole 64-byte pieces, and converts each number once; the step's piece of W goes through LDS (two
// buffers, one barrier a step), and what the next step needs is in flight while this one is multiplied.  The last
// step begins 32 positions before the end; the weights of positions that an earlier step had are zero there.
//
// Lane l holds A row (or column of W) l % 16 and inner positions 4 (l / 16) + {0 ... 3, 16 ... 19} of a step.
//
// 262 144 x 602 times 602 x 128: the GEMM library's fp32 product 358 us (113 TFLOP/s; the fp32 matrix cores give at most
// 157), this one 255: 950 TFLOP/s of bf16 products, where a large bf16 product of the library reaches 1200, with the
// conversions and 765 MB of A and C (150 us at copy rate) beside it.  One instead of two steps in flight, one accumulator
// instead of two, blocks of 8 waves and blocks that stay over several sets of rows all came out within 5 % of it;
// splitting W in every block instead of once per call took 300 us.  Error against float64 (2-norm, relative): 1.4e-7,
// the library's 4.4e-7.
//
// Results that the pieces do not carry are computed again on the fp32 matrix cores, 32 rows of 16 columns at a time: where one
// is not finite (infinities split into infinity and NaN, numbers next to the largest round to infinity) or so small that
// products of pieces may have been lost below the smallest normal number.  Pieces of numbers below 2^-100 may be lost
// there, too, up to 2^-125 of a number and with it that much of the largest number it is multiplied by, k times over at
// most: results are computed again that are not 2^26 times as large.  Only waves that hold such a number, or whose weights
// do, look for the largest ones, so that one among ordinary numbers costs next to nothing (262 144 x 602 x 128: 270 us with such
// a weight, 274 with such a number in one row of 64, 263 without; 576 where these rows hold nothing larger, 705 where
// all results are that small).
// ------------------------------------------------------------------------------------------
template <bool B> struct Truth { static constexpr bool value = B; };
constexpr int kSplitBlock = 256, kSplitRows = 128, kSplitStep = 32;   // 4 waves of 32 rows

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// The pieces of 8 numbers.
struct SplitFrag { bf16x8 p[3]; };

__device__ __forceinline__ SplitFrag split8(const float* x) {
    typedef float f2 __attribute__((ext_vector_type(2)));
    SplitFrag f;
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        f2 r = {x[e], x[e + 1]};
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const bf16x2 b = __builtin_convertvector(r, bf16x2);
            f.p[q][e] = b[0];
            f.p[q][e + 1] = b[1];
            if (q < 2) { r[0] -= (float)b[0]; r[1] -= (float)b[1]; }
        }
    }
    return f;
}

// Order of |x| in which zero is the largest; keys below kSplitTiny are numbers other than zero below 2^-100.
constexpr unsigned kSplitTiny = (27u << 24) - 1u;
__device__ __forceinline__ unsigned tiny_key(float x) { return (__float_as_uint(x) << 1) - 1u; }

// A barrier that orders LDS only: loads from memory stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__host__ __device__ constexpr int split_steps(int k) { return (k + kSplitStep - 1) / kSplitStep; }

// Pieces of W: frag[((step * tiles + tile) * 3 + piece) * 64 + lane], tile = 16 columns; columns past the last repeat it.
// tiny[step * tiles + tile]: whether a weight is that small.  sizes[(step * tiles + tile) * 16 + column]: the largest weight of
// the column, the sign bit set where one is that small.  One wave per step and tile.
constexpr size_t kSplitBytes = 192 * sizeof(bf16x8) + 17 * sizeof(int);   // of the workspace, for a step and tile

__global__ __launch_bounds__(64) void dense_split_weights_kernel(int k, int n, const float* __restrict__ W, long wk, long wn,
                                                                 bf16x8* __restrict__ frag, unsigned* __restrict__ sizes, int* __restrict__ tiny)
{
    const int step = blockIdx.x, tile = blockIdx.y, tiles = gridDim.y, lane = threadIdx.x;
    const int p0 = min(step * kSplitStep, k - kSplitStep) + 4 * (lane >> 4);
    const float* __restrict__ w = W + (long)min(tile * 16 + (lane & 15), n - 1) * wn;
    float x[8];
    unsigned least = ~0u, most = 0u;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int p = p0 + (e & 3) + 16 * (e >> 2);
        x[e] = w[(long)p * wk];
        x[e] = p >= step * kSplitStep ? x[e] : 0.f;
        least = min(least, tiny_key(x[e]));
        most = max(most, __float_as_uint(x[e]) & 0x7fffffffu);
    }
    const SplitFrag f = split8(x);
    const long at = (long)step * tiles + tile;
#pragma unroll
    for (int q = 0; q < 3; ++q) frag[(at * 3 + q) * 64 + lane] = f.p[q];
#pragma unroll
    for (int d = 16; d <= 32; d *= 2) {
        least = min(least, (unsigned)__shfl_xor((int)least, d));
        most = max(most, (unsigned)__shfl_xor((int)most, d));
    }
    if (lane < 16) sizes[at * 16 + lane] = most | (least < kSplitTiny ? 0x80000000u : 0u);
    const bool any = __any(least < kSplitTiny);
    if (lane == 0) tiny[at] = any;
}

// NT tiles of 16 columns.  k >= 32; `tiles` tiles to a step of `frag`.
template <int NT>
__global__ __launch_bounds__(kSplitBlock, 2) void dense_split_kernel(
    int rows, int n, int k, const float* __restrict__ A, long lda, const float* __restrict__ W, long wk, long wn,
    const bf16x8* __restrict__ frag, const unsigned* __restrict__ sizes, const int* __restrict__ tiny, int tiles, float* __restrict__ C,
    long ldc)
{
    constexpr int kFrags = 3 * NT * 64;                    // 16-byte pieces of a step
    constexpr int WL = (kFrags + kSplitBlock - 1) / kSplitBlock;
    __shared__ bf16x8 buf[2][kFrags];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = lane & 15, h = lane >> 4;
    const int tile0 = blockIdx.y * NT, n0 = tile0 * 16;
    const int steps = split_steps(k);
    // the tiles of the last column block that do not exist read the last one that does
    const bf16x8* __restrict__ wsrc[WL];
    bool wuse[WL];
#pragma unroll
    for (int j = 0; j < WL; ++j) {
        const int at = threadIdx.x + j * kSplitBlock;
        wuse[j] = at < kFrags;
        const int tile = min(tile0 + at / 192, tiles - 1);
        wsrc[j] = frag + (long)tile * 192 + at % 192;
    }
    bool w_tiny = false;
    for (int s = lane; s < steps * tiles; s += 64) w_tiny |= tiny[s] != 0;
    w_tiny = __any(w_tiny);

    float x[16];
    bf16x8 w[WL];
    auto fetch_w = [&](int s) {
#pragma unroll
        for (int j = 0; j < WL; ++j) w[j] = wsrc[j][(long)s * tiles * 192];
    };
    const long first = (long)blockIdx.x * kSplitRows + wave * 32 + i;
    const float* __restrict__ arow[2] = {A + min(first, (long)rows - 1) * lda + 4 * h, A + min(first + 16, (long)rows - 1) * lda + 4 * h};
    auto fetch_a = [&](int s) {
        const int p = min(s * kSplitStep, k - kSplitStep);
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const float4 v = load4(arow[r] + p + 16 * q);
                x[8 * r + 4 * q] = v.x; x[8 * r + 4 * q + 1] = v.y; x[8 * r + 4 * q + 2] = v.z; x[8 * r + 4 * q + 3] = v.w;
            }
    };
    mfma_acc big[2][NT], small[2][NT];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t) big[r][t] = small[r][t] = mfma_acc{0.f, 0.f, 0.f, 0.f};
    unsigned least[2] = {~0u, ~0u}, most[2] = {0u, 0u};   // of the rows' numbers; most only if w_tiny
    fetch_w(0);
    fetch_a(0);
    for (int s = 0; s < steps; ++s) {
        bf16x8* __restrict__ b = buf[s & 1];
#pragma unroll
        for (int j = 0; j < WL; ++j) if (WL * kSplitBlock == kFrags || wuse[j]) b[threadIdx.x + j * kSplitBlock] = w[j];
        SplitFrag a[2];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            a[r] = split8(x + 8 * r);
#pragma unroll
            for (int q = 0; q < 8; ++q) least[r] = min(least[r], tiny_key(x[8 * r + q]));
        }
        if (w_tiny) {
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int q = 0; q < 8; ++q) most[r] = max(most[r], __float_as_uint(x[8 * r + q]) & 0x7fffffffu);
        }
        fetch_w(min(s + 1, steps - 1));                // in flight across the barrier and the matrix instructions
        fetch_a(min(s + 1, steps - 1));
        lds_barrier();                                 // the other buffer's readers are past the barrier before this one
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const bf16x8 w0 = b[(t * 3) * 64 + lane], w1 = b[(t * 3 + 1) * 64 + lane], w2 = b[(t * 3 + 2) * 64 + lane];
            auto dot = [&](bf16x8 u, int piece, mfma_acc (&c)[2][NT]) {
#pragma unroll
                for (int r = 0; r < 2; ++r) c[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(u, a[r].p[piece], c[r][t], 0, 0, 0);
            };
            dot(w0, 0, big);
            dot(w0, 2, small);
            dot(w1, 1, small);
            dot(w2, 0, small);
            dot(w0, 1, small);
            dot(w1, 0, small);
        }
    }

    // sizes of results, sign dropped: other than zero below 2^-90, not finite
    constexpr unsigned kResultTiny = (37u << 24) - 1u, kResultMost = 0xfefffffeu;
    unsigned low = ~0u, high = 0u;
    auto look = [&](const mfma_acc& x) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            low = min(low, tiny_key(x[q]));
            high = max(high, __float_as_uint(x[q]) << 1);
        }
    };
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            big[r][t] += small[r][t];
            look(big[r][t]);
        }
    unsigned again = 0u;                                   // bit t: tile t
    if (__any((low < kResultTiny) | (high > kResultMost))) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            low = ~0u;
            high = 0u;
            look(big[0][t]);
            look(big[1][t]);
            again |= (unsigned)((low < kResultTiny) | (high > kResultMost)) << t;
        }
    }
    if (w_tiny || __any(min(least[0], least[1]) < kSplitTiny)) {
        float row_most[2];                                 // what tiny weights may have lost is that much times 2^-125
        bool row_tiny[2];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
#pragma unroll
            for (int d = 16; d <= 32; d *= 2) {
                least[r] = min(least[r], (unsigned)__shfl_xor((int)least[r], d));
                most[r] = max(most[r], (unsigned)__shfl_xor((int)most[r], d));
            }
            row_most[r] = __uint_as_float(most[r]);
            row_tiny[r] = least[r] < kSplitTiny;
        }
        const float per = (float)k * 1.5777218e-30f;       // 2^-99
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const unsigned* __restrict__ of_tile = sizes + (long)min(tile0 + t, tiles - 1) * 16 + 4 * h;
            unsigned col_most[4] = {0u, 0u, 0u, 0u}, col_tiny = 0u;
            for (int s = i; s < steps; s += 16)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const unsigned x = of_tile[(long)s * tiles * 16 + q];
                    col_most[q] = max(col_most[q], x & 0x7fffffffu);
                    col_tiny |= (x >> 31) << q;
                }
#pragma unroll
            for (int d = 1; d <= 8; d *= 2) {
                col_tiny |= (unsigned)__shfl_xor((int)col_tiny, d);
#pragma unroll
                for (int q = 0; q < 4; ++q) col_most[q] = max(col_most[q], (unsigned)__shfl_xor((int)col_most[q], d));
            }
            float spare = 0.f;                             // below zero where a result is too small
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float a = row_tiny[r] ? __uint_as_float(col_most[q]) : 0.f, b = (col_tiny >> q & 1u) ? row_most[r] : 0.f;
                    spare = fminf(spare, fabsf(big[r][t][q]) - per * fmaxf(a, b));
                }
            again |= (unsigned)(spare < 0.f) << t;
        }
    }
    if (__any(again != 0u)) {
        unsigned redo = 0u;
#pragma unroll
        for (int t = 0; t < NT; ++t) redo |= __any(again >> t & 1u) ? 1u << t : 0u;
        // 16 positions at a time, 4 of them a lane's own; the last ones begin 16 before the end and leave out what was there.
        // From three tiles on all of them: loads of all tiles are then in flight together.
        auto fp32 = [&](auto all) {
            constexpr bool ALL = decltype(all)::value;
#pragma unroll
            for (int t = 0; t < NT; ++t)
                if (ALL || (redo >> t & 1u)) big[0][t] = big[1][t] = mfma_acc{0.f, 0.f, 0.f, 0.f};
            for (int p0 = 0; p0 < k; p0 += 16) {
                const int p = min(p0, k - 16) + 4 * h;
                float u[2][4], v[NT][4];
                auto fetch = [&](int t) {
                    const float* __restrict__ wcol = W + (long)min(n0 + 16 * t + i, n - 1) * wn;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[t][e] = wcol[(long)(p + e) * wk];
                };
                auto multiply = [&](int t) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float x = p + e >= p0 ? v[t][e] : 0.f;
#pragma unroll
                        for (int r = 0; r < 2; ++r) big[r][t] = mfma16(x, u[r][e], big[r][t]);
                    }
                };
                if constexpr (ALL)
#pragma unroll
                    for (int t = 0; t < NT; ++t) fetch(t);
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const float4 x4 = load4(arow[r] - 4 * h + p);
                    u[r][0] = x4.x; u[r][1] = x4.y; u[r][2] = x4.z; u[r][3] = x4.w;
#pragma unroll
                    for (int e = 0; e < 4; ++e) u[r][e] = p + e >= p0 ? u[r][e] : 0.f;
                }
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    if constexpr (ALL) multiply(t);
                    else if (redo >> t & 1u) { fetch(t); multiply(t); }
                }
            }
        };
        if (__popc(redo) > 2) fp32(Truth<true>{});
        else fp32(Truth<false>{});
    }
    typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        if (first + 16 * r >= rows) continue;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int col = n0 + 16 * t + 4 * h;
            float* __restrict__ c = C + (first + 16 * r) * ldc + col;
            if (col + 4 <= n) {
                *reinterpret_cast<f4*>(c) = f4{big[r][t][0], big[r][t][1], big[r][t][2], big[r][t][3]};
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) if (col + q < n) c[q] = big[r][t][q];
            }
        }
    }
}

}  // namespace daspmm
