// Rows that hold a good part of all columns ("heavy" rows: a few hundred of 20 000 to 100 000 entries in a matrix of
// 524 288 columns, the popular nodes in the transpose of a power-law graph).  Every row of B is then used by dozens of
// them, but the EB kernels fetch it anew for every stored entry, and that rate, 64 bytes a clock and CU from the
// vector L1, is what bounds them (33 M entries, N = 64: 460 us).
//
// heavy_rows_kernel turns the loops round: a block owns a range of columns and heavy rows of similar length (up to 576).  It
// brings its rows of B into LDS once, a band at a time in two buffers, and walks the stored entries of all its heavy
// rows that lie in the band, with the rows' sums in registers from the first band to the last; they are added to C
// atomically once per block.  The same matrix takes 326 us at N = 64, EB 445 (under
// the profiler 265 here and 98 for the other rows), 121 and 172 at N = 8 (85 and 41), 217 and 268 at N = 32.  What bounds it: the vector
// units, busy in 76 % of the cycles at N = 64 (6 operations for 4 entries and 64 columns, some 25 for a batch of 64
// entries), LDS in 35 %, without bank conflicts; at N = 8 63 and 26 %, besides the stream of entries (50 us).
//
// Lane groups of 16 walk one row each, 16 entries at a time, one per lane; an entry's column and value reach the
// lanes by DPP broadcasts, the column as an operand of the address addition.  An entry takes the 16 lanes, or a
// quarter of them (GL = 4, up to 8 columns).  Lane j of them owns columns j, j + GL, ... of the tile, side by side in
// LDS, so that one read of 4 V bytes serves V columns and additions to C cover neighbouring elements.  Rows of similar
// length share a wave (in storage order: 318 us instead of 270 at N = 64).  Two buffers of 64 KiB; 8 instead of 4 entries
// read ahead at V = 4 take more steps for the last entries of a band: 288 us.
//
// The plan (da_spmm_prepare) lists the heavy rows and, per row and cell of columns, the position at which the cell's
// entries begin.  As everywhere, a plan only steers: positions are clamped to the row, so that whatever they hold the
// entries of a row are dealt to the blocks exactly once; an entry whose column is not in the band takes its operand
// from memory; a listed row that is not heavy any more is left to the other rows' kernel, which leaves out a row only if it
// is heavy by its present length and listed.  All that is slow: long rows that are not listed are added up row by row
// (33 M entries, N = 64: 22 ms, 1.3 in the EB kernels), entries outside the band one after another.  So both kernels
// mark a plan that does not describe the matrix, and later products do without it.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "da_dense_kernels.hip"
#include "da_spmm_kernels.hip"

namespace daspmm {

constexpr int kHeavyBlock = 1024, kHeavyWaves = kHeavyBlock / 64;
constexpr int kHeavyQuads = 9;                             // sets of 4 rows a wave holds
constexpr int kHeavyRows = kHeavyWaves * 4 * kHeavyQuads;  // heavy rows of a block
template <int GL, int V> constexpr int kHeavyBand = 16384 / (GL * V);   // rows of B in a buffer of 64 KiB
constexpr size_t kHeavyLds = 2 * 65536 + 256;              // two buffers and a row of zeros

struct HeavyPlan {
    const int* rows;     // count row numbers, by length
    const int* at;       // at[h * (cells + 1) + c]: position of the first entry of row h with column >= c * cell
    int count, cells, cell, min_len, nnz;
    int* stale;          // in host memory
};

// Blocks of a launch: group i has the rows row[i] ... row[i + 1] - 1 of the plan and the blocks block[i] ... block[i + 1] - 1,
// each with the rows' entries in per[i] cells.
constexpr int kHeavyGroups = 16;
struct HeavyGroups {
    int count, block[kHeavyGroups + 1], row[kHeavyGroups + 1], per[kHeavyGroups];
};

// Rows of at least min_len entries, in no order (count[0], list[] up to `most`), and of the others the sum of squared
// lengths (sums[0]) and the longest (sums[1]).  All cleared before.
__global__ __launch_bounds__(256) void heavy_rows_list_kernel(int m, const int* __restrict__ rowptr, int min_len, int most,
                                                              int* __restrict__ list, unsigned long long* __restrict__ sums,
                                                              int* __restrict__ count)
{
    unsigned long long sq = 0, mx = 0;
    for (long r = (long)blockIdx.x * 256 + threadIdx.x; r < m; r += (long)gridDim.x * 256) {
        const int len = rowptr[r + 1] - rowptr[r];
        if (len >= min_len) {
            const int at = atomicAdd(count, 1);
            if (at < most) list[at] = (int)r;
        } else {
            sq += (unsigned long long)len * len;
            mx = max(mx, (unsigned long long)len);
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        sq += __shfl_down(sq, d);
        mx = max(mx, __shfl_down(mx, d));
    }
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(&sums[0], sq);
        atomicMax(&sums[1], mx);
    }
}

// Where the listed rows begin and end.
__global__ __launch_bounds__(256) void heavy_row_ends_kernel(int count, const int* __restrict__ list, const int* __restrict__ rowptr,
                                                             int* __restrict__ pairs)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= count) return;
    pairs[2 * i] = rowptr[list[i]];
    pairs[2 * i + 1] = rowptr[list[i] + 1];
}

// Positions of the cells in the listed rows, and the rows' bits; unsorted[0] = 1 where columns of a row descend.
__global__ __launch_bounds__(256) void heavy_cells_kernel(const int* __restrict__ rowptr, const int* __restrict__ colind,
                                                          const int* __restrict__ rows, int cells, int cell, int* __restrict__ at,
                                                          unsigned* __restrict__ bits, int* __restrict__ unsorted)
{
    const int h = blockIdx.x, r = rows[h];
    const int s = rowptr[r], e = rowptr[r + 1];
    int* __restrict__ mine = at + (long)h * (cells + 1);
    if (blockIdx.y == 0 && threadIdx.x == 0) atomicOr(&bits[r >> 5], 1u << (r & 31));
    bool bad = false;
    for (int p = s + blockIdx.y * 256 + threadIdx.x; p <= e; p += gridDim.y * 256) {
        const int prev = p == s ? -1 : colind[p - 1], c = p == e ? 0x7fffffff : colind[p];
        bad |= c < prev;
        // cells that begin behind the entry before and not behind this one
        const int lo = prev < 0 ? 0 : prev / cell + 1, hi = p == e ? cells : min(c / cell, cells);
        for (int q = lo; q <= hi; ++q) mine[q] = p;
    }
    if (__any(bad) && (threadIdx.x & 63) == 0) unsorted[0] = 1;
}

// Lane n of the caller's group of GL lanes, 4 or 16.
template <int GL, int n>
__device__ __forceinline__ int group_lane(int x) {
    return __builtin_amdgcn_update_dpp(0, x, GL == 16 ? 0x150 + n : n * 0x55, 0xf, 0xf, true);   // row_newbcast:n, quad_perm
}

// Entries n0 ... n0 + L - 1 of the groups' batches: reads of their rows of B in LDS first, then the multiply-adds.
template <int GL, int V, int n0, int L>
struct HeavySteps {
    typedef float vec __attribute__((ext_vector_type(V)));
    vec b[L];
    template <int n>
    __device__ __forceinline__ void read(const char* lds, int off, int lane_off) {
        if constexpr (n < L) {
            b[n] = *reinterpret_cast<const vec*>(lds + (group_lane<GL, n0 + n>(off) + lane_off));
            read<n + 1>(lds, off, lane_off);
        }
    }
    template <int n>
    __device__ __forceinline__ void fma(float val, float (&acc)[V]) const {
        if constexpr (n < L) {
            const float s = __int_as_float(group_lane<GL, n0 + n>(__float_as_int(val)));
#pragma unroll
            for (int v = 0; v < V; ++v) acc[v] = fmaf(s, b[n][v], acc[v]);
            fma<n + 1>(val, acc);
        }
    }
    static __device__ __forceinline__ void run(const char* lds, int off, float val, int lane_off, float (&acc)[V]) {
        HeavySteps x;
        x.template read<0>(lds, off, lane_off);
        x.template fma<0>(val, acc);
    }
};

template <int GL, int V>
__global__ __launch_bounds__(kHeavyBlock) void heavy_rows_kernel(
    int m, int k, int N, Strides sd, const int* __restrict__ rowptr, const int* __restrict__ colind, const float* __restrict__ vals,
    const float* __restrict__ B, float* __restrict__ C, HeavyPlan plan, HeavyGroups groups)
{
    if (rowptr[m] != plan.nnz) {                           // a plan of another matrix: the other rows' kernel takes everything
        if (threadIdx.x == 0) *plan.stale = 1;
        return;
    }
    bool strayed = false;                                  // whether the wave met an entry outside its band
    extern __shared__ __align__(16) char heavy_lds[];
    char* const lds = heavy_lds;
    constexpr int kBand = kHeavyBand<GL, V>, kRow = 4 * GL * V;              // rows of a band; bytes of a row in LDS
    constexpr int kZero = 2 * 65536;                       // offset of the row of zeros
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = lane >> 4, j = lane & 15, jc = lane & (GL - 1);
    int group = 0;
    while (group + 1 < groups.count && (int)blockIdx.x >= groups.block[group + 1]) ++group;
    const int slab = blockIdx.x - groups.block[group], row0 = groups.row[group], row1 = groups.row[group + 1];
    const int quads = (row1 - row0 + kHeavyWaves * 4 - 1) / (kHeavyWaves * 4);
    const int tile0 = blockIdx.y * GL * V;
    const int cell0 = slab * groups.per[group], cell1 = min(cell0 + groups.per[group], plan.cells);
    const int col0 = cell0 * plan.cell;
    const int col1 = cell1 == plan.cells ? k : cell1 * plan.cell;

    // rows of B, in four parts: thread t brings rows t / GL + kBlock / GL * p of the band, columns jc + GL v
    constexpr int kParts = 4, kPasses = 16 / V / kParts, kStep = kHeavyBlock / GL;
    static_assert(kPasses >= 1, "at most 4 columns a lane");
    float stage[kPasses * V];
    int bcol[V];
#pragma unroll
    for (int v = 0; v < V; ++v) bcol[v] = min(tile0 + jc + GL * v, N - 1);
    auto fetch = [&](int first, int part) {
#pragma unroll
        for (int p = 0; p < kPasses; ++p) {
            const long row = min(first + (int)threadIdx.x / GL + kStep * (part * kPasses + p), col1 - 1);
#pragma unroll
            for (int v = 0; v < V; ++v) stage[p * V + v] = B[row * sd.rb + (long)bcol[v] * sd.cb];
        }
    };
    auto put = [&](int buffer, int part) {
        typedef float vec __attribute__((ext_vector_type(V)));
#pragma unroll
        for (int p = 0; p < kPasses; ++p) {
            vec x;
#pragma unroll
            for (int v = 0; v < V; ++v) x[v] = stage[p * V + v];
            *reinterpret_cast<vec*>(lds + buffer * 65536 + ((int)threadIdx.x / GL + kStep * (part * kPasses + p)) * kRow + jc * 4 * V) = x;
        }
    };
    if (threadIdx.x < 64) reinterpret_cast<float*>(lds + kZero)[threadIdx.x] = 0.f;
    fetch(col0, 0);

    // rows of the lane groups; blocks begin at different rows so that their additions to C do not meet
    int pos[kHeavyQuads], stop[kHeavyQuads];
    float acc[kHeavyQuads][V];
    auto index = [&](int i) {
        int q = wave + kHeavyWaves * i + (int)(slab * 5u % (unsigned)(kHeavyWaves * quads));
        if (q >= kHeavyWaves * quads) q -= kHeavyWaves * quads;
        return row0 + 4 * q + g;
    };
#pragma unroll
    for (int i = 0; i < kHeavyQuads; ++i) {
        pos[i] = stop[i] = 0;
#pragma unroll
        for (int v = 0; v < V; ++v) acc[i][v] = 0.f;
        if (i < quads) {
            const int h = index(i);
            if (h < row1) {
                const int r = plan.rows[h];
                const int s = rowptr[r], e = rowptr[r + 1];
                const int* at = plan.at + (long)h * (plan.cells + 1);
                if (e - s >= plan.min_len) {
                    pos[i] = cell0 == 0 ? s : min(max(at[cell0], s), e);
                    stop[i] = cell1 == plan.cells ? e : min(max(at[cell1], pos[i]), e);
                }
            }
        }
    }
#pragma unroll
    for (int q = 0; q < kParts; ++q) { put(0, q); if (q + 1 < kParts) fetch(col0, q + 1); }
    __syncthreads();
    struct Entry { int c; float v; };
    auto request = [&](int p, int end) {                   // the lane's entry of a batch; past the end any entry
        const unsigned at = p + j < end ? (unsigned)(p + j) * 4u : 0u;
        Entry e;
        e.c = *reinterpret_cast<const int*>(reinterpret_cast<const char*>(colind) + at);
        e.v = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(vals) + at);
        return e;
    };
    constexpr int D = GL * V == 64 ? 2 : 4, L = GL * V == 32 ? 8 : 4;      // batches in flight; entries read together
    Entry next[D];
    auto request_first = [&](int p, int end) {
#pragma unroll
        for (int d = 0; d < D; ++d) next[d] = request(p + 16 * d, end);
    };
    request_first(pos[0], stop[0]);
    int buffer = 0;
    for (int first = col0; first < col1; first += kBand) {
        const bool last = first + kBand >= col1;           // the last band takes what is left
        if (!last) fetch(first + kBand, 0);
        const unsigned here = (unsigned)min(kBand, col1 - first);              // rows of the band
        const int base = buffer * 65536, lane_off = jc * 4 * V;
#pragma unroll
        for (int i = 0; i < kHeavyQuads; ++i) {
            if (i < quads) {
                Entry e[D];
#pragma unroll
                for (int d = 0; d < D; ++d) e[d] = next[d];
                int p = pos[i];
                const int end = stop[i];
                // the next set's first batches are on their way while this one is worked on
                if (i + 1 < kHeavyQuads && i + 1 < quads) request_first(pos[(i + 1) % kHeavyQuads], stop[(i + 1) % kHeavyQuads]);
                int limit = last ? 0x7fffffff : first + kBand;
                auto batch = [&](Entry& ahead) {           // whether some group took all of its batch
                    const Entry now = ahead;
                    ahead = request(p + 16 * D, end);
                    // leading entries of the batch that lie in the band or before it
                    bool take = p + j < end && now.c < limit;
                    unsigned long long bits = __ballot(take);
                    if (bits & ~(bits << 1 | 0x0001000100010001ull)) {         // columns out of order
                        const unsigned m16 = (unsigned)(bits >> (16 * g)) & 0xffffu;
                        take = j < __builtin_ctz(~m16);
                        bits = __ballot(take);
                    }
                    const unsigned half = lane & 32 ? (unsigned)(bits >> 32) : (unsigned)bits;
                    const int cnt = __popc((half >> (lane & 16)) & 0xffffu);
                    const int local = now.c - first;
                    const bool inside = take && (unsigned)local < here;
                    const int off = inside ? base + local * kRow : kZero;
                    const float val = inside ? now.v : 0.f;
                    const unsigned any = ((unsigned)bits | (unsigned)(bits >> 16) | (unsigned)(bits >> 32) | (unsigned)(bits >> 48)) & 0xffffu;
                    float sum[V];
#pragma unroll
                    for (int w = 0; w < V; ++w) sum[w] = 0.f;
                    if constexpr (GL == 16) {
                        if (any) HeavySteps<GL, V, 0, L>::run(lds, off, val, lane_off, sum);
                        if constexpr (L == 4) { if (any & 0xfff0u) HeavySteps<GL, V, 4, L>::run(lds, off, val, lane_off, sum); }
                        if (any & 0xff00u) HeavySteps<GL, V, 8, L>::run(lds, off, val, lane_off, sum);
                        if constexpr (L == 4) { if (any & 0xf000u) HeavySteps<GL, V, 12, L>::run(lds, off, val, lane_off, sum); }
                    } else {
                        HeavySteps<GL, V, 0, L>::run(lds, off, val, lane_off, sum);
                    }
#pragma unroll
                    for (int w = 0; w < V; ++w) acc[i][w] += sum[w];           // one rounding of the long sum for 16 entries
                    if (__any(take && !inside)) {          // columns out of order, or a plan of another matrix
                        strayed = true;
                        for (int n = 0; n < 16; ++n) {
                            const int cn = __shfl(now.c, 16 * g + n);
                            const float vn = __shfl(now.v, 16 * g + n);
                            if (__shfl((int)(take && !inside), 16 * g + n) && (GL == 16 || j / GL == n / GL)) {
#pragma unroll
                                for (int w = 0; w < V; ++w) acc[i][w] = fmaf(vn, B[(long)cn * sd.rb + (long)bcol[w] * sd.cb], acc[i][w]);
                            }
                        }
                    }
                    p += cnt;
                    if (cnt < 16) limit = (int)0x80000000; // this group is done with the band
                    return (any & 0x8000u) != 0;
                };
                if constexpr (D == 2) while (batch(e[0]) && batch(e[1])) {}
                else while (batch(e[0]) && batch(e[1]) && batch(e[2]) && batch(e[3])) {}
                pos[i] = p;
                // the next band's parts follow one another, two sets of rows apart
                if (!last && i % 2 == 1 && i / 2 + 1 < kParts) { put(buffer ^ 1, i / 2); fetch(first + kBand, i / 2 + 1); }
            }
        }
        if (!last) {
            request_first(pos[0], stop[0]);
#pragma unroll
            for (int q = 0; q < kParts; ++q) {
                if (q < quads / 2 && q + 1 < kParts) continue;                 // done above
                put(buffer ^ 1, q);
                if (q + 1 < kParts) fetch(first + kBand, q + 1);
            }
            lds_barrier();
            buffer ^= 1;
        }
    }
    if (strayed && lane == 0) *plan.stale = 1;
#pragma unroll
    for (int i = 0; i < kHeavyQuads; ++i) {
        if (i < quads) {
            const int h = index(i);
            if (h < row1) {
                const int r = plan.rows[h];
                if (rowptr[r + 1] - rowptr[r] >= plan.min_len) {
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        if constexpr (GL == 4) {           // the four groups of 4 lanes have a quarter of the entries each
                            acc[i][v] = dpp_add<0x128>(acc[i][v]);
                            acc[i][v] = dpp_add<0x124>(acc[i][v]);
                        }
                        const int n = tile0 + jc + GL * v;
                        if (n < N && j < GL) unsafeAtomicAdd(C + (long)r * sd.rc + (long)n * sd.cc, acc[i][v]);
                    }
                }
            }
        }
    }
}

}  // namespace daspmm
