// Rows that hold a good part of all columns ("heavy" rows: a few hundred of 20 000 to 100 000 entries in a matrix of
// 524 288 columns, the popular nodes in the transpose of a power-law graph).  Every row of B is then used by dozens of
// them, but the EB kernels fetch it anew for every stored entry, and that rate, 64 bytes a clock and CU from the
// vector L1, is what bounds them (33 M entries, N = 64: 460 us).
//
// heavy_rows_kernel turns the loops round: a block owns a range of columns and heavy rows of similar length (up to 576).  It
// brings its rows of B into LDS once, a band at a time in two buffers, and walks the stored entries of all its heavy
// rows that lie in the band, with the rows' sums in registers from the first band to the last; they are added to C
// atomically once per block.  The same matrix takes 294 us at N = 64, EB 458; 207 and 278 at N = 32, 166 and 228 at N = 16, 115 and 176
// at N = 8.  What bounds it: latency.  The waves wait in half of their cycles; LDS is busy in 38 % of them at N = 64, the
// vector units in about half (4 entries and 64 columns take two operations with DPP, 4 cycles each, and four multiply-adds, 2 each; a
// batch of 64 entries some 20 operations).
//
// One wave does nothing but bring B, 16 bytes a lane: from memory to LDS directly where rows of B are such pieces, through registers
// where they are not (N = 41: 288 us; 492 directly, 4 bytes a lane).  While every wave brought a share through its registers, in parts
// between its rows, each part's entries waited for B's latency, since loads come back in order (N = 64: 338 us, N = 41: 322, N = 8: 117); it
// stays so where B is column-major or has less than four columns, see heavy_loader.  Two waves at N = 8: 110, one 108.  Lanes in order of
// memory: with the columns of a lane side by side in LDS, 64 bytes apart in memory, the kernel took 324 us under the profiler where it
// then took 235.
//
// Lane groups of 16 walk one row each, 16 entries at a time, one per lane; an entry's column and value reach the
// lanes by DPP broadcasts, the column as an operand of the address addition (the value as an operand of the multiply-adds: DPP
// halves their rate, no gain).  An entry takes the 16 lanes, or a quarter of them (GL = 4, up to 8 columns).  Lane j of them owns
// V neighbouring columns, one read of 4 V bytes; before the additions to C the lanes exchange their sums, so that an
// addition covers neighbouring elements (up to 8 columns all of them: 72 rows of 24 000, whose lines of C every block adds to, N = 2
// 29 -> 20 us, N = 8 31 -> 24).  Rows of similar length share a wave (in storage order: 318 us instead of 270 at N = 64).
// Two buffers of 64 KiB.  More requests for entries ahead (4 batches at V = 4, 8 at GL = 4) or two entries a lane: no gain.
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

constexpr int kHeavyBlock = 1024;
// Waves of a block that walk rows.
constexpr int heavy_waves(bool loader) { return kHeavyBlock / 64 - loader; }
constexpr int kHeavyQuads = 9;                             // sets of 4 rows a wave holds
template <int GL, int V> constexpr int kHeavyBand = 16384 / (GL * V);   // rows of B in a buffer of 64 KiB
constexpr size_t kHeavyLds = 2 * 65536 + 256 + heavy_waves(false) * 1024;   // two buffers, a row of zeros, and a row's sums per lane group

struct HeavyPlan {
    const int* rows;     // count row numbers, by length
    const int* at;       // at[h * (cells + 1) + c]: position of the first entry of row h with column >= c * cell
    int count, cells, cell, min_len, nnz;
    int* stale;          // in host memory
};

// Blocks of a launch: group i has the rows row[i] ... row[i + 1] - 1 of the plan and the blocks block[i] ... block[i + 1] - 1,
// each with the rows' entries in per[i] cells.
constexpr int kHeavyGroups = 17;
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

// Entries n0 ... n0 + L - 1 of the groups' batches: their rows of B from LDS, and the multiply-adds with them.
template <int GL, int V, int L>
struct HeavySteps {
    typedef float vec __attribute__((ext_vector_type(V)));
    vec b[L];
    template <int n0, int n = 0>
    __device__ __forceinline__ void read(const char* lds, int off, int lane_off) {
        if constexpr (n < L) {
            b[n] = *reinterpret_cast<const vec*>(lds + (group_lane<GL, n0 + n>(off) + lane_off));
            read<n0, n + 1>(lds, off, lane_off);
        }
    }
    template <int n0, int n = 0>
    __device__ __forceinline__ void fma(float val, float (&acc)[V]) const {
        if constexpr (n < L) {
            const float s = __int_as_float(group_lane<GL, n0 + n>(__float_as_int(val)));
#pragma unroll
            for (int v = 0; v < V; ++v) acc[v] = fmaf(s, b[n][v], acc[v]);
            fma<n0, n + 1>(val, acc);
        }
    }
};

// A batch of 16 entries, as far as the leading ones that `any` tells of, from n0 on.  Up to two columns a lane the next L
// entries' reads are on their way during the multiply-adds of L; with four there are no registers for them.
template <int GL, int V, int L, int n0>
__device__ __forceinline__ void heavy_batch(HeavySteps<GL, V, L>& now, unsigned any, const char* lds, int off, float val, int lane_off,
                                            float (&sum)[V]) {
    if constexpr (V == 4) now.template fma<n0>(val, sum);
    if constexpr (n0 + L < GL) {
        if (any >> (n0 + L)) {
            HeavySteps<GL, V, L> next;
            next.template read<n0 + L>(lds, off, lane_off);
            if constexpr (V < 4) now.template fma<n0>(val, sum);
            heavy_batch<GL, V, L, n0 + L>(next, any, lds, off, val, lane_off, sum);
            return;
        }
    }
    if constexpr (V < 4) now.template fma<n0>(val, sum);
}

// Calls batch with 0, 1, ... D - 1 until it returns false.
template <int D, int d = 0, class BATCH>
__device__ __forceinline__ bool each_batch(BATCH& batch) {
    if (!batch(Count<d>{})) return false;
    if constexpr (d + 1 < D) return each_batch<D, d + 1>(batch);
    return true;
}

template <int GL, int V, bool LOADER>
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
    constexpr int kWaves = heavy_waves(LOADER);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int g = lane >> 4, j = lane & 15, jc = lane & (GL - 1);
    int group = 0;
    while (group + 1 < groups.count && (int)blockIdx.x >= groups.block[group + 1]) ++group;
    const int slab = blockIdx.x - groups.block[group], row0 = groups.row[group], row1 = groups.row[group + 1];
    const int quads = (row1 - row0 + kWaves * 4 - 1) / (kWaves * 4);
    const int tile0 = blockIdx.y * GL * V;
    const int cell0 = slab * groups.per[group], cell1 = min(cell0 + groups.per[group], plan.cells);
    const int col0 = cell0 * plan.cell;
    const int col1 = cell1 == plan.cells ? k : cell1 * plan.cell;

    if constexpr (LOADER) {
        if (wave == kWaves) {
            // Lanes one after another, 16 bytes each: from memory to LDS where rows of B are whole 16-byte pieces, through
            // registers where they are not.
            typedef float four __attribute__((ext_vector_type(4), aligned(4)));
            typedef float four_in_lds __attribute__((ext_vector_type(4)));
            constexpr int kLanes = GL * V / 4, kPer = 64 / kLanes, kLoads = kBand / kPer, kAtOnce = 16;
            static_assert(kLoads == 64, "1 KB each");
            const int col = tile0 + lane % kLanes * 4, r = lane / kLanes;
            const int past = col + 4 - N;                  // the four numbers come from column N - 4 on where they would end behind N - 1
            const float* const mine = B + min(col, N - 4);
            const bool whole = ((unsigned long long)B % 16 | N % 4 | sd.rb % 4) == 0;
            auto from = [&](int first, int i) { return mine + (long)min(first + i * kPer + r, col1 - 1) * sd.rb; };
            reinterpret_cast<float*>(lds + kZero)[lane] = 0.f;
            int buffer = 0;
            for (int first = col0; first < col1; first += kBand, buffer ^= 1) {
                char* const to = lds + buffer * 65536;
                if (whole) {
#pragma unroll 1    // 294 us, 298 in loops of 4 and more (N = 64)
                    for (int i = 0; i < kLoads; ++i)
                        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)from(first, i),
                                                         (__attribute__((address_space(3))) void*)(to + i * 1024), 16, 0, 0);
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                } else {
                    for (int i = 0; i < kLoads; i += kAtOnce) {
                        four x[kAtOnce];
#pragma unroll
                        for (int q = 0; q < kAtOnce; ++q) x[q] = *reinterpret_cast<const four*>(from(first, i + q));
#pragma unroll
                        for (int q = 0; q < kAtOnce; ++q) {
                            four y = x[q];                 // columns from N on are never read out
                            if (past > 0 && past & 1) y = four{y[1], y[2], y[3], y[3]};
                            if (past > 0 && past & 2) y = four{y[2], y[3], y[3], y[3]};
                            *reinterpret_cast<four_in_lds*>(to + (i + q) * 1024 + lane * 16) = four_in_lds{y[0], y[1], y[2], y[3]};
                        }
                    }
                }
                lds_barrier();
            }
            return;
        }
    }
    // Without a loader a band's rows of B come through registers, in four parts of four numbers a thread; GL lanes on a row.
    constexpr int kParts = 4, kEach = 4;
    static_assert(kParts * kEach * kHeavyBlock == 16384, "a band");
    float stage[kEach];
    auto place = [&](int n, unsigned t, int* row, int* col) {
        *row = t / GL + kHeavyBlock / GL * (n / V);
        *col = t % GL + GL * (n % V);
    };
    auto fetch = [&](int first, int part) {
        unsigned t = threadIdx.x;
        asm volatile("" : "+v"(t));                        // nothing of this is worth registers from part to part
#pragma unroll
        for (int q = 0; q < kEach; ++q) {
            int row, col;
            place(part * kEach + q, t, &row, &col);
            stage[q] = B[(long)min(first + row, col1 - 1) * sd.rb + (long)min(tile0 + col, N - 1) * sd.cb];
        }
    };
    auto put = [&](int buffer, int part) {
        unsigned t = threadIdx.x;
        asm volatile("" : "+v"(t));
#pragma unroll
        for (int q = 0; q < kEach; ++q) {
            int row, col;
            place(part * kEach + q, t, &row, &col);
            reinterpret_cast<float*>(lds + buffer * 65536)[row * GL * V + col] = stage[q];
        }
    };
    if constexpr (!LOADER) {
        if (wave == 0) reinterpret_cast<float*>(lds + kZero)[lane] = 0.f;
        fetch(col0, 0);
    }
    int bcol[V];                                           // the lane's columns
#pragma unroll
    for (int v = 0; v < V; ++v) bcol[v] = min(tile0 + jc * V + v, N - 1);

    // rows of the lane groups; blocks begin at different rows so that their additions to C do not meet
    unsigned pos[kHeavyQuads], stop[kHeavyQuads];          // byte offsets: of the lane's next entry, and of the row's end
    float acc[kHeavyQuads][V];
    auto index = [&](int i) {
        int q = wave + kWaves * i + (int)(slab * 5u % (unsigned)(kWaves * quads));
        if (q >= kWaves * quads) q -= kWaves * quads;
        return row0 + 4 * q + g;
    };
#pragma unroll
    for (int i = 0; i < kHeavyQuads; ++i) {
        int from = 0, to = 0;
#pragma unroll
        for (int v = 0; v < V; ++v) acc[i][v] = 0.f;
        if (i < quads) {
            const int h = index(i);
            if (h < row1) {
                const int r = plan.rows[h];
                const int s = rowptr[r], e = rowptr[r + 1];
                const int* at = plan.at + (long)h * (plan.cells + 1);
                if (e - s >= plan.min_len) {
                    from = cell0 == 0 ? s : min(max(at[cell0], s), e);
                    to = cell1 == plan.cells ? e : min(max(at[cell1], from), e);
                }
            }
        }
        pos[i] = (unsigned)(from + j) * 4u;
        stop[i] = (unsigned)to * 4u;
    }
    struct Entry { int c; float v; };
    // The entry at byte offset p + ahead; past the last one of the matrix zeros.  From the row's end on, which is at `end`, any: the one
    // there, which all lanes share, saves bytes (8000 rows of 700, N = 4: 51 -> 41 us, N = 8: 50 -> 39); with four columns a lane the
    // operation costs more on long rows (524 of 20 000 to 100 000, N = 64: 298 -> 305) than it saves.
    const unsigned bytes = (unsigned)plan.nnz * 4u;        // plans end at 2^30 entries, 32 bits of bytes
    const __amdgpu_buffer_rsrc_t cols = __builtin_amdgcn_make_buffer_rsrc(const_cast<int*>(colind), 0, bytes, 0x00027000);
    const __amdgpu_buffer_rsrc_t numbers = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(vals), 0, bytes, 0x00027000);
    auto request = [&](unsigned p, unsigned ahead, unsigned end) {
        Entry e;
        p = (V < 4 ? min(p, end - ahead) : p) + ahead;
        e.c = (int)__builtin_amdgcn_raw_buffer_load_b32(cols, (int)p, 0, 0);
        e.v = __int_as_float((int)__builtin_amdgcn_raw_buffer_load_b32(numbers, (int)p, 0, 0));
        return e;
    };
    constexpr int D = V == 4 ? 2 : 4, L = 4;               // batches in flight; entries read together
    Entry next[D];
    auto request_first = [&](unsigned p, unsigned end) {
#pragma unroll
        for (int d = 0; d < D; ++d) next[d] = request(p, 64 * d, end);
    };
    if constexpr (!LOADER) {
#pragma unroll
        for (int q = 0; q < kParts; ++q) { put(0, q); if (q + 1 < kParts) fetch(col0, q + 1); }
    }
    request_first(pos[0], stop[0]);
    int buffer = 0;
    for (int first = col0; first < col1; first += kBand) {
        const bool last = first + kBand >= col1;           // the last band takes what is left
        lds_barrier();                                     // the band is here
        if (!LOADER && !last) fetch(first + kBand, 0);
        const unsigned here = (unsigned)min(kBand, col1 - first);              // rows of the band
        const int base = buffer * 65536, lane_off = jc * 4 * V;
#pragma unroll
        for (int i = 0; i < kHeavyQuads; ++i) {
            if (i < quads) {
                Entry e[D];
#pragma unroll
                for (int d = 0; d < D; ++d) e[d] = next[d];
                unsigned p = pos[i];
                const unsigned end = stop[i];
                unsigned long long alive = ~0ull;          // lanes of groups that are not done with the band
                // the next set's first batches are on their way while this one is worked on
                if (i + 1 < kHeavyQuads && i + 1 < quads) request_first(pos[(i + 1) % kHeavyQuads], stop[(i + 1) % kHeavyQuads]);
                const int limit = last ? 0x7fffffff : first + kBand;
                auto batch = [&](auto which) {
                    constexpr int d = decltype(which)::value;
                    const Entry now = e[d];
                    e[d] = request(p, 64 * D, end);
                    asm volatile("; batch %0" ::"n"(d));   // one loop over batches of changing registers would wait for each request
                    // leading entries of the batch that lie in the band or before it
                    unsigned long long bits = alive & __builtin_amdgcn_ballot_w64(p < end) & __builtin_amdgcn_ballot_w64(now.c < limit);
                    if (bits & ~(bits << 1 | 0x0001000100010001ull)) {         // columns out of order
                        const unsigned m16 = (unsigned)(bits >> (16 * g)) & 0xffffu;
                        bits = __builtin_amdgcn_ballot_w64(j < __builtin_ctz(~m16));
                    }
                    const int local = now.c - first;
                    const unsigned long long within = bits & __builtin_amdgcn_ballot_w64((unsigned)local < here);
                    const bool inside = __builtin_amdgcn_inverse_ballot_w64(within);
                    const int off = inside ? base + local * kRow : kZero;
                    const float val = inside ? now.v : 0.f;
                    const unsigned any = ((unsigned)bits | (unsigned)(bits >> 16) | (unsigned)(bits >> 32) | (unsigned)(bits >> 48)) & 0xffffu;
                    float sum[V];
#pragma unroll
                    for (int w = 0; w < V; ++w) sum[w] = 0.f;
                    if (GL == 4 || any) {
                        HeavySteps<GL, V, L> steps;
                        steps.template read<0>(lds, off, lane_off);
                        heavy_batch<GL, V, L, 0>(steps, any, lds, off, val, lane_off, sum);
                    }
#pragma unroll
                    for (int w = 0; w < V; ++w) acc[i][w] += sum[w];           // one rounding of the long sum for 16 entries
                    if (within != bits) {                  // columns out of order, or a plan of another matrix
                        strayed = true;
                        const int far = (int)__builtin_amdgcn_inverse_ballot_w64(bits & ~within);
                        for (int n = 0; n < 16; ++n) {
                            const int cn = __shfl(now.c, 16 * g + n);
                            const float vn = __shfl(now.v, 16 * g + n);
                            if (__shfl(far, 16 * g + n) && (GL == 16 || j / GL == n / GL)) {
#pragma unroll
                                for (int w = 0; w < V; ++w) acc[i][w] = fmaf(vn, B[(long)cn * sd.rb + (long)bcol[w] * sd.cb], acc[i][w]);
                            }
                        }
                    }
                    if (bits == ~0ull) {
                        p += 64;
                    } else {
                        const unsigned half = lane & 32 ? (unsigned)(bits >> 32) : (unsigned)bits;
                        const unsigned cnt = __popc((half >> (lane & 16)) & 0xffffu);
                        p += 4 * cnt;
                        alive &= __builtin_amdgcn_ballot_w64(cnt == 16);
                    }
                    return (any & 0x8000u) != 0;
                };
                while (each_batch<D>(batch)) {}
                pos[i] = p;
                // the next band's parts follow one another, two sets of rows apart
                if (!LOADER && !last && i % 2 == 1 && i / 2 + 1 < kParts) { put(buffer ^ 1, i / 2); fetch(first + kBand, i / 2 + 1); }
            }
        }
        if (!last) {
            request_first(pos[0], stop[0]);
            if constexpr (!LOADER) {
#pragma unroll
                for (int q = 0; q < kParts; ++q) {
                    if (q < quads / 2 && q + 1 < kParts) continue;             // done above
                    put(buffer ^ 1, q);
                    if (q + 1 < kParts) fetch(first + kBand, q + 1);
                }
            }
        }
        buffer ^= 1;
    }
    if (strayed && lane == 0) *plan.stale = 1;
#pragma unroll
    for (int i = 0; i < kHeavyQuads; ++i) {
        if (i < quads) {
            if constexpr (GL == 16 && V > 1) {             // the sums of 16 lanes change hands, so that an addition covers neighbouring columns
                float* turn = reinterpret_cast<float*>(lds + kZero + 256) + (wave * 4 + g) * GL * V;
#pragma unroll
                for (int v = 0; v < V; ++v) turn[j * V + v] = acc[i][v];
                wave_lds_sync();
#pragma unroll
                for (int v = 0; v < V; ++v) acc[i][v] = turn[j + GL * v];
                wave_lds_sync();
            }
            const int h = index(i);
            if (h < row1) {
                const int r = plan.rows[h];
                if (rowptr[r + 1] - rowptr[r] >= plan.min_len) {
                    if constexpr (GL == 4) {               // the four groups of 4 lanes have a quarter of the entries each
                        static_assert(V == 2, "columns of lanes 0 ... 7");
                        const int from = (lane & 48) + (j >> 1 & 3);
                        const float even = __shfl(dpp_add<0x124>(dpp_add<0x128>(acc[i][0])), from);
                        const float odd = __shfl(dpp_add<0x124>(dpp_add<0x128>(acc[i][1])), from);
                        const float sum = j % 2 == 0 ? even : odd;
                        if (j < 8 && tile0 + j < N) unsafeAtomicAdd(C + (long)r * sd.rc + (long)(tile0 + j) * sd.cc, sum);
                    } else {
#pragma unroll
                        for (int v = 0; v < V; ++v) {
                            const int n = tile0 + j + GL * v;
                            if (n < N) unsafeAtomicAdd(C + (long)r * sd.rc + (long)n * sd.cc, acc[i][v]);
                        }
                    }
                }
            }
        }
    }
}

}  // namespace daspmm
