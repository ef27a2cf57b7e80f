// CSR transpose for gfx950 (wave64): the CSR arrays of A^T from those of A, needed by the backward
// pass of a graph-convolution layer (the GCN application of Sec. 6), where the gradient of
// <G, A.X> with respect to X is A^T.G and is computed by the same SpMM kernels on A^T.
//
// Row j of A^T lists the stored entries of column j of A with ascending row numbers.  CSR stores
// entries row after row, so a STABLE sort of the entries by column index is exactly that order,
// and it is deterministic (no atomic cursors on global memory).
//
// Two radix sorts live here.
//
// (1) The transpose proper (transpose_* kernels): least-significant-digit radix sort in one or two
//     passes of at most 10 bits, for k <= 2^20.  What bounds it is memory traffic, so it moves as little
//     as possible: the first pass drops the digit it has sorted by and packs the rest of the column
//     index with the row number into one word, the second pass unpacks it, so an entry is 8 bytes
//     between the passes and full column indices are never written.  One pass is
//         transpose_count_kernel    digit histograms of a group of tiles, as prefixes inside the group
//         transpose_scan_kernel     exclusive prefix over the groups, per digit, and digit totals
//         transpose_scatter_kernel  stable placement of a tile
//     and transpose_rowptr_kernel derives the row pointers of A^T from the histograms: after the first
//     pass the entries are ordered by the low digit, so row pointer (high, low) is the position at which
//     the second pass puts the first entry at or behind the start of `low` with digit `high`.
// (2) A general sort of (key, id, payload) triples with digits of at most 8 bits (radix_* kernels), used
//     for the EB schedules, and for the transpose when k > 2^20 or when row number and high digit do
//     not fit one word together.
//
// In both, each wave owns a contiguous run of entries and walks it 64 entries at a time; the lanes
// that hold the same digit find each other with one ballot per digit bit, so the rank of an entry
// among its peers is a population count and only one lane per distinct digit touches the wave's
// running counter in LDS.  The block first orders its tile by digit in LDS and then copies it out, so
// that entries with the same digit leave as contiguous runs (coalesced stores) rather than as single
// 4-byte stores.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "da_dense_kernels.hip"
#include "da_spmm_kernels.hip"

namespace daspmm {

constexpr int kRadixBits = 8;                            // widest digit
constexpr int kBins = 1 << kRadixBits;
constexpr int kSortBlock = 256;                          // one thread per bin in the bookkeeping steps
constexpr int kSortWaves = kSortBlock / 64;
constexpr int kSortRounds = 16;                          // 64-entry rounds per wave and block
constexpr int kSortWaveRun = kSortRounds * 64;           // consecutive entries owned by one wave
constexpr int kSortTile = kSortWaves * kSortWaveRun;     // entries per block
constexpr int kScanPerThread = 16;
constexpr int kScanChunk = kSortBlock * kScanPerThread;  // ints per block in the scan kernels

static_assert(kBins == kSortBlock, "bookkeeping maps one thread to one bin");

__device__ __forceinline__ int digit_of(int key, int shift, int mask) { return (key >> shift) & mask; }

// Lanes of the wave that are valid and hold the same digit as the caller (meaningless for a lane
// that is not valid).  Every lane of the wave must call it.
__device__ __forceinline__ unsigned long long digit_peers(int d, bool valid) {
    unsigned long long peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < kRadixBits; ++b) {
        const bool bit = (d >> b) & 1;
        const unsigned long long vote = __ballot(bit && valid);
        peers &= bit ? vote : ~vote;
    }
    return peers;
}

__device__ __forceinline__ int wave_inclusive_scan(int v, int lane) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int t = __shfl_up(v, d);
        if (lane >= d) v += t;
    }
    return v;
}

// Exclusive prefix of v over the 256 threads of the block; *total receives the block sum.
// sh: kSortWaves ints of LDS.  All threads must call it.
__device__ __forceinline__ int block_exclusive_scan(int v, int* sh, int* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int inc = wave_inclusive_scan(v, lane);
    __syncthreads();                                     // sh may still be read from a previous call
    if (lane == 63) sh[wave] = inc;
    __syncthreads();
    int off = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) {
        const int s = sh[w];
        if (w < wave) off += s;
        tot += s;
    }
    *total = tot;
    return off + inc - v;
}

// ------------------------------------------------------------------------------------------
// exclusive prefix sum of an int array, in place: reduce per chunk, scan the chunk sums in one
// block, then scan every chunk with its base
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ void scan_reduce_body(unsigned bx, const int* __restrict__ data, long len,
                                                 int* __restrict__ part)
{
    __shared__ int sh[kSortWaves];
    const long base = (long)bx * kScanChunk;
    int s = 0;
    for (int j = 0; j < kScanPerThread; ++j) {
        const long i = base + j * kSortBlock + threadIdx.x;
        if (i < len) s += data[i];
    }
    int total;
    block_exclusive_scan(s, sh, &total);
    if (threadIdx.x == 0) part[bx] = total;
}

__global__ __launch_bounds__(kSortBlock) void scan_reduce_kernel(const int* __restrict__ data, long len,
                                                                 int* __restrict__ part)
{
    scan_reduce_body(blockIdx.x, data, len, part);
}

__device__ __forceinline__ void scan_top_body(int* __restrict__ part, int count)
{
    __shared__ int sh[kSortWaves];
    int carry = 0;
    for (int base = 0; base < count; base += kSortBlock) {
        const int i = base + threadIdx.x;
        const int v = i < count ? part[i] : 0;
        int total;
        const int ex = block_exclusive_scan(v, sh, &total);
        if (i < count) part[i] = carry + ex;
        carry += total;
    }
}

__global__ __launch_bounds__(kSortBlock) void scan_top_kernel(int* __restrict__ part, int count)
{
    scan_top_body(part, count);
}

__device__ __forceinline__ void scan_apply_body(unsigned bx, int* __restrict__ data, long len,
                                                const int* __restrict__ part)
{
    __shared__ int sh[kSortWaves];
    const long first = (long)bx * kScanChunk + (long)threadIdx.x * kScanPerThread;
    int x[kScanPerThread];
    int s = 0;
#pragma unroll
    for (int j = 0; j < kScanPerThread; ++j) {
        x[j] = first + j < len ? data[first + j] : 0;
        s += x[j];
    }
    int total;
    int run = part[bx] + block_exclusive_scan(s, sh, &total);
#pragma unroll
    for (int j = 0; j < kScanPerThread; ++j) {
        if (first + j < len) data[first + j] = run;
        run += x[j];
    }
}

__global__ __launch_bounds__(kSortBlock) void scan_apply_kernel(int* __restrict__ data, long len,
                                                                const int* __restrict__ part)
{
    scan_apply_body(blockIdx.x, data, len, part);
}

// Smallest r in [lo, hi] with rowptr[r+1] > e: the row that owns stored entry e, given that it
// lies in [lo, hi].
__device__ __forceinline__ int owner_row(const int* __restrict__ rowptr, int lo, int hi, int e) {
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (rowptr[mid + 1] > e) hi = mid; else lo = mid + 1;
    }
    return lo;
}

// ------------------------------------------------------------------------------------------
// one radix pass; digit = (key >> shift) & mask with mask < kBins
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ void radix_count_body(unsigned bx, const int* __restrict__ keys, int n, int shift, int mask,
                                                 int* __restrict__ hist, int nblocks)
{
    __shared__ int cnt[kBins];
    cnt[threadIdx.x] = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long wbase = (long)bx * kSortTile + (long)wave * kSortWaveRun;
    int key[kSortRounds];
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {               // all loads of the lane in flight together;
        const long e = wbase + r * 64 + lane;             // clamped, so that they need no branch
        key[r] = keys[e < n ? e : n - 1];
    }
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const bool valid = wbase + r * 64 + lane < n;
        const int d = digit_of(key[r], shift, mask);
        const unsigned long long peers = digit_peers(d, valid);
        if (valid && lane == __ffsll((long long)peers) - 1) atomicAdd(&cnt[d], __popcll(peers));
        __builtin_amdgcn_sched_barrier(0);                // keep the ballots of one round together
    }
    __syncthreads();
    hist[(long)threadIdx.x * nblocks + bx] = cnt[threadIdx.x];
}

__global__ __launch_bounds__(kSortBlock) void radix_count_kernel(const int* __restrict__ keys, int n, int shift, int mask,
                                                                 int* __restrict__ hist, int nblocks)
{
    radix_count_body(blockIdx.x, keys, n, shift, mask, hist, nblocks);
}

// hist holds the exclusive prefix sums of the pass's histograms.  FIRST: the input is the matrix
// itself (keys_in = colind, vals_in = vals) and the row number of an entry is derived from rowptr;
// otherwise rows_in carries it.  The outputs of the last pass are the arrays of A^T.
template <bool FIRST>
__device__ __forceinline__ void radix_scatter_body(
    unsigned bx, const int* __restrict__ keys_in, const int* __restrict__ rows_in, const float* __restrict__ vals_in, int n,
    int shift, int mask, const int* __restrict__ hist, int nblocks,
    int* __restrict__ keys_out, int* __restrict__ rows_out, float* __restrict__ vals_out,
    const int* __restrict__ rowptr, int m)
{
    __shared__ int wcnt[kSortWaves][kBins];              // per wave and digit: count, then next slot in the tile
    __shared__ int gbase[kBins];                          // global position minus tile slot, per digit
    __shared__ int sh[kSortWaves];
    __shared__ int skey[kSortTile];
    __shared__ int srow[kSortTile];
    __shared__ float sval[kSortTile];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) wcnt[w][threadIdx.x] = 0;
    const long tbase = (long)bx * kSortTile;
    const long wbase = tbase + (long)wave * kSortWaveRun;
    const int tile_count = (int)min((long)kSortTile, (long)n - tbase);
    // the lane's 16 entries: every load is issued before the first one is used (indices clamped to
    // the last entry instead of branching; `valid` masks the surplus lanes of the last block)
    int key[kSortRounds], row[kSortRounds];
    float val[kSortRounds];
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const long e = wbase + r * 64 + lane;
        const long ec = e < n ? e : n - 1;
        key[r] = keys_in[ec];
        val[r] = vals_in[ec];
        if constexpr (!FIRST) row[r] = rows_in[ec];
    }
    if constexpr (FIRST) {
        // rows of the wave's run lie in [row_lo, row_hi]; the 16 searches of a lane advance together
        // so that their probes overlap
        int lo[kSortRounds], hi[kSortRounds];
        const long last = min(wbase + kSortWaveRun - 1, (long)n - 1);
        int row_lo = 0, row_hi = 0;
        if (wbase < n) {
            row_lo = owner_row(rowptr, 0, m - 1, (int)wbase);
            row_hi = owner_row(rowptr, row_lo, m - 1, (int)last);
        }
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) { lo[r] = row_lo; hi[r] = row_hi; }
        for (int span = row_hi - row_lo; span > 0; span >>= 1) {      // ceil(log2(span + 1)) steps
#pragma unroll
            for (int r = 0; r < kSortRounds; ++r) {
                const long e = wbase + r * 64 + lane;
                const int ec = (int)(e < last ? e : last);
                const int mid = (lo[r] + hi[r]) >> 1;
                if (rowptr[mid + 1] > ec) hi[r] = mid; else lo[r] = mid + 1;
            }
        }
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) row[r] = lo[r];
    }
    __syncthreads();
    // digits per wave; the peer masks are kept for the placement step
    unsigned long long peers[kSortRounds];
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const bool valid = wbase + r * 64 + lane < n;
        const int d = digit_of(key[r], shift, mask);
        peers[r] = valid ? digit_peers(d, valid) : 0ull;
        if (valid && lane == __ffsll((long long)peers[r]) - 1) atomicAdd(&wcnt[wave][d], __popcll(peers[r]));
        __builtin_amdgcn_sched_barrier(0);                // keep the ballots of one round together
    }
    __syncthreads();
    // thread d: counts of digit d -> first tile slot of every (wave, d), and the offset that turns
    // a tile slot of digit d into its global position
    {
        const int d = threadIdx.x;
        int c[kSortWaves], total = 0;
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w) { c[w] = wcnt[w][d]; total += c[w]; }
        int all;
        int slot = block_exclusive_scan(total, sh, &all);
        gbase[d] = hist[(long)d * nblocks + bx] - slot;
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w) { wcnt[w][d] = slot; slot += c[w]; }
    }
    __syncthreads();
    // stable placement inside the tile: rounds in order, peers ranked by lane number
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const bool valid = peers[r] != 0ull;              // a valid lane is its own peer
        const int d = digit_of(key[r], shift, mask);
        const int leader = __ffsll((long long)peers[r]) - 1;
        int first = 0;
        if (valid && lane == leader) first = atomicAdd(&wcnt[wave][d], __popcll(peers[r]));
        first = __shfl(first, leader & 63);
        if (valid) {
            const int slot = first + __popcll(peers[r] & ((1ull << lane) - 1ull));
            skey[slot] = key[r];
            srow[slot] = row[r];
            sval[slot] = val[r];
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    // copy out: neighbouring tile slots of one digit are neighbouring global positions
    for (int i = threadIdx.x; i < tile_count; i += kSortBlock) {
        const int k2 = skey[i];
        const int pos = gbase[digit_of(k2, shift, mask)] + i;
        keys_out[pos] = k2;
        rows_out[pos] = srow[i];
        vals_out[pos] = sval[i];
    }
}

template <bool FIRST>
__global__ __launch_bounds__(kSortBlock) void radix_scatter_kernel(
    const int* __restrict__ keys_in, const int* __restrict__ rows_in, const float* __restrict__ vals_in, int n,
    int shift, int mask, const int* __restrict__ hist, int nblocks,
    int* __restrict__ keys_out, int* __restrict__ rows_out, float* __restrict__ vals_out,
    const int* __restrict__ rowptr, int m)
{
    radix_scatter_body<FIRST>(blockIdx.x, keys_in, rows_in, vals_in, n, shift, mask, hist, nblocks, keys_out, rows_out,
                              vals_out, rowptr, m);
}

// Sort keys of the EB schedule for unit u (the stored entries [u*unit, (u+1)*unit)), in [0, 2k).
// A unit inside one row covers a narrow column range and is keyed by the middle of that range,
// k + (first + last column index)/2: these units are swept over B in column order.  A unit that
// touches several rows is keyed by its first column index alone (units that start at the same
// place of rows of similar length walk the column range in step, so this aligns them too; for
// units of many short rows no order matters): all such units sort before the others and form a
// first segment of the schedule.  They walk row ends (stores, atomics, a row-pointer load each) and
// are latency-bound where the single-row units are bandwidth-bound; a wave that holds both kinds
// runs at the pace of the slower, so the kinds are kept apart, and the launch deals each segment
// to all XCDs.  count (one int, cleared first) receives the number of units of that segment.
// ids = 0, 1, 2, ...; the value slot of the triples the radix passes move carries, as a bit pattern,
// the row that owns the unit's first entry, so that the sort also delivers those rows in schedule order;
// rows_by_unit (may be null) receives the same rows indexed by unit number.
//
// Several schedules (one per chunk size) are built side by side: every kernel of the pipeline takes
// up to kMaxSortJobs jobs and blockIdx.y selects the job, so that the orders for all chunk sizes of
// a matrix cost the launches of one.
constexpr int kMaxSortJobs = 5;

struct SortJob {                       // one radix pass of one job (pointers change from pass to pass)
    const int* keys_in; const int* rows_in; const float* vals_in;
    int* keys_out; int* rows_out; float* vals_out;
    int* hist; int* part;
    long hist_len;
    int n, nblocks, parts;
};
struct SortJobs { SortJob j[kMaxSortJobs]; };

struct KeyJob {                        // key generation of one schedule
    int unit, nunits;
    int* keys; int* ids; float* pad; int* count; int* rows_by_unit;
};
struct KeyJobs { KeyJob j[kMaxSortJobs]; };

__global__ void schedule_clear_kernel(KeyJobs jobs, int njobs) {
    if ((int)threadIdx.x < njobs) *jobs.j[threadIdx.x].count = 0;
}

__global__ __launch_bounds__(kSortBlock) void radix_count_jobs_kernel(SortJobs jobs, int shift, int mask) {
    const SortJob J = jobs.j[blockIdx.y];
    if ((int)blockIdx.x < J.nblocks) radix_count_body(blockIdx.x, J.keys_in, J.n, shift, mask, J.hist, J.nblocks);
}
__global__ __launch_bounds__(kSortBlock) void scan_reduce_jobs_kernel(SortJobs jobs) {
    const SortJob J = jobs.j[blockIdx.y];
    if ((int)blockIdx.x < J.parts) scan_reduce_body(blockIdx.x, J.hist, J.hist_len, J.part);
}
__global__ __launch_bounds__(kSortBlock) void scan_top_jobs_kernel(SortJobs jobs) {
    const SortJob J = jobs.j[blockIdx.x];
    scan_top_body(J.part, J.parts);
}
__global__ __launch_bounds__(kSortBlock) void scan_apply_jobs_kernel(SortJobs jobs) {
    const SortJob J = jobs.j[blockIdx.y];
    if ((int)blockIdx.x < J.parts) scan_apply_body(blockIdx.x, J.hist, J.hist_len, J.part);
}
__global__ __launch_bounds__(kSortBlock) void radix_scatter_jobs_kernel(SortJobs jobs, int shift, int mask) {
    const SortJob J = jobs.j[blockIdx.y];
    if ((int)blockIdx.x < J.nblocks)
        radix_scatter_body<false>(blockIdx.x, J.keys_in, J.rows_in, J.vals_in, J.n, shift, mask, J.hist, J.nblocks, J.keys_out,
                                  J.rows_out, J.vals_out, nullptr, 0);
}

__global__ __launch_bounds__(kSortBlock) void schedule_keys_kernel(int m, int k, int nnz, const int* __restrict__ rowptr,
                                                                   const int* __restrict__ colind, KeyJobs jobs)
{
    const KeyJob J = jobs.j[blockIdx.y];
    const int unit = J.unit, nunits = J.nunits;
    int* __restrict__ keys = J.keys;
    int* __restrict__ ids = J.ids;
    float* __restrict__ pad = J.pad;
    int* __restrict__ count = J.count;
    int* __restrict__ rows_by_unit = J.rows_by_unit;
    const long u = (long)blockIdx.x * kSortBlock + threadIdx.x;
    if ((long)blockIdx.x * kSortBlock >= nunits) return;          // whole block beyond this job's units
    bool several = false;
    if (u < nunits) {
        const long c0 = u * unit;
        const long c1 = min(c0 + unit, (long)nnz) - 1;
        const int r0 = owner_row(rowptr, 0, m - 1, (int)c0);
        several = rowptr[r0 + 1] <= c1;
        keys[u] = several ? colind[c0] : k + (int)(((long)colind[c0] + (long)colind[c1]) >> 1);
        ids[u] = (int)u;
        pad[u] = __int_as_float(r0);
        if (rows_by_unit) rows_by_unit[u] = r0;
    }
    const unsigned long long vote = __ballot(several);
    if ((threadIdx.x & 63) == 0 && vote) atomicAdd(count, __popcll(vote));
}

// t_rowptr[c] = number of stored entries with column index < c, for c = 0..k.
__global__ __launch_bounds__(kSortBlock) void rowptr_from_sorted_kernel(const int* __restrict__ keys, int n, int k,
                                                                        int* __restrict__ t_rowptr)
{
    const long c = (long)blockIdx.x * kSortBlock + threadIdx.x;
    if (c > k) return;
    int lo = 0, hi = n;                                   // first position whose key is >= c
    while (lo < hi) {
        const int mid = (int)(((long)lo + hi) >> 1);
        if (keys[mid] < c) lo = mid + 1; else hi = mid;
    }
    t_rowptr[c] = lo;
}

// ------------------------------------------------------------------------------------------
// the transpose in one or two passes
// ------------------------------------------------------------------------------------------
constexpr int kDigitBitsMax = 10;
constexpr int kDigitBinsMax = 1 << kDigitBitsMax;
constexpr int kGroupMax = 8;                             // tiles counted by one block
constexpr int kCountBlock = 512;
constexpr int kScanDigits = 16;                          // digits per block of transpose_scan_kernel

// One pass.  Entries come from the matrix (colind, vals, row numbers from rowptr) in the first pass and
// from (mid_in, vals_in) in the second.  mid = row | (column >> low digit's bits) << row_bits.
struct TransposePass {
    const int* colind;
    const int* rowptr;
    const unsigned* mid_in;
    const float* vals_in;
    unsigned* mid_out;
    int* t_colind;
    float* vals_out;
    int* hist;               // [tile][digit]: entries of the digit in the earlier tiles of the group
    int* group_hist;         // [group][digit]: entries of the digit in the group, then in the groups before it
    int* total;              // [digit]
    int* tile_row;           // [tile]: row of the tile's first entry, and behind the last tile the last entry's
    int m, n, ntiles;
    int group;               // tiles per group
    int bits;                // width of this pass's digit
    int row_bits;
};

// Tiles are dealt to the XCDs in contiguous groups: the runs that neighbouring tiles write for one
// digit are neighbours in memory, and the L2 of one XCD merges them into whole lines.
__device__ __forceinline__ int tile_of_block(int ntiles) {
    const int per = (ntiles + 7) >> 3;
    return (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
}

template <bool FIRST>
__device__ __forceinline__ unsigned pass_digit(unsigned key, const TransposePass& P) {
    return FIRST ? key & ((1u << P.bits) - 1u) : key >> P.row_bits;
}

// The row that owns entry q, found by the 64 lanes of a wave together (64 probes per step).
__device__ __forceinline__ int owner_row_wave(const int* __restrict__ rowptr, int lo, int hi, int q, int lane) {
    while (lo < hi) {
        const long len = hi - lo;
        const int r = lo + (int)((len * (lane + 1)) / 65);
        const int low = 64 - __popcll(__ballot(rowptr[r + 1] > q));   // probes 0 .. low-1 lie before the owner
        const int nlo = low == 0 ? lo : lo + (int)((len * low) / 65) + 1;
        hi = low == 64 ? hi : lo + (int)((len * (low + 1)) / 65);
        lo = nlo;
    }
    return lo;
}

// cnt[d] += 1 for every valid lane.  The lanes that agree with the first valid one are added at once: the
// entries of a popular column lie together after the first pass, and 64 additions to one LDS word take
// 64 turns (count of the second pass 33 -> 18 us on a power-law matrix of 13 M entries).
__device__ __forceinline__ void count_digit(int* cnt, unsigned d, bool valid) {
    if (!valid) return;
    const unsigned d0 = (unsigned)__builtin_amdgcn_readfirstlane((int)d);
    const unsigned long long same = __ballot(d == d0);
    const unsigned below = __builtin_amdgcn_mbcnt_hi((unsigned)(same >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)same, 0u));
    if (d != d0) atomicAdd(&cnt[d], 1);
    else if (below == 0) atomicAdd(&cnt[d], __popcll(same));
}

// A block counts the tiles of one group, so that what remains to be scanned is one row of counts per group (one row
// per tile took as long to scan as the tiles take to count).  Every tile has counters of its own, so that nothing waits
// between the group's request for all of its keys and the sums over its tiles (22 us at 13 M entries, 23 with one set of
// counters and two barriers a tile).
template <int ROUNDS, bool FIRST>
__global__ __launch_bounds__(kCountBlock) void transpose_count_kernel(TransposePass P)
{
    constexpr int THREADS = kCountBlock, T = kSortBlock * ROUNDS, PER = T / THREADS;
    static_assert(PER * THREADS == T && kGroupMax <= THREADS / 64, "whole loads per tile, one wave per tile's row search");
    typedef unsigned keys_of_tile __attribute__((ext_vector_type(PER), aligned(4)));
    __shared__ int cnt[kGroupMax * kDigitBinsMax];
    const int bins = 1 << P.bits;
    const int tile0 = blockIdx.x * P.group, tiles = min(P.group, P.ntiles - tile0);
    const long base = (long)tile0 * T;
    const int count = (int)min((long)tiles * T, (long)P.n - base);
    const unsigned* __restrict__ keys = (FIRST ? reinterpret_cast<const unsigned*>(P.colind) : P.mid_in) + base;
    const int own = (int)threadIdx.x * PER;
    keys_of_tile key[kGroupMax];
#pragma unroll
    for (int g = 0; g < kGroupMax; ++g) {
        if ((g + 1) * T <= count) {
            key[g] = *reinterpret_cast<const keys_of_tile*>(keys + g * T + own);
        } else {
#pragma unroll
            for (int i = 0; i < PER; ++i) key[g][i] = g * T + own + i < count ? keys[g * T + own + i] : 0u;
        }
    }
    for (int d = threadIdx.x; d < tiles * bins; d += THREADS) cnt[d] = 0;
    if constexpr (FIRST) {                                // the scatter kernel starts its row walk from here
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        if (w < tiles) {
            const int tile = tile0 + w;
            const int r = owner_row_wave(P.rowptr, 0, P.m - 1, (int)((long)tile * T), lane);
            if (lane == 0) P.tile_row[tile] = r;
            if (tile == P.ntiles - 1) {
                const int l = owner_row_wave(P.rowptr, r, P.m - 1, P.n - 1, lane);
                if (lane == 0) P.tile_row[P.ntiles] = l;
            }
        }
    }
    lds_barrier();
#pragma unroll
    for (int g = 0; g < kGroupMax; ++g) {
        if (g < tiles) {
#pragma unroll
            for (int i = 0; i < PER; ++i) count_digit(cnt + g * bins, pass_digit<FIRST>(key[g][i], P), g * T + own + i < count);
        }
    }
    lds_barrier();
    for (int d = threadIdx.x; d < bins; d += THREADS) {
        int before = 0;
        for (int g = 0; g < tiles; ++g) {
            P.hist[(long)(tile0 + g) * bins + d] = before;
            before += cnt[g * bins + d];
        }
        P.group_hist[(long)blockIdx.x * bins + d] = before;
    }
}

// Exclusive prefix over the groups for every digit, in place, and the digit totals.  A block owns 16
// digits (64-byte pieces of the rows) and cuts the groups into 64 stretches, one per thread and digit.
__global__ __launch_bounds__(1024) void transpose_scan_kernel(int* __restrict__ hist, int rows, int bins, int* __restrict__ total)
{
    constexpr int U = 8;
    __shared__ int part[64][kScanDigits + 1];
    const int dl = threadIdx.x & (kScanDigits - 1), ch = threadIdx.x / kScanDigits;
    const int per = (rows + 63) >> 6;
    const int t0 = min(ch * per, rows), t1 = min(t0 + per, rows);
    int* __restrict__ h = hist + blockIdx.x * kScanDigits + dl;
    int sum = 0;
    for (int t = t0; t < t1; t += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) sum += t + u < t1 ? h[(long)(t + u) * bins] : 0;
    }
    part[ch][dl] = sum;
    __syncthreads();
    {
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;      // wave w scans the stretches of digit w
        const int v = part[lane][w];
        const int inc = wave_inclusive_scan_dpp(v);
        part[lane][w] = inc - v;
        if (lane == 63) total[blockIdx.x * kScanDigits + w] = inc;
    }
    __syncthreads();
    int run = part[ch][dl];
    for (int t = t0; t < t1; t += U) {
        int v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = t + u < t1 ? h[(long)(t + u) * bins] : 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (t + u < t1) h[(long)(t + u) * bins] = run;
            run += v[u];
        }
    }
}

// Exclusive prefix sums over 1024 values spread 4 to a thread in order (value i of thread t belongs to
// index 4 t + i) of a block of 256.  sh: 4 ints.  All threads must call it.
__device__ __forceinline__ void block_scan_bins(int (&v)[4], int* sh) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int sum = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) { const int x = v[i]; v[i] = sum; sum += x; }
    const int inc = wave_inclusive_scan_dpp(sum);
    lds_barrier();
    if (lane == 63) sh[wave] = inc;
    lds_barrier();
    const int s0 = sh[0], s1 = sh[1], s2 = sh[2];
    const int off = inc - sum + (wave > 0 ? s0 : 0) + (wave > 1 ? s1 : 0) + (wave > 2 ? s2 : 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] += off;
}

// Values 4 t ... 4 t + 3 of p for thread t, zeros at and behind `bins`, a multiple of 4; p on a 16-byte boundary.
__device__ __forceinline__ void load_bins(const int* __restrict__ p, int bins, int (&v)[4]) {
    const bool own = (int)threadIdx.x * 4 < bins;
    const int4 x = *reinterpret_cast<const int4*>(p + (own ? threadIdx.x * 4 : 0));
    v[0] = own ? x.x : 0; v[1] = own ? x.y : 0; v[2] = own ? x.z : 0; v[3] = own ? x.w : 0;
}

// Lanes of the wave that hold the same digit, among the lanes of `valid`.  The width is known to the compiler, so that the
// votes are straight code and no branch stands around every bit.
template <int BITS>
__device__ __forceinline__ unsigned long long digit_peers_of(unsigned d, unsigned long long valid) {
    unsigned lo = (unsigned)valid, hi = (unsigned)(valid >> 32);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const int m = __builtin_amdgcn_sbfe((int)d, b, 1);            // all ones when the bit is set
        const unsigned long long vote = __builtin_amdgcn_ballot_w64(m < 0);
        lo &= ~((unsigned)vote ^ (unsigned)m);
        hi &= ~((unsigned)(vote >> 32) ^ (unsigned)m);
    }
    return (unsigned long long)hi << 32 | lo;
}

// LDS of a scatter block in bytes: tile (key, value, digit), digit offsets, 16-bit counters per wave.
template <int ROUNDS>
constexpr size_t transpose_scatter_lds(int bins) {
    return (size_t)kSortBlock * ROUNDS * 10 + (size_t)bins * 4 + (size_t)bins * 2 * kSortWaves + kSortWaves * 8;
}

// Inclusive maximum over the lanes of a wave.
__device__ __forceinline__ unsigned wave_inclusive_max(unsigned v) {
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));   // row_shr:1
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));   // row_shr:2
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));   // row_shr:4
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));   // row_shr:8
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));   // row_bcast:15
    return max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));   // row_bcast:31
}

// Stable placement of one tile.  FIRST: input is the matrix; LAST: output is the arrays of A^T.  WIDE: byte offsets of
// entries do not fit 32 bits.  BITS: at least P.bits; the votes of bits that no digit has change nothing.
//
// Row numbers (FIRST): the rows that begin inside the tile leave a mark at their first entry, in a
// coalesced walk over their row pointers, and an entry's row is the last mark at or before it.  (A binary
// search per entry took as long as the rest of the pass: 175 against 82 us at 13 M entries.)  A tile that
// spans very many rows without entries searches after all.
//
// What bounds a pass: memory (8 bytes in and out per entry) and, close behind, the vector instructions of the ranking;
// small tiles keep enough waves resident to overlap the two (13 M entries, k = 262 144: 68 and 46 us; with the row
// pointers behind the ranking 76, with a branch around every vote 79 and 51 before that).  The tiles that an XCD has in hand at a
// time are neighbours: blocks that stay and take several neighbouring tiles one after another, the next one's entries on their
// way, took 125 and 80 us where the kernel then took 74 and 49, since their runs meet in L2 only when many lines have left it half full.
template <int ROUNDS, bool FIRST, bool LAST, int BITS, bool WIDE>
__global__ __launch_bounds__(kSortBlock) void transpose_scatter_kernel(TransposePass P)
{
    constexpr int THREADS = kSortBlock, T = THREADS * ROUNDS, WAVES = kSortWaves, RUN = ROUNDS * 64;
    static_assert(THREADS == 256 && kDigitBinsMax == 1024 && T <= 0xffff, "4 digits a thread, counters of 16 bits");
    extern __shared__ __align__(16) int lds[];
    const int tile = tile_of_block(P.ntiles);
    if (tile >= P.ntiles) return;
    const int bins = 1 << P.bits;
    int* skey = lds;                                      // [T]
    float* sval = reinterpret_cast<float*>(lds + T);      // [T]
    int* gofs = lds + 2 * T;                              // [bins]: global position minus tile slot, per digit
    unsigned* wcnt = reinterpret_cast<unsigned*>(gofs + bins);                       // [WAVES][bins / 2]: count, then first slot
    unsigned short* sdig = reinterpret_cast<unsigned short*>(wcnt + WAVES * (bins / 2));   // [T]
    int* sh = reinterpret_cast<int*>(sdig + T);           // [WAVES], and the waves' last marks
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long base = (long)tile * T;
    const int count = (int)min((long)T, (long)P.n - base);
    const unsigned own = wave * RUN + lane;               // the thread's first entry
    auto request = [&](const auto* from, auto& x) {
        typedef std::remove_reference_t<decltype(*from)> number;
        const char* p = reinterpret_cast<const char*>(from + base);
        if (count == T) {
#pragma unroll
            for (int q = 0; q < ROUNDS; ++q) x[q] = *reinterpret_cast<number*>(p + own * 4u + q * 256);
        } else {
            const unsigned last = (unsigned)count - 1;
#pragma unroll
            for (int q = 0; q < ROUNDS; ++q) x[q] = *reinterpret_cast<number*>(p + min(own + q * 64, last) * 4u);
        }
    };
    unsigned key[ROUNDS];
    float val[ROUNDS];
    request(FIRST ? reinterpret_cast<const unsigned*>(P.colind) : P.mid_in, key);
    request(P.vals_in, val);
    // thread t owns digits 4 t ... 4 t + 3: the global position of the tile's first entry of the digit
    const bool owner = (int)threadIdx.x * 4 < bins;
    int gpos[4], before[4], in_group[4];
    load_bins(P.total, bins, gpos);
    load_bins(P.group_hist + (long)(tile / P.group) * bins, bins, before);
    load_bins(P.hist + (long)tile * bins, bins, in_group);
    if (owner) {
#pragma unroll
        for (int w = 0; w < WAVES; ++w) *reinterpret_cast<uint2*>(&wcnt[w * (bins / 2) + 2 * threadIdx.x]) = make_uint2(0u, 0u);
    }
    // FIRST: the pointers of the rows that begin in the tile, one a thread, are on their way during the ranking
    const int* __restrict__ rowptr = P.rowptr;
    const int row_lo = FIRST ? P.tile_row[tile] : 0, row_hi = FIRST ? P.tile_row[tile + 1] : 0;
    const bool marked = FIRST && row_hi - row_lo <= 8 * T;
    int begins = 0;
    if (marked) {
        begins = rowptr[min(row_lo + 1 + (int)threadIdx.x, row_hi)];
#pragma unroll
        for (int q = 0; q < ROUNDS; ++q) skey[q * THREADS + threadIdx.x] = 0;
    }
    lds_barrier();
    // rank of every entry among the wave's entries of the same digit
    unsigned* counter = wcnt + wave * (bins / 2);
    const unsigned short* counted = reinterpret_cast<const unsigned short*>(counter);
    unsigned rank[ROUNDS];
#pragma unroll
    for (int q = 0; q < ROUNDS; ++q) {
        const bool valid = (int)own + q * 64 < count;
        const unsigned d = pass_digit<FIRST>(key[q], P);
        const unsigned long long peers = digit_peers_of<BITS>(d, __builtin_amdgcn_ballot_w64(valid));
        const unsigned below = __builtin_amdgcn_mbcnt_hi((unsigned)(peers >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)peers, 0u));
        // every lane reads, then one lane per digit adds: the LDS unit serves a wave's requests in issue order, so that
        // no round waits for the one before
        rank[q] = counted[d] + below;
        wave_lds_sync();
        if (valid && below == 0) atomicAdd(&counter[d >> 1], (unsigned)__popcll(peers) << ((d & 1u) * 16));
        wave_lds_sync();
        __builtin_amdgcn_sched_barrier(0);            // keep the votes of one round together
    }
    if (marked) {
        for (int r = row_lo + 1 + (int)threadIdx.x; r <= row_hi; r += THREADS) {
            const int p = begins - (int)base;             // row_hi may begin with the next tile
            if (p < count) atomicMax(&skey[p], r - row_lo);
            if (r + THREADS <= row_hi) begins = rowptr[r + THREADS];
        }
    }
    lds_barrier();
    int row[ROUNDS];
    if constexpr (FIRST) {
        if (marked) {
            // marks ascend: the last one at or before an entry is the largest
            unsigned upto = 0;
#pragma unroll
            for (int q = 0; q < ROUNDS; ++q) {
                const unsigned v = max(wave_inclusive_max((unsigned)skey[own + q * 64]), upto);
                row[q] = (int)v;
                upto = (unsigned)__builtin_amdgcn_readlane((int)v, 63);
            }
            if (lane == 0) sh[WAVES + wave] = (int)upto;
        } else {
#pragma unroll
            for (int q = 0; q < ROUNDS; ++q) row[q] = owner_row(rowptr, row_lo, row_hi, (int)base + min((int)own + q * 64, count - 1));
        }
    }
    block_scan_bins(gpos, sh);                        // digit totals -> first positions
    {
        // two digits to a word: no sum of a tile's counts leaves 16 bits
        uint2 c[WAVES], sum = make_uint2(0u, 0u);
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            c[w] = owner ? *reinterpret_cast<const uint2*>(&wcnt[w * (bins / 2) + 2 * threadIdx.x]) : make_uint2(0u, 0u);
            sum.x += c[w].x;
            sum.y += c[w].y;
        }
        int slot[4] = {(int)(sum.x & 0xffffu), (int)(sum.x >> 16), (int)(sum.y & 0xffffu), (int)(sum.y >> 16)};
        block_scan_bins(slot, sh);
        if (owner) {
            *reinterpret_cast<int4*>(&gofs[4 * threadIdx.x]) =
                make_int4(gpos[0] + before[0] + in_group[0] - slot[0], gpos[1] + before[1] + in_group[1] - slot[1],
                          gpos[2] + before[2] + in_group[2] - slot[2], gpos[3] + before[3] + in_group[3] - slot[3]);
            uint2 run = make_uint2((unsigned)slot[0] | (unsigned)slot[1] << 16, (unsigned)slot[2] | (unsigned)slot[3] << 16);
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                *reinterpret_cast<uint2*>(&wcnt[w * (bins / 2) + 2 * threadIdx.x]) = run;
                run.x += c[w].x;
                run.y += c[w].y;
            }
        }
    }
    if constexpr (FIRST) {
        if (marked) {                                     // the scans' barriers lie between
            int carry = 0;
#pragma unroll
            for (int w = 0; w < WAVES - 1; ++w) { const int x = sh[WAVES + w]; if (w < wave) carry = max(carry, x); }
#pragma unroll
            for (int q = 0; q < ROUNDS; ++q) row[q] = row_lo + max(row[q], carry);
        }
    }
    lds_barrier();
#pragma unroll
    for (int q = 0; q < ROUNDS; ++q) {
        if ((int)own + q * 64 < count) {
            const unsigned d = pass_digit<FIRST>(key[q], P);
            const unsigned slot = counted[d] + rank[q];
            unsigned out = key[q];
            if constexpr (FIRST) out = LAST ? (unsigned)row[q] : (unsigned)row[q] | (key[q] >> P.bits) << P.row_bits;
            skey[slot] = (int)out;
            sval[slot] = val[q];
            if constexpr (FIRST) sdig[slot] = (unsigned short)d;
        }
    }
    lds_barrier();
    // copy out: neighbouring tile slots of one digit are neighbouring global positions
    const unsigned row_mask = (1u << P.row_bits) - 1u;
    char* out_keys = reinterpret_cast<char*>(LAST ? reinterpret_cast<unsigned*>(P.t_colind) : P.mid_out);
    char* out_vals = reinterpret_cast<char*>(P.vals_out);
#pragma unroll
    for (int q = 0; q < ROUNDS; ++q) {
        const int i = q * THREADS + (int)threadIdx.x;
        if (i < count) {
            const unsigned x = (unsigned)skey[i];
            const int d = FIRST ? (int)sdig[i] : (int)(x >> P.row_bits);
            const unsigned pos = (unsigned)(gofs[d] + i);
            const size_t at = WIDE ? (size_t)pos * 4 : (size_t)(pos * 4u);
            *reinterpret_cast<unsigned*>(out_keys + at) = LAST && !FIRST ? x & row_mask : x;
            *reinterpret_cast<float*>(out_vals + at) = sval[i];
        }
    }
}

// Row pointers of A^T after two passes.  Block `low` finds where the first pass's output begins to hold
// that low digit and counts the high digits between the beginning of that tile of the second pass and
// there; what lies before the tile is in the second pass's prefixes.
template <int T>
__global__ __launch_bounds__(256) void transpose_rowptr_kernel(
    const unsigned* __restrict__ mid, int n, int k, int row_bits, int low_bits, int high_bits,
    const int* __restrict__ low_total, const int* __restrict__ hist, const int* __restrict__ group_hist,
    const int* __restrict__ high_total, int ntiles, int group, int* __restrict__ t_rowptr)
{
    __shared__ int cnt[kDigitBinsMax];
    __shared__ int sh[4];
    __shared__ int start;
    const int low = blockIdx.x, low_bins = 1 << low_bits, high_bins = 1 << high_bits;
    int first[4], lows[4];
    load_bins(high_total, high_bins, first);
    load_bins(low_total, low_bins, lows);
#pragma unroll
    for (int i = 0; i < 4; ++i) cnt[threadIdx.x * 4 + i] = 0;
    block_scan_bins(lows, sh);
#pragma unroll
    for (int i = 0; i < 4; ++i) if ((int)threadIdx.x * 4 + i == low) start = lows[i];
    block_scan_bins(first, sh);
    __syncthreads();
    const int pos = start;                                // entries with a smaller low digit
    const int tile = min(pos / T, ntiles - 1);            // pos == n: the last tile is counted whole
    const int count = pos - tile * T;                     // 0 ... T
    const unsigned* __restrict__ keys = mid + (long)tile * T;
#pragma unroll
    for (int r = 0; r < T / 256; ++r) {
        const int e = r * 256 + (int)threadIdx.x;
        count_digit(cnt, e < count ? keys[e] >> row_bits : 0u, e < count);
    }
    __syncthreads();
    int before[4], in_group[4];
    load_bins(group_hist + (long)(tile / group) * high_bins, high_bins, before);
    load_bins(hist + (long)tile * high_bins, high_bins, in_group);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int d = threadIdx.x * 4 + i;
        const long c = ((long)d << low_bits) | low;
        if (d < high_bins && c < k) t_rowptr[c] = first[i] + before[i] + in_group[i] + cnt[d];
    }
    if (low == 0 && threadIdx.x == 0) t_rowptr[k] = n;
}

// Row pointers of A^T after one pass: the digits' places themselves.
__global__ __launch_bounds__(256) void transpose_rowptr_one_kernel(const int* __restrict__ total, int bins, int n, int k,
                                                                   int* __restrict__ t_rowptr)
{
    __shared__ int sh[4];
    int first[4];
    load_bins(total, bins, first);
    block_scan_bins(first, sh);
#pragma unroll
    for (int i = 0; i < 4; ++i) { const int d = threadIdx.x * 4 + i; if (d < k) t_rowptr[d] = first[i]; }
    if (threadIdx.x == 0) t_rowptr[k] = n;
}

}  // namespace daspmm
