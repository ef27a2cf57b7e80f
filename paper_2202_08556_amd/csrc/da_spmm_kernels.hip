// HIP kernels of the DA-SpMM algorithm space for gfx950 (MI355X, wave64).
//
// Four kernel templates cover the 8 algorithms of the paper's Table 1:
//
//                     K-loop SR (Sec. 3.4 K1)        K-loop PR (Sec. 3.4 K2, Sec. 4)
//   M-loop RB (M1)    rb_sr_kernel<V,G,NV>           rb_pr_kernel<V,G,NV>
//   M-loop EB (M2)    eb_sr_kernel<V,G,NV>           eb_pr_kernel<V,G,NV>  (conditional reduction)
//
// The N-loop axis (Sec. 3.3) is the lane mapping, set by the template parameters:
//   G   neighbouring lanes that share one stored entry and hold neighbouring column vectors of
//       the B row it points to.  RM mapping: G > 1 (a lane group reads one contiguous B row
//       segment, coalesced).  CM mapping: G = 1 (neighbouring lanes hold different rows / entries).
//   V   consecutive columns a lane loads at once (the float2/float4 technique of Sec. 4): 1 or 4.
//   NV  vectors of V columns a lane walks one after another, G*V columns apart (CM: the lane's own
//       strip of columns; RM uses NV = 1).
// A lane group covers G*V*NV columns; further column tiles are further blocks (see block_map).
// B and C are row-major in memory in every case.
//
// Memory-level parallelism: the hot loops fetch U entries' B segments back to back into registers
// before the first multiply-add consumes them, so that every wave keeps U gathers in flight; row
// bookkeeping (EB) happens while those loads are outstanding.
//
// No MFMA anywhere: every multiply-add consumes a freshly gathered B operand, there is no dense
// tile to contract.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace daspmm {

constexpr int kWave = 64;
constexpr int kBlock = 256;                 // 4 waves
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kU = 8;                       // gathers in flight per lane (4 ... 16 measured within 1 % on EB+RM+SR)

// Element strides of the dense operands: B(r, n) is at B[r*rb + n*cb], C(i, n) at C[i*rc + n*cc].
// Row-major storage has cb = cc = 1 and rb, rc = leading dimension; column-major storage has
// rb = rc = 1 and cb, cc = leading dimension.  Vector loads / stores (V = 4) need cb = cc = 1 and N >= 4,
// no alignment: the hardware takes 16-byte accesses at any multiple of 4 bytes.
struct Strides {
    long rb, cb, rc, cc;
};

// Order in which the EB workers take the chunks of stored entries: worker u takes chunk order[u]
// instead of chunk u.  The order is a permutation of 0..units-1 built for a matrix with `nnz`
// stored entries and the chunk size of the launch; a kernel that finds another nnz on the device
// ignores it (order == nullptr: no schedule).
// stripe > 0: the schedule is dealt in stripes to the XCDs that work on it (see sweep_block): all 8,
// or the 8 / pin_tiles XCDs that share a column tile when tiles are pinned to XCDs (nx_log2 = log2
// of that number).  The schedule may consist of two segments that are dealt separately, blocks
// [0, split) in stripes of `stripe` blocks and the rest in stripes of `stripe_b`, so that every XCD
// gets the same share of both (split == 0: one segment).  per_a = blocks of the first segment per
// XCD, rounded up to whole stripes; vblocks = number of block positions to walk (XCDs * blocks per
// XCD over both segments; positions that fall outside a segment find no chunk).  The grid's x
// extent must be a multiple of 8 so that a block stays on its XCD when it makes more than one pass.
struct Schedule {
    const int* order;
    int units;
    int nnz;
    int stripe, split, per_a, stripe_b, vblocks, nx_log2;
    // first_row[u] (may be null): the row that owned the first entry of chunk order[u] when the
    // order was built.  A hint only: a worker checks it against the row pointers it finds (two
    // independent loads) and searches when it does not hold, so stale contents cost speed, never
    // correctness.
    const int* first_row;
    // row_by_chunk[c] (may be null): the same hint indexed by chunk number; a worker on chunk c
    // reads row_by_chunk[c + 1], the row at the boundary that follows its chunk
    const int* row_by_chunk;
};

// The row that owns stored entry q according to the hint r, or -1 when the hint does not hold.
// *start / *end receive the row's pointers when it does.
__device__ __forceinline__ int hinted_row(const int* __restrict__ rowptr, int m, int r, int q, int* start, int* end) {
    if (r < 0 || r >= m) return -1;
    const int a = rowptr[r], b = rowptr[r + 1];
    if (a > q || q >= b) return -1;
    *start = a;
    *end = b;
    return r;
}

// ------------------------------------------------------------------------------------------
// small helpers
// ------------------------------------------------------------------------------------------
typedef float floatx4 __attribute__((ext_vector_type(4), aligned(4)));

template <int V>
__device__ __forceinline__ void load_vec(const float* __restrict__ p, float (&x)[V]) {
    if constexpr (V == 4) {
        const floatx4 t = *reinterpret_cast<const floatx4*>(p);
        x[0] = t.x; x[1] = t.y; x[2] = t.z; x[3] = t.w;
    } else {
        static_assert(V == 1, "V is 1 or 4");
        x[0] = *p;
    }
}

// C is written once and never read back by the kernels: its stores are marked non-temporal so
// that they do not push B rows out of L2.
template <int V>
__device__ __forceinline__ void store_vec(float* __restrict__ p, const float (&x)[V]) {
    if constexpr (V == 4) {
        floatx4 t = {x[0], x[1], x[2], x[3]};
        __builtin_nontemporal_store(t, reinterpret_cast<floatx4*>(p));
    } else {
        __builtin_nontemporal_store(x[0], p);
    }
}

// Rows shared between workers are combined with hardware fp32 atomic adds (Sec. 4: "atomic_add"
// for rows assigned to different workers); the return value is not used.  The first `skip` components
// belong to another lane as well (Cols): harmless to store twice, not to add twice.
template <int V>
__device__ __forceinline__ void emit_vec(float* __restrict__ p, const float (&x)[V], bool atomic, int skip) {
    if (atomic) {
#pragma unroll
        for (int v = 0; v < V; ++v)
            if (V == 1 || v >= skip) unsafeAtomicAdd(p + v, x[v]);
    } else {
        store_vec<V>(p, x);
    }
}

// The columns of a lane: nvec vectors of V columns, vector i at column n0 + i*G*V.  When N is not a
// multiple of V = 4 the last vector of the row is moved left by `shift` columns so that it ends with
// the row; its first `shift` columns are then also its left neighbour's, who computes the same values.
// (One column per lane instead, as before, issues four times the loads: N = 41 took twice as long on
// matrices that fit the caches.)
template <int V, int G, int NV>
struct Cols {
    int n0, nvec, shift;
    __device__ __forceinline__ Cols(int tile, int j, int N) {
        n0 = (tile * NV * G + j) * V;
        const int left = N - n0;
        nvec = left <= 0 ? 0 : min(NV, (left - 1) / (G * V) + 1);
        shift = 0;
        if constexpr (V > 1) {
            if (nvec > 0) shift = max(0, n0 + (nvec - 1) * G * V + V - N);
            if constexpr (NV == 1) n0 -= shift;
        }
    }
    // column offset of vector i from n0; vectors past nvec repeat the first one (valid memory)
    __device__ __forceinline__ int offset(int i) const {
        if constexpr (NV == 1) return 0;
        if constexpr (V == 1) return (i < nvec ? i : 0) * G * V;
        const int moved = i == nvec - 1 ? shift : 0;
        return i < nvec ? i * G * V - moved : (nvec == 1 ? -shift : 0);
    }
    __device__ __forceinline__ int skip(int i) const { return i == nvec - 1 ? shift : 0; }
};

// A lane's accumulators, laid out like its columns.
template <int V, int G, int NV>
struct Acc {
    typedef Cols<V, G, NV> C;
    float a[NV][V];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
            for (int v = 0; v < V; ++v) a[i][v] = 0.f;
    }
    // Branch-free gather of the lane's vectors of one B row (c.nvec >= 1).  Values of vectors past nvec
    // are never written out.  cs = column stride.
    __device__ __forceinline__ void load(const float* __restrict__ p, const C& c, long cs) {
#pragma unroll
        for (int i = 0; i < NV; ++i) load_vec<V>(p + (V == 1 ? c.offset(i) * cs : c.offset(i)), a[i]);
    }
    __device__ __forceinline__ void fma(float s, const Acc& b) {
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
            for (int v = 0; v < V; ++v) a[i][v] = fmaf(s, b.a[i][v], a[i][v]);
    }
    __device__ __forceinline__ void scale(float s) {
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
            for (int v = 0; v < V; ++v) a[i][v] *= s;
    }
    __device__ __forceinline__ void add(const Acc& b) {
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
            for (int v = 0; v < V; ++v) a[i][v] += b.a[i][v];
    }
    // b = bias of the column that vector 0 would begin at (in memory or LDS), or null
    template <class END> __device__ __forceinline__ void finish(const END& after, const float* b, const C& c) {
        static_assert(NV == 1, "one vector per lane");
#pragma unroll
        for (int v = 0; v < V; ++v) a[0][v] = after(a[0][v], b != nullptr ? b[v] : 0.f);
    }
    __device__ __forceinline__ void emit(float* __restrict__ p, const C& c, bool atomic, long cs) const {
#pragma unroll
        for (int i = 0; i < NV; ++i)
            if (i < c.nvec) emit_vec<V>(p + (V == 1 ? c.offset(i) * cs : c.offset(i)), a[i], atomic, c.skip(i));
    }
};

// What happens to a sum on its way to C: nothing, or a layer's bias (may be null) and rectification.  In the
// product kernel this costs the rows that one worker owns no memory traffic; a pass over C of its own reads and writes
// all of it once more (two layers on 262 144 nodes, 602 -> 128 -> 41: 982 us with such passes, 924 without; gradients of
// a layer 96 -> 64 on 100 003 nodes: 294 and 286).  Rows that several workers add to get theirs from
// eb_finish_kernel after the product.
struct PlainSums { static constexpr bool layer = false; };
struct LayerSums {
    static constexpr bool layer = true;
    const float* bias;
    int relu;
    __device__ __forceinline__ float operator()(float x, float b) const {
        x += b;
        return relu ? (x > 0.f || x != x ? x : 0.f) : x;   // NaN stays NaN
    }
};

// EB: the bias of the tile's columns waits in LDS, four columns to the left of the tile included (Cols::shift).  A load
// from memory at a row's end would wait for the stores before it.
template <class END, int TILE>
struct TileBias {
    static constexpr int kSize = END::layer ? TILE + 4 : 1;
    __device__ static __forceinline__ void fill(float* lds, const END& after, int tile0, int N) {
        if constexpr (END::layer) {
            for (int i = threadIdx.x; i < kSize; i += kBlock) {
                const int n = tile0 - 4 + i;
                lds[i] = after.bias != nullptr && n >= 0 && n < N ? after.bias[n] : 0.f;
            }
            __syncthreads();
        }
    }
};

// Orders LDS traffic of the lanes of one wave: the LDS unit serves one wave's requests in issue
// order, so only the compiler has to be kept from moving accesses across this point.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A lane group adds its sums of one row of C atomically.  With 16-byte vectors the four additions of a lane
// would each touch every fourth element of the row, four requests to a line where one does: the group's
// sums pass through LDS (`turn`, 4*G floats of the group's own) so that each addition of the G lanes covers
// G neighbouring elements.  (On a matrix with rows of 40 000 entries EB+RM+SR at N = 64 went from 164 to
// 84 us, and to the rate of the mapping with one column per lane.)  Every lane of the group must call it;
// crow = first column of the group's tile in the row, left = columns of B from there on.
template <int V, int G, int NV>
__device__ __forceinline__ void add_row(float* __restrict__ crow, const Acc<V, G, NV>& x, const Cols<V, G, NV>& c, int j,
                                        int left, long cs, float* turn) {
    if constexpr (V == 4 && G >= 4 && NV == 1) {
        const int at = j * V - c.shift;
        if (c.nvec > 0) {
#pragma unroll
            for (int v = 0; v < V; ++v)
                if (at + v >= 0) turn[at + v] = x.a[0][v];  // the row's last vector may begin before the tile
        }
        wave_lds_sync();
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const int n = v * G + j;
            if (n < left) unsafeAtomicAdd(crow + n, turn[n]);
        }
        wave_lds_sync();
    } else {
        if (c.nvec > 0) x.emit(crow + (long)(j * V - (NV == 1 ? c.shift : 0)) * cs, c, true, cs);
    }
}

// Address of the lane's first column in a row of B.  The gather address is the only per-entry
// integer work of the kernels, and in 64-bit form (sign extension, 64 x 64-bit multiply, 64-bit
// adds: about ten VALU operations, several of them quarter rate) it costs more issue slots than the
// four multiply-adds a 16-byte gather feeds.  WIDE = false: k < 2^24, row pitch < 16 MiB and B
// smaller than 4 GiB (checked by the host): byte offset = col * pitch + lane offset in one 24-bit
// multiply-add, added to the wave-uniform base by the load instruction itself.
template <bool WIDE>
struct BRows {
    const float* base;
    long rb;
    unsigned pitch_bytes, lane_bytes;
    __device__ __forceinline__ BRows(const float* __restrict__ B, int n0, const Strides& sd) {
        if constexpr (WIDE) {
            base = B + (long)n0 * sd.cb; rb = sd.rb; pitch_bytes = 0; lane_bytes = 0;
        } else {
            base = B; rb = 0;
            pitch_bytes = (unsigned)sd.rb * 4u;
            lane_bytes = (unsigned)n0 * (unsigned)sd.cb * 4u;
        }
    }
    __device__ __forceinline__ const float* row(int col) const {
        if constexpr (WIDE) {
            return base + (long)col * rb;
        } else {
            const unsigned off = __umul24((unsigned)col, pitch_bytes) + lane_bytes;
            return reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + off);
        }
    }
};

// Sum over the lanes of a wave that share lane % G (the slots of a PR kernel); every lane ends up
// with the total.  Butterfly steps at distance 32 and 16 use the gfx950 lane-swap instructions,
// the steps inside a 16-lane row use DPP rotations fused into the add: no LDS round trips.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
    return x + __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), CTRL, 0xf, 0xf, false));
}

template <int G>
__device__ __forceinline__ float slot_allreduce(float x) {
    if constexpr (G <= 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    if constexpr (G <= 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    if constexpr (G <= 8) x = dpp_add<0x128>(x);   // row_ror:8
    if constexpr (G <= 4) x = dpp_add<0x124>(x);   // row_ror:4
    if constexpr (G <= 2) x = dpp_add<0x122>(x);   // row_ror:2
    if constexpr (G <= 1) x = dpp_add<0x121>(x);   // row_ror:1
    return x;
}

// y[l] = x[l + D] for the lanes l < 64 - D of a wave (the other lanes receive unspecified values):
// the data movement of one step of the conditional reduction (Sec. 4, Fig. 6(e)), where a slot
// takes in the partial result of the slot D lanes to its right.  Distance 32 is one lane swap,
// distance 16 two swaps and a select, distance 1 a single DPP wave shift: no LDS round trip.
__device__ __forceinline__ unsigned lane_shift_down_32(unsigned x) {
    return __builtin_amdgcn_permlane32_swap(x, x, false, false)[1];      // lanes 0..31 <- lanes 32..63
}
__device__ __forceinline__ unsigned lane_shift_down_16(unsigned x) {
    // rows of 16 lanes [x0 x1 x2 x3] -> [x1 x2 x3 .]
    const unsigned z = lane_shift_down_32(x);                             // [x2 x3 x2 x3]
    const auto r = __builtin_amdgcn_permlane16_swap(x, z, false, false);  // [x0 x2 x2 x2], [x1 x3 x3 x3]
    return (threadIdx.x & 16) ? r[0] : r[1];
}
template <int D>
__device__ __forceinline__ float lane_shift_down(float xf) {
    static_assert(D == 1 || D == 2 || D == 4 || D == 8 || D == 16 || D == 32, "power of two below 64");
    const unsigned x = __float_as_uint(xf);
    if constexpr (D == 32) {
        return __uint_as_float(lane_shift_down_32(x));
    } else if constexpr (D == 16) {
        return __uint_as_float(lane_shift_down_16(x));
    } else if constexpr (D == 1) {
        return __uint_as_float(__builtin_amdgcn_update_dpp(0u, x, 0x130, 0xf, 0xf, false));   // wave_shl:1
    } else {
        // Distances 2, 4, 8 would take a DPP row rotation plus the rotation of the next row for the
        // lanes that wrap around (five operations); the LDS crossbar moves them in one and measured
        // faster (EB+RM+PR on the power-law matrix at N = 32: 249 against 261 us).
        return __shfl_down(xf, D, kWave);
    }
}

// The log-step network of the conditional reduction over the S = 64/G slots of a wave: in step DS
// (1, 2, 4, ...) slot s adds the value of slot s + DS when that slot belongs to the same run of
// equal row indices, i.e. when DS <= dist, the number of slots from s to the end of its run.
template <int G, int DS>
__device__ __forceinline__ void conditional_steps(float& x, int dist) {
    if constexpr (DS * G < kWave) {
        const float o = lane_shift_down<DS * G>(x);
        if (DS <= dist) x += o;
        conditional_steps<G, DS * 2>(x, dist);
    }
}

// Smallest r in [lo, hi] with rowptr[r+1] > q: the row that owns stored entry q (rows without
// entries are skipped).  Requires rowptr[lo] <= q < rowptr[hi+1].
__device__ __forceinline__ int row_of_entry(const int* __restrict__ rowptr, int lo, int hi, int q) {
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (rowptr[mid + 1] > q) hi = mid; else lo = mid + 1;
    }
    return lo;
}

// The same search done by the G lanes of a group together: every step probes G rows at once and
// narrows [lo, hi] to 1/(G+1) of its width, so it takes log_{G+1}(m) dependent loads instead of
// log_2(m).  All lanes of the group must call it together with the same q; j = lane index inside
// the group, shift = index of the group's first lane in the wave.
template <int G>
__device__ __forceinline__ int row_of_entry_group(const int* __restrict__ rowptr, int lo, int hi, int q,
                                                  int j, int shift) {
    if constexpr (G < 4) {
        return row_of_entry(rowptr, lo, hi, q);
    } else {
        while (lo < hi) {
            const long len = hi - lo;
            const int r = lo + (int)((len * (j + 1)) / (G + 1));       // lo <= r < hi
            const bool above = rowptr[r + 1] > q;                      // owner row is <= r
            unsigned long long bits = __ballot(above) >> shift;
            if constexpr (G < 64) bits &= (1ull << G) - 1;
            const int nfalse = G - __popcll(bits);                     // probes 0..nfalse-1 are too low
            const int new_lo = nfalse == 0 ? lo : lo + (int)((len * nfalse) / (G + 1)) + 1;
            const int new_hi = nfalse == G ? hi : lo + (int)((len * (nfalse + 1)) / (G + 1));
            lo = new_lo;
            hi = new_hi;
        }
        return lo;
    }
}

// entries a lane group stages per batch
template <int G> struct StageBatch { static constexpr int value = G < 8 ? kU : (G < 32 ? 32 : G); };

template <int U> struct Count { static constexpr int value = U; };

// A lane's share of a staged batch of SB stored entries (lane j of the group holds entries j, j+G,
// ...).  The next batch is fetched into registers while the current one is being consumed from LDS,
// so the (colind, val) round trip is off the critical path.
template <int G, int SB>
struct BatchRegs {
    int2 e[SB / G];
    __device__ __forceinline__ void fetch(const int* __restrict__ colind, const float* __restrict__ vals,
                                          int p0, int end, int j) {
#pragma unroll
        for (int i = 0; i < SB / G; ++i) {
            const int p = p0 + j + i * G;
            e[i] = make_int2(0, 0);
            if (p < end) { e[i].x = colind[p]; e[i].y = __float_as_int(vals[p]); }
        }
    }
    __device__ __forceinline__ void put(int2* st, int j) const {
#pragma unroll
        for (int i = 0; i < SB / G; ++i) st[j + i * G] = e[i];
    }
};

// Which column tile a block works on and its rank among the blocks of that tile.
//   pin_tiles == 0: 2-D grid, blockIdx.y = tile.
//   pin_tiles in {2,4,8}: 1-D grid whose size is a multiple of 8.  Consecutive workgroups go to
//     consecutive XCDs (8 per device, each with its own L2), so tile = (blockIdx.x % 8) % pin_tiles
//     keeps every XCD on one tile: its L2 then caches only that tile's slice of B.
struct BlockMap { int tile; long bx; long nbx; };
__device__ __forceinline__ BlockMap block_map(int pin_tiles) {
    BlockMap b;
    if (pin_tiles <= 0) {
        b.tile = blockIdx.y; b.bx = blockIdx.x; b.nbx = gridDim.x;
    } else {
        const int xcd = blockIdx.x & 7, per = 8 / pin_tiles;
        b.tile = xcd % pin_tiles;
        b.bx = (long)(blockIdx.x >> 3) * per + xcd / pin_tiles;
        b.nbx = (long)(gridDim.x >> 3) * per;
    }
    return b;
}

// Position in the schedule of (virtual) block vb when the schedule is swept by nx XCDs together
// (nx = 8, or 8 / pin_tiles for the XCDs that share a pinned column tile).  Workgroups go
// round-robin to the 8 XCDs and block_map numbers the blocks of one tile so that block vb runs on
// the (vb % nx)-th of these XCDs and is that XCD's (vb / nx)-th block.  Stripe t of XCD x is stripe
// nx t + x of the segment: at any time the XCDs work on nx neighbouring stripes, each on its own,
// and the rows of B that one L2 has to hold are an nx-th of the band all running workers cover.
// Returns -1 for a position outside its segment.
__device__ __forceinline__ long sweep_block(long vb, const Schedule& sch) {
    const unsigned nx = 1u << sch.nx_log2;
    const unsigned x = (unsigned)vb & (nx - 1u);          // block counts fit 32 bits
    unsigned l = (unsigned)(vb >> sch.nx_log2);
    if (l < (unsigned)sch.per_a) {
        const unsigned st = (unsigned)sch.stripe, t = l / st;
        const long sb = (long)(t * nx + x) * st + (l - t * st);
        return (sch.split > 0 && sb >= sch.split) ? -1 : sb;
    }
    l -= (unsigned)sch.per_a;
    const unsigned st = (unsigned)sch.stripe_b, t = l / st;
    return sch.split + (long)(t * nx + x) * st + (l - t * st);
}

// Calls f(Count<UU>, t) for t covering [begin, cnt) in blocks of UMAX, then 8, 4, 2, 1 entries, so that
// every block is straight-line code of a compile-time size: its gathers carry no predicates and
// are all in flight before the first one is consumed.
template <int UMAX, class F>
__device__ __forceinline__ void for_blocks(int begin, int cnt, F&& f) {
    int t = begin;
    for (; t + UMAX <= cnt; t += UMAX) f(Count<UMAX>{}, t);
    static_assert(UMAX <= 16, "the remainder is covered by blocks of 8, 4, 2, 1");
    if constexpr (UMAX > 8) { if (t + 8 <= cnt) { f(Count<8>{}, t); t += 8; } }
    if constexpr (UMAX > 4) { if (t + 4 <= cnt) { f(Count<4>{}, t); t += 4; } }
    if constexpr (UMAX > 2) { if (t + 2 <= cnt) { f(Count<2>{}, t); t += 2; } }
    if constexpr (UMAX > 1) { if (t < cnt) f(Count<1>{}, t); }
}
template <int UMAX, class F>
__device__ __forceinline__ void for_blocks(int cnt, F&& f) { for_blocks<UMAX>(0, cnt, f); }

// Rows whose sums another kernel adds to C (heavy_rows_kernel): one bit a row, for rows of at least min_len entries in
// a matrix of nnz (the number at `end`); they are written as zeros.  rows == nullptr: none.  *stale (in host memory)
// becomes 1 where another row has more than `longest` entries: the list is of another matrix.
struct LeftOut {
    const unsigned* rows;
    const int* end;
    int min_len, nnz, longest;
    int* stale;
};

// ------------------------------------------------------------------------------------------
// RB + SR : a lane group owns a row and adds its products one after another
// (Sec. 3.2 design M1, Sec. 3.4 design K1).  For G > 1 the group's lanes load a batch of stored
// entries with coalesced requests and pass them round through LDS, so that every entry is fetched
// once and reused for all columns of the tile (the sparse-element cache of Sec. 4).
// ------------------------------------------------------------------------------------------
template <int V, int G, int NV, bool WIDE, class END>
__global__ __launch_bounds__(kBlock) void rb_sr_kernel(
    int m, int N, Strides sd, const int* __restrict__ rowptr, const int* __restrict__ colind,
    const float* __restrict__ vals, const float* __restrict__ B, float* __restrict__ C, int pin_tiles, LeftOut out,
    END after)
{
    constexpr int RPW = kWave / G;                       // rows per wave
    constexpr int SB = StageBatch<G>::value;
    constexpr int UL = G == 1 ? kU / NV : kU;            // entries whose gathers are issued together
    __shared__ int2 stage[G > 1 ? kWavesPerBlock * RPW * SB : 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = lane / G, j = lane % G;
    const BlockMap bm = block_map(pin_tiles);
    const long row = (bm.bx * kWavesPerBlock + wave) * RPW + g;
    const Cols<V, G, NV> cols(bm.tile, j, N);
    const int n0 = cols.n0, nvec = cols.nvec;
    int start = 0, end = 0;
    if (row < m) { start = rowptr[row]; end = rowptr[row + 1]; }
    if (out.rows != nullptr && end - start > out.longest) {
        if (end - start >= out.min_len && (out.rows[row >> 5] >> (row & 31) & 1u) && *out.end == out.nnz) end = start;
        else *out.stale = 1;
    }
    Acc<V, G, NV> acc;
    acc.clear();
    const BRows<WIDE> brow(B, n0, sd);

    if constexpr (G == 1) {
        if (nvec > 0) {
            for_blocks<UL>(end - start, [&](auto uc, int t) {
                constexpr int UU = decltype(uc)::value;
                const int p0 = start + t;
                int c[UU];
                float a[UU];
                Acc<V, G, NV> b[UU];
#pragma unroll
                for (int u = 0; u < UU; ++u) { c[u] = colind[p0 + u]; a[u] = vals[p0 + u]; }
#pragma unroll
                for (int u = 0; u < UU; ++u) b[u].load(brow.row(c[u]), cols, sd.cb);
#pragma unroll
                for (int u = 0; u < UU; ++u) acc.fma(a[u], b[u]);
            });
        }
    } else {
        int2* st = stage + (wave * RPW + g) * SB;
        BatchRegs<G, SB> next;
        next.fetch(colind, vals, start, end, j);
        // The last entries of a row in one block, whose gathers behind the end fetch row 0 and give way to zeros, or exactly, in
        // blocks of 4, 2 and 1, each a round trip that the wave's other rows wait for.  Lanes of one column gain from one block
        // (27-point stencil of 64 x 128 x 128, N = 8 91 -> 87 us, N = 16 145 -> 138; 2 entries a row, 300 000 rows, N = 16 24.1 -> 21.4;
        // lognormal rows of 10, N = 16 17.2 -> 16.4; groups of 32 and 64 little: lognormal rows of 40, N = 17 61.1 -> 59.8, N = 33 90.8 -> 89.8;
        // rows of 60, N = 24 11.7 -> 11.5; 0.99 to 1.005 elsewhere over 8 matrices and N = 17 ... 130), but for groups of four (the stencil,
        // N = 4: 86 and 88); four columns a lane lose by the gathers (the stencil, N = 32: 168 and 172), also where only waves of
        // short rows take it.
        constexpr bool kInOne = V == 1 && G >= 8;
        for (int p0 = start; p0 < end; p0 += SB) {
            next.put(st, j);
            wave_lds_sync();
            if (p0 + SB < end) next.fetch(colind, vals, p0 + SB, end, j);
            if (nvec > 0) {
                const int cnt = min(SB, end - p0);
                auto block = [&](auto uc, auto whole, int t) {
                    constexpr int UU = decltype(uc)::value;
                    int2 e[UU];
                    Acc<V, G, NV> b[UU];
#pragma unroll
                    for (int u = 0; u < UU; ++u) e[u] = st[t + u];
#pragma unroll
                    for (int u = 0; u < UU; ++u) b[u].load(brow.row(e[u].x), cols, sd.cb);
#pragma unroll
                    for (int u = 0; u < UU; ++u) {
                        if (!decltype(whole)::value && u >= UU / 2 - (UU == 4)) {
#pragma unroll
                            for (int v = 0; v < V; ++v) b[u].a[0][v] = t + u < cnt ? b[u].a[0][v] : 0.f;
                        }
                        acc.fma(__int_as_float(e[u].y), b[u]);
                    }
                };
                if constexpr (kInOne) {
                    int t = 0;
                    for (; t + UL <= cnt; t += UL) block(Count<UL>{}, Count<1>{}, t);
                    if (cnt - t > UL / 2) block(Count<UL>{}, Count<0>{}, t);
                    else if (cnt > t) block(Count<UL / 2>{}, Count<0>{}, t);
                } else {
                    for_blocks<UL>(cnt, [&](auto uc, int t) { block(uc, Count<1>{}, t); });
                }
            }
            wave_lds_sync();
        }
    }
    if constexpr (END::layer)
        if (row < m && nvec > 0) acc.finish(after, after.bias ? after.bias + n0 : nullptr, cols);
    if (row < m && nvec > 0) acc.emit(C + row * sd.rc + (long)n0 * sd.cc, cols, false, sd.cc);
}

// ------------------------------------------------------------------------------------------
// RB + PR : a wave owns a row; its 64 lanes form S = 64/G slots along the row's stored entries
// (times G lanes along n).  Rows longer than S are walked with a for-loop (technique 1 of Sec. 4),
// lanes load V consecutive columns at once (technique 2), the wave's entries are fetched once and
// shared through LDS (technique 3), and the slots are combined by a reduction tree (Sec. 3.4 K2).
// In a batch of 64 staged entries slot s takes entries s, s+S, s+2S, ...
// With 4 slots (groups of 16 lanes) and N no multiple of four, which ran with 8 slots of one-column lanes before it took
// 16-byte lanes, a slot adds four products to each other before it adds them to its sum, which then
// takes fewer additions than with 8 slots (N = 41, rows of 400: error 1.9e-7 with one addition an entry, 1.4e-7 with 8
// slots, 1.1e-7 now).  Two sums instead, of the even and the odd entries, cost registers: 27-point stencil, N = 41:
// 45 -> 54 us; multiples of four keep one addition an entry (GROUPED = false; rows of 1000, N = 36: 46 us, 49 with
// groups, and as many with the choice made at run time).
// ------------------------------------------------------------------------------------------
template <int V, int G, int NV, bool WIDE, bool GROUPED, class END>
__global__ __launch_bounds__(kBlock) void rb_pr_kernel(
    int m, int N, Strides sd, const int* __restrict__ rowptr, const int* __restrict__ colind,
    const float* __restrict__ vals, const float* __restrict__ B, float* __restrict__ C, int pin_tiles, END after)
{
    constexpr int S = kWave / G;
    constexpr int UL = G == 1 ? (NV > 2 ? 2 : 4) : (G < kU ? G : kU);
    __shared__ int2 stage[G > 1 ? kBlock : 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int s = lane / G, j = lane % G;
    const BlockMap bm = block_map(pin_tiles);
    const long row = bm.bx * kWavesPerBlock + wave;
    if (row >= m) return;                                 // whole wave leaves together
    const Cols<V, G, NV> cols(bm.tile, j, N);
    const int n0 = cols.n0, nvec = cols.nvec;
    const int start = rowptr[row], end = rowptr[row + 1];
    Acc<V, G, NV> acc;
    acc.clear();
    const BRows<WIDE> brow(B, n0, sd);

    if constexpr (G == 1) {
        if (nvec > 0) {
            // steps in which all 64 lanes hold an entry, then one ragged step
            const int len = end - start;
            for_blocks<UL>(len / kWave, [&](auto uc, int t) {
                constexpr int UU = decltype(uc)::value;
                const int p0 = start + t * kWave + lane;
                int c[UU];
                float a[UU];
                Acc<V, G, NV> b[UU];
#pragma unroll
                for (int u = 0; u < UU; ++u) { c[u] = colind[p0 + u * kWave]; a[u] = vals[p0 + u * kWave]; }
#pragma unroll
                for (int u = 0; u < UU; ++u) b[u].load(brow.row(c[u]), cols, sd.cb);
#pragma unroll
                for (int u = 0; u < UU; ++u) acc.fma(a[u], b[u]);
            });
            const int p = start + (len / kWave) * kWave + lane;
            if (p < end) {
                Acc<V, G, NV> b;
                b.load(brow.row(colind[p]), cols, sd.cb);
                acc.fma(vals[p], b);
            }
        }
    } else {
        int2* st = stage + wave * kWave;
        BatchRegs<kWave, kWave> next;
        next.fetch(colind, vals, start, end, lane);
        for (int p0 = start; p0 < end; p0 += kWave) {
            next.put(st, lane);
            wave_lds_sync();
            if (p0 + kWave < end) next.fetch(colind, vals, p0 + kWave, end, lane);
            const int cnt = min(kWave, end - p0);
            if (nvec > 0) {
                // The last step may be ragged: slots behind the last entry gather row 0 and take zeros in its place.  A step of
                // its own was one more round trip to memory (lognormal rows of 23, k = 61 417, N = 64: 54.6 -> 47 us, N = 32
                // 33.1 -> 29.7; 25 entries a row, N = 32 18.2 -> 16.1; 27-point stencil of 30^3, N = 32 11.5 -> 10.0).
                for_blocks<UL>((cnt + S - 1) / S, [&](auto uc, int t) {
                    constexpr int UU = decltype(uc)::value;
                    int2 ee[UU];
                    Acc<V, G, NV> b[UU];
#pragma unroll
                    for (int u = 0; u < UU; ++u) ee[u] = st[(t + u) * S + s];
#pragma unroll
                    for (int u = 0; u < UU; ++u) b[u].load(brow.row(ee[u].x), cols, sd.cb);
                    const bool held = (t + UU - 1) * S + s < cnt;
#pragma unroll
                    for (int i = 0; i < NV; ++i)
#pragma unroll
                        for (int v = 0; v < V; ++v) b[UU - 1].a[i][v] = held ? b[UU - 1].a[i][v] : 0.f;
#pragma unroll
                    for (int u = 0; u < UU; ++u) {
                        if (!GROUPED || UU == 1) {
                            acc.fma(__int_as_float(ee[u].y), b[u]);
                        } else if (u % 2 == 0) {           // UU is a power of two
                            b[u].scale(__int_as_float(ee[u].y));
                            b[u].fma(__int_as_float(ee[(u + 1) % UU].y), b[(u + 1) % UU]);
                            if (UU < 4) acc.add(b[u]);
                            else if (u % 4 == 2) { b[u].add(b[(u + UU - 2) % UU]); acc.add(b[u]); }
                        }
                    }
                });
            }
            wave_lds_sync();
        }
    }
    // reduction tree over the slots: lanes with equal j
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
        for (int v = 0; v < V; ++v) acc.a[i][v] = slot_allreduce<G>(acc.a[i][v]);
    if constexpr (END::layer)
        if (s == 0 && nvec > 0) acc.finish(after, after.bias ? after.bias + n0 : nullptr, cols);
    if (s == 0 && nvec > 0) acc.emit(C + row * sd.rc + (long)n0 * sd.cc, cols, false, sd.cc);
}

// ------------------------------------------------------------------------------------------
// RB on a column-major B (columns contiguous, rb = 1): L lanes share a row and take its entries in turn, each for the NC
// columns of the tile; neighbouring lanes hold neighbouring rows.  A load then fetches one column of B for the entries of
// 64 / L rows, which lie side by side in a banded or stencil matrix.  Lanes along N instead, as the row-major
// kernels have them, fetch every element from a line of its own, and write C in 4-byte pieces where its columns
// are contiguous, too.  What bounds it: the lines a load touches.  27-point stencil of 64^3, N = 8: 58 us with lanes along N,
// 25 here (52 with the L lanes of a row side by side, 27 with every lane reading its own entries: a third of the
// time), N = 16: 197 and 45; 12 random columns a row, N = 8: 43 and 43, N = 20: 206 and 102.
// Sums: a lane adds n / L entries one after another, then the lanes' sums are added in a tree.
// ------------------------------------------------------------------------------------------
template <int L, int NC>
__global__ __launch_bounds__(kBlock) void rb_columns_kernel(
    int m, int N, Strides sd, const int* __restrict__ rowptr, const int* __restrict__ colind,
    const float* __restrict__ vals, const float* __restrict__ B, float* __restrict__ C)
{
    constexpr int U = 4, R = kWave / L;                    // entries of a lane in flight, rows of a wave
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane / R;
    const long row0 = ((long)blockIdx.x * kWavesPerBlock + wave) * R, row = row0 + lane % R;
    const int n0 = blockIdx.y * NC, left = min(N - n0, NC);
    // Entries are read by L neighbouring lanes to a row, in the order of memory, and change lanes once: the lane of
    // row r and turn j receives the one that lane r * L + j read.
    const int source = (lane % R) * L + j;
    unsigned start = 0, end = 0, from = 0, to = 0;        // the last steps pass 2^31 where nnz is next to it
    if (row < m) { start = rowptr[row]; end = rowptr[row + 1]; }
    if (row0 + lane / L < m) { from = rowptr[row0 + lane / L] + lane % L; to = rowptr[row0 + lane / L + 1]; }
    const float* __restrict__ Bn = B + (long)n0 * sd.cb;
    float acc[NC];
#pragma unroll
    for (int n = 0; n < NC; ++n) acc[n] = 0.f;
    for (unsigned p = start + j; __any(p < end); p += U * L, from += U * L) {
        int c[U];
        float a[U], b[U][NC];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            c[u] = 0;
            a[u] = 0.f;
            if (from + u * L < to) { c[u] = colind[from + u * L]; a[u] = vals[from + u * L]; }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) { c[u] = __shfl(c[u], source); a[u] = __shfl(a[u], source); }
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int n = 0; n < NC; ++n) b[u][n] = 0.f;
            if (p + u * L < end) {                         // zeros otherwise: no product with what column 0 holds
#pragma unroll
                for (int n = 0; n < NC; ++n) if (n < left) b[u][n] = Bn[n * sd.cb + (unsigned)c[u]];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int n = 0; n < NC; ++n) acc[n] = fmaf(a[u], b[u][n], acc[n]);
    }
#pragma unroll
    for (int n = 0; n < NC; ++n) {
        const float x = slot_allreduce<R>(acc[n]);
        if (j == n % L && row < m && n < left) __builtin_nontemporal_store(x, C + row * sd.rc + (long)(n0 + n) * sd.cc);
    }
}

// ------------------------------------------------------------------------------------------
// EB pre-pass.  EB workers own fixed-size chunks of consecutive stored entries (Sec. 3.2 design
// M2).  A row whose entries all fall into one chunk is written by exactly one worker with a plain
// store; a row that straddles a chunk boundary receives atomic additions from several workers and
// must start from zero; a row without entries is touched by no worker.  This pass zeroes exactly
// those two kinds of rows so that C needs no full memset.  `chunk` is the number of entries per
// worker of the product kernel that follows.  own_short: that kernel gives every row of at most
// `chunk` entries to a single worker (see eb_sr_kernel), so only longer rows are shared.  A wave inspects 64 rows (one per lane) and then
// clears the flagged ones together: one row at a time with full-width stores when a row takes
// more than 32 stores, several rows per store instruction otherwise.
// A layer (LayerSums): rows without entries get what bias and rectification make of zero at once, the product kernel finishes
// the rows of one worker, and eb_finish_kernel after it those that several workers add to.  Reading rows without entries
// again after the product costs more than it looks, since loads wait where stores do not (150 000 rows, 3000 of them
// stored, 40 -> 32 -> 37: 102 us, 76 as here; 86 with a pass over all of C).
// ------------------------------------------------------------------------------------------
struct EbRow { bool empty, split; };
__device__ __forceinline__ EbRow eb_row(int m, long row, const int* __restrict__ rowptr, int chunk, int own_short) {
    if (row >= m) return EbRow{false, false};
    const int start = rowptr[row], end = rowptr[row + 1];
    return EbRow{end == start, end != start && start / chunk != (end - 1) / chunk && (!own_short || end - start > chunk)};
}

// The flagged ones of the wave's 64 rows: what `rows` reads of up to U pieces of V columns, then what it writes.
template <int V, int U, class ROWS>
__device__ __forceinline__ void for_flagged_rows(long base, int N, bool flagged, ROWS rows) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long mask = __ballot(flagged);
    if (mask == 0) return;
    const int vecs = (N + V - 1) / V;                     // stores per row
    if (vecs > kWave / 2) {
        for (int n0 = lane * V; n0 < N; n0 += kWave * V) {
            rows.columns(n0);
            for (unsigned long long left = mask; left; left &= left - 1) {
                const long row = base + __ffsll((long long)left) - 1;
                rows.read(row, 0);
                rows.write(row, 0);
            }
        }
    } else {
        // short rows of C: T lanes per row, 64/T flagged rows per store instruction.  The flagged
        // lanes list themselves in LDS in lane order; lane group s then takes list entries
        // s, s + 64/T, ...
        __shared__ unsigned char listed[kWavesPerBlock][kWave];
        const int count = __popcll(mask);
        if (flagged) listed[wave][__popcll(mask & ((1ull << lane) - 1ull))] = (unsigned char)lane;
        wave_lds_sync();
        const int T = vecs <= 1 ? 1 : 1 << (32 - __clz(vecs - 1));   // power of two >= vecs, <= 32
        const int n0 = (lane & (T - 1)) * V;
        if (n0 >= N) return;
        rows.columns(n0);
        for (int s = lane / T; s < count; s += kWave / T * U) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (s + kWave / T * u < count) rows.read(base + listed[wave][s + kWave / T * u], u);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (s + kWave / T * u < count) rows.write(base + listed[wave][s + kWave / T * u], u);
        }
    }
}

// Rows of C that become zero, or what a layer makes of zero.
template <int V, class END>
struct FillRows {
    int N;
    const Strides& sd;
    float* C;
    END after;
    float* at;
    float z[V];
    __device__ __forceinline__ void columns(int n0) {
        const int n = min(n0, N - V);
        at = C + (long)n * sd.cc;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            z[v] = 0.f;
            if constexpr (END::layer) z[v] = after(0.f, after.bias ? after.bias[n + v] : 0.f);
        }
    }
    __device__ __forceinline__ void read(long, int) {}
    __device__ __forceinline__ void write(long row, int) { store_vec<V>(at + row * sd.rc, z); }
};

template <int V, class END>
__global__ __launch_bounds__(kBlock) void eb_zero_kernel(
    int m, int N, Strides sd, const int* __restrict__ rowptr, float* __restrict__ C, int chunk, int own_short, END after)
{
    const long base = ((long)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6)) * kWave;
    if (base >= m) return;
    const EbRow r = eb_row(m, base + (threadIdx.x & 63), rowptr, chunk, own_short);
    if constexpr (END::layer) for_flagged_rows<V, 1>(base, N, r.empty, FillRows<V, END>{N, sd, C, after});
    for_flagged_rows<V, 1>(base, N, r.split || (!END::layer && r.empty), FillRows<V, PlainSums>{N, sd, C, PlainSums{}});
}

// Bias and rectification of rows that are complete.  Where N is no multiple of V the last lane of a row begins
// left of its columns and writes its own ones only, so that every element is finished once.
template <int V, int U>
struct FinishRows {
    int N;
    const Strides& sd;
    float* C;
    LayerSums after;
    float* at;
    int skip;
    float b[V], x[U][V];
    __device__ __forceinline__ void columns(int n0) {
        const int n = min(n0, N - V);
        at = C + (long)n * sd.cc;
        skip = n0 - n;
#pragma unroll
        for (int v = 0; v < V; ++v) b[v] = after.bias ? after.bias[n + v] : 0.f;
    }
    __device__ __forceinline__ void read(long row, int u) { load_vec<V>(at + row * sd.rc, x[u]); }
    __device__ __forceinline__ void write(long row, int u) {
#pragma unroll
        for (int v = 0; v < V; ++v) x[u][v] = after(x[u][v], b[v]);
        if (skip == 0) return store_vec<V>(at + row * sd.rc, x[u]);
#pragma unroll
        for (int v = 0; v < V; ++v) if (v >= skip) at[row * sd.rc + v * sd.cc] = x[u][v];
    }
};

template <int V>
__global__ __launch_bounds__(kBlock) void eb_finish_kernel(
    int m, int N, Strides sd, const int* __restrict__ rowptr, float* __restrict__ C, int chunk, int own_short, LayerSums after)
{
    const long base = ((long)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6)) * kWave;
    if (base >= m) return;
    const bool split = eb_row(m, base + (threadIdx.x & 63), rowptr, chunk, own_short).split;
    for_flagged_rows<V, 4>(base, N, split, FinishRows<V, 4>{N, sd, C, after});
}

// ------------------------------------------------------------------------------------------
// EB + SR : a lane group owns `chunk` consecutive stored entries and walks them in order,
// keeping (partial sum, row).  When the row changes the partial is written: plain store if the
// row lies wholly inside the chunk, atomic add for the first / last row when it is shared with the
// neighbouring chunk (the "partial sum aggregation among workers" of Sec. 3.2).  The row of the
// chunk's first entry is found by binary search in rowptr (the "row index calculation" overhead
// named there).  Workers stride over the chunks so that the grid size does not depend on nnz,
// which only the device knows.  With own_short the chunk boundaries give way to short rows: a row
// of at most `chunk` entries that straddles a boundary goes whole to the worker in whose chunk it
// starts, so that only rows longer than a chunk take atomic additions (eb_zero_kernel is told).
// ------------------------------------------------------------------------------------------
// Lane groups for which EB+SR can keep short rows whole (own_short): measured to pay for groups of
// 16 and 32 lanes (power-law N = 128 468 -> 460 us); for groups of 8 the extra bookkeeping costs
// registers and occupancy (power-law N = 32 144 -> 148 us), so those kernels are built without it.
template <int G> constexpr bool kOwnShortRows = G >= 16;

// Bound for 6 waves per SIMD: groups of 8 lanes with 16-byte vectors would take registers for 5 and spill 2 instead
// (4 with wide addresses); with 5 waves the power-law graph takes 113 us at N = 32 instead of 111, but rows of 1000
// entries 36.5 instead of 38.4.  No other instantiation spills.
template <int V, int G, int NV, bool WIDE, class END>
__global__ __launch_bounds__(kBlock, 6) void eb_sr_kernel(
    int m, int N, Strides sd, const int* __restrict__ rowptr, const int* __restrict__ colind,
    const float* __restrict__ vals, const float* __restrict__ B, float* __restrict__ C, int chunk,
    int pin_tiles, Schedule sch, int own_short, END after)
{
    constexpr int GPW = kWave / G;                        // workers per wave
    constexpr int SB = StageBatch<G>::value;
    constexpr int UL = G == 1 ? kU / NV : kU;             // entries whose gathers are issued together
    __shared__ int2 stage[G > 1 ? kWavesPerBlock * GPW * SB : 1];
    __shared__ float turns[V == 4 && G >= 4 ? kBlock * V : 1];
    typedef TileBias<END, G * V * NV> Bias;
    __shared__ float bias[Bias::kSize];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = lane / G, j = lane % G;
    const BlockMap bm = block_map(pin_tiles);
    const Cols<V, G, NV> cols(bm.tile, j, N);
    const int n0 = cols.n0, nvec = cols.nvec;
    const BRows<WIDE> brow(B, n0, sd);
    const int tile0 = bm.tile * G * V * NV;                // first column of the tile
    float* __restrict__ Ct = C + (long)tile0 * sd.cc;
    Bias::fill(bias, after, tile0, N);
    // a layer's row that this worker alone owns (sums without one keep to emit: through here, power-law graph, N = 32, 134 us for 131)
    auto put_row = [&](long row, Acc<V, G, NV> x) {
        if constexpr (END::layer) x.finish(after, bias + 4 + (n0 - tile0), cols);
        x.emit(Ct + row * sd.rc + (long)(n0 - tile0) * sd.cc, cols, false, sd.cc);
    };
    float* turn = turns + (V == 4 && G >= 4 ? (wave * GPW + g) * G * V : 0);
    const int nnz = rowptr[m];
    int2* st = stage + (G > 1 ? (wave * GPW + g) * SB : 0);

    const long nunits = ((unsigned)nnz + (unsigned)chunk - 1u) / (unsigned)chunk;   // nnz < 2^31
    const bool scheduled = sch.order != nullptr && sch.nnz == nnz && sch.units == nunits;
    const bool striped = scheduled && sch.stripe > 0;
    constexpr long WPB = kWavesPerBlock * GPW;            // workers per block
    const long nvb = striped ? sch.vblocks : (nunits + WPB - 1) / WPB;   // block positions to walk
    for (long vb = bm.bx; vb < nvb; vb += bm.nbx) {
        const long sb = striped ? sweep_block(vb, sch) : vb;
        const long u = sb * WPB + wave * GPW + g;
        if (sb < 0 || u >= nunits) continue;
        const long cid = scheduled ? (long)sch.order[u] : u;
        const long c0l = cid * chunk;
        const int c0 = (int)c0l;
        const int c1 = (int)min(c0l + chunk, (long)nnz);
        // the chunk's first row: from the plan's hint when it holds (one round trip), else by the
        // group's search (log_{G+1} m dependent loads)
        int row_start = 0, row_end = 0;
        int row = (scheduled && sch.first_row != nullptr) ? hinted_row(rowptr, m, sch.first_row[u], c0, &row_start, &row_end) : -1;
        if (row < 0) {
            row = row_of_entry_group<G>(rowptr, 0, m - 1, c0, j, g * G);
            row_start = rowptr[row];
            row_end = rowptr[row + 1];
        }
        BatchRegs<G, SB> next;
        // the first batch is fetched before the worker knows where exactly its entries begin and end
        if constexpr (G > 1) next.fetch(colind, vals, c0, (int)min(c0l + 2l * chunk, (long)nnz), j);
        // Rows of at most `chunk` entries are never split (own_short): the one that straddles the
        // chunk's end is finished by this worker, the one that straddles its start was finished by
        // the worker before.  Both workers read the same row pointers, so they agree; a worker then
        // owns the entries [lo, hi), between 0 and 2 * chunk - 1 of them, and only rows longer than a
        // chunk are combined with atomic additions.
        int lo = c0, hi = c1;
        if (kOwnShortRows<G> && own_short) {
            if (c1 < nnz) {
                int bs = 0, be = 0;
                int rb = (scheduled && sch.row_by_chunk != nullptr)
                             ? hinted_row(rowptr, m, sch.row_by_chunk[cid + 1], c1, &bs, &be) : -1;
                if (rb < 0) {
                    rb = row_of_entry_group<G>(rowptr, row, m - 1, c1, j, g * G);
                    bs = rowptr[rb];
                    be = rowptr[rb + 1];
                }
                if (bs < c1 && be - bs <= chunk) hi = be;
            }
            if (row_start < c0 && row_end - row_start <= chunk) {
                lo = row_end;
                if (lo < hi) {                                 // the next row with entries starts at lo
                    int walked = 0;
                    do { ++row; row_end = rowptr[row + 1]; } while (row_end <= lo && ++walked < 4);
                    if (row_end <= lo) {
                        row = row_of_entry_group<G>(rowptr, row + 1, m - 1, lo, j, g * G);
                        row_end = rowptr[row + 1];
                    }
                    row_start = lo;
                }
            }
        }
        if (lo >= hi) continue;
        bool shared_with_prev = row_start < lo;            // only the worker's first row can be
        Acc<V, G, NV> acc;
        acc.clear();

        int q0 = c0, skip = lo - c0;                       // entries of the first batch that are not ours
        if (skip >= SB) {                                  // the first batch holds none of ours: fetch again
            q0 = lo;
            skip = 0;
            if constexpr (G > 1) next.fetch(colind, vals, q0, hi, j);
        }
        for (; q0 < hi; q0 += SB, skip = 0) {
            if constexpr (G > 1) {
                next.put(st, j);
                wave_lds_sync();
                if (q0 + SB < hi) next.fetch(colind, vals, q0 + SB, hi, j);
            }
            for_blocks<UL>(skip, min(SB, hi - q0), [&](auto uc, int t) {
                constexpr int UU = decltype(uc)::value;
                int2 e[UU];
                Acc<V, G, NV> b[UU];
#pragma unroll
                for (int u = 0; u < UU; ++u) {
                    if constexpr (G > 1) e[u] = st[t + u];
                    else e[u] = make_int2(colind[q0 + t + u], __float_as_int(vals[q0 + t + u]));
                }
                if (nvec > 0) {
#pragma unroll
                    for (int u = 0; u < UU; ++u) b[u].load(brow.row(e[u].x), cols, sd.cb);
                }
                if (row_end > q0 + t + UU) {
                    // the common case: the whole block lies inside the current row
                    if (nvec > 0) {
#pragma unroll
                        for (int u = 0; u < UU; ++u) acc.fma(__int_as_float(e[u].y), b[u]);
                    }
                } else {
                    // All products first, so that every gather has been waited for before the
                    // first store or atomic is issued: stores share the in-order memory counter
                    // with loads, and a store issued between a gather and its use would make the
                    // wave wait for the store's acknowledgement.
                    if (nvec > 0) {
#pragma unroll
                        for (int u = 0; u < UU; ++u) b[u].scale(__int_as_float(e[u].y));
                    }
#pragma unroll
                    for (int u = 0; u < UU; ++u) {
                        if (nvec > 0) acc.add(b[u]);
                        const int next = q0 + t + u + 1;
                        if (next == row_end) {                 // the row is complete
                            if (shared_with_prev) add_row(Ct + (long)row * sd.rc, acc, cols, j, N - tile0, sd.cc, turn);
                            else if (nvec > 0) {
                                if constexpr (END::layer) put_row(row, acc);
                                else acc.emit(Ct + (long)row * sd.rc + (long)(n0 - tile0) * sd.cc, cols, false, sd.cc);
                            }
                            acc.clear();
                            shared_with_prev = false;
                            if (next < hi) {
                                // the next row with entries: usually row + 1; after a few rows
                                // without entries search instead of walking (a run of thousands
                                // of empty rows would otherwise cost a dependent load each)
                                int walked = 0;
                                do { ++row; row_end = rowptr[row + 1]; } while (row_end <= next && ++walked < 4);
                                if (row_end <= next) {
                                    row = row_of_entry_group<G>(rowptr, row + 1, m - 1, next, j, g * G);
                                    row_end = rowptr[row + 1];
                                }
                            }
                        }
                    }
                }
            });
            if constexpr (G > 1) wave_lds_sync();
        }
        if (row_end > hi)                                  // last row continues with the next worker
            add_row(Ct + (long)row * sd.rc, acc, cols, j, N - tile0, sd.cc, turn);
    }
}

// ------------------------------------------------------------------------------------------
// EB + PR : a wave owns `chunk` consecutive stored entries and takes them 64 at a time.  The
// lanes form S = 64/G slots (times G lanes along n); in one step slot s holds the product vector
// of one entry together with that entry's row index.
//
// A step whose entries all belong to one row needs no cross-lane traffic: every slot adds its
// product to its own partial sum of the current row (as the RB+PR kernel does); the slots are
// combined only when the row ends.  A step that contains a row boundary is combined with the
// CONDITIONAL REDUCTION of Sec. 4 (Fig. 6(e)): a log-step network in which slot s adds the value
// of slot s+d only if both belong to the same row.  Because entries are stored row after row,
// afterwards the leftmost slot of every run of equal row indices holds the sum of the run (the
// validity rule of Sec. 4); whether slot s+d is in the same run is decided once, from a ballot of
// the run heads, instead of comparing shuffled row indices in every step of the network.  The run
// that starts the step is merged with the partial sums carried so far, runs that end inside the
// step are written by their leftmost slot, and the run that reaches the end of the step
// unfinished becomes the new set of per-slot partial sums.  Rows that are complete inside the
// chunk get one plain store; only the first and last row of a chunk, when shared with the
// neighbouring chunks, are combined with atomic adds.
// ------------------------------------------------------------------------------------------
template <int V, int G, int NV>
__device__ __forceinline__ Acc<V, G, NV> slots_allreduce(Acc<V, G, NV> x) {
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
        for (int v = 0; v < V; ++v) x.a[i][v] = slot_allreduce<G>(x.a[i][v]);
    return x;
}

// Inclusive prefix sum of v over the 64 lanes of a wave: log-step scan inside the rows of 16 lanes
// with DPP row shifts (zeros shifted in), then the totals of the rows below are added.
__device__ __forceinline__ int wave_inclusive_scan_dpp(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);    // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);    // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);    // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);    // row_shr:8
    const int t0 = __builtin_amdgcn_readlane(v, 15), t1 = __builtin_amdgcn_readlane(v, 31),
              t2 = __builtin_amdgcn_readlane(v, 47);
    const int row = (threadIdx.x >> 4) & 3;
    return v + (row >= 1 ? t0 : 0) + (row >= 2 ? t1 : 0) + (row >= 3 ? t2 : 0);
}

constexpr int kStagedChunk = 512;   // EB+PR: largest chunk whose row starts are staged in LDS

// Six waves per SIMD up to 80 registers: with 81 the kernel takes five, and rows shorter than a chunk a tenth longer.  Steps inside
// one row, without selects and with half of the additions in multiply-adds: A^T of a power-law graph, 4.5 M entries, N = 64 101 -> 96 us;
// rows of 200, N = 64 17.2 -> 15.7, N = 128 23.1 -> 21.0.
template <int V, int G, int NV, bool WIDE, class END>
__global__ __launch_bounds__(kBlock, V == 4 && G >= 4 ? 6 : 1) void eb_pr_kernel(
    int m, int N, Strides sd, const int* __restrict__ rowptr, const int* __restrict__ colind,
    const float* __restrict__ vals, const float* __restrict__ B, float* __restrict__ C, int chunk,
    int pin_tiles, Schedule sch, END after)
{
    constexpr int S = kWave / G;
    constexpr int UU = G < 4 ? G : 4;                     // steps whose gathers are issued together (8 measured slower)
    __shared__ int4 stage[G > 1 ? kBlock : 1];
    __shared__ int starts[kWavesPerBlock][kStagedChunk + 2];
    __shared__ float turns[V == 4 && G >= 4 ? kBlock * V : 1];
    typedef TileBias<END, G * V * NV> Bias;
    __shared__ float bias[Bias::kSize];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int s = lane / G, j = lane % G;
    const BlockMap bm = block_map(pin_tiles);
    const Cols<V, G, NV> cols(bm.tile, j, N);
    const int n0 = cols.n0, nvec = cols.nvec;
    const BRows<WIDE> brow(B, n0, sd);
    const int tile0 = bm.tile * G * V * NV;                // first column of the tile
    float* __restrict__ Ct = C + (long)tile0 * sd.cc;
    Bias::fill(bias, after, tile0, N);
    // a layer's row that this worker alone owns (sums without one keep to emit: through here, power-law graph, N = 32, 134 us for 131)
    auto put_row = [&](long row, Acc<V, G, NV> x) {
        if constexpr (END::layer) x.finish(after, bias + 4 + (n0 - tile0), cols);
        x.emit(Ct + row * sd.rc + (long)(n0 - tile0) * sd.cc, cols, false, sd.cc);
    };
    float* turn = turns + (V == 4 && G >= 4 ? (wave * kWave + s * G) * V : 0);
    const int nnz = rowptr[m];
    int4* st = stage + (G > 1 ? wave * kWave : 0);
    int* cnt = starts[wave];

    const long nunits = ((unsigned)nnz + (unsigned)chunk - 1u) / (unsigned)chunk;   // nnz < 2^31
    const bool scheduled = sch.order != nullptr && sch.nnz == nnz && sch.units == nunits;
    const bool striped = scheduled && sch.stripe > 0;
    const long nvb = striped ? sch.vblocks : (nunits + kWavesPerBlock - 1) / kWavesPerBlock;   // block positions to walk
    for (long vb = bm.bx; vb < nvb; vb += bm.nbx) {
        const long sb = striped ? sweep_block(vb, sch) : vb;
        const long u = sb * kWavesPerBlock + wave;
        if (sb < 0 || u >= nunits) continue;
        const long c0l = (scheduled ? (long)sch.order[u] : u) * chunk;
        const int c0 = (int)c0l;
        const int c1 = (int)min(c0l + chunk, (long)nnz);
        int hint_start, hint_end;
        int row_lo = (scheduled && sch.first_row != nullptr) ? hinted_row(rowptr, m, sch.first_row[u], c0, &hint_start, &hint_end) : -1;
        if (row_lo < 0) row_lo = row_of_entry_group<kWave>(rowptr, 0, m - 1, c0, lane, 0);
        const int row_hi = row_of_entry_group<kWave>(rowptr, row_lo, m - 1, c1 - 1, lane, 0);
        Acc<V, G, NV> acc;                                    // per-slot partial sums of row `cur`
        acc.clear();
        int cur = -1;                                      // row being accumulated (wave-uniform)
        bool cur_started = false;                          // its first entry lies in this chunk

        // The row of every entry ("row index calculation" of Sec. 3.2).  The rows after the first
        // that begin inside the chunk are counted per chunk position in LDS, one coalesced pass
        // over their row pointers; the row of the entry at position p is then the first row plus
        // the number of row starts at positions 1..p, a prefix sum over the wave, and an entry is
        // the first / last of its row when a row starts at its own / the next position.  cnt[0]
        // holds whether the first row starts with the chunk, cnt[c1 - c0] whether the last one ends
        // with it.  A row range too long to stage (runs of rows without entries) falls back to a
        // binary search per entry; a chunk inside one row needs none of this.
        const int len = c1 - c0;
        const bool single = row_hi == row_lo;                  // the chunk lies inside one row (wave-uniform)
        const bool staged = !single && chunk <= kStagedChunk && row_hi - row_lo <= 4 * kStagedChunk;
        const int single_start = single ? rowptr[row_lo] : 0, single_end = single ? rowptr[row_lo + 1] : 0;
        int row_base = 0, carried = 0;
        if (staged) {
            for (int i = lane; i <= len; i += kWave) cnt[i] = 0;
            wave_lds_sync();
            for (int r = row_lo + 1 + lane; r <= row_hi; r += kWave) atomicAdd(&cnt[rowptr[r] - c0], 1);
            const int first_here = rowptr[row_lo] == c0 ? 1 : 0;
            if (lane == 0) { cnt[0] = first_here; cnt[len] = rowptr[row_hi + 1] == c1 ? 1 : 0; }
            wave_lds_sync();
            row_base = row_lo - first_here;
        }
        auto lookup = [&](int q) {
            int4 e = make_int4(0, 0, -1, 0);
            if (single) {
                if (q < c1) {
                    e.x = colind[q];
                    e.y = __float_as_int(vals[q]);
                    e.z = row_lo;
                    e.w = (q == single_start ? 1 : 0) | (q + 1 == single_end ? 2 : 0);
                }
            } else if (staged) {
                const bool valid = q < c1;
                const int here = valid ? cnt[q - c0] : 0, next = valid ? cnt[q - c0 + 1] : 0;
                const int upto = wave_inclusive_scan_dpp(here);
                if (valid) {
                    e.x = colind[q];
                    e.y = __float_as_int(vals[q]);
                    e.z = row_base + carried + upto;
                    e.w = (here > 0 ? 1 : 0) | (next > 0 ? 2 : 0);
                }
                carried += __builtin_amdgcn_readlane(upto, kWave - 1);
            } else if (q < c1) {
                const int r = row_of_entry(rowptr, row_lo, row_hi, q);
                e.x = colind[q];
                e.y = __float_as_int(vals[q]);
                e.z = r;
                e.w = (q == rowptr[r] ? 1 : 0) | (q + 1 == rowptr[r + 1] ? 2 : 0);
            }
            return e;
        };
        for (int q0 = c0; q0 < c1; q0 += kWave) {
            const int4 mine = lookup(q0 + lane);
            if constexpr (G > 1) { st[lane] = mine; wave_lds_sync(); }
            const int cnt = min(kWave, c1 - q0);

            for (int tb = 0; tb * S < cnt; tb += UU) {
                int4 e[UU];
                Acc<V, G, NV> b[UU];
#pragma unroll
                for (int u = 0; u < UU; ++u) {
                    if constexpr (G > 1) e[u] = st[((tb + u) * S + s) & (kWave - 1)]; else e[u] = mine;
                }
                // branch-free gathers: slots past the end of the chunk hold column 0
                if (nvec > 0) {
#pragma unroll
                    for (int u = 0; u < UU; ++u) b[u].load(brow.row(e[u].x), cols, sd.cb);
                }
                // all steps in one row that does not end here: their products are added to each other first, so that
                // a slot's sum takes one addition for four entries and no step looks for row boundaries (N = 65, rows of
                // 400: error 2.3e-7 with an addition each, 1.3e-7 now, as with 8 slots; 296 -> 182 us).  Every slot holds an
                // entry then, and two of the products are multiply-adds.
                if constexpr (UU == 4) {
                    const int row0 = __builtin_amdgcn_readfirstlane(e[0].z);
                    if ((tb + UU) * S <= cnt && row0 == __builtin_amdgcn_readlane(e[UU - 1].z, (S - 1) * G) &&
                        (__builtin_amdgcn_readlane(e[UU - 1].w, (S - 1) * G) & 2) == 0) {
                        if (cur < 0) { cur = row0; cur_started = (__builtin_amdgcn_readfirstlane(e[0].w) & 1) != 0; }
                        b[0].scale(__int_as_float(e[0].y));
                        b[0].fma(__int_as_float(e[1].y), b[1]);
                        b[2].scale(__int_as_float(e[2].y));
                        b[2].fma(__int_as_float(e[3].y), b[3]);
                        b[0].add(b[2]);
                        acc.add(b[0]);
                        continue;
                    }
                }
                // all products first: no store or atomic is issued while a gather is outstanding
                // (stores share the in-order memory counter with loads)
#pragma unroll
                for (int u = 0; u < UU; ++u) {
                    if ((tb + u) * S + s >= cnt) e[u].z = -1;
                    const bool ok = e[u].z >= 0 && nvec > 0;
                    const float a = __int_as_float(e[u].y);
#pragma unroll
                    for (int i = 0; i < NV; ++i)
#pragma unroll
                        for (int v = 0; v < V; ++v) b[u].a[i][v] = ok ? a * b[u].a[i][v] : 0.f;
                }
#pragma unroll
                for (int u = 0; u < UU; ++u) {
                    const int t0 = (tb + u) * S;                       // first entry of this step
                    if (t0 >= cnt) break;                              // wave-uniform
                    const int er = e[u].z;
                    const bool evalid = er >= 0;
                    const int nv = min(S, cnt - t0);                   // valid slots in this step
                    const int first_row = __builtin_amdgcn_readfirstlane(er);
                    const int first_flags = __builtin_amdgcn_readfirstlane(e[u].w);
                    const int last_row = __builtin_amdgcn_readlane(er, (nv - 1) * G);
                    const int last_flags = __builtin_amdgcn_readlane(e[u].w, (nv - 1) * G);

                    if (first_row == last_row) {
                        // one row in the whole step: no cross-lane work
                        if (cur < 0) { cur = first_row; cur_started = (first_flags & 1) != 0; }
                        acc.add(b[u]);
                        if (last_flags & 2) {                           // the row ends here
                            const Acc<V, G, NV> total = slots_allreduce<V, G, NV>(acc);
                            if (s == 0) {
                                if (!cur_started) add_row(Ct + (long)cur * sd.rc, total, cols, j, N - tile0, sd.cc, turn);
                                else if (nvec > 0) {
                                    if constexpr (END::layer) put_row(cur, total);
                                    else total.emit(Ct + (long)cur * sd.rc + (long)(n0 - tile0) * sd.cc, cols, false, sd.cc);
                                }
                            }
                            acc.clear();
                            cur = -1;
                        }
                    } else {
                        // a row boundary inside the step: conditional reduction
                        const Acc<V, G, NV> p = b[u];                      // this slot's product
                        Acc<V, G, NV> x = p;
                        // run heads: a slot whose entry is the first of its row (entries are stored
                        // row after row, so its left neighbour then holds another row); the first
                        // slot past the valid ones counts as a head so that the last run ends there
                        const bool head = s <= nv && (s == 0 || s == nv || (e[u].w & 1) != 0);
                        const unsigned long long heads = __ballot(head);
                        // slots from s to the end of its run
                        int dist = S - 1 - s;
                        if (s < S - 1) {
                            const unsigned long long above = heads >> ((s + 1) * G);
                            if (above) dist = (__ffsll((long long)above) - 1) / G;
                        }
#pragma unroll
                        for (int i = 0; i < NV; ++i)
#pragma unroll
                            for (int v = 0; v < V; ++v) conditional_steps<G, 1>(x.a[i][v], dist);
                        // the run that starts the step continues the row accumulated so far
                        bool started = true;                            // runs that begin inside the step
                        if (cur >= 0) {
                            const Acc<V, G, NV> total = slots_allreduce<V, G, NV>(acc);
                            if (s == 0) { x.add(total); started = cur_started; }
                        } else if (s == 0) {
                            started = (first_flags & 1) != 0;
                        }
                        const bool last_ended = (last_flags & 2) != 0;
                        const bool in_last_run = evalid && er == last_row;
                        if (head && evalid && (!in_last_run || last_ended)) {
                            if (!started) add_row(Ct + (long)er * sd.rc, x, cols, j, N - tile0, sd.cc, turn);
                            else if (nvec > 0) {
                                if constexpr (END::layer) put_row(er, x);
                                else x.emit(Ct + (long)er * sd.rc + (long)(n0 - tile0) * sd.cc, cols, false, sd.cc);
                            }
                        }
                        if (last_ended) {
                            acc.clear();
                            cur = -1;
                        } else {                                        // unfinished run -> new partial sums
#pragma unroll
                            for (int i = 0; i < NV; ++i)
#pragma unroll
                                for (int v = 0; v < V; ++v) acc.a[i][v] = in_last_run ? p.a[i][v] : 0.f;
                            cur = last_row;
                            cur_started = true;
                        }
                    }
                }
            }
            if constexpr (G > 1) wave_lds_sync();
        }
        if (cur >= 0) {                                       // row continues in the next chunk
            const Acc<V, G, NV> total = slots_allreduce<V, G, NV>(acc);
            if (s == 0) add_row(Ct + (long)cur * sd.rc, total, cols, j, N - tile0, sd.cc, turn);
        }
    }
}

// ------------------------------------------------------------------------------------------
// Input characteristics (Sec. 5.1, Table 2): sum of squared row lengths and the longest row,
// reduced exactly in integers.  The block that finishes last writes them and nnz straight into pinned
// host memory, followed by `ticket`, and leaves the device scratch (sum, longest, finished blocks) zero
// for the next call: no allocation, clearing or copy around the kernel.
// ------------------------------------------------------------------------------------------
struct FeatureScratch { unsigned long long sq, mx, done; };
struct FeatureResult { unsigned long long sq, mx, nnz, ticket; };

__global__ __launch_bounds__(kBlock) void features_kernel(
    int m, const int* __restrict__ rowptr, FeatureScratch* __restrict__ scratch, FeatureResult* __restrict__ result,
    unsigned long long ticket)
{
    constexpr int U = 8;
    __shared__ unsigned long long s_sq[kWavesPerBlock];
    __shared__ unsigned long long s_mx[kWavesPerBlock];
    unsigned long long sq = 0, mx = 0;
    const long stride = (long)gridDim.x * kBlock;
    for (long i = (long)blockIdx.x * kBlock + threadIdx.x; i < m; i += U * stride) {
        int a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {                     // all loads in flight together
            const long r = i + u * stride < m ? i + u * stride : m - 1;
            a[u] = rowptr[r];
            b[u] = rowptr[r + 1];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned long long len = i + u * stride < m ? (unsigned long long)(b[u] - a[u]) : 0ull;
            sq += len * len;
            mx = len > mx ? len : mx;
        }
    }
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1) {
        sq += __shfl_down(sq, d, kWave);
        const unsigned long long o = __shfl_down(mx, d, kWave);
        mx = o > mx ? o : mx;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) { s_sq[wave] = sq; s_mx[wave] = mx; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kWavesPerBlock; ++w) { sq += s_sq[w]; mx = s_mx[w] > mx ? s_mx[w] : mx; }
        if (gridDim.x > 1) {
            atomicAdd(&scratch->sq, sq);
            atomicMax(&scratch->mx, mx);
            __threadfence();
            if (atomicAdd(&scratch->done, 1ull) != gridDim.x - 1) return;
            __threadfence();
            sq = atomicExch(&scratch->sq, 0ull);
            mx = atomicExch(&scratch->mx, 0ull);
            atomicExch(&scratch->done, 0ull);
        }
        result->sq = sq;
        result->mx = mx;
        result->nnz = (unsigned long long)rowptr[m];
        __threadfence_system();
        __hip_atomic_store(&result->ticket, ticket, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// ------------------------------------------------------------------------------------------
// Well-formedness checks of the CSR arrays (debug aid).  flags[0] collects violation bits,
// flags[1] receives rowptr[m].  The column check must only run after the row-pointer check
// passed: it trusts rowptr[m] as the number of stored entries.
// ------------------------------------------------------------------------------------------
enum : unsigned { kBadFirst = 1u, kBadOrder = 2u, kBadColumn = 4u };

__global__ __launch_bounds__(kBlock) void validate_rowptr_kernel(int m, const int* __restrict__ rowptr,
                                                                 unsigned* __restrict__ flags)
{
    unsigned bad = 0;
    for (long i = (long)blockIdx.x * kBlock + threadIdx.x; i < m; i += (long)gridDim.x * kBlock)
        if (rowptr[i + 1] < rowptr[i]) bad |= kBadOrder;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (rowptr[0] != 0) bad |= kBadFirst;
        flags[1] = (unsigned)rowptr[m];
    }
    if (bad) atomicOr(flags, bad);
}

__global__ __launch_bounds__(kBlock) void validate_colind_kernel(int nnz, int k, const int* __restrict__ colind,
                                                                 unsigned* __restrict__ flags)
{
    unsigned bad = 0;
    for (long p = (long)blockIdx.x * kBlock + threadIdx.x; p < nnz; p += (long)gridDim.x * kBlock) {
        const int c = colind[p];
        if (c < 0 || c >= k) bad |= kBadColumn;
    }
    if (bad) atomicOr(flags, bad);
}

}  // namespace daspmm
