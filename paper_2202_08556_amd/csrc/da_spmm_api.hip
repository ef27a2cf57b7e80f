// Host side of libdaspmm.so: argument checks, choice of launch geometry, dispatch of the
// algorithm id to a kernel instantiation, the feature-extraction helper and the selector.
// The C ABI is declared and documented in include/da_spmm.h.
#include "da_spmm.h"
#include "da_spmm_kernels.hip"
#include "da_transpose_kernels.hip"
#include "da_dense_kernels.hip"
#include "da_heavy_kernels.hip"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <vector>

namespace {

using namespace daspmm;

thread_local char g_err[256] = "";

int fail(int code, const char* fmt, const char* a = "") {
    std::snprintf(g_err, sizeof g_err, fmt, a);
    return code;
}

int hip_fail(hipError_t e, const char* where) {
    std::snprintf(g_err, sizeof g_err, "%s: %s", where, hipGetErrorString(e));
    return DA_ERR_HIP;
}

// number of compute units of the current device (cached per device ordinal)
int cu_count() {
    static std::atomic<int> cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int c = cached[dev].load(std::memory_order_relaxed);
    if (c == 0) {
        if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || c <= 0)
            c = 256;
        cached[dev].store(c, std::memory_order_relaxed);
    }
    return c;
}

int pow2_ceil(long x) {
    int p = 1;
    while (p < x) p <<= 1;
    return p;
}

struct Problem {
    int m, N;
    Strides sd;
    const int* rowptr;
    const int* colind;
    const float* vals;
    const float* B;
    float* C;
    hipStream_t stream;
    int64_t k;
    LeftOut left_out;    // RB_SR: rows that heavy_rows_kernel sums
    LayerSums* layer;    // what C takes besides the sums; null: nothing
    bool* finished;      // set when the product's kernels have done that
};

enum Family { RB_SR, RB_PR, EB_SR, EB_PR };

// Launch geometry of one call: lane mapping (V, G, NV as in da_spmm_kernels.hip) and, for EB,
// the number of stored entries per worker.
struct Geometry {
    int V, G, NV, chunk;
    int pin;    // pin column tiles to XCDs when the tile count is 2, 4 or 8: 1 yes, 0 no, -1 as launch_w finds it best
    int stripe; // blocks per stripe when a prepared matrix's chunk order is dealt to the XCDs (0: off)
    bool order; // take a prepared matrix's chunk order
};

constexpr int kSweepStripe = 256;

constexpr int kMaxGridY = 65535;
constexpr int64_t kMaxGridX = (1LL << 32) / kBlock - 1;   // blocks; of 2^32 threads and more the high bits are lost
constexpr int kMaxGroupPR = 32;        // PR needs at least two slots along the entries
constexpr int kDefaultGroupPR = 8;     // 4-byte accesses: at least 8 slots along the entries
constexpr int kEntriesPerWavePR = 512; // EB+PR: stored entries per wave and pass

int env_int(const char* name, int fallback) {
    const char* v = std::getenv(name);
    return (v && *v) ? std::atoi(v) : fallback;
}

bool is_pow2(int x) { return x > 0 && (x & (x - 1)) == 0; }

// What is known of matrices whose features were extracted or that were prepared, keyed by (rowptr address,
// m): nnz, and the length of the row that an average entry lies in (sum of squared row lengths over nnz;
// 0 = unknown).  da_spmm uses both only for the launch geometry; the EB kernels stride over all chunks
// whatever the grid size, so a stale or missing hint costs speed, never correctness.
struct MatrixHint { const void* rowptr; int64_t m; int64_t nnz; double seen_len; };
std::mutex g_hint_mu;
MatrixHint g_hints[16];
int g_hint_next = 0;

void remember_matrix(const void* rowptr, int64_t m, int64_t nnz, double seen_len) {
    std::lock_guard<std::mutex> lk(g_hint_mu);
    for (auto& h : g_hints)
        if (h.rowptr == rowptr && h.m == m) { h.nnz = nnz; h.seen_len = seen_len; return; }
    g_hints[g_hint_next] = MatrixHint{rowptr, m, nnz, seen_len};
    g_hint_next = (g_hint_next + 1) % 16;
}

MatrixHint lookup_matrix(const void* rowptr, int64_t m) {
    std::lock_guard<std::mutex> lk(g_hint_mu);
    for (const auto& h : g_hints)
        if (h.rowptr == rowptr && h.m == m) return h;
    return MatrixHint{nullptr, 0, -1, 0.0};
}

// Chunk schedules of matrices prepared with da_spmm_prepare, keyed like the nnz hints.  The
// orders live in one library-owned device allocation per matrix, held through a reference count:
// a product call copies the reference under the mutex, launches outside it and drops the reference
// after the launch, so that a concurrent release / re-prepare / eviction can free the memory only
// once no call is between its lookup and its launch (hipFree itself waits for launched kernels).
constexpr int kPlans = 5;
constexpr int kPlanUnits[kPlans] = {32, 64, 128, 256, 512};     // plan_info reads number 3, 256
constexpr int64_t kSmallPlanMaxNnz = 4 << 20;   // beyond, launches never take the smallest chunks: no order for them
struct DeviceBlock {
    void* p = nullptr;
    ~DeviceBlock() { if (p) (void)hipFree(p); if (pinned) (void)hipHostFree(pinned); }
    int* pinned = nullptr;
};
struct Plan {
    const void* rowptr = nullptr;
    const void* colind = nullptr;
    int64_t m = 0, nnz = 0;
    int* order[kPlans] = {};
    int* first_row[kPlans] = {};   // per schedule position: row of the chunk's first entry (hint)
    int* row_by_chunk[kPlans] = {}; // the same rows indexed by chunk number
    int units[kPlans] = {};
    int first_units[kPlans] = {};   // chunks of the first schedule segment (multi-row chunks)
    std::shared_ptr<DeviceBlock> block;
    HeavyPlan heavy{};                   // count > 0: rows that heavy_rows_kernel takes from EB+RM+SR
    int64_t heavy_k = 0;                 // columns that the cells of `heavy` cover
    const unsigned* heavy_bits = nullptr;
    double rest_len = 0.0;               // length of the row that an average entry of the other rows lies in
    int rest_longest = 0;                // the longest of them
    std::shared_ptr<const std::vector<int64_t>> heavy_sums;   // entries of the first 0, 1, ... heavy rows by length
    std::shared_ptr<DeviceBlock> heavy_block;
    bool captured = false;               // a stream capture recorded a kernel that reads the orders
};
std::mutex g_plan_mu;
Plan g_plans[16];
int g_plan_next = 0;

// What the launch geometry wants to know of a matrix's plan: whether there is one, and the share of the
// entries that lie in chunks of 256 inside one row (rows much longer than a chunk).
struct PlanInfo { bool found; double long_rows; };

PlanInfo plan_info(const void* rowptr, const void* colind, int64_t m) {
    std::lock_guard<std::mutex> lk(g_plan_mu);
    for (const auto& pl : g_plans)
        if (pl.block && pl.rowptr == rowptr && pl.colind == colind && pl.m == m)
            return PlanInfo{true, 1.0 - (double)pl.first_units[3] / (double)pl.units[3]};
    return PlanInfo{false, 0.0};
}

// Schedule of a prepared matrix for this chunk size; split holds the CHUNKS of the first segment
// here, the launch turns it into blocks.  *keep receives a reference to the plan's memory, to be
// held until the kernel that reads the order has been launched.  capturing: the launch is being
// recorded into a HIP graph, which will read the order on every replay: such a plan is never
// evicted or replaced behind the caller's back, only da_spmm_release frees it.
Schedule lookup_schedule(const void* rowptr, const void* colind, int64_t m, int chunk, bool capturing,
                         std::shared_ptr<DeviceBlock>* keep) {
    std::lock_guard<std::mutex> lk(g_plan_mu);
    for (auto& pl : g_plans)
        if (pl.block && pl.rowptr == rowptr && pl.colind == colind && pl.m == m)
            for (int i = 0; i < kPlans; ++i)
                if (kPlanUnits[i] == chunk && pl.order[i]) {
                    *keep = pl.block;
                    if (capturing) pl.captured = true;
                    return Schedule{pl.order[i], pl.units[i], (int)pl.nnz, 0, pl.first_units[i], 0, 0, 0, 3, pl.first_row[i], pl.row_by_chunk[i]};
                }
    return Schedule{nullptr, 0, 0, 0, 0, 0, 0, 0, 3, nullptr, nullptr};
}

bool is_capturing(hipStream_t s) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cap) != hipSuccess) { (void)hipGetLastError(); cap = hipStreamCaptureStatusNone; }
    return cap == hipStreamCaptureStatusActive;
}

// The heavy rows of a prepared matrix; references and captures as for lookup_schedule.  The kernel reads every row of B
// that the cells cover, used or not: products that declare other columns than da_spmm_prepare did go without, and so do
// those after one that found the list to be of another matrix.
struct HeavyLookup {
    HeavyPlan plan{};
    const unsigned* bits = nullptr;
    double rest_len = 0.0;
    int rest_longest = 0;
    std::shared_ptr<const std::vector<int64_t>> sums;
    std::shared_ptr<DeviceBlock> keep;
};
HeavyLookup lookup_heavy(const void* rowptr, const void* colind, int64_t m, int64_t k, hipStream_t stream) {
    HeavyLookup out;
    std::lock_guard<std::mutex> lk(g_plan_mu);
    for (auto& pl : g_plans)
        if (pl.block && pl.rowptr == rowptr && pl.colind == colind && pl.m == m && pl.heavy.count > 0 && pl.heavy_k == k &&
            __atomic_load_n(pl.heavy.stale, __ATOMIC_RELAXED) == 0) {
            out.plan = pl.heavy;
            out.bits = pl.heavy_bits;
            out.rest_len = pl.rest_len;
            out.rest_longest = pl.rest_longest;
            out.sums = pl.heavy_sums;
            out.keep = pl.heavy_block;
            if (is_capturing(stream)) pl.captured = true;
            break;
        }
    return out;
}

// SR from 17 columns, where rows of B and C are not whole 16-byte pieces: whether a wave is better off with 8, 4 or 2
// workers of 16-byte lanes than with 2 or 1 of one column per lane.
// RB: a wave waits for its longest row.  Where rows are short and of one length the loads decide (27-point
// stencil, N = 24: 19 us against 27; 12 entries a row, N = 17: 20 and 25; 15 +- 7: 21 and 23), beyond that the
// waiting does (25 +- 12: 24 and 23; 40 +- 20: 36 and 31; lognormal rows of 23, coefficient 1.3: 61 and 47;
// power-law: 198 and 131), at any width up to 63 (power-law N = 63: 202 and 167).  Above 64 columns one column per
// lane takes a second pass over the row (N = 65, lognormal: 92 and 108), which pays only where one row of very many
// entries sets the time (N = 65, rows of 1000: 118 and 99; power-law A^T: 974 and 797).
// EB: without a plan a chunk begins with a search that a wave's workers make one after another (power-law
// N = 24: 202 and 186; skewed: 887 and 835), which some million entries in rows of some hundred pay back with smaller
// chunks (4.5 M in rows of 616, N = 24: 72 and 80; 3.6 M of 914: 65 and 74; 2 M of 1090, N = 50: 41 and 47).  With
// one the loads decide (power-law N = 24: 145 and 161, N = 41: 210 and 242), unless the matrix has too few entries for that many workers (105 000: 19 and 13), or so many in
// long rows that the workers end their chunks with additions to the same lines (A^T of a power-law graph with 1.2 M
// entries, N = 17: 44 and 31) -- which 12 waves per SIMD hide (33 M entries in rows of 60 000, N = 24: 316 and
// 354; 13 M: 152 and 134).  From 25 columns the one-column lanes are nearly all in use, and rows of B that
// begin anywhere cost 16-byte lanes more lines (power-law A^T with 4.5 M entries, N = 31: 100 and 72).
bool wide_lanes_pay(bool eb, int64_t N, const MatrixHint& hint, const PlanInfo& plan) {
    if (N > 64) return eb || hint.seen_len < 800.0;
    if (!eb) return hint.seen_len > 0.0 && hint.seen_len < 28.0;
    if (hint.nnz < 0 || (N >= 25 && N <= 32)) return false;
    if (!plan.found) return hint.nnz >= 1500000 && hint.nnz <= 6000000 && hint.seen_len >= 200.0 && hint.seen_len <= 1500.0;
    const int64_t waves = hint.nnz / 256 / (N <= 32 ? 8 : 4);
    return waves >= (int64_t)cu_count() * 4 * 12 || (hint.nnz >= 600000 && hint.seen_len >= 16.0 && hint.seen_len <= 1500.0);
}

// Entries of a matrix that are many and lie in rows of uneven length: tiles on XCDs of their own wait for each other.
bool uneven_rows(int64_t m, const MatrixHint& hint) { return hint.nnz >= 2000000 && hint.seen_len * (double)m > 1.5 * (double)hint.nnz; }

// RB tiles of tile_cols columns on XCDs of their own, see launch_w.
bool slices_fit_l2(int64_t k, int64_t N, int64_t tile_cols) { return k * tile_cols * 4 <= 12 << 20 && k * N * 4 > 9 << 19; }

// RB+PR with whole 128-byte pieces of B: whether tiles of 32 columns beat tiles of 64.  They give a row 8 slots instead of 4, and an L2
// slices of B half as wide, but a row of A twice the waves.  Measured over 1300 products, tiles of 64 and of 32 as they run now, in us;
// (23, 61) are lognormal rows of 23 with coefficient 1.3, in which an average entry sees 61; so (28, 62), (50, 90), (90, 180).
// - Rows of n entries and more columns than 1.25 M / n: the slices decide, however many rows there are.  60 000 rows, N = 64: (23, 61),
//   k = 26 000 41.7 and 43.3, 80 000 56.4 -> 49.1; (50, 90), 18 000 51.6 and 50.9, 26 000 63.7 -> 52.3, 40 000 83.5 -> 58.4; rows of 60, 18 000
//   46.2 and 51.4, 26 000 61.5 -> 51.8.  120 000 rows, N = 128: (50, 90), 26 000 206 -> 185.  They end where slices of 32 columns do not
//   fit either: rows of 45, N = 64, k = 150 000 228 -> 208, 210 000 313 -> 304, 260 000 314 and 318; N = 96, whose second tile of 64 is half empty,
//   150 000 330 -> 326, 180 000 403 and 415.
// - Fewer columns: only while a few rows per wave of the chip are left, whose longest sets the time, and rows are uneven.  k = 14 000, N = 64: (23,
//   61), 10 000 rows 17.3 -> 9.7, 28 000 21.3 and 22.5, 100 000 47.1 and 61.2; (90, 180), 40 000 rows 58.4 -> 55.1, 100 000 112 and 117; N = 96, (28, 62),
//   28 000 rows 30.4 and 30.5, (90, 180), 100 000 186 and 166.  More columns, more rows: (35, 98), k = 31 000, 31 000 rows, N = 64 49.0 -> 32.9.
// - Not while tiles of 64 have XCDs of their own and slices of up to 6 MB (rows of 45, k = 22 000, N = 128 34.2 and 36.1; 11 000, N = 256 27.7
//   and 34.5), and not where rows are very uneven: most are then short or empty (20 000 rows of 180 among a million: N = 64 168 and 316), and in
//   graphs popular columns go with that (power-law, N = 64: 104 and 115, N = 128 175 and 205).
bool narrow_tiles_pay(int64_t m, int64_t k, int64_t N, const MatrixHint& hint) {
    if (N % 32 != 0 || N > 32L * kMaxGridY || hint.nnz <= 0 || hint.seen_len < 55.0) return false;   // tiles of 64 reach twice as far
    const double mean = (double)hint.nnz / (double)m, unevenness = hint.seen_len / mean;
    if (unevenness > 3.0 || k * 128 > (N % 64 == 0 ? 28 << 20 : 20 << 20)) return false;
    if ((N == 128 || N == 256 || N == 512) && slices_fit_l2(k, N, 64) && !uneven_rows(m, hint) && k * 256 <= 6 << 20) return false;
    if (k * 256 > 4 << 20 && (double)k * mean > 1.25e6) return true;
    const double most = 1.3e6 * std::max(1.0, hint.seen_len / 60.0) * (N % 64 == 0 ? 1.0 : 2.0) * std::max(1.0, (double)k / 16384.0);
    return unevenness >= 1.4 && (double)m * (double)N <= most;
}

// Rounding error of a row of n entries that is summed in chunks of c entries, relative to n: every chunk is summed
// one entry after another by each of `chains` partial sums, and the chunks are added one after another.  For
// products of random sign the errors of a sum of c terms grow with c, for products of one sign with c^2.
double random_error(double c, double chains, double n) { return c / chains + n / c; }
double one_sign_error(double c, double chains, double n) { return c * c / (chains * chains) + n * n / c; }

// Stored entries per worker of the EB ids.
//
// Without a plan: 256 entries for SR lane groups of 16 or more and fewer for narrow ones, whose search costs more per
// entry; 512 for the waves of PR.  Small matrices: shrunk until there are about four waves of workers per SIMD, so
// that the chunk walk, a chain of dependent memory round trips, does not set the run time.  PR, and SR above 64
// columns, count the lanes of one column there where rows of B are not whole 16-byte pieces.
//
// With a plan a chunk is cheap to begin (row hints) and with coalesced atomic additions cheap to end, and the orders
// exist for powers of two only.  SR: 64 entries keep the workers closer together in the sweep over B (power-law
// N = 128: 449 us at 256, 399 at 64; rows of 175 entries, N = 64: 350 and 167), 32 where 64 leaves too few workers
// (1.2 M entries in rows of 40, N = 64: 37 and 29), 128 up to 64 columns where more than a fifth of the entries are
// in rows much longer than a chunk, whose chunks all add to the same few lines of C, and 128 still makes 12 waves
// per SIMD (power-law, 13 M entries, N = 24: 145 at 64, 141 at 128; N = 32: 118 and 110; N = 64: 205 and 198; with
// 4.5 M entries, N = 24: 59 and 67).  One column per lane in groups of 16 and more: 128, 256 on rows of more than
// 16 000 entries, 64 up to 4 M entries, and not more than the size without a plan (power-law N = 16: 120 at 64, 111
// at 128; rows of 30 000, N = 41: 120 at 256, 130 at 128; 1.4 M entries, N = 16: 32 us at 32, 28 at 64, 29 at 88).
// PR: the size without a plan, rounded down (0.64 M entries, N = 32: 34 us at 64, 30 at 128; 1.9 M in rows of 16 000,
// N = 32: 39 at 256, 65 at 512).
//
// Smaller chunks split a row into more parts.  Rows of up to some thousand entries lose nothing by that, a chunk
// of 256 being the longer sum; the error of longer ones grows with the number of chunks (1.9 M entries in rows of
// 16 000, N = 17: 3.0e-7 of the result at 232, 4.2e-7 at 64).  So the size is doubled while the row length that
// an average entry sees makes the error for random signs larger than at the size without a plan (a twentieth of it is
// less than the order of the atomic additions changes from run to run), or that for one sign by more than 1.4.
int chunk_size(bool cm, bool pr, int64_t N, bool whole, const Geometry& g, const MatrixHint& hint, const PlanInfo& plan) {
    const int64_t cols = whole ? (N + 3) / 4 : N;
    const int lanes = cm ? 1 : (!plan.found && !pr && N < 64 ? g.G : std::min(pow2_ceil(cols), whole ? 32 : (pr ? kDefaultGroupPR : kWave)));
    const int most = pr ? kEntriesPerWavePR : (lanes >= 16 ? 256 : (lanes == 8 ? (plan.found ? 128 : 256) : (lanes == 4 ? 128 : 64)));
    if (hint.nnz < 0) return most;
    const int least = pr ? 64 : (lanes >= 8 ? 32 : most);
    const int64_t workers = (int64_t)cu_count() * 16 * (pr ? 1 : kWave / lanes);
    const int64_t spread = (hint.nnz / workers + 7) / 8 * 8;
    const int plain = (int)std::min<int64_t>(most, std::max<int64_t>(least, spread));
    if (!plan.found || (!pr && (cm || lanes < 8))) return plain;

    int near = 32;                                                    // plain rounded down to a power of two
    while (near * 2 <= plain) near *= 2;
    int c;
    if (pr) c = std::min(kEntriesPerWavePR, std::max(64, near));
    else if (g.V == 1 && g.G >= 16) c = std::min(hint.nnz <= kSmallPlanMaxNnz ? 64 : (hint.seen_len <= 16384.0 ? 128 : 256), near);
    else if (hint.nnz > kSmallPlanMaxNnz)
        c = g.V == 4 && N <= 64 && plan.long_rows > 0.2 && hint.nnz / 128 / (kWave / g.G) >= (int64_t)cu_count() * 4 * 12 ? 128 : 64;
    else c = hint.nnz / 64 < (g.G == 8 ? 48 : 28) * 1024 ? 32 : 64;
    // partial sums of a chunk, now and in lanes of one column; PR adds its products four at a time in groups of 4 and more
    const double n = hint.seen_len, ours = pr ? (g.G >= 4 ? 4.0 : 1.0) * (kWave / g.G) : 1.0, theirs = pr ? (double)(kWave / lanes) : 1.0;
    while (c < plain && (random_error(c, ours, n) > 1.12 * random_error(plain, theirs, n) ||
                         one_sign_error(c, ours, n) > 2.0 * one_sign_error(plain, theirs, n)))
        c *= 2;
    return c;
}

// Default geometry per algorithm family and N.  Measured on MI355X: 16-byte and 4-byte gathers run at
// full rate, 8-byte gathers at about half.  SR narrows to one column per lane for N <= 16: lane groups of
// 4 lanes or fewer walk 16 or more rows or chunks per wave and wait for the longest (power-law N = 8,
// EB+RM+SR: 110 us with 8 lanes of one column, 176 with 2 lanes of 4).  PR has no such spread, its slots
// share a row: there 16-byte gathers win or tie at any width (power-law N = 16, RB+RM+PR: 159 us against 265; at N = 4,
// where a lane then takes an entry of its own like in CM: RB+RM+PR on rows of 175 entries 51 and 51, EB+RM+PR on 12
// entries a row 25 and 29, on lognormal rows 26 and 27).
// Between (17 ... 31 columns, and up to 63 where rows of B are not whole 16-byte pieces) 16-byte gathers
// issue fewer loads but put 8 or 4 workers on a wave instead of 2 or 1, see wide_lanes_pay.
// Setting DA_SPMM_TUNE=1 lets DA_SPMM_V / _G / _NV / _CHUNK override the choice (for tuning runs only;
// invalid combinations are rejected).
//
// Small matrices of mostly empty rows do without their plan up to 32 columns: the stored rows are short and far
// apart, few rows of B are read twice, and chunks in the order of their columns scatter the additions to neighbouring rows of
// C over the XCDs.  SR from 5 columns: fewer than 3 entries a row (0.64 M entries, 1.6 a row, N = 8: 33 us with the plan, 27 without;
// 0.4 M, 0.4 a row, N = 24: 86 and 60; N = 64: 48 and 52; 0.2 M, 6.7 a row, N = 8: 18 and 20).  PR: fewer than 8 where
// the size without a plan is none of the plan's (0.64 M, 1.6 a row, N = 16, EB+CM+PR: 39 and 34; 2 M, 6.7 a row,
// N = 4: 30 and 25; 0.2 M, 6.7 a row, N = 8, with chunks of 64 either way: 14 and 16).
int pick_geometry(bool cm, bool pr, bool eb, int64_t m, int64_t k, int64_t N, const Strides& sd, bool aligned,
                  const MatrixHint& hint, PlanInfo plan, Geometry* out) {
    const bool vec4_ok = N >= 4 && sd.cb == 1 && sd.cc == 1;      // 16-byte accesses, at any alignment
    Geometry g{1, 1, 1, 0, -1, kSweepStripe, true};
    if (plan.found && N <= 32 && hint.nnz >= 0) {
        const int64_t waves = (int64_t)cu_count() * 16;
        const bool bare = pr ? hint.nnz < 8 * m && hint.nnz > 64 * waves && hint.nnz < kEntriesPerWavePR * waves
                             : !cm && N > 4 && hint.nnz < 3 * m && hint.nnz <= kSmallPlanMaxNnz;
        if (bare) { plan.found = false; g.order = false; }
    }
    if (cm) {
        g.V = vec4_ok ? 4 : 1;
        const long vecs = (N + g.V - 1) / g.V;
        g.NV = vecs >= 4 ? 4 : pow2_ceil(vecs);
        g.G = 1;
    } else {
        const bool whole = aligned && N >= 32 && N % 4 == 0;
        g.V = (vec4_ok && (pr || whole || (N > 16 && wide_lanes_pay(eb, N, hint, plan)))) ? 4 : 1;
        g.G = pow2_ceil((N + g.V - 1) / g.V);
        // SR: at most 128 columns per tile (32 lanes of 4): at N = 256 two passes over 512-byte row
        // segments keep more rows of B in L2 than one pass over 1 KB rows and were never slower
        // PR keeps slots along the entries: with 16-byte accesses 2 under EB (wave per chunk; the
        // conditional reduction gets shallower as the group widens: power-law N = 128 823 / 645 /
        // 574 us for groups of 8 / 16 / 32) and 4 under RB (wave per row: 629 / 559 / 636 us)
        const int cap = g.V == 4 ? ((pr && !eb) ? 16 : 32) : (pr ? kDefaultGroupPR : kWave);
        if (g.G > cap) g.G = cap;
        if (pr && !eb && whole && N >= 64 && narrow_tiles_pay(m, k, N, hint)) g.G = 8;
        g.NV = 1;
    }
    static const bool tune = std::getenv("DA_SPMM_TUNE") != nullptr;
    if (tune) {
        g.V = env_int("DA_SPMM_V", g.V);
        g.G = env_int("DA_SPMM_G", g.G);
        g.NV = env_int("DA_SPMM_NV", g.NV);
        g.pin = env_int("DA_SPMM_PIN", -1);
        g.stripe = env_int("DA_SPMM_STRIPE", g.stripe);
        if (g.stripe < 0 || g.stripe > 4096) return fail(DA_ERR_UNSUPPORTED, "DA_SPMM_STRIPE outside 0..4096%s");
        if ((g.V != 1 && g.V != 4) || (g.V == 4 && !vec4_ok) || !is_pow2(g.G) || g.G > kWave ||
            (pr && g.G > kMaxGroupPR) || (g.NV != 1 && g.NV != 2 && g.NV != 4) || (g.G > 1 && g.NV != 1))
            return fail(DA_ERR_UNSUPPORTED, "DA_SPMM_V/_G/_NV override is not a supported combination%s");
    }
    if (eb) {
        const bool whole = vec4_ok && aligned && N >= 32 && N % 4 == 0;
        g.chunk = chunk_size(cm, pr, N, whole, g, hint, plan);
        if (tune) g.chunk = env_int("DA_SPMM_CHUNK", g.chunk);
        if (g.chunk < 8 || g.chunk > (1 << 20)) return fail(DA_ERR_UNSUPPORTED, "bad DA_SPMM_CHUNK%s");
    }
    *out = g;
    return DA_OK;
}

constexpr long kLayerElements = 2L << 20;   // of C, for layers that EB kernels finish

// Calls launch with the whole product or, where its rows make more than max_blocks blocks, with one part of them after
// another (67 M rows of a wave each).
template <class F>
void for_row_parts(const Problem& p, int64_t rows_per_block, int64_t max_blocks, F launch) {
    const int64_t most = max_blocks * rows_per_block / 64 * 64;        // whole words of LeftOut's bits
    for (int64_t first = 0; first < p.m; first += most) {
        Problem part = p;
        part.m = (int)std::min<int64_t>(most, p.m - first);
        part.rowptr += first;
        part.C += first * p.sd.rc;
        if (part.left_out.rows) part.left_out.rows += first / 32;
        launch(part);
    }
}

template <int V, int G, int NV, bool WIDE>
int launch_w(Family fam, const Problem& p, const Geometry& geo) {
    const int chunk = geo.chunk;
    const long tile_cols = (long)G * V * NV;
    const long tiles_l = (p.N + tile_cols - 1) / tile_cols;
    if (tiles_l > kMaxGridY) return fail(DA_ERR_UNSUPPORTED, "N needs more than 65535 column tiles%s");
    const unsigned tiles = (unsigned)tiles_l;
    // RB with 2, 4 or 8 about equal tiles: each tile on XCDs of its own, whose L2s then hold its slice of B alone.  It pays
    // while a good part of the slice fits the 4 MB of an L2 and all of B does not (RB+RM+PR, random columns, 23 entries a
    // row, k = 12 000: N = 128 13.3 -> 10.9 us, N = 256 23.3 -> 19.2; 24 000: 26.3 -> 23.2 and 47.9 -> 42.4; 40 000, slices of 10 MB:
    // 49.6 -> 48.0 and 94.8 -> 92.9; 61 417, 15.7 MB: 105 and 101, with 100 entries a row 328 and 334.  RB+RM+SR, N = 256:
    // 5000 11.3 -> 9.3, 24 000 62.2 -> 60.9, 27-point stencil of 28^3 28.6 -> 24.2.  4096 columns, N = 256, 4.2 MB: 6.1 and 6.2).
    // Not where many entries lie in rows of uneven length, whose XCDs then wait for each other (50 000 lognormal rows of 60,
    // PR, N = 256: k = 6000 133 and 140, 49 152 331 and 345; 5000 such rows, 12 000: 37 and 20).
    // Tiles of 32 columns (narrow_tiles_pay): slices of up to 6 MB and not of a very small B (lognormal rows of 50, coefficient 0.9: N = 64,
    // k = 5000, 10 000 rows 11.7 -> 10.1, 11 000 15.5 -> 13.2, 44 000 47.2 -> 45.6, 75 000 97 and 95; N = 128, 2500 8.9 and 9.1, 6000 15.5 -> 13.9), uneven
    // rows too but for eight tiles (rows of 90, coefficient 1, 31 000: N = 64 53.1 -> 49.5, N = 128 90.7 -> 88.5, N = 256 166 and 195).
    const bool narrow = G == 8 && fam == RB_PR;
    const bool slices_fit = V == 4 && (G >= 16 || narrow) && (fam == RB_SR || fam == RB_PR) && p.sd.cb == 1 &&
                            tiles_l * tile_cols - p.N <= tile_cols / 8 &&
                            (narrow ? p.k * tile_cols * 4 <= 6 << 20 && (p.k > 3072 || (long)p.k * p.N * 4 > 2 << 20) : slices_fit_l2(p.k, p.N, tile_cols)) &&
                            !((!narrow || tiles == 8) && uneven_rows(p.m, lookup_matrix(p.rowptr, p.m)));
    const int pin = ((geo.pin < 0 ? slices_fit : geo.pin != 0) && (tiles == 2 || tiles == 4 || tiles == 8)) ? (int)tiles : 0;
    // grid for `bx` blocks per column tile
    auto grid_for = [&](long bx) {
        if (pin) { const long per = 8 / pin; return dim3((unsigned)(8 * ((bx + per - 1) / per)), 1); }
        return dim3((unsigned)bx, tiles);
    };
    const int64_t max_blocks = pin ? kMaxGridX / 8 * (8 / pin) : kMaxGridX;
    const dim3 block(kBlock);
    // Bias and rectification in the product kernel: groups of 8 and more lanes of one column, of 4 and more of four.  EB needs
    // eb_finish_kernel after it, which takes as long as the pass over a small C (30 000 rows, 64 -> 64 -> 32: 87.3 us, 85.3 with
    // the pass; 60 000 rows, 64 -> 64 -> 24: 114.7 and 119.4): from 2 M elements on.
    constexpr bool kLayers = !WIDE && NV == 1 && G >= (V == 4 ? 4 : 8);
    const bool layer = kLayers && p.layer != nullptr && (fam == RB_SR || fam == RB_PR || (long)p.m * p.N >= kLayerElements);
    if (layer) *p.finished = true;
    auto ended = [&](auto launch_with) {
        if constexpr (kLayers)
            if (layer) return launch_with(*p.layer);
        launch_with(PlainSums{});
    };
    switch (fam) {
    case RB_SR: {
        const long rows_per_block = (long)kWavesPerBlock * (kWave / G);
        ended([&](auto after) {
            for_row_parts(p, rows_per_block, max_blocks, [&](const Problem& q) {
                hipLaunchKernelGGL((rb_sr_kernel<V, G, NV, WIDE, decltype(after)>), grid_for((q.m + rows_per_block - 1) / rows_per_block),
                                   block, 0, q.stream, q.m, q.N, q.sd, q.rowptr, q.colind, q.vals, q.B, q.C, pin, q.left_out, after);
            });
        });
        break;
    }
    case RB_PR: {
        if constexpr (G <= kMaxGroupPR) {
            ended([&](auto after) {
                auto go = [&](auto kernel) {
                    for_row_parts(p, kWavesPerBlock, max_blocks, [&](const Problem& q) {
                        hipLaunchKernelGGL(kernel, grid_for(((int64_t)q.m + kWavesPerBlock - 1) / kWavesPerBlock),
                                           block, 0, q.stream, q.m, q.N, q.sd, q.rowptr, q.colind, q.vals, q.B, q.C, pin, after);
                    });
                };
                if (V == 4 && G >= 16 && p.N % 4 != 0) go(rb_pr_kernel<V, G, NV, WIDE, V == 4 && G >= 16, decltype(after)>);
                else go(rb_pr_kernel<V, G, NV, WIDE, false, decltype(after)>);
            });
        }
        break;
    }
    case EB_SR:
    case EB_PR: {
        // entries per block and pass: a lane group (SR) or a whole wave (PR) owns `chunk` entries
        const long entries_per_block = fam == EB_SR ? (long)chunk * kWavesPerBlock * (kWave / G)
                                                    : (long)chunk * kWavesPerBlock;
        // One chunk per worker when nnz is known from an earlier da_spmm_features call (the
        // hardware dispatcher then balances the blocks); otherwise nnz is known only on the
        // device and the grid is sized for a few waves of blocks over the whole machine, bounded
        // by what the matrix could hold at most.
        long blocks;
        const int64_t known = lookup_matrix(p.rowptr, p.m).nnz;
        if (known >= 0) {
            blocks = (known + entries_per_block - 1) / entries_per_block;
            if (blocks > (1L << 20)) blocks = 1L << 20;
        } else {
            long max_nnz = (long)p.m * (p.k < 1 ? 1 : p.k);
            if (max_nnz > 0x7fffffffL) max_nnz = 0x7fffffffL;
            blocks = (max_nnz + entries_per_block - 1) / entries_per_block;
            const long full = (long)cu_count() * 8 * 4;
            if (blocks > full) blocks = full;
        }
        if (blocks < 1) blocks = 1;
        // chunk order of a prepared matrix (column sweep), if one exists for this chunk size
        std::shared_ptr<DeviceBlock> keep;                 // dropped after the launch
        Schedule sch = !geo.order || env_int("DA_SPMM_NO_SCHEDULE", 0)
                           ? Schedule{nullptr, 0, 0, 0, 0, 0, 0, 0, 3, nullptr, nullptr}
                           : lookup_schedule(p.rowptr, p.colind, p.m, chunk, is_capturing(p.stream), &keep);
        // EB+SR on a prepared matrix never splits rows of at most a chunk (the plan's row hints make
        // the second boundary look-up cheap); the zero pass and the product kernel are told alike
        const int own_short = (fam == EB_SR && kOwnShortRows<G> && sch.order != nullptr &&
                               env_int("DA_SPMM_SPLIT_SHORT_ROWS", 0) == 0) ? 1 : 0;
        // pre-pass: the rows that receive atomic additions, and the rows without entries
        const dim3 zgrid((unsigned)((p.m + kBlock - 1) / kBlock));
        ended([&](auto after) {
            hipLaunchKernelGGL((eb_zero_kernel<V, decltype(after)>), zgrid, block, 0, p.stream, p.m, p.N, p.sd, p.rowptr, p.C, chunk,
                               own_short, after);
        });
        const int first_chunks = sch.split;
        sch.split = 0;
        if (sch.order && geo.stripe > 0) {
            // Deal the schedule in stripes (sweep_block) to the XCDs that work on it: all 8, or the
            // 8 / pin that share a pinned column tile.  Stripe length near geo.stripe such that whole
            // rounds of stripes cover a segment with next to no surplus (all XCDs then get the same
            // number of stripes).  When the schedule starts with a segment of multi-row chunks, that
            // segment and the rest are dealt separately: the two kinds of chunk cost differently,
            // and every XCD should get the same share of both.
            const long nx = pin ? 8 / pin : 8;
            sch.nx_log2 = nx == 8 ? 3 : (nx == 4 ? 2 : (nx == 2 ? 1 : 0));
            const long wpb = fam == EB_SR ? (long)kWavesPerBlock * (kWave / G) : (long)kWavesPerBlock;
            const long nvb = (sch.units + wpb - 1) / wpb;
            auto deal = [&](long nb, int* stripe_out) {        // blocks per XCD, rounded up to whole stripes
                const long per_xcd = (nb + nx - 1) / nx;
                long rounds = (per_xcd + geo.stripe / 2) / geo.stripe;
                if (rounds < 1) rounds = 1;
                *stripe_out = (int)((per_xcd + rounds - 1) / rounds);
                return (long)*stripe_out * rounds;
            };
            long split = env_int("DA_SPMM_NO_SPLIT", 0) ? 0 : first_chunks / wpb;
            if (split < 16 || nvb - split < 16) split = 0;
            if (nvb >= 16) {
                long per_b = 0;
                sch.split = (int)split;
                sch.per_a = (int)deal(split > 0 ? split : nvb, &sch.stripe);
                if (split > 0) per_b = deal(nvb - split, &sch.stripe_b); else sch.stripe_b = 1;
                sch.vblocks = (int)(nx * (sch.per_a + per_b));
                if (blocks >= nvb) blocks = sch.vblocks;      // one chunk per worker
            }
            if (!pin) blocks = (blocks + 7) / 8 * 8;       // block b stays on XCD b % 8 on every pass
        }
        ended([&](auto after) {
            if (fam == EB_SR) {
                hipLaunchKernelGGL((eb_sr_kernel<V, G, NV, WIDE, decltype(after)>), grid_for(blocks), block, 0, p.stream,
                                   p.m, p.N, p.sd, p.rowptr, p.colind, p.vals, p.B, p.C, chunk, pin, sch, own_short, after);
            } else {
                if constexpr (G <= kMaxGroupPR)
                    hipLaunchKernelGGL((eb_pr_kernel<V, G, NV, WIDE, decltype(after)>), grid_for(blocks), block, 0, p.stream,
                                       p.m, p.N, p.sd, p.rowptr, p.colind, p.vals, p.B, p.C, chunk, pin, sch, after);
            }
        });
        if (layer)
            hipLaunchKernelGGL((eb_finish_kernel<V>), zgrid, block, 0, p.stream, p.m, p.N, p.sd, p.rowptr, p.C, chunk, own_short,
                               *p.layer);
        break;
    }
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "kernel launch");
    return DA_OK;
}

// 32-bit gather offsets (BRows<false>) need column indices below 2^24, a row pitch below 16 MiB and
// every element of B within 4 GiB of its base; anything larger takes the 64-bit kernels.
template <int V, int G, int NV>
int launch(Family fam, const Problem& p, const Geometry& geo) {
    const unsigned long long last = (unsigned long long)(p.k > 0 ? p.k - 1 : 0) * (unsigned long long)p.sd.rb +
                                    (unsigned long long)(p.N > 0 ? p.N - 1 : 0) * (unsigned long long)p.sd.cb;
    const bool narrow = p.k <= (1 << 24) && p.sd.rb * 4 < (1 << 24) && (last + 4) * 4 < (1ull << 32) &&
                        env_int("DA_SPMM_WIDE", 0) == 0;
    return narrow ? launch_w<V, G, NV, false>(fam, p, geo) : launch_w<V, G, NV, true>(fam, p, geo);
}

// Column-major B under the RB ids whose sums rb_columns_kernel makes at least as exact (SR; RM+PR from 5 columns on, which
// has 8 slots).  Lanes per row by the length of the row that an average entry lies in: 4 below 7 (3 a row, N = 1: 6.7 us,
// with 8 lanes 7.9, with lanes along N 6.8), 16 from 40 on (rows of 170, N = 8: 93 us with 8, 87 with 16, lanes along N: SR 105,
// PR 99; 27-point stencil: 25 with 8, 35 with 16), 64 from 200 on, where a few rows are much longer than the others
// (power-law, N = 8: 71 with 16, 59 with 64, PR along N 63).  Unknown: 8.
// Whether rb_columns_kernel beats the lanes along N: algo is one of those three ids, mean and len are the lengths of an average row
// and of the row that an average entry lies in.  Its lanes wait for memory a row at a time, so rows want some entries (1 M
// rows of 1: SR, N = 1 7.3 us along N, 10.6 here), and lanes of neighbouring rows write a row-major C in pieces of 4 bytes (SR, rows of
// 3, N = 8: 12.2 and 14.1; of 10: 34.7 and 35.8; from 16 and 24 columns on the loads decide: N = 24, rows of 2 333 and 240, N = 32, of 10 365 and 142).  Nine or ten
// columns are a tile of 8 and one of next to nothing (SR, rows of 3, N = 9: 15.3 and 16.7).  CM has a lane for a row, which is good
// where rows are even and short and 8 columns of B do not fit an L2 (300 000 random rows of 5, N = 8: 91 and 123; 200 000 of 13, N = 16:
// 255 and 279, N = 5 100 and 60; 100 000 of 10, N = 8: 46 and 35) and waits for the longest of 64 where they are not (lognormal rows
// of 8, N = 8: 147 and 55).  PR has a wave for a row and 8 slots along it already: short rows leave them empty (rows of 1, N = 8: 185
// and 49; of 10: 41 and 35; lognormal rows of 60: 40 and 50; 500 rows of 40, N = 64: 8.2 and 4.9; few very long ones, N = 16: 155 and
// 115), above 64 columns it is as good with uneven ones (few very long ones, N = 128: 363 and 396).  Of a
// matrix that nothing is known of every law is possible: the ids keep their lanes along N (PR on 64 rows of 8000, N = 12: 61 and
// 345; SR on 1 M rows of 1, N = 1: 7.4 and 22) but for SR with a column-major C from 24 columns on (1 M rows of 1, N = 24: 400 and 149;
// 64 rows of 8000: 670 and 350; lognormal rows of 25: 123 and 132).
bool columns_pay(int algo, int64_t m, int64_t k, int64_t N, bool c_by_rows, const MatrixHint& hint) {
    const bool sr = algo == DA_RB_RM_SR;
    if (hint.nnz < 0 || hint.seen_len <= 0.0) return sr && !c_by_rows && N >= 24;
    const double mean = (double)hint.nnz / (double)m, len = hint.seen_len;
    if (algo == DA_RB_RM_PR) {
        const bool even = len < 1.15 * mean;
        if (len >= 200.0) return c_by_rows ? N <= 64 && (len >= 2000.0 || (mean < 2.0 && N <= 8)) : N <= 64 || even;
        if (c_by_rows) return (len < 28.0 && (N <= 12 || mean >= 20.0)) || (mean < 2.0 && N <= 8);
        return len < 28.0 || mean < 2.0 || (N > 8 && ((len < 40.0 && len < 2.0 * mean) || even));
    }
    if (!sr) return len >= 35.0 || mean >= 15.0 || (mean >= 3.0 && k <= 1 << 17) || (mean >= 5.0 && N <= 5) ||
                    (c_by_rows && mean < 3.5 && N >= 16);
    if (N >= 24) return mean >= 2.0 || !c_by_rows;
    if (N == 9 || N == 10) return mean >= (c_by_rows ? 20.0 : 8.0) || (len >= 200.0 && mean >= 8.0);
    if (c_by_rows) return mean >= 12.0 || (N >= 16 && mean >= 4.0 && len < 6.0 * mean);
    return mean >= (N > 10 ? 2.0 : 2.5) || (N >= 16 && len < 35.0);
}

int launch_columns(const Problem& p, const MatrixHint& hint) {
    auto go = [&](auto l, auto nc) {
        constexpr int L = decltype(l)::value, NC = decltype(nc)::value;
        const long rows = (long)kWavesPerBlock * (kWave / L);
        for_row_parts(p, rows, kMaxGridX, [&](const Problem& q) {
            hipLaunchKernelGGL((rb_columns_kernel<L, NC>), dim3((unsigned)((q.m + rows - 1) / rows), (unsigned)((q.N + NC - 1) / NC)),
                               dim3(kBlock), 0, q.stream, q.m, q.N, q.sd, q.rowptr, q.colind, q.vals, q.B, q.C);
        });
    };
    auto by_columns = [&](auto l) {
        if (p.N >= 5) go(l, Count<8>{});
        else if (p.N >= 3) go(l, Count<4>{});
        else if (p.N == 2) go(l, Count<2>{});
        else go(l, Count<1>{});
    };
    const double len = hint.seen_len > 0.0 ? hint.seen_len : 8.0;
    if (len < 7.0 && p.N < 5) by_columns(Count<4>{});
    else if (len < 40.0) by_columns(Count<8>{});
    else if (len < 200.0) by_columns(Count<16>{});
    else by_columns(Count<64>{});
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "kernel launch");
    return DA_OK;
}

// How the heavy rows' part of a product is dealt to the blocks.  A block has 147 KB of LDS and 16 waves, one to a CU: as many
// ranges of columns as make one block per CU over all groups of rows and column tiles.  Every block's part of a row is one
// more rounding of the row's sum, as every chunk of EB+SR is: a group has no more ranges than its shortest row's sum
// takes.  Rows of similar length make a group, so that the ranges of long rows need not be as few as those of short ones,
// and the ranges are as many as the group's entries want.  524 rows of 20 000 to 100 000, N = 64: 61, 90 and 103 ranges for
// 180, 180 and 164 rows, whose blocks take 186, 181 and 188 us (before, with the ranges in cells twice as large and less for a
// row's turn, two groups' 198 and 170).
struct HeavyLaunch {
    HeavyGroups groups;
    double load;         // entries, and work of as much time, of the block that has most
};

constexpr double kHeavyLeast = 5000.0;   // work of a block that is worth a range of its own (40 rows of 16 000, N = 8: 16 us, 18 in twice as many)

// Entries that take as long as a row's turn in a band of B, by the times of blocks with short and with long rows.
constexpr double kHeavyVisit = 12.0;

constexpr int heavy_tile(int64_t N) { return N <= 8 ? 8 : (N <= 16 ? 16 : (N <= 32 ? 32 : 64)); }

// Whether a wave of each block brings B, 16 bytes a lane.  Rows of B that are column-major or have less than 16 bytes all
// waves bring together (524 rows of 20 000 to 100 000, N = 41: 492 us with 4 bytes a lane by one wave, 322 by all waves, 302 by one wave with
// 16 bytes a lane; N = 8: 117 by all waves, 110 by two, 108 by one).
bool heavy_loader(int64_t N, const Strides& sd) { return sd.cb == 1 && N >= 4; }

// Entries of a heavy row of n entries that a block has to add up, at least, for a sum as exact as EB's in chunks of c: as
// one_sign_error, with sums of 16 entries that are added one after another inside a part.
double heavy_part(double n, double c) {
    const double bound = one_sign_error(c, 1.0, n) - 256.0;
    double part = n * n / bound;
    for (int i = 0; i < 3; ++i) part = n * n / (bound - part * part / 16.0);
    return part;
}

HeavyLaunch deal_heavy_rows(const HeavyPlan& pl, const std::vector<int64_t>& sums, int64_t k, int64_t N, int chunk, bool loader) {
    const int tile = heavy_tile(N), band = 16384 / tile;
    const int64_t tiles = (N + tile - 1) / tile;
    const int waves = heavy_waves(loader), quads = (pl.count + 3) / 4, most = waves * kHeavyQuads, least = (quads + most - 1) / most;
    HeavyLaunch best{};
    auto deal = [&](int n, int unit) {                      // n groups of whole units of 4 * unit rows
        HeavyLaunch x{};
        x.groups.count = n;
        const int64_t blocks = std::max<int64_t>(cu_count() / tiles, n);
        const int units = (quads + unit - 1) / unit;
        double cost[kHeavyGroups], all = 0.0;
        int fewest[kHeavyGroups];                           // cells of a range, at least
        for (int i = 0; i <= n; ++i) x.groups.row[i] = std::min(pl.count, 4 * unit * (int)((int64_t)units * i / n));
        for (int i = 0; i < n; ++i) {
            const int r0 = x.groups.row[i], r1 = x.groups.row[i + 1], here = (r1 - r0 + 3) / 4;
            const double entries = (double)(sums[r1] - sums[r0]) + kHeavyVisit * (r1 - r0) * ((double)k / band);
            // a CU needs some 12 of its waves to be busy
            const double longest = entries * ((here + waves - 1) / waves) / here;
            cost[i] = std::max(entries, 12.0 * longest) + 2.0 * (double)k;
            all += cost[i];
            const double shortest = (double)(sums[r0 + 1] - sums[r0]);
            const int ranges = std::max(1, (int)(shortest / heavy_part(shortest, chunk)));
            fewest[i] = (pl.cells + ranges - 1) / ranges;
        }
        for (double target = std::max(kHeavyLeast, all / (double)blocks);; target *= 1.02) {
            x.load = 0.0;
            for (int i = 0; i < n; ++i) {
                const int per = std::max(fewest[i], std::max(1, (int)(std::min(target / cost[i], 1.0) * pl.cells)));
                x.groups.per[i] = per;
                x.groups.block[i + 1] = x.groups.block[i] + (pl.cells + per - 1) / per;
                x.load = std::max(x.load, cost[i] * per / pl.cells);
            }
            if (x.groups.block[n] <= blocks) break;
        }
        if (best.groups.count == 0 || x.load < 0.97 * best.load) best = x;
    };
    // every wave of a block with as many rows as the others, as far as that goes
    deal(least, 1);
    for (int n = least; n <= std::min(kHeavyGroups, least + 3); ++n) {
        if (n * waves <= quads) deal(n, waves);
        else if (n == 2 && quads >= 2) deal(n, 1);
    }
    return best;
}

// Whether the heavy rows' kernel beats EB, which has all rows in one kernel and as many blocks as it likes.  share: the load of
// the block that has most, in shares of a CU of all entries.  EB's additions to the same few lines of C are what costs it
// most, so that few rows of many entries always gain up to 32 columns (72 rows of 24 000, N = 32: 72 us in EB, 34 here; 300
// of 2300, N = 8: 20.3 and 15.3, N = 24: 27.6 and 24.3; 1000 of 20 000, share 1.34, N = 32: 123 and 131, the most that is lost).
// Up to four columns EB has 16 and more workers to a wave and waits for them (4000 rows of 1000, N = 4: 47 and 39).  Beyond 128 the
// entries are read for every tile in EB, too (N = 130: 12 M 520 and 390, 33 M 1540 and 833).  Column-major B gathers every element
// from a line of its own in EB (300 heavy rows, N = 32: 92 and 76; 5000 of 8000: 2756 and 451).
// Between, many rows are EB's unless they fill the CUs evenly, and EB's time for an entry grows with their number (N = 64: 10.4 us a
// million at 12 M, 12.7 at 50 M): the share that still pays grows with it.  Fitted over 70 matrices of 72 to 8000 heavy rows, 0.8 to 50 M
// entries; on either side of the line, EB and here:
//   N <= 8           1500 of 8000, 12.3 M, share 1.14: 58 and 50; 6000 of 6000, 36 M, 1.26: 163 and 131; 8000 of 700, 5.8 M, 1.25: 36 and 39
//   N <= 16          1500 of 17 000, 26 M, 1.30: 128 and 118; 5000 of 3000, 15 M, 1.33: 85 and 95; 3500 of 5000, 18 M, 1.32: 98 and 104
//   N < 32           2000 of 6000, 12 M, 1.31, N = 24: 109 and 89; 1500 of 17 000, 1.47: 175 and 180; 8000 of 1300, 11 M, 1.80: 89 and 134
//   N = 32           5000 of 4000 to 12 000, 41 M, 1.43: 314 and 281; 4000 of 4000, 16 M, 1.33: 98 and 118
//   N <= 64          8000 of 3000, 24 M, 1.67, N = 64: 239 and 199; 1500 of 17 000, 1.84: 313 and 254; 1500 of 8000, 12 M, 1.84: 128 and
//                    147; 5000 of 5000, 26 M, 2.32: 277 and 324; 3000 of 10 000, 31 M, 2.29: 391 and 360
//   the same, rows of B not whole 16-byte pieces, which EB gathers in twice the time
//                    1500 of 5000, 7.6 M, 1.99, N = 41: 112 and 87; 3500 of 5000, 18 M, 2.03: 196 and 216
// Beyond 64 the entries are read for every tile (N = 96: 5 M 88 and 88, 12 M 286 and 216, 25 M 512 and 412), and beyond 32
// the rows that are not heavy cost more in a kernel of their own (12 M entries, 300 000 rows, N = 64: 142 and 149).
bool heavy_rows_pay(int64_t m, int64_t N, bool row_major, bool whole, int count, int64_t nnz, double share) {
    const bool many = nnz >= 10000000;
    if (!row_major) return (N > 8 || count <= 2048 || many) && (N <= 32 || count >= 256);
    if (N <= 4) return true;
    const double millions = (double)nnz * 1e-6;
    if (N <= 8) return count <= 1024 || share <= 1.1 + millions / 20.0;
    if (N <= 16) return count <= 1024 || share <= 1.0 + millions / 60.0;
    if (N <= 32) return count <= 1024 || share <= (N < 32 ? 1.5 + millions / 120.0 : 1.05 + millions / 70.0);
    if (count < 256) return false;
    if (N > 128) return true;
    if (nnz / 48 < m) return false;
    return N <= 64 ? count <= 640 || share <= std::max(1.45 + millions / 34.0, whole ? 0.0 : 2.0) : many;
}

// The heavy rows' part of a product whose other rows are on the stream already.
// Lanes: 4 of two columns up to 8 columns (N = 8: 90 us, 16 lanes of one column 114), 16 beyond (N = 16, 1.6 M entries: 16 us,
// 4 lanes of four columns, whose random 64-byte reads meet in the banks of LDS, 33).
int launch_heavy(const Problem& p, const HeavyPlan& pl, const HeavyGroups& groups) {
    const int tile = heavy_tile(p.N);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)groups.block[groups.count], (unsigned)((p.N + tile - 1) / tile)), dim3(kHeavyBlock), kHeavyLds,
                           p.stream, p.m, (int)p.k, p.N, p.sd, p.rowptr, p.colind, p.vals, p.B, p.C, pl, groups);
    };
    auto by_tile = [&](auto loader) {
        constexpr bool LOADER = decltype(loader)::value;
        switch (tile) {
        case 8: go(heavy_rows_kernel<4, 2, LOADER>); break;
        case 16: go(heavy_rows_kernel<16, 1, LOADER>); break;
        case 32: go(heavy_rows_kernel<16, 2, LOADER>); break;
        default: go(heavy_rows_kernel<16, 4, LOADER>);
        }
    };
    if (heavy_loader(p.N, p.sd)) by_tile(Truth<true>{});
    else by_tile(Truth<false>{});
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "kernel launch");
    return DA_OK;
}

template <int V>
int dispatch_v(Family fam, const Geometry& g, const Problem& p) {
    if (g.G == 1) {
        switch (g.NV) {
        case 1: return launch<V, 1, 1>(fam, p, g);
        case 2: return launch<V, 1, 2>(fam, p, g);
        case 4: return launch<V, 1, 4>(fam, p, g);
        }
    } else if (g.NV == 1) {
        switch (g.G) {
        case 2: return launch<V, 2, 1>(fam, p, g);
        case 4: return launch<V, 4, 1>(fam, p, g);
        case 8: return launch<V, 8, 1>(fam, p, g);
        case 16: return launch<V, 16, 1>(fam, p, g);
        case 32: return launch<V, 32, 1>(fam, p, g);
        case 64: return launch<V, 64, 1>(fam, p, g);
        }
    }
    return fail(DA_ERR_UNSUPPORTED, "unsupported lane mapping%s");
}

int dispatch(Family fam, const Geometry& g, const Problem& p) {
    if ((fam == RB_PR || fam == EB_PR) && g.G > kMaxGroupPR)
        return fail(DA_ERR_UNSUPPORTED, "PR lane group too wide%s");
    return g.V == 4 ? dispatch_v<4>(fam, g, p) : dispatch_v<1>(fam, g, p);
}

const char* const kNames[DA_NUM_ALGOS] = {
    "RB+RM+SR", "RB+RM+PR", "RB+CM+SR", "RB+CM+PR", "EB+RM+SR", "EB+RM+PR", "EB+CM+SR", "EB+CM+PR"};

// Workspace of da_csr_transpose: two buffers each of keys, row numbers and values (nnz elements)
// for the ping-pong of the radix passes, the per-block digit histograms of one pass, and the chunk
// sums of their prefix scan.  Every part starts on a 256-byte boundary.
struct TransposePlan {
    int passes, digit_bits, nblocks;
    long hist_len, parts;
    size_t off_keys[2], off_rows[2], off_vals[2], off_hist, off_part, bytes;
};

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

TransposePlan plan_transpose(int64_t k, int64_t nnz) {
    TransposePlan t{};
    int bits = 1;
    while (bits < 31 && (int64_t(1) << bits) < k) ++bits;             // column indices are < 2^bits
    t.passes = (bits + kRadixBits - 1) / kRadixBits;
    t.digit_bits = (bits + t.passes - 1) / t.passes;                  // equal digits, at most kRadixBits wide
    t.nblocks = (int)((nnz + kSortTile - 1) / kSortTile);
    t.hist_len = (long)kBins * t.nblocks;
    t.parts = (t.hist_len + kScanChunk - 1) / kScanChunk;
    size_t off = 0;
    const size_t per = align256((size_t)nnz * 4);
    for (int i = 0; i < 2; ++i) { t.off_keys[i] = off; off += per; }
    for (int i = 0; i < 2; ++i) { t.off_rows[i] = off; off += per; }
    for (int i = 0; i < 2; ++i) { t.off_vals[i] = off; off += per; }
    t.off_hist = off; off += align256((size_t)t.hist_len * sizeof(int));
    t.off_part = off; off += align256((size_t)t.parts * sizeof(int));
    t.bytes = off > 0 ? off : 256;
    return t;
}

// Plan of the transpose in one or two passes (transpose_* kernels), for k <= 2^20 when the row number
// and the second digit fit one word.  Tiles of 1024 entries while that leaves a chip of 256 CUs less than
// full, of 2048 beyond (1024 ... 4096 measured within 7 %).  Groups of up to 8 tiles, at least 512 of them where
// there are as many tiles.
struct TransposeFast {
    bool usable;
    int passes, bits[2], row_bits, tile, ntiles, group, ngroups;
    size_t off_mid, off_vals, off_hist, off_group, off_total, off_rows, bytes;
};

int bits_for(int64_t values) {                            // smallest b with 2^b >= values, at least 1
    int b = 1;
    while (b < 31 && (int64_t(1) << b) < values) ++b;
    return b;
}

TransposeFast plan_transpose_fast(int64_t m, int64_t k, int64_t nnz) {
    TransposeFast t{};
    const int bits = bits_for(k);
    t.row_bits = bits_for(m);
    t.passes = bits <= kDigitBitsMax ? 1 : 2;
    t.bits[0] = t.passes == 1 ? bits : (bits + 1) / 2;
    t.bits[1] = t.passes == 1 ? 0 : bits - t.bits[0];
    t.usable = t.bits[0] <= kDigitBitsMax && t.row_bits + t.bits[1] <= 32;
    for (int i = 0; i < t.passes; ++i) if (t.bits[i] < 4) t.bits[i] = 4;     // transpose_scan_kernel takes 16 digits a block
    t.tile = kSortBlock * (nnz < 1024 * 1024 ? 4 : 8);
    t.ntiles = (int)((nnz + t.tile - 1) / t.tile);
    t.group = t.ntiles <= 512 ? 1 : (t.ntiles >= kGroupMax * 512 ? kGroupMax : t.ntiles / 512);
    t.ngroups = (t.ntiles + t.group - 1) / t.group;
    size_t off = 0;
    const size_t per = align256((size_t)nnz * 4);
    const int widest = t.bits[0] > t.bits[1] ? t.bits[0] : t.bits[1];
    t.off_mid = off; off += per;
    t.off_vals = off; off += per;
    t.off_hist = off; off += align256(((size_t)t.ntiles << widest) * sizeof(int));
    t.off_group = off; off += align256(((size_t)t.ngroups << widest) * sizeof(int));
    t.off_total = off; off += align256(2 * kDigitBinsMax * sizeof(int));
    t.off_rows = off; off += align256(((size_t)t.ntiles + 1) * sizeof(int));
    t.bytes = off;
    return t;
}

// One schedule to build: da_eb_schedule's outputs, and optionally the row of every chunk's first
// entry in schedule order (first_rows[u] belongs to chunk order[u]) and indexed by chunk number
// (rows_by_unit); all device pointers, the last three may be null
struct ScheduleJob {
    int unit;
    int32_t* order; int32_t* first_segment; int32_t* first_rows; int32_t* rows_by_unit;
    void* workspace; size_t workspace_bytes;
};
int enqueue_schedules(int64_t m, int64_t k, int64_t nnz, const int32_t* rowptr, const int32_t* colind,
                      const ScheduleJob* jobs, int njobs, void* stream);
int check_transpose_args(int64_t m, int64_t k, int64_t nnz, const int32_t* rowptr, const int32_t* colind,
                         const float* vals, int32_t* t_rowptr, int32_t* t_colind, float* t_vals);
int enqueue_transpose(int64_t m, int64_t k, int64_t nnz, const int32_t* rowptr, const int32_t* colind,
                      const float* vals, int32_t* t_rowptr, int32_t* t_colind, float* t_vals,
                      void* workspace, size_t workspace_bytes, void* stream);

// The size a transpose asks for and needs: the general sort's.  The packed passes run where their scratch fits
// into it, which it does from about a thousand entries on (about 16 B per entry at most against 24).
size_t transpose_workspace_bytes(int64_t k, int64_t nnz) { return plan_transpose(k, nnz).bytes; }

// Scratch memory of the entry point that allocates nothing (da_csr_transpose_noalloc): a static
// device array, one copy per GPU, held from the moment the library is loaded on that GPU until the
// process ends.  In host code the array's name is only a handle for the runtime, not a device
// address: the address on the current device is asked for once per device and kept.
constexpr size_t kScratchBytes = size_t(32) << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];

int scratch_address(void** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return fail(DA_ERR_UNSUPPORTED, "device ordinal beyond 63%s");
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
        if (!p || reinterpret_cast<uintptr_t>(p) % 256 != 0) return fail(DA_ERR_HIP, "static scratch has no usable device address%s");
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return DA_OK;
}

// Device scratch and pinned host memory of da_spmm_features, kept between calls (allocating, clearing,
// copying and freeing them took ten times as long as the reduction).  A call owns one slot from start to
// end, so calls of several threads and streams do not meet; at most kFeatureSlots idle ones are kept per
// device, the rest is freed when the call returns.
constexpr size_t kFeatureSlots = 8;
struct FeatureSlot {
    FeatureScratch* scratch = nullptr;
    FeatureResult* result = nullptr;
    unsigned long long ticket = 0;
};
std::mutex g_feature_mu;
std::vector<FeatureSlot> g_feature_slots[kMaxDevices];

void free_slot(const FeatureSlot& s) {
    if (s.scratch) (void)hipFree(s.scratch);
    if (s.result) (void)hipHostFree(s.result);
}

// A new slot is cleared on the stream of the call that takes it, whose kernel follows; nothing waits for other streams.
hipError_t take_slot(int dev, hipStream_t stream, FeatureSlot* out) {
    {
        std::lock_guard<std::mutex> lk(g_feature_mu);
        auto& pool = g_feature_slots[dev];
        if (!pool.empty()) {
            *out = pool.back();
            pool.pop_back();
            return hipSuccess;
        }
    }
    FeatureSlot s;
    hipError_t e = hipMalloc(&s.scratch, sizeof(FeatureScratch));
    if (e == hipSuccess) e = hipMemsetAsync(s.scratch, 0, sizeof(FeatureScratch), stream);
    if (e == hipSuccess) e = hipHostMalloc(&s.result, sizeof(FeatureResult), hipHostMallocMapped | hipHostMallocCoherent);
    if (e != hipSuccess) { free_slot(s); return e; }
    s.result->ticket = 0;
    *out = s;
    return hipSuccess;
}

void give_slot(int dev, const FeatureSlot& s) {
    {
        std::lock_guard<std::mutex> lk(g_feature_mu);
        auto& pool = g_feature_slots[dev];
        if (pool.size() < kFeatureSlots) { pool.push_back(s); return; }
    }
    free_slot(s);
}

// Enqueues the reduction over the row pointers; its result is in slot->result once the ticket is there.  The slot is
// the caller's to give back, or to free after an error.
hipError_t start_features(int64_t m, const int32_t* rowptr, hipStream_t stream, int* dev, FeatureSlot* slot) {
    hipError_t e = hipGetDevice(dev);
    if (e == hipSuccess && (*dev < 0 || *dev >= kMaxDevices)) e = hipErrorInvalidDevice;
    if (e == hipSuccess) e = take_slot(*dev, stream, slot);
    if (e != hipSuccess) return e;
    ++slot->ticket;
    // 8 row pointers a thread: enough blocks to hide their latency, few enough for the shared counters
    long blocks = (m + 8 * kBlock - 1) / (8 * kBlock);
    const long cap = (long)cu_count() * 4;
    if (blocks > cap) blocks = cap;
    hipLaunchKernelGGL(features_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, stream, (int)m, rowptr, slot->scratch, slot->result,
                       slot->ticket);
    return hipGetLastError();
}

bool arrived(const FeatureSlot& s) { return __atomic_load_n(&s.result->ticket, __ATOMIC_ACQUIRE) == s.ticket; }

// DA_SPMM_DEBUG_VALIDATE=1 makes da_spmm / da_spmm_ex / da_csr_transpose check the CSR arrays on
// the device before they launch anything (this synchronises the stream)
bool debug_validate() {
    const char* v = std::getenv("DA_SPMM_DEBUG_VALIDATE");
    return v && *v && std::strcmp(v, "0") != 0;
}

}  // namespace

extern "C" {

int da_csr_validate(int64_t m, int64_t k, int64_t nnz, const int32_t* rowptr, const int32_t* colind, void* stream)
{
    if (m < 0 || k < 0 || nnz < -1) return fail(DA_ERR_INVALID_ARG, "negative size%s");
    if (m > 0x7ffffffeLL || k > 0x7fffffffLL || nnz > 0x7fffffffLL)
        return fail(DA_ERR_INVALID_ARG, "size beyond the int32 index range%s");
    if (m == 0) return nnz > 0 ? fail(DA_ERR_INVALID_ARG, "stored entries in a matrix without rows%s") : DA_OK;
    if (!rowptr) return fail(DA_ERR_INVALID_ARG, "null rowptr%s");
    hipStream_t st = (hipStream_t)stream;
    unsigned* dflags = nullptr;
    hipError_t e = hipMalloc(&dflags, 2 * sizeof(unsigned));
    if (e != hipSuccess) return hip_fail(e, "hipMalloc");
    unsigned h[2] = {0, 0};
    const long cap = (long)cu_count() * 8;
    auto blocks_for = [&](long n) { long b = (n + kBlock - 1) / kBlock; return (unsigned)(b > cap ? cap : (b < 1 ? 1 : b)); };
    e = hipMemsetAsync(dflags, 0, sizeof h, st);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(validate_rowptr_kernel, dim3(blocks_for(m)), dim3(kBlock), 0, st, (int)m, rowptr, dflags);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(h, dflags, sizeof h, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    int status = DA_OK;
    if (e == hipSuccess) {
        const int64_t dev_nnz = (int64_t)(int32_t)h[1];
        if (h[0] & kBadFirst) status = fail(DA_ERR_INVALID_ARG, "malformed CSR: rowptr[0] != 0%s");
        else if (h[0] & kBadOrder) status = fail(DA_ERR_INVALID_ARG, "malformed CSR: rowptr decreases%s");
        else if (nnz >= 0 && dev_nnz != nnz) status = fail(DA_ERR_INVALID_ARG, "malformed CSR: rowptr[m] differs from nnz%s");
        else if (dev_nnz > 0 && !colind) status = fail(DA_ERR_INVALID_ARG, "null colind with stored entries%s");
        else if (dev_nnz > 0) {
            hipLaunchKernelGGL(validate_colind_kernel, dim3(blocks_for(dev_nnz)), dim3(kBlock), 0, st, (int)dev_nnz, (int)k,
                               colind, dflags);
            e = hipGetLastError();
            if (e == hipSuccess) e = hipMemcpyAsync(h, dflags, sizeof h, hipMemcpyDeviceToHost, st);
            if (e == hipSuccess) e = hipStreamSynchronize(st);
            if (e == hipSuccess && (h[0] & kBadColumn))
                status = fail(DA_ERR_INVALID_ARG, "malformed CSR: column index outside [0, k)%s");
        }
    }
    (void)hipFree(dflags);
    if (e != hipSuccess) return hip_fail(e, "da_csr_validate");
    return status;
}

}  // extern "C"

namespace {

// da_spmm_ex; with a layer also what C takes besides the sums, if *finished comes back true.
int product(int64_t m, int64_t k, int64_t N, const int32_t* rowptr, const int32_t* colind,
            const float* vals, const float* B, int64_t ldb, int layout_b, float* C, int64_t ldc,
            int layout_c, int algo, void* stream, LayerSums* layer, bool* finished)
{
    if (m < 0 || k < 0 || N < 0) return fail(DA_ERR_INVALID_ARG, "negative size%s");
    if (m > 0x7ffffffeLL || k > 0x7fffffffLL || N > 0x7fffffffLL)
        return fail(DA_ERR_INVALID_ARG, "size beyond the int32 index range%s");
    if (algo < 0 || algo >= DA_NUM_ALGOS) return fail(DA_ERR_BAD_ALGO, "algorithm id outside 0..7%s");
    if ((layout_b != DA_ROW_MAJOR && layout_b != DA_COL_MAJOR) || (layout_c != DA_ROW_MAJOR && layout_c != DA_COL_MAJOR))
        return fail(DA_ERR_INVALID_ARG, "layout is neither DA_ROW_MAJOR nor DA_COL_MAJOR%s");
    if (ldb < (layout_b == DA_ROW_MAJOR ? N : k) || ldc < (layout_c == DA_ROW_MAJOR ? N : m))
        return fail(DA_ERR_INVALID_ARG, "leading dimension smaller than the extent it strides over%s");
    if (m == 0 || N == 0) return DA_OK;
    if (!rowptr || !C) return fail(DA_ERR_INVALID_ARG, "null rowptr or C%s");
    // colind, vals and B are read only through stored entries; they may be null when nnz == 0,
    // which only the device knows
    if (debug_validate()) {
        const int v = da_csr_validate(m, k, -1, rowptr, colind, stream);
        if (v != DA_OK) return v;
    }

    Strides sd;
    sd.rb = layout_b == DA_ROW_MAJOR ? ldb : 1;
    sd.cb = layout_b == DA_ROW_MAJOR ? 1 : ldb;
    sd.rc = layout_c == DA_ROW_MAJOR ? ldc : 1;
    sd.cc = layout_c == DA_ROW_MAJOR ? 1 : ldc;
    Problem p{(int)m, (int)N, sd, rowptr, colind, vals, B, C, (hipStream_t)stream, k, LeftOut{}, nullptr, nullptr};
    const bool eb = algo >= DA_EB_RM_SR;
    const bool cm = (algo & 2) != 0;
    const bool pr = (algo & 1) != 0;
    Geometry g;
    const uintptr_t ends = reinterpret_cast<uintptr_t>(B) | reinterpret_cast<uintptr_t>(C) | (uintptr_t)(sd.rb * 4) | (uintptr_t)(sd.rc * 4);
    p.layer = layer;
    p.finished = finished;
    const bool tuned = std::getenv("DA_SPMM_TUNE") != nullptr;        // the launch geometry is that of the ids' own kernels
    if (sd.rb == 1 && N <= 8L * kMaxGridY && (algo == DA_RB_RM_SR || algo == DA_RB_CM_SR || (algo == DA_RB_RM_PR && N >= 5)) && !tuned) {
        // a single column of C lies the same way in either order
        const MatrixHint hint = lookup_matrix(rowptr, m);
        if (columns_pay(algo, m, k, N, sd.rc != 1, hint)) return launch_columns(p, hint);
    }
    const bool ask = eb || (pr && !cm && N >= 64 && N % 32 == 0) || (!cm && !pr && N > 16 && (N < 32 || N % 4 != 0 || ends % 16 != 0));   // RB: only where the lanes depend on it
    const int st = pick_geometry(cm, pr, eb, m, k, N, sd, ends % 16 == 0, ask ? lookup_matrix(rowptr, m) : MatrixHint{nullptr, 0, -1, 0.0},
                                 eb ? plan_info(rowptr, colind, m) : PlanInfo{false, 0.0}, &g);
    if (st != DA_OK) return st;
    if (algo == DA_EB_RM_SR && N <= 64L * kMaxGridY && !tuned && env_int("DA_SPMM_NO_HEAVY", 0) == 0) {
        // Heavy rows in a kernel of their own, the others, which are short and even, row by row.  A row is then added up
        // entry by entry; EB does that with up to a chunk of them.
        const HeavyLookup heavy = lookup_heavy(rowptr, colind, m, k, p.stream);
        const int64_t known = lookup_matrix(rowptr, m).nnz;              // the features may have been taken of another matrix since
        if (heavy.plan.count > 0 && heavy.rest_longest <= g.chunk && (known < 0 || known == heavy.plan.nnz)) {
            const HeavyLaunch dealt = deal_heavy_rows(heavy.plan, *heavy.sums, k, N, g.chunk, heavy_loader(N, sd));
            if (heavy_rows_pay(m, N, sd.cb == 1, ends % 16 == 0 && N % 4 == 0, heavy.plan.count, heavy.plan.nnz, dealt.load * cu_count() / heavy.plan.nnz)) {
                Problem q = p;
                q.layer = nullptr;
                Geometry rest;
                const int rs = pick_geometry(false, false, false, m, k, N, sd, ends % 16 == 0, MatrixHint{rowptr, m, heavy.plan.nnz, heavy.rest_len},
                                             PlanInfo{false, 0.0}, &rest);
                if (rs != DA_OK) return rs;
                q.left_out = LeftOut{heavy.bits, rowptr + m, heavy.plan.min_len, heavy.plan.nnz, std::min(g.chunk, heavy.plan.min_len - 1),
                                     heavy.plan.stale};
                const int done = dispatch(RB_SR, rest, q);
                return done != DA_OK ? done : launch_heavy(q, heavy.plan, dealt.groups);
            }
        }
    }
    const Family fam = eb ? (pr ? EB_PR : EB_SR) : (pr ? RB_PR : RB_SR);
    return dispatch(fam, g, p);
}

}  // namespace

extern "C" {

int da_spmm_ex(int64_t m, int64_t k, int64_t N, const int32_t* rowptr, const int32_t* colind,
               const float* vals, const float* B, int64_t ldb, int layout_b, float* C, int64_t ldc,
               int layout_c, int algo, void* stream)
{
    return product(m, k, N, rowptr, colind, vals, B, ldb, layout_b, C, ldc, layout_c, algo, stream, nullptr, nullptr);
}

int da_spmm_layer(int64_t m, int64_t k, int64_t N, const int32_t* rowptr, const int32_t* colind, const float* vals,
                  const float* B, int64_t ldb, float* C, const float* bias, int relu, int algo, void* stream)
{
    LayerSums after{bias, relu};
    const bool sums_only = bias == nullptr && relu == 0;
    bool finished = sums_only;
    const int st = product(m, k, N, rowptr, colind, vals, B, ldb, DA_ROW_MAJOR, C, N, DA_ROW_MAJOR, algo, stream,
                           sums_only ? nullptr : &after, &finished);
    return st != DA_OK || finished ? st : da_spmm_bias_relu(m, N, C, bias, relu, stream);
}

int da_spmm(int64_t m, int64_t k, int64_t N, const int32_t* rowptr, const int32_t* colind,
            const float* vals, const float* B, float* C, int algo, void* stream)
{
    if (N < 0) return fail(DA_ERR_INVALID_ARG, "negative size%s");
    return da_spmm_ex(m, k, N, rowptr, colind, vals, B, N, DA_ROW_MAJOR, C, N, DA_ROW_MAJOR, algo, stream);
}

int da_spmm_features(int64_t m, int64_t N, const int32_t* rowptr, void* stream, da_features* out)
{
    if (!out) return fail(DA_ERR_INVALID_ARG, "null output%s");
    if (m < 0 || N < 0 || m > 0x7ffffffeLL) return fail(DA_ERR_INVALID_ARG, "bad size%s");
    std::memset(out, 0, sizeof *out);
    out->N = N;
    if (m == 0) return DA_OK;
    if (!rowptr) return fail(DA_ERR_INVALID_ARG, "null rowptr%s");
    hipStream_t st = (hipStream_t)stream;
    // the call waits for its result, which a recorded kernel would not deliver
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &capture) != hipSuccess) { (void)hipGetLastError(); capture = hipStreamCaptureStatusNone; }
    if (capture != hipStreamCaptureStatusNone) return hip_fail(hipErrorStreamCaptureUnsupported, "da_spmm_features");
    int dev = 0;
    FeatureSlot slot;
    hipError_t e = start_features(m, rowptr, st, &dev, &slot);
    if (e == hipErrorInvalidDevice) return fail(DA_ERR_UNSUPPORTED, "device ordinal beyond 63%s");
    if (e == hipSuccess) {
        // The result arrives in host memory: look for it a while (a stream that is idle answers within
        // microseconds), then wait for the stream.
        bool here = false;
        for (int i = 0; i < 20000 && !here; ++i) {
            here = arrived(slot);
            if (!here) __builtin_ia32_pause();
        }
        if (!here) e = hipStreamSynchronize(st);
        if (e == hipSuccess && !arrived(slot)) e = hipErrorUnknown;
    }
    if (e != hipSuccess) { free_slot(slot); return hip_fail(e, "da_spmm_features"); }
    const unsigned long long h[3] = {slot.result->sq, slot.result->mx, slot.result->nnz};
    give_slot(dev, slot);
    // population variance = (m * sum len^2 - nnz^2) / m^2, formed exactly in 128-bit integers
    const unsigned __int128 num = (unsigned __int128)(unsigned long long)m * h[0]
                                  - (unsigned __int128)h[2] * h[2];
    const double md = (double)m;
    const double mean = (double)h[2] / md;
    const double var = (double)num / (md * md);
    out->rows = m;
    out->nnz = (int64_t)h[2];
    remember_matrix(rowptr, m, out->nnz, h[2] ? (double)h[0] / (double)h[2] : 0.0);
    out->row_nnz_mean = mean;
    out->row_nnz_std = std::sqrt(var);
    out->row_nnz_max = (double)h[1];
    return DA_OK;
}

int da_csr_transpose_workspace(int64_t m, int64_t k, int64_t nnz, size_t* bytes)
{
    if (!bytes) return fail(DA_ERR_INVALID_ARG, "null bytes%s");
    if (m < 0 || k < 0 || nnz < 0) return fail(DA_ERR_INVALID_ARG, "negative size%s");
    if (m > 0x7ffffffeLL || k > 0x7ffffffeLL || nnz > 0x7fffffffLL)
        return fail(DA_ERR_INVALID_ARG, "size beyond the int32 index range%s");
    *bytes = transpose_workspace_bytes(k, nnz);
    return DA_OK;
}

int da_csr_transpose(int64_t m, int64_t k, int64_t nnz, const int32_t* rowptr, const int32_t* colind,
                     const float* vals, int32_t* t_rowptr, int32_t* t_colind, float* t_vals,
                     void* workspace, size_t workspace_bytes, void* stream)
{
    const int st = check_transpose_args(m, k, nnz, rowptr, colind, vals, t_rowptr, t_colind, t_vals);
    if (st != DA_OK) return st;
    if (debug_validate() && m > 0) {
        const int v = da_csr_validate(m, k, nnz, rowptr, colind, stream);
        if (v != DA_OK) return v;
    }
    return enqueue_transpose(m, k, nnz, rowptr, colind, vals, t_rowptr, t_colind, t_vals, workspace, workspace_bytes, stream);
}

int da_csr_transpose_noalloc(int64_t m, int64_t k, int64_t nnz, const int32_t* rowptr, const int32_t* colind,
                             const float* vals, int32_t* t_rowptr, int32_t* t_colind, float* t_vals, void* stream)
{
    const int st = check_transpose_args(m, k, nnz, rowptr, colind, vals, t_rowptr, t_colind, t_vals);
    if (st != DA_OK) return st;
    if (plan_transpose(k, nnz).bytes > kScratchBytes)
        return fail(DA_ERR_UNSUPPORTED,
                    "da_csr_transpose_noalloc: the sort needs more than the library's 32 MiB static scratch "
                    "(about 24 bytes per stored entry); use da_csr_transpose with a workspace%s");
    void* ptr = nullptr;
    const int sp = scratch_address(&ptr);
    if (sp != DA_OK) return sp;
    return enqueue_transpose(m, k, nnz, rowptr, colind, vals, t_rowptr, t_colind, t_vals, ptr, kScratchBytes, stream);
}

}  // extern "C"

namespace {

int check_transpose_args(int64_t m, int64_t k, int64_t nnz, const int32_t* rowptr, const int32_t* colind,
                         const float* vals, int32_t* t_rowptr, int32_t* t_colind, float* t_vals)
{
    if (m < 0 || k < 0 || nnz < 0) return fail(DA_ERR_INVALID_ARG, "negative size%s");
    if (m > 0x7ffffffeLL || k > 0x7ffffffeLL || nnz > 0x7fffffffLL)
        return fail(DA_ERR_INVALID_ARG, "size beyond the int32 index range%s");
    if (!t_rowptr) return fail(DA_ERR_INVALID_ARG, "null t_rowptr%s");
    if (nnz > 0 && (m == 0 || k == 0)) return fail(DA_ERR_INVALID_ARG, "stored entries in a matrix without rows or columns%s");
    if (nnz > 0 && (!rowptr || !colind || !vals || !t_colind || !t_vals))
        return fail(DA_ERR_INVALID_ARG, "null array with nnz > 0%s");
    return DA_OK;
}

template <int ROUNDS>
void launch_transpose_passes(const TransposeFast& t, TransposePass P, int64_t k, int32_t* t_rowptr, float* t_vals,
                             char* ws, hipStream_t s) {
    const dim3 grid((unsigned)(8 * ((t.ntiles + 7) / 8))), block(kSortBlock);
    const bool wide = ROUNDS == 8 && P.n >= (1 << 30);      // as many entries always lie in the larger tiles
    unsigned* mid = reinterpret_cast<unsigned*>(ws + t.off_mid);
    float* mid_vals = reinterpret_cast<float*>(ws + t.off_vals);
    int* totals = reinterpret_cast<int*>(ws + t.off_total);
    P.hist = reinterpret_cast<int*>(ws + t.off_hist);
    P.tile_row = reinterpret_cast<int*>(ws + t.off_rows);
    P.group_hist = reinterpret_cast<int*>(ws + t.off_group);
    P.ntiles = t.ntiles; P.group = t.group;
    const float* vals = P.vals_in;
    for (int p = 0; p < t.passes; ++p) {
        const bool last = p == t.passes - 1;
        const int bins = 1 << t.bits[p];
        const size_t lds = transpose_scatter_lds<ROUNDS>(bins);
        P.bits = t.bits[p];
        P.total = totals + p * kDigitBinsMax;
        P.mid_in = mid;
        P.mid_out = mid;
        P.vals_in = p == 0 ? vals : mid_vals;
        P.vals_out = last ? t_vals : mid_vals;
        if (p == 0) hipLaunchKernelGGL((transpose_count_kernel<ROUNDS, true>), dim3((unsigned)t.ngroups), dim3(kCountBlock), 0, s, P);
        else hipLaunchKernelGGL((transpose_count_kernel<ROUNDS, false>), dim3((unsigned)t.ngroups), dim3(kCountBlock), 0, s, P);
        hipLaunchKernelGGL(transpose_scan_kernel, dim3((unsigned)(bins / kScanDigits)), dim3(1024), 0, s, P.group_hist, t.ngroups, bins,
                           P.total);
        // digits of 6 and 7 bits, A with few columns: all passes of 2 M entries, k = 50 22.5 us, 22.9 with the votes of 8 bits; k = 4000 47.6 and
        // 48.5; of 13 M, k = 50 60.9 and 62.7, k = 16 000 137.5 and 138.2
        auto scatter = [&](auto width, auto far) {
            constexpr int BITS = decltype(width)::value;
            constexpr bool WIDE = decltype(far)::value;
            if (p == 0 && last) hipLaunchKernelGGL((transpose_scatter_kernel<ROUNDS, true, true, BITS, WIDE>), grid, block, lds, s, P);
            else if (p == 0) hipLaunchKernelGGL((transpose_scatter_kernel<ROUNDS, true, false, BITS, WIDE>), grid, block, lds, s, P);
            else hipLaunchKernelGGL((transpose_scatter_kernel<ROUNDS, false, true, BITS, WIDE>), grid, block, lds, s, P);
        };
        if (wide) {
            if constexpr (ROUNDS == 8) scatter(Count<kDigitBitsMax>{}, Truth<true>{});
        } else if (P.bits <= 6) scatter(Count<6>{}, Truth<false>{});
        else if (P.bits == 7) scatter(Count<7>{}, Truth<false>{});
        else if (P.bits == 8) scatter(Count<8>{}, Truth<false>{});
        else if (P.bits == 9) scatter(Count<9>{}, Truth<false>{});
        else scatter(Count<kDigitBitsMax>{}, Truth<false>{});
    }
    if (t.passes == 1)
        hipLaunchKernelGGL(transpose_rowptr_one_kernel, dim3(1), dim3(256), 0, s, totals, 1 << t.bits[0], P.n, (int)k, t_rowptr);
    else
        hipLaunchKernelGGL((transpose_rowptr_kernel<kSortBlock * ROUNDS>), dim3(1u << t.bits[0]), dim3(256), 0, s, mid, P.n, (int)k, t.row_bits,
                           t.bits[0], t.bits[1], totals, P.hist, P.group_hist, totals + kDigitBinsMax, t.ntiles, t.group, t_rowptr);
}

// The radix passes of the transpose on the given scratch memory.  Every part of the scratch that
// a kernel reads was written earlier in the same call (entries between the passes, the whole
// histogram, totals or chunk sums), so stale contents of a reused buffer are never seen.
int enqueue_transpose(int64_t m, int64_t k, int64_t nnz, const int32_t* rowptr, const int32_t* colind,
                      const float* vals, int32_t* t_rowptr, int32_t* t_colind, float* t_vals,
                      void* workspace, size_t workspace_bytes, void* stream)
{
    if (nnz > 0 && (!workspace || workspace_bytes < plan_transpose(k, nnz).bytes))
        return fail(DA_ERR_INVALID_ARG, "workspace missing or smaller than da_csr_transpose_workspace reports%s");
    if (nnz > 0 && reinterpret_cast<uintptr_t>(workspace) % 256 != 0)
        return fail(DA_ERR_INVALID_ARG, "workspace is not 256-byte aligned%s");
    if (nnz > 0) {
        const TransposeFast f = plan_transpose_fast(m, k, nnz);
        if (f.usable && f.bytes <= workspace_bytes) {
            TransposePass P{};
            P.colind = colind; P.rowptr = rowptr; P.vals_in = vals; P.t_colind = t_colind;
            P.m = (int)m; P.n = (int)nnz; P.row_bits = f.row_bits;
            char* ws = static_cast<char*>(workspace);
            hipStream_t s = (hipStream_t)stream;
            if (f.tile == kSortBlock * 4) launch_transpose_passes<4>(f, P, k, t_rowptr, t_vals, ws, s);
            else launch_transpose_passes<8>(f, P, k, t_rowptr, t_vals, ws, s);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return hip_fail(e, "da_csr_transpose launch");
            return DA_OK;
        }
    }
    const TransposePlan t = plan_transpose(k, nnz);
    hipStream_t s = (hipStream_t)stream;
    const int n = (int)nnz;
    char* ws = static_cast<char*>(workspace);
    const int* sorted_keys = nullptr;
    if (n > 0) {
        int* keys[2] = {reinterpret_cast<int*>(ws + t.off_keys[0]), reinterpret_cast<int*>(ws + t.off_keys[1])};
        int* rows[2] = {reinterpret_cast<int*>(ws + t.off_rows[0]), reinterpret_cast<int*>(ws + t.off_rows[1])};
        float* vbuf[2] = {reinterpret_cast<float*>(ws + t.off_vals[0]), reinterpret_cast<float*>(ws + t.off_vals[1])};
        int* hist = reinterpret_cast<int*>(ws + t.off_hist);
        int* part = reinterpret_cast<int*>(ws + t.off_part);
        const int mask = (1 << t.digit_bits) - 1;
        const int* keys_in = colind;
        const int* rows_in = nullptr;
        const float* vals_in = vals;
        for (int p = 0; p < t.passes; ++p) {
            const int shift = p * t.digit_bits;
            const bool last = p == t.passes - 1;
            int* keys_out = keys[p & 1];
            int* rows_out = last ? t_colind : rows[p & 1];
            float* vals_out = last ? t_vals : vbuf[p & 1];
            hipLaunchKernelGGL(radix_count_kernel, dim3(t.nblocks), dim3(kSortBlock), 0, s, keys_in, n, shift, mask, hist,
                               t.nblocks);
            hipLaunchKernelGGL(scan_reduce_kernel, dim3((unsigned)t.parts), dim3(kSortBlock), 0, s, hist, t.hist_len, part);
            hipLaunchKernelGGL(scan_top_kernel, dim3(1), dim3(kSortBlock), 0, s, part, (int)t.parts);
            hipLaunchKernelGGL(scan_apply_kernel, dim3((unsigned)t.parts), dim3(kSortBlock), 0, s, hist, t.hist_len, part);
            if (p == 0)
                hipLaunchKernelGGL(radix_scatter_kernel<true>, dim3(t.nblocks), dim3(kSortBlock), 0, s, keys_in, rows_in,
                                   vals_in, n, shift, mask, hist, t.nblocks, keys_out, rows_out, vals_out, rowptr, (int)m);
            else
                hipLaunchKernelGGL(radix_scatter_kernel<false>, dim3(t.nblocks), dim3(kSortBlock), 0, s, keys_in, rows_in,
                                   vals_in, n, shift, mask, hist, t.nblocks, keys_out, rows_out, vals_out, rowptr, (int)m);
            keys_in = keys_out;
            rows_in = rows_out;
            vals_in = vals_out;
        }
        sorted_keys = keys_in;
    }
    hipLaunchKernelGGL(rowptr_from_sorted_kernel, dim3((unsigned)((k + 1 + kSortBlock - 1) / kSortBlock)), dim3(kSortBlock),
                       0, s, sorted_keys, n, (int)k, t_rowptr);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "da_csr_transpose launch");
    return DA_OK;
}

}  // namespace

extern "C" {

int da_eb_schedule_workspace(int64_t k, int64_t nnz, int unit, size_t* bytes)
{
    if (!bytes) return fail(DA_ERR_INVALID_ARG, "null bytes%s");
    if (k < 0 || nnz < 0 || unit < 1) return fail(DA_ERR_INVALID_ARG, "negative size or unit < 1%s");
    if (k > 0x7ffffffeLL || nnz > 0x7fffffffLL) return fail(DA_ERR_INVALID_ARG, "size beyond the int32 index range%s");
    if (k > (1LL << 30)) return fail(DA_ERR_UNSUPPORTED, "more than 2^30 columns%s");
    *bytes = plan_transpose(2 * k, (nnz + unit - 1) / unit).bytes;        // sort keys lie in [0, 2k)
    return DA_OK;
}

int da_eb_schedule(int64_t m, int64_t k, int64_t nnz, const int32_t* rowptr, const int32_t* colind, int unit,
                   int32_t* order, int32_t* first_segment, void* workspace, size_t workspace_bytes, void* stream)
{
    const ScheduleJob job{unit, order, first_segment, nullptr, nullptr, workspace, workspace_bytes};
    return enqueue_schedules(m, k, nnz, rowptr, colind, &job, 1, stream);
}

}  // extern "C"

namespace {

// Builds up to kMaxSortJobs schedules of one matrix side by side: every stage is one launch whose
// blockIdx.y selects the schedule, so four chunk sizes cost the launches of one.  The number of
// radix passes depends on k alone and is therefore the same for every job.
int enqueue_schedules(int64_t m, int64_t k, int64_t nnz, const int32_t* rowptr, const int32_t* colind,
                      const ScheduleJob* jobs, int njobs, void* stream)
{
    if (m < 0 || k < 0 || nnz < 0) return fail(DA_ERR_INVALID_ARG, "negative size or unit < 1%s");
    if (m > 0x7ffffffeLL || k > 0x7ffffffeLL || nnz > 0x7fffffffLL)
        return fail(DA_ERR_INVALID_ARG, "size beyond the int32 index range%s");
    if (k > (1LL << 30)) return fail(DA_ERR_UNSUPPORTED, "more than 2^30 columns%s");
    if (njobs < 1 || njobs > kMaxSortJobs) return fail(DA_ERR_INVALID_ARG, "number of schedules out of range%s");
    for (int i = 0; i < njobs; ++i)
        if (jobs[i].unit < 1) return fail(DA_ERR_INVALID_ARG, "negative size or unit < 1%s");
    if (nnz == 0) return DA_OK;
    if (m == 0) return fail(DA_ERR_INVALID_ARG, "stored entries in a matrix without rows%s");
    if (!rowptr || !colind) return fail(DA_ERR_INVALID_ARG, "null rowptr, colind or order%s");
    TransposePlan t[kMaxSortJobs];
    int n[kMaxSortJobs];
    int *keys[kMaxSortJobs][2], *ids[kMaxSortJobs][2];
    float* pad[kMaxSortJobs][2];
    KeyJobs kj{};
    unsigned max_units_blocks = 0, max_nblocks = 0, max_parts = 0;
    for (int i = 0; i < njobs; ++i) {
        const ScheduleJob& J = jobs[i];
        if (!J.order) return fail(DA_ERR_INVALID_ARG, "null rowptr, colind or order%s");
        const int64_t nunits = (nnz + J.unit - 1) / J.unit;
        t[i] = plan_transpose(2 * k, nunits);
        if (!J.workspace || J.workspace_bytes < t[i].bytes)
            return fail(DA_ERR_INVALID_ARG, "workspace missing or smaller than da_eb_schedule_workspace reports%s");
        if (reinterpret_cast<uintptr_t>(J.workspace) % 256 != 0)
            return fail(DA_ERR_INVALID_ARG, "workspace is not 256-byte aligned%s");
        char* ws = static_cast<char*>(J.workspace);
        for (int b = 0; b < 2; ++b) {
            keys[i][b] = reinterpret_cast<int*>(ws + t[i].off_keys[b]);
            ids[i][b] = reinterpret_cast<int*>(ws + t[i].off_rows[b]);
            pad[i][b] = reinterpret_cast<float*>(ws + t[i].off_vals[b]);
        }
        n[i] = (int)nunits;
        int* part = reinterpret_cast<int*>(ws + t[i].off_part);
        // without a caller's counter the chunk sums serve: they are free until the first scan
        kj.j[i] = KeyJob{J.unit, n[i], keys[i][0], ids[i][0], pad[i][0], J.first_segment ? J.first_segment : part, J.rows_by_unit};
        const unsigned ub = (unsigned)((n[i] + kSortBlock - 1) / kSortBlock);
        max_units_blocks = ub > max_units_blocks ? ub : max_units_blocks;
        max_nblocks = (unsigned)t[i].nblocks > max_nblocks ? (unsigned)t[i].nblocks : max_nblocks;
        max_parts = (unsigned)t[i].parts > max_parts ? (unsigned)t[i].parts : max_parts;
    }
    hipStream_t s = (hipStream_t)stream;
    const unsigned nj = (unsigned)njobs;
    hipLaunchKernelGGL(schedule_clear_kernel, dim3(1), dim3(64), 0, s, kj, njobs);
    hipLaunchKernelGGL(schedule_keys_kernel, dim3(max_units_blocks, nj), dim3(kSortBlock), 0, s, (int)m, (int)k, (int)nnz, rowptr,
                       colind, kj);
    const int mask = (1 << t[0].digit_bits) - 1;
    for (int p = 0; p < t[0].passes; ++p) {
        const int shift = p * t[0].digit_bits;
        const int in = p & 1, out = in ^ 1;
        const bool last = p == t[0].passes - 1;
        SortJobs sj{};
        for (int i = 0; i < njobs; ++i) {
            char* ws = static_cast<char*>(jobs[i].workspace);
            SortJob& S = sj.j[i];
            S.keys_in = keys[i][in]; S.rows_in = ids[i][in]; S.vals_in = pad[i][in];
            S.keys_out = keys[i][out];
            S.rows_out = last ? jobs[i].order : ids[i][out];
            // the last pass delivers the first rows of the chunks, in schedule order, where the caller wants them
            S.vals_out = (last && jobs[i].first_rows) ? reinterpret_cast<float*>(jobs[i].first_rows) : pad[i][out];
            S.hist = reinterpret_cast<int*>(ws + t[i].off_hist);
            S.part = reinterpret_cast<int*>(ws + t[i].off_part);
            S.hist_len = t[i].hist_len;
            S.n = n[i]; S.nblocks = t[i].nblocks; S.parts = (int)t[i].parts;
        }
        hipLaunchKernelGGL(radix_count_jobs_kernel, dim3(max_nblocks, nj), dim3(kSortBlock), 0, s, sj, shift, mask);
        hipLaunchKernelGGL(scan_reduce_jobs_kernel, dim3(max_parts, nj), dim3(kSortBlock), 0, s, sj);
        hipLaunchKernelGGL(scan_top_jobs_kernel, dim3(nj), dim3(kSortBlock), 0, s, sj);
        hipLaunchKernelGGL(scan_apply_jobs_kernel, dim3(max_parts, nj), dim3(kSortBlock), 0, s, sj);
        hipLaunchKernelGGL(radix_scatter_jobs_kernel, dim3(max_nblocks, nj), dim3(kSortBlock), 0, s, sj, shift, mask);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "da_eb_schedule launch");
    return DA_OK;
}

}  // namespace

extern "C" {

int da_spmm_release(const int32_t* rowptr)
{
    // the references are dropped outside the mutex: the last one frees device memory, which waits
    // for the device
    std::shared_ptr<DeviceBlock> dropped[32];
    {
        std::lock_guard<std::mutex> lk(g_plan_mu);
        int n = 0;
        for (auto& pl : g_plans)
            if (pl.block && (!rowptr || pl.rowptr == rowptr)) {
                dropped[n++] = std::move(pl.block);
                dropped[n++] = std::move(pl.heavy_block);
                pl = Plan{};
            }
    }
    return DA_OK;
}

}  // extern "C"

namespace {

// Heavy rows: a 32nd of all columns and more (at fewer, a row has so few entries in a band of B that the walk over the
// rows costs more than the entries).  Worth a kernel of their own where they hold most entries, every row of B serves
// at least 8 of them, and the other rows are even enough to be taken one by one.
constexpr int64_t kHeavyShare = 32, kHeavyMinCols = 16384, kHeavyMinEntries = 400000, kHeavyUses = 8;
constexpr int kHeavyMost = 8192, kHeavyCells = 2048, kRestLongest = 1024;   // at more than half as many rows half as many cells: 32 MB
constexpr double kRestLen = 64.0;

// Without the memory for it there is no list: it steers the launches of products, the orders do without it.
int no_heavy_rows() { (void)hipGetLastError(); return DA_OK; }

int plan_heavy_rows(int64_t m, int64_t k, int64_t nnz, const int32_t* rowptr, const int32_t* colind, hipStream_t s, Plan* pl)
try {
    if (k < kHeavyMinCols || nnz < kHeavyMinEntries || nnz >= (1LL << 30)) return DA_OK;
    const int min_len = (int)(k / kHeavyShare);
    DeviceBlock tmp;                                       // count and flag, sums, list
    const size_t tmp_bytes = 64 + kHeavyMost * sizeof(int);
    hipError_t e = hipMalloc(&tmp.p, tmp_bytes);
    if (e != hipSuccess) return no_heavy_rows();
    int* count = static_cast<int*>(tmp.p);
    unsigned long long* sums = reinterpret_cast<unsigned long long*>(count + 4);
    int* list = count + 16;
    struct { int count, unsorted, pad[2]; unsigned long long sq, mx; } host{};
    std::vector<int> rows;
    e = hipMemsetAsync(tmp.p, 0, 64, s);
    if (e == hipSuccess) {
        const long blocks = std::min<long>((m + 255) / 256, (long)cu_count() * 8);
        hipLaunchKernelGGL(heavy_rows_list_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (int)m, rowptr, min_len, kHeavyMost, list, sums, count);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(&host, tmp.p, sizeof host, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(e, "da_spmm_prepare");
    if (host.count < 1 || host.count > kHeavyMost || host.mx > (unsigned long long)kRestLongest) return DA_OK;
    // the lengths come with the rows' pointers, two at a time
    rows.resize(host.count);
    e = hipMemcpyAsync(rows.data(), list, rows.size() * sizeof(int), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    std::vector<int> ptr(2 * rows.size());
    DeviceBlock pairs;
    if (e == hipSuccess && hipMalloc(&pairs.p, 2 * rows.size() * sizeof(int)) != hipSuccess) return no_heavy_rows();
    if (e == hipSuccess) {
        hipLaunchKernelGGL(heavy_row_ends_kernel, dim3((unsigned)((rows.size() + 255) / 256)), dim3(256), 0, s, (int)rows.size(), list, rowptr,
                           static_cast<int*>(pairs.p));
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(ptr.data(), pairs.p, ptr.size() * sizeof(int), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(e, "da_spmm_prepare");
    int64_t entries = 0;
    std::vector<std::pair<int, int>> by_length(rows.size());
    for (size_t i = 0; i < rows.size(); ++i) {
        by_length[i] = {ptr[2 * i + 1] - ptr[2 * i], rows[i]};
        entries += by_length[i].first;
    }
    const double rest_len = nnz > entries ? (double)host.sq / (double)(nnz - entries) : 0.0;
    if (entries < kHeavyMinEntries || 2 * entries < nnz || entries < kHeavyUses * k || rest_len > kRestLen) return DA_OK;
    std::sort(by_length.begin(), by_length.end());         // neighbours walk side by side: rows of one length
    auto row_sums = std::make_shared<std::vector<int64_t>>(rows.size() + 1, 0);
    for (size_t i = 0; i < rows.size(); ++i) {
        rows[i] = by_length[i].second;
        (*row_sums)[i + 1] = (*row_sums)[i] + by_length[i].first;
    }

    const int64_t finest = rows.size() <= kHeavyMost / 2 ? kHeavyCells : kHeavyCells / 2;
    const int cell = (int)((k + finest - 1) / finest), cells = (int)((k + cell - 1) / cell);
    const size_t words = (size_t)(m + 31) / 32, n = rows.size();
    auto block = std::make_shared<DeviceBlock>();
    const size_t ints = ((n + 63) & ~size_t(63)) + ((words + 63) & ~size_t(63)) + n * (size_t)(cells + 1);
    if (hipMalloc(&block->p, ints * sizeof(int)) != hipSuccess ||
        hipHostMalloc(reinterpret_cast<void**>(&block->pinned), sizeof(int), hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) return no_heavy_rows();
    *block->pinned = 0;
    int* drows = static_cast<int*>(block->p);
    unsigned* bits = reinterpret_cast<unsigned*>(drows + ((n + 63) & ~size_t(63)));
    int* at = reinterpret_cast<int*>(bits + ((words + 63) & ~size_t(63)));
    e = hipMemsetAsync(bits, 0, words * sizeof(unsigned), s);
    if (e == hipSuccess) e = hipMemcpyAsync(drows, rows.data(), n * sizeof(int), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(heavy_cells_kernel, dim3((unsigned)n, 8), dim3(256), 0, s, rowptr, colind, drows, cells, cell, at, bits, count + 1);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(&host, tmp.p, sizeof host, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(e, "da_spmm_prepare");
    if (host.unsorted) return DA_OK;
    pl->heavy = HeavyPlan{drows, at, (int)n, cells, cell, min_len, (int)nnz, block->pinned};
    pl->heavy_k = k;
    pl->heavy_bits = bits;
    pl->rest_len = rest_len;
    pl->rest_longest = (int)host.mx;
    pl->heavy_sums = row_sums;
    pl->heavy_block = block;
    return DA_OK;
} catch (const std::bad_alloc&) {
    return DA_OK;
}

}  // namespace

extern "C" {

int da_spmm_prepare(int64_t m, int64_t k, int64_t nnz, const int32_t* rowptr, const int32_t* colind, void* stream)
{
    if (m < 0 || k < 0 || nnz < 0) return fail(DA_ERR_INVALID_ARG, "negative size%s");
    if (m > 0x7ffffffeLL || k > 0x7ffffffeLL || nnz > 0x7fffffffLL)
        return fail(DA_ERR_INVALID_ARG, "size beyond the int32 index range%s");
    if (m == 0 || nnz == 0) return DA_OK;
    if (!rowptr || !colind) return fail(DA_ERR_INVALID_ARG, "null rowptr or colind%s");
    if (debug_validate()) {
        const int v = da_csr_validate(m, k, nnz, rowptr, colind, stream);
        if (v != DA_OK) return v;
    }
    if (k > (1LL << 30)) { remember_matrix(rowptr, m, nnz, 0.0); return DA_OK; }    // no schedule for such widths
    Plan pl;
    pl.rowptr = rowptr; pl.colind = colind; pl.m = m; pl.nnz = nnz;
    size_t ints = 64, ws_bytes = 0, ws_off[kPlans];        // the first ints receive the segment sizes
    const int first_plan = nnz > kSmallPlanMaxNnz ? 1 : 0;
    for (int i = first_plan; i < kPlans; ++i) {
        pl.units[i] = (int)((nnz + kPlanUnits[i] - 1) / kPlanUnits[i]);
        ints += 3 * (size_t)((pl.units[i] + 63) & ~63);     // the order and, twice, the first rows of the chunks
        ws_off[i] = ws_bytes;                               // the sorts run side by side, each in its own part
        ws_bytes += align256(plan_transpose(2 * k, pl.units[i]).bytes);
    }
    pl.block = std::make_shared<DeviceBlock>();
    DeviceBlock ws;
    hipError_t e = hipMalloc(&pl.block->p, ints * sizeof(int));
    if (e != hipSuccess) return hip_fail(e, "hipMalloc");
    e = hipMalloc(&ws.p, ws_bytes);
    if (e != hipSuccess) return hip_fail(e, "hipMalloc");
    size_t off = 64;
    int* seg = static_cast<int*>(pl.block->p);
    ScheduleJob jobs[kPlans];
    for (int i = first_plan; i < kPlans; ++i) {
        pl.order[i] = seg + off;
        off += (size_t)((pl.units[i] + 63) & ~63);
        pl.first_row[i] = seg + off;
        off += (size_t)((pl.units[i] + 63) & ~63);
        pl.row_by_chunk[i] = seg + off;
        off += (size_t)((pl.units[i] + 63) & ~63);
        jobs[i] = ScheduleJob{kPlanUnits[i], pl.order[i], seg + i, pl.first_row[i], pl.row_by_chunk[i],
                              static_cast<char*>(ws.p) + ws_off[i], ws_bytes - ws_off[i]};
    }
    int status = enqueue_schedules(m, k, nnz, rowptr, colind, jobs + first_plan, kPlans - first_plan, stream);
    e = hipSuccess;
    int dev = 0;
    FeatureSlot sums;                                      // row lengths, for the launch geometry
    if (status == DA_OK) e = start_features(m, rowptr, (hipStream_t)stream, &dev, &sums);
    const bool summed = e == hipSuccess && status == DA_OK;
    if (e == hipErrorInvalidDevice) e = hipSuccess;        // no slots for that many devices: lengths stay unknown
    if (status == DA_OK && e == hipSuccess)
        e = hipMemcpyAsync(pl.first_units, seg, sizeof pl.first_units, hipMemcpyDeviceToHost, (hipStream_t)stream);
    if (e == hipSuccess) e = hipStreamSynchronize((hipStream_t)stream);
    if (status == DA_OK && e != hipSuccess) status = hip_fail(e, "da_spmm_prepare");
    double seen_len = 0.0;
    if (status == DA_OK && summed && arrived(sums)) seen_len = (double)sums.result->sq / (double)nnz;
    if (status == DA_OK && summed) give_slot(dev, sums); else free_slot(sums);
    if (status != DA_OK) return status;
    remember_matrix(rowptr, m, nnz, seen_len);
    if (seen_len >= (double)(k / kHeavyShare)) {
        const int hs = plan_heavy_rows(m, k, nnz, rowptr, colind, (hipStream_t)stream, &pl);
        if (hs != DA_OK) return hs;
    }
    std::shared_ptr<DeviceBlock> old, old_heavy;           // freed after the mutex is released
    {
        std::lock_guard<std::mutex> lk(g_plan_mu);
        Plan* slot = nullptr;
        for (auto& q : g_plans)
            if (q.block && q.rowptr == rowptr && q.m == m) { slot = &q; break; }  // an older plan of this matrix
        if (slot && slot->captured) {
            // A recorded graph reads the old orders on every replay: they stay.  When they describe
            // the same matrix shape the old plan simply remains in use; otherwise the new one takes
            // another slot and the old one lives on until da_spmm_release.
            if (slot->colind == colind && slot->nnz == nnz) return DA_OK;
            slot->rowptr = nullptr;                        // no longer found by lookups; memory kept
            slot = nullptr;
        }
        if (!slot) {
            for (int tries = 0; tries < 16 && !slot; ++tries) {
                Plan* cand = &g_plans[g_plan_next];
                g_plan_next = (g_plan_next + 1) % 16;
                if (!(cand->block && cand->captured)) slot = cand;
            }
            if (!slot) return DA_OK;                       // every slot is pinned by a graph: no plan for this matrix
        }
        old = std::move(slot->block);
        old_heavy = std::move(slot->heavy_block);
        *slot = pl;
    }
    return DA_OK;
}

namespace {
constexpr int64_t kDenseMaxRows = 1 << 30;         // the kernels count rows, and a block's rows past the end, in 32 bits
constexpr int64_t kDenseMaxCols = 1 << 20, kSumsMaxCols = 1 << 22;
constexpr int64_t kSplitMaxInner = 1 << 20, kSplitMaxCols = 1 << 14;

// Row blocks of the weight gradient: two blocks to a CU over all tiles, and no fewer than 64 rows each.
int weight_grad_blocks(int64_t rows, int64_t tiles) {
    int64_t nb = 2 * cu_count() / tiles;
    const int64_t most = (rows + 63) / 64;
    if (nb > most) nb = most;
    return (int)(nb < 1 ? 1 : nb);
}
int64_t weight_grad_tiles(int64_t fin, int64_t fout) {
    return ((fin + kWgTile - 1) / kWgTile) * ((fout + kWgTile - 1) / kWgTile);
}
}  // namespace

int da_spmm_weight_grad_workspace(int64_t rows, int64_t fin, int64_t fout, size_t* bytes)
{
    if (!bytes) return fail(DA_ERR_INVALID_ARG, "null bytes%s");
    if (rows < 0 || fin < 0 || fout < 0) return fail(DA_ERR_INVALID_ARG, "negative size%s");
    if (rows > kDenseMaxRows || fin > kDenseMaxCols || fout > kDenseMaxCols) return fail(DA_ERR_UNSUPPORTED, "size too large%s");
    const int64_t tiles = weight_grad_tiles(fin, fout);
    if (tiles > kMaxGridY) return fail(DA_ERR_UNSUPPORTED, "more than 65535 tiles%s");
    *bytes = tiles == 0 ? 0 : (size_t)tiles * weight_grad_blocks(rows, tiles) * kWgPart * sizeof(float);
    return DA_OK;
}

int da_spmm_weight_grad(int64_t rows, int64_t fin, int64_t fout, const float* X, int64_t ldx, const float* G, int64_t ldg,
                        float* dW, void* workspace, size_t workspace_bytes, void* stream)
{
    size_t need = 0;
    const int st = da_spmm_weight_grad_workspace(rows, fin, fout, &need);
    if (st != DA_OK) return st;
    if (fin < 4 || fout < 4) return fail(DA_ERR_UNSUPPORTED, "fewer than 4 columns%s");
    if (rows < 1) return fail(DA_ERR_UNSUPPORTED, "no rows%s");
    if (ldx < fin || ldg < fout) return fail(DA_ERR_INVALID_ARG, "leading dimension smaller than the extent it strides over%s");
    if (!X || !G || !dW) return fail(DA_ERR_INVALID_ARG, "null X, G or dW%s");
    if (!workspace || workspace_bytes < need || reinterpret_cast<uintptr_t>(workspace) % 16 != 0)
        return fail(DA_ERR_INVALID_ARG, "workspace missing, misaligned or smaller than da_spmm_weight_grad_workspace reports%s");
    const int64_t tiles = weight_grad_tiles(fin, fout);
    const int nb = weight_grad_blocks(rows, tiles);
    const int64_t per = ((rows + nb - 1) / nb + 15) / 16 * 16;      // whole turns of a wave, 16 rows
    hipStream_t s = (hipStream_t)stream;
    float* part = static_cast<float*>(workspace);
    hipLaunchKernelGGL(weight_grad_kernel, dim3((unsigned)nb, (unsigned)tiles), dim3(kWgBlock), 0, s, (int)rows, (int)fin,
                       (int)fout, X, (long)ldx, G, (long)ldg, (int)per, part);
    hipLaunchKernelGGL(weight_grad_sum_kernel, dim3(kWgTile, (unsigned)tiles), dim3(1024), 0, s, part, nb, (int)fin,
                       (int)fout, dW);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "da_spmm_weight_grad launch");
    return DA_OK;
}

// Row blocks of the column sums, and columns per block
static int column_sums_blocks(int64_t rows) {
    int64_t nb = 2 * cu_count();
    const int64_t most = (rows + 63) / 64;
    if (nb > most) nb = most;
    return (int)(nb < 1 ? 1 : nb);
}

int da_spmm_column_sums_workspace(int64_t rows, int64_t n, size_t* bytes)
{
    if (!bytes) return fail(DA_ERR_INVALID_ARG, "null bytes%s");
    if (rows < 0 || n < 0) return fail(DA_ERR_INVALID_ARG, "negative size%s");
    if (rows > kDenseMaxRows || n > kSumsMaxCols) return fail(DA_ERR_UNSUPPORTED, "size too large%s");
    *bytes = (size_t)column_sums_blocks(rows) * (size_t)n * sizeof(float);
    return DA_OK;
}

int da_spmm_column_sums(int64_t rows, int64_t n, const float* G, int64_t ldg, float* sums, void* workspace,
                        size_t workspace_bytes, void* stream)
{
    size_t need = 0;
    const int st = da_spmm_column_sums_workspace(rows, n, &need);
    if (st != DA_OK) return st;
    if (n == 0) return DA_OK;
    if (ldg < n) return fail(DA_ERR_INVALID_ARG, "leading dimension smaller than the extent it strides over%s");
    if ((rows > 0 && !G) || !sums) return fail(DA_ERR_INVALID_ARG, "null G or sums%s");
    if (!workspace || workspace_bytes < need || reinterpret_cast<uintptr_t>(workspace) % 16 != 0)
        return fail(DA_ERR_INVALID_ARG, "workspace missing, misaligned or smaller than da_spmm_column_sums_workspace reports%s");
    const int nb = column_sums_blocks(rows), lanes = n >= kCsBlock ? kCsBlock : pow2_ceil(n);
    const int64_t ny = (n + lanes - 1) / lanes;
    const int per = (int)((rows + nb - 1) / nb);
    hipStream_t s = (hipStream_t)stream;
    float* part = static_cast<float*>(workspace);
    hipLaunchKernelGGL(column_sums_kernel, dim3((unsigned)nb, (unsigned)ny), dim3(kCsBlock), 0, s, (int)rows, (int)n, lanes, G,
                       (long)ldg, per, part);
    hipLaunchKernelGGL(column_sums_sum_kernel, dim3((unsigned)((n + 63) / 64)), dim3(1024), 0, s, part, nb, (int)n, sums);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "da_spmm_column_sums launch");
    return DA_OK;
}

int da_spmm_bias_relu(int64_t rows, int64_t n, float* Z, const float* bias, int relu, void* stream)
{
    if (rows < 0 || n < 0 || n > 0x7fffffffLL) return fail(DA_ERR_INVALID_ARG, "bad size%s");
    if (rows == 0 || n == 0 || (!bias && !relu)) return DA_OK;
    if (!Z) return fail(DA_ERR_INVALID_ARG, "null Z%s");
    long blocks = (rows * n / 4 + 255) / 256;
    const long most = (long)cu_count() * 16;
    if (blocks > most) blocks = most;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(bias_relu_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, (long)rows, (int)n, Z, bias, relu);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "da_spmm_bias_relu launch");
    return DA_OK;
}

int da_spmm_dense(int64_t rows, int64_t k, int64_t n, const float* A, int64_t lda, const float* W, int64_t wk, int64_t wn,
                  float* C, int64_t ldc, void* stream)
{
    if (rows < 0 || k < 0 || n < 0) return fail(DA_ERR_INVALID_ARG, "negative size%s");
    if (rows > kDenseMaxRows || n > kDenseMaxCols) return fail(DA_ERR_UNSUPPORTED, "size too large%s");
    if (rows == 0 || n == 0) return DA_OK;
    if (k < 1) return fail(DA_ERR_UNSUPPORTED, "no columns in A%s");
    if (lda < k || ldc < n || wk < 1 || wn < 1) return fail(DA_ERR_INVALID_ARG, "leading dimension smaller than the extent it strides over%s");
    if (!A || !W || !C) return fail(DA_ERR_INVALID_ARG, "null A, W or C%s");
    hipStream_t s = (hipStream_t)stream;
    if (k > 256) return fail(DA_ERR_UNSUPPORTED, "weight matrix beyond what a block keeps in LDS%s");   // 130 KiB at 128 columns
    auto go = [&](auto nt, auto kmax) {
        constexpr int NT = decltype(nt)::value, KS = decltype(kmax)::value;
        const size_t lds = dense_lds<NT>((int)k);
        // blocks that are resident together (LDS, and 3 of 4 waves per SIMD by registers), each wave with
        // several sets of rows if there are as many
        const int64_t resident = (int64_t)cu_count() * std::min<int64_t>(3, (160 << 10) / (int64_t)lds);
        const int64_t ny = (n + 16 * NT - 1) / (16 * NT);
        int64_t nx = (rows + 63) / 64;
        if (nx * ny > resident) nx = std::max<int64_t>(1, resident / ny);
        hipLaunchKernelGGL((dense_product_kernel<NT, KS>), dim3((unsigned)nx, (unsigned)ny), dim3(kDpBlock), lds, s, (int)rows,
                           (int)n, (int)k, A, (long)lda, W, (long)wk, (long)wn, C, (long)ldc);
    };
    auto by_k = [&](auto nt) {
        if (k <= 64) go(nt, Count<4>{});
        else if (k <= 128) go(nt, Count<8>{});
        else go(nt, Count<16>{});
    };
    if (n <= 16) by_k(Count<1>{});
    else if (n <= 32) by_k(Count<2>{});
    else if (n <= 48) by_k(Count<3>{});
    else if (n <= 64) by_k(Count<4>{});
    else if (n <= 96) by_k(Count<6>{});
    else by_k(Count<8>{});
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "da_spmm_dense launch");
    return DA_OK;
}

int da_spmm_dense_split_workspace(int64_t k, int64_t n, size_t* bytes)
{
    if (!bytes) return fail(DA_ERR_INVALID_ARG, "null bytes%s");
    if (k < 0 || n < 0) return fail(DA_ERR_INVALID_ARG, "negative size%s");
    if (k > kSplitMaxInner || n > kSplitMaxCols) return fail(DA_ERR_UNSUPPORTED, "size too large%s");
    const size_t pieces = (size_t)split_steps((int)k) * (size_t)((n + 15) / 16);
    *bytes = pieces * kSplitBytes;
    return DA_OK;
}

int da_spmm_dense_split(int64_t rows, int64_t k, int64_t n, const float* A, int64_t lda, const float* W, int64_t wk, int64_t wn,
                        float* C, int64_t ldc, void* workspace, size_t workspace_bytes, void* stream)
{
    if (rows < 0) return fail(DA_ERR_INVALID_ARG, "negative size%s");
    size_t need = 0;
    const int st = da_spmm_dense_split_workspace(k, n, &need);
    if (st != DA_OK) return st;
    if (rows > kDenseMaxRows) return fail(DA_ERR_UNSUPPORTED, "size too large%s");
    if (rows == 0 || n == 0) return DA_OK;
    if (k < kSplitStep) return fail(DA_ERR_UNSUPPORTED, "fewer than 32 columns in A%s");
    if (lda < k || ldc < n || wk < 1 || wn < 1) return fail(DA_ERR_INVALID_ARG, "leading dimension smaller than the extent it strides over%s");
    if (!A || !W || !C) return fail(DA_ERR_INVALID_ARG, "null A, W or C%s");
    if (!workspace || workspace_bytes < need || reinterpret_cast<uintptr_t>(workspace) % 16 != 0)
        return fail(DA_ERR_INVALID_ARG, "workspace missing, misaligned or smaller than da_spmm_dense_split_workspace reports%s");
    hipStream_t s = (hipStream_t)stream;
    const int steps = split_steps((int)k), tiles = (int)((n + 15) / 16);
    bf16x8* frag = static_cast<bf16x8*>(workspace);
    unsigned* sizes = reinterpret_cast<unsigned*>(frag + (size_t)steps * tiles * 192);
    int* tiny = reinterpret_cast<int*>(sizes + (size_t)steps * tiles * 16);
    hipLaunchKernelGGL(dense_split_weights_kernel, dim3((unsigned)steps, (unsigned)tiles), dim3(64), 0, s, (int)k, (int)n, W, (long)wk,
                       (long)wn, frag, sizes, tiny);
    auto go = [&](auto nt) {
        constexpr int NT = decltype(nt)::value;
        hipLaunchKernelGGL((dense_split_kernel<NT>), dim3((unsigned)((rows + kSplitRows - 1) / kSplitRows), (unsigned)((tiles + NT - 1) / NT)),
                           dim3(kSplitBlock), 0, s, (int)rows, (int)n, (int)k, A, (long)lda, W, (long)wk, (long)wn, frag, sizes, tiny, tiles, C,
                           (long)ldc);
    };
    if (tiles <= 2) go(Count<2>{});
    else if (tiles <= 4) go(Count<4>{});
    else if (tiles <= 6) go(Count<6>{});
    else go(Count<8>{});
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "da_spmm_dense_split launch");
    return DA_OK;
}

const char* da_spmm_algo_name(int algo)
{
    return (algo >= 0 && algo < DA_NUM_ALGOS) ? kNames[algo] : nullptr;
}

const char* da_spmm_last_error(void) { return g_err; }

}  // extern "C"
