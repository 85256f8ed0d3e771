// Host side of libdgsp: argument checks, launch geometry, the selector.
// The C-ABI is documented in include/dgsp.h.
#include "../../include/dgsp.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <map>
#include <mutex>
#include <type_traits>
#include <utility>

#include "call_numbers.hpp"
#include "dgsp_internal.h"
#include "dgsp_kernels.hpp"
#include "stat_pool.hpp"

namespace {

using namespace dgsp;

// ---------------------------------------------------------------- device facts
struct DeviceInfo {
    int cus = 0;
};

DeviceInfo device_info() {
    static std::mutex mu;
    static DeviceInfo cache[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return DeviceInfo{256};
    std::lock_guard<std::mutex> lock(mu);
    if (cache[dev].cus == 0) {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
            cus = 256;
        cache[dev].cus = cus;
    }
    return cache[dev];
}

inline int ilog2_ceil(long long v) {   // smallest l with 2^l >= v  (v >= 1)
    int l = 0;
    while ((1LL << l) < v) ++l;
    return l;
}

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

inline unsigned clamp_blocks(long long want, long long cap) {
    if (want < 1) want = 1;
    return (unsigned)(want < cap ? want : cap);
}

// resident waves per CU assumed when sizing machine-filling grids
constexpr int kBlocksPerCu = 8;

static_assert((1 << kNbSrLogTile) == kNbSrTile, "tile must be a power of two");

// Rows count as "about equally long" for the launch geometry of the row-split sequential kernel when the
// caller's statistics give a coefficient of variation up to this (a property of the kernel's schedule, fixed
// here; the selector's thresholds are separate state and do not reach the launch code).
constexpr double kEvenRowsCvMax = 0.3;
// largest leading dimension of Y the balanced kernels take (a tile's rows are stored through 32-bit byte offsets)
constexpr int64_t kBalancedLdyMax = 1 << 20;

// What a caller's row statistics tell the launch code (nothing, when it passed none).
struct Hints {
    double col_span = 0.0;
    double cv_row = -1.0;
    int64_t max_row = -1;
    int64_t size = -1;          // a bound of the entry count
    bool chosen = false;        // the kernel is the library's choice from these statistics, not the caller's
    double saved_share = 0.0;   // what column blocks half as wide would save (kSavedShareMin); 0 = unknown
    const uint32_t* hot_columns = nullptr;      // the hot runs of a matrix of `hot_K` columns
    int64_t hot_K = 0;
    const dgsp_internal_hints_t* more = nullptr;     // for its workspace
    Hints() = default;
    explicit Hints(const dgsp_features_t* f, const dgsp_internal_hints_t* more = nullptr) : more(more) {
        if (f) { col_span = f->col_span; cv_row = f->cv_row; max_row = f->max_row; }
        if (more) saved_share = more->saved_share;
        if (f && more) { hot_columns = more->hot_columns; hot_K = f->K; }
    }
};

struct Problem {
    int M, N;
    int ldx, ldy;       // leading dimensions of X and Y in elements (>= N)
    long long K, nnz;   // nnz < 0: unknown on the host
    const int* rowptr; const int* colidx; const float* vals; const float* X; float* Y;
    hipStream_t stream;
    int phase = DGSP_PHASE_ALL;
    double col_span = 0.0;   // mean column span of a row / K; 0 = unknown
    double cv_row = -1.0;    // coefficient of variation of the row lengths; < 0 = unknown
    long long max_row = -1;  // entries of the longest row; < 0 = unknown
    long long size = -1;     // the entry count or, for launch geometry, a bound of it; < 0 = unknown
    double saved_share = 0.0;  // see Hints
    const uint32_t* hot_columns = nullptr;
    const dgsp_internal_hints_t* more = nullptr;
    int switches = 0;        // DGSP_ABL_* (measurement aids)
    bool scaled = false;     // Y = alpha * A X + beta * Y instead of Y = A X
    float alpha = 1.0f, beta = 0.0f;
};

// Vector width of the comparison kernel without LDS staging (rs_sr_direct_kernel) only: it uses plain
// float2 / float4 accesses, which need N, the leading dimensions and the addresses of X and Y to fit.
// The four kernels proper do not depend on alignment (see pr_vector_width, rs_sr_shape).
inline int direct_kernel_vector_width(const Problem& p) {
    if (p.switches & DGSP_ABL_SCALAR_DENSE_LOADS) return 1;
    int v = 1;
    if (p.N % 4 == 0 && aligned(p.X, 16) && aligned(p.Y, 16)) v = 4;
    else if (p.N % 2 == 0 && aligned(p.X, 8) && aligned(p.Y, 8)) v = 2;
    while (v > 1 && (p.ldx % v != 0 || p.ldy % v != 0)) v >>= 1;     // every row must start aligned
    return v;
}

// Dense columns per lane and pass of the parallel-reduction kernels: the widest of 4, 3, 2 that divides N (one
// dwordx4 / x3 / x2 access, taken at any dword address, so alignment and leading dimensions do not matter).
inline int pr_vector_width(int64_t N, int switches) {
    if (switches & DGSP_ABL_SCALAR_DENSE_LOADS) return 1;
    return N % 4 == 0 ? 4 : N % 3 == 0 ? 3 : N % 2 == 0 ? 2 : 1;
}
inline int pr_vector_width(const Problem& p) { return pr_vector_width(p.N, p.switches); }
// The same for the balanced parallel kernel, which also has eight columns per lane (two dwordx4 accesses): when 8
// divides N - one pass over A instead of two - and for N = 5, 6, 7 with the two groups of four overlapping.
inline int nb_pr_lane_width(int64_t N, int switches) {
    const int v = pr_vector_width(N, switches);
    if (v == 4 && N % 8 == 0) return 8;
    if (N >= 5 && N <= 7 && !(switches & DGSP_ABL_SCALAR_DENSE_LOADS)) return 8;
    return v;
}

#define DGSP_LAUNCH(kernel, grid, ...) DGSP_LAUNCH_THREADS(kernel, grid, kBlock, __VA_ARGS__)
#define DGSP_LAUNCH_THREADS(kernel, grid, threads, ...)                                       \
    do {                                                                                      \
        hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, p.stream, __VA_ARGS__);            \
        if (hipGetLastError() != hipSuccess) return DGSP_ERR_LAUNCH;                          \
    } while (0)

// ---------------------------------------------------------------- launch geometry helpers
// Workgroups of `kernel` that one CU keeps resident (registers and LDS decide).  The balanced
// kernels cut the work into equal shares per wave, so their grid must not exceed what runs at
// once: a workgroup that waits for a slot would start its share when the others are done.
template <typename K>
int resident_blocks_per_cu(K kernel) {
    static std::mutex mu;
    static std::map<std::pair<const void*, int>, int> cache;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 4;
    const auto key = std::make_pair(reinterpret_cast<const void*>(kernel), dev);
    std::lock_guard<std::mutex> lock(mu);
    auto it = cache.find(key);
    if (it != cache.end()) return it->second;
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, kBlock, 0) != hipSuccess || n <= 0) n = 4;
    cache[key] = n;
    return n;
}

// ---------------------------------------------------------------- row-split launches
// Workgroups whose waves stride over `groups` groups of rows: at most `cap`, and so many that the rounds are equal.  An
// incomplete last round would be neighbouring groups, which xcd_contiguous gives to one or two XCDs, and would take as long
// as a full one.  `cap` workgroups against equal rounds: 573 735 rows of 60 at N = 2 326 -> 219 us, 27-point stencil on
// 106^3 at N = 1 / 2 76 / 90 -> 54 / 64 us, on 84^3 at N = 21 146 -> 97 us.
inline unsigned even_round_blocks(long long groups, long long cap) {
    const long long blocks = (groups + kWavesPerBlock - 1) / kWavesPerBlock;
    const long long rounds = blocks > cap ? (blocks + cap - 1) / cap : 1;
    return clamp_blocks((blocks + rounds - 1) / rounds, cap);
}

// X can be addressed with 32-bit byte offsets (through a buffer descriptor)
constexpr unsigned long long kL2BytesPerXcd = 4ull << 20;      // gfx950: 4 MB of L2 per XCD

inline bool x_fits_descriptor(const Problem& p) {
    return dense_bytes(p.K, p.ldx, p.N) <= 0xffffffffull;
}

template <int V, bool XBUF>
int launch_rs_pr_v(const Problem& p) {
    const int logG = p.nnz >= 0 ? pr_lanes_log2(p.nnz, p.M) : -1;
    // one wave per row group when lanes-per-row is known; else assume the
    // finest split the kernel may choose (2 lanes per row) and let waves stride
    const int rows_per_wave = (kWave >> (logG >= 0 ? logG : 1)) * kRsPrUnroll;
    const long long groups = ((long long)p.M + rows_per_wave - 1) / rows_per_wave;
    const long long cap = (long long)device_info().cus * kBlocksPerCu * 8;
    const dim3 grid(even_round_blocks(groups, cap));
    if (p.scaled) {
        DGSP_LAUNCH((rs_pr_kernel<V, XBUF, true>), grid, p.M, p.K, p.N, p.ldx, p.ldy, p.rowptr, p.colidx, p.vals, p.X,
                    p.Y, logG, Scaling{p.alpha, p.beta});
        return DGSP_OK;
    }
    DGSP_LAUNCH((rs_pr_kernel<V, XBUF>), grid, p.M, p.K, p.N, p.ldx, p.ldy, p.rowptr, p.colidx, p.vals, p.X, p.Y, logG);
    return DGSP_OK;
}

int launch_rs_pr(const Problem& p) {
    const bool xb = x_fits_descriptor(p);
    switch (pr_vector_width(p)) {
        case 4: return xb ? launch_rs_pr_v<4, true>(p) : launch_rs_pr_v<4, false>(p);
        case 3: return xb ? launch_rs_pr_v<3, true>(p) : launch_rs_pr_v<3, false>(p);
        case 2: return xb ? launch_rs_pr_v<2, true>(p) : launch_rs_pr_v<2, false>(p);
        default: return xb ? launch_rs_pr_v<1, true>(p) : launch_rs_pr_v<1, false>(p);
    }
}

// lanes per row of the sequential kernels: enough lanes of width V to span N, at most a wave
inline int sr_lanes_log2(long long N, int V, int cap = 6) {
    const long long need = (N + V - 1) / V;
    const int lg = ilog2_ceil(need);
    return lg > cap ? cap : lg;
}

// Column blocks of the sequential kernels.  A group of G lanes (a power of two) walks the entries once per block,
// so a call costs about blocks * G lane-steps per entry, and every further pass over the matrix costs more than
// its share (measured +15 ... +33 % per extra pass at equal blocks * G).  The blocks are made equally wide (three
// blocks for N = 300 are 100 + 100 + 100, not 128 + 128 + 44).  `narrow`: N is a multiple of 64 and the caller
// wants blocks of 64 columns, all lanes busy in every block (see the launch functions for when that pays).
struct SrColumns { int logG; int cols_per_block; unsigned blocks; };
inline SrColumns sr_columns(long long N, int V, bool narrow) {
    const long long lanes = (N + V - 1) / V;
    long long blocks = 1;
    if (narrow && N % 64 == 0) {
        blocks = N / 64;
    } else {
        double best = 0.0;
        for (int lg = 0; lg <= 6; ++lg) {
            const long long b = (lanes + (1ll << lg) - 1) >> lg;
            const double cost = (double)(b << lg) * (1.0 + 0.3 * (double)(b - 1));
            if (lg == 0 || cost <= best) { best = cost; blocks = b; }         // ties: the wider group, fewer passes
        }
    }
    const long long per = (((N + blocks - 1) / blocks + V - 1) / V) * V;        // a multiple of V
    return {sr_lanes_log2(per, V), (int)per, (unsigned)((N + per - 1) / per)};
}

// Dense-row loads in flight per lane of the sequential kernels: enough to fill, not to overflow,
// the L1 when rows of X are scattered (about 1 KB per wave: 4 / V loads), four when the matrix is
// known to be banded (neighbouring rows then share their rows of X and mostly hit in cache).
inline bool even_rows(const Problem& p) { return p.cv_row >= 0.0 && p.cv_row <= kEvenRowsCvMax; }
constexpr double kBandedSpan = 0.05;
inline bool banded(const Problem& p) { return p.col_span > 0.0 && p.col_span <= kBandedSpan; }

// The sequential kernels give a lane four dense columns whenever a row has four: the memory pipeline takes
// dwordx2 / dwordx4 accesses at any dword address, so neither the alignment of X and Y nor their leading
// dimensions restrict the width.  When N is not a multiple of four the last lane of a row takes the row's last
// four columns; those it shares with its neighbour are the neighbour's to add or to scale (RAGGED).
struct SrShape { int v; bool ragged; };
// dense-row loads in flight per lane of the balanced kernel at one and two columns (see banded())
template <int V> constexpr int sr_depth_scattered() { return V == 2 ? 2 : 4; }

// Lines of 128 bytes that `cols` consecutive columns of a row of X touch, on average over the rows.
inline double lines_per_row(long long cols, long long ldx) {
    const long long bytes = cols * 4, pitch = ldx * 4;
    if (pitch % 128 == 0 || 128 % pitch == 0) return (double)((bytes + 127) / 128);
    return (double)(bytes - 4) / 128.0 + 1.0;
}

// Do the rows sweep X in step?  Row-split waves that start together, one lane group per row and one dense-row load in
// flight each, walk their (ascending, scattered) columns at the same pace, so that at any time they touch a narrow band of
// X and find it in the L2; more loads in flight, or several lanes on a row's entries, widen the band until it no longer
// fits.  In step, a call is a chain of dependent loads; out of step it is bound by the lines that the gathers fetch, the
// dearer the more of them the L2 (4 MB) misses.  Both costs are fitted, to 15 % or so, on random columns of X from 3 to
// 40 MB, N = 1 to 128, 65 536 to 524 288 rows (`occ`: share of the wave slots in use, `part`: lines per wave / 64):
//   a step in step      0.1 us + 0.4 us * (1 - occ) + part * (2.6 us * occ + 1.5 us * missed)
//   a line out of step  5.7 ps + 5 ps * missed + 6 ps * missed^2
// 262 144 rows of 30, X of 2 / 4 / 8 / 16 MB at N = 4, in step against out of step: 45 / 49 / 59 / 75 against 40 / 47 / 78 /
// 109 us; X of 0.25 / 1 / 4 MB at N = 1 37 / 44 / 49 against 34 / 39 / 46 us; 131 072 rows of 60 at N = 33 (17 MB) 108 against
// 203 us, 262 144 Poisson rows of 12 there 103 against 92 us; 131 072 rows of 60 at N = 1 (1 MB) 105 against 38 us.  On 94
// matrices of such rows (X of 0.25 to 268 MB, N = 1 to 64) the choice loses 0.6 % to the better of the two (always out of step
// 10 %, always in step 24 %; the worst, Poisson rows of 12 with 8 MB of X, 16 %).
constexpr double kWaveSlotsPerCu = 32.0;
inline bool rows_in_step(const Problem& p, const SrColumns& cols) {
    const double lines = lines_per_row(cols.cols_per_block, p.ldx);
    // columns of a wider matrix come with the lines around them (64 378 rows of 15, 18 of 33 columns, N * K of 4.6 MB, lines of
    // 8.5 MB: in step 13.9, out of step 18.0 us)
    const double x_bytes = (double)p.K * std::fmin(p.ldx * 4.0, lines * cols.blocks * 128.0);
    const double missed = x_bytes > (double)kL2BytesPerXcd ? 1.0 - (double)kL2BytesPerXcd / x_bytes : 0.0;
    if (banded(p) || p.nnz == 0) return false;
    if (p.nnz < 0) return missed > 0.0;                        // entry count unknown: rows taken to be long and alike
    const double avg = (double)p.nnz / (double)p.M;
    const double longest = p.cv_row > 0.0 ? avg * (1.0 + 2.5 * p.cv_row) : avg;      // of the rows a wave walks together
    const double rows_per_wave = (double)(kWave >> cols.logG);
    const double rounds = (double)p.M / rows_per_wave * cols.blocks / (device_info().cus * kWaveSlotsPerCu);
    const double occ = std::fmin(rounds, 1.0);
    const double part = rows_per_wave * lines / 64.0;
    const double step = 0.1 + 0.4 * (1.0 - occ) + part * (2.6 * occ + 1.5 * missed);
    // a wave's rows beyond four rounds of its LDS tile: too few of them walk at a time
    const double overflow = std::fmax(1.0, rows_per_wave * avg / (4.0 * kRsSrTile));
    const double in_us = step * longest * std::fmax(rounds, 1.0) * std::pow(overflow, 0.75);
    const double out_us = (double)p.nnz * lines * cols.blocks * (5.7e-6 + (5.0e-6 + 6.0e-6 * missed) * missed);
    return 1.05 * in_us < out_us;
}

// log2 of the lanes that share a row's entries (H) when 2^logG lanes span its columns.  A wave's rows should fit one
// round of the LDS tile: with 64 rows of 27 a round holds 19 of them and the other lanes wait (27-point stencil on 128^3,
// H = 1 / 2 / 4 / 8: N = 1 117 / 100 / 94 / 119 us, N = 4 174 / 132 / 114 / 125 us).  A matrix that leaves the machine half
// empty is split further while a lane keeps two entries (4500 rows of 30: H = 2 / 4 / 8 4.9 / 3.8 / 3.7 us), uneven rows for
// the longest one's sake (32 768 lognormal rows of 8 at N = 4: H = 4 / 8 / 16 15.7 / 9.9 / 7.8 us).  On 3665 drawn matrices
// the choice loses 3.1 % to the best of H = 1 ... 16 (H = 1 92 %); 10 % of them lose more than 10 %.
// dense-row loads in flight per lane out of step; at one column per lane eight are as many registers as two at four
// columns (stencil 128^3 at N = 1: 94 us with four or eight)
constexpr int rs_sr_depth(int v) { return v == 1 ? 8 : 4; }
constexpr double kRowGroupCvMax = 0.6;
inline int rs_sr_split_log2(const Problem& p, int logG) {
    if (p.nnz < 0 || p.M == 0) return 0;
    const double avg = (double)p.nnz / (double)p.M;
    int logH = 0;
    for (; logG + logH < 6; ++logH) {
        const int rows = kWave >> (logG + logH);
        if (p.max_row >= 0 && (double)rows * (double)p.max_row <= (double)kRsSrTile) break;
        const double spread = p.cv_row >= 0.0 ? 2.0 * p.cv_row * avg * std::sqrt((double)rows) : 0.1 * rows * avg;
        if (rows * avg + spread <= (double)kRsSrTile) break;
    }
    // waves: two per SIMD, or with uneven rows, whose longest keep their lanes busy when the others are done, as many as fit
    const double few = device_info().cus * (p.cv_row > kRowGroupCvMax ? kWaveSlotsPerCu : 8.0);
    while (logG + logH < 6 && (double)p.M * (double)(1 << (logG + logH)) < few * kWave &&
           (avg >= (double)(4 << logH) || p.max_row >= (16ll << logH))) ++logH;
    return logH;
}

// Do waves that stage go before those that walk (rs_sr_kernel)?  Where the gathers go past the L1, yes; on a band the
// neighbours' walks find their lines in the L1 while they are at it, and what there is to wait for are the streams.  Staging
// level with the walk / first: 262 144 rows of 64 uniform columns at N = 1 / 2 / 4 85 / 91 / 103 against 76 / 79 / 93 us,
// 50 001 Poisson rows of 40 over 8000 columns at N = 4 / 16 13.3 / 15.6 against 11.0 / 13.8 us; 27-point stencil on 81^3 at
// N = 2 / 4 / 5 / 8 / 12 / 16 / 32 27.6 / 30.3 / 36.5 / 38.4 / 51.0 / 56.4 / 93.5 against
// 31.2 / 33.2 / 37.5 / 38.7 / 49.8 / 53.9 / 91.1 us. Unknown columns are taken for a band.
inline bool staging_first(const Problem& p, int logG) { return p.col_span > kBandedSpan || logG >= 2; }

template <int V, bool XBUF, int DEPTH, bool RAGGED>
int launch_rs_sr_v(const Problem& p, const SrColumns& cols, int logH) {
    const int logG = cols.logG;
    const unsigned col_blocks = cols.blocks;
    if (col_blocks > 65535u) return DGSP_ERR_INVALID_ARG;
    const int rows_per_wave = kWave >> (logG + logH);
    const long long groups = ((long long)p.M + rows_per_wave - 1) / rows_per_wave;
    const long long cap = (long long)device_info().cus * kBlocksPerCu * 8;
    const dim3 grid(even_round_blocks(groups, cap), col_blocks);
    const int first = staging_first(p, logG);
    if (p.scaled) {
        DGSP_LAUNCH((rs_sr_kernel<V, XBUF, DEPTH, true, RAGGED>), grid, p.M, p.K, p.N, p.ldx, p.ldy, p.rowptr, p.colidx, p.vals,
                    p.X, p.Y, logG, logH, cols.cols_per_block, first, Scaling{p.alpha, p.beta});
        return DGSP_OK;
    }
    DGSP_LAUNCH((rs_sr_kernel<V, XBUF, DEPTH, false, RAGGED>), grid, p.M, p.K, p.N, p.ldx, p.ldy, p.rowptr, p.colidx, p.vals, p.X,
                p.Y, logG, logH, cols.cols_per_block, first);
    return DGSP_OK;
}

template <int V>
int launch_rs_sr_direct_v(const Problem& p) {
    // the same column blocks as the kernel it is compared with
    const SrColumns cols = sr_columns(p.N, V, even_rows(p) && p.N >= 128);
    const int logG = cols.logG;
    const unsigned col_blocks = cols.blocks;
    if (col_blocks > 65535u) return DGSP_ERR_INVALID_ARG;
    const int rows_per_wave = kWave >> logG;
    const long long groups = ((long long)p.M + rows_per_wave - 1) / rows_per_wave;
    const long long cap = (long long)device_info().cus * kBlocksPerCu * 8;
    const dim3 grid(even_round_blocks(groups, cap), col_blocks);
    DGSP_LAUNCH((rs_sr_direct_kernel<V>), grid, p.M, p.N, p.ldx, p.ldy, p.rowptr, p.colidx, p.vals, p.X, p.Y, logG,
                cols.cols_per_block);
    return DGSP_OK;
}

// Dense columns per lane of the row-split sequential kernel: four, the last lane's window overlapping its neighbour's
// when four does not divide N; three where it divides N = 3 or 6 (N = 3 as three lanes of one column, one lane of four
// idle: stencil 80^3 42 us, against 37 us at N = 4).
inline SrShape rs_sr_shape(const Problem& p) {
    if (p.switches & DGSP_ABL_SCALAR_DENSE_LOADS) return {1, false};
    if (p.N == 3 || p.N == 6) return {3, false};
    if (p.N < 4) return {p.N, false};
    return {4, p.N % 4 != 0};
}

// Where the library chooses: may the row-group kernel (rs_sr_kernel) take the place of the kernel that the selection rules
// name?  Its H lanes on a row's entries are a parallel reduction too, it needs no search, no row marks, no prepare launch and
// no atomics, and its entries arrive coalesced through LDS; it does nothing against rows longer than the others but give a
// row more lanes.
//   Rows more or less alike, up to four columns: equal runs of rows are equal shares of entries.  Against rs_pr: 4096 rows
//   of 8 at N = 4 5.9 -> 3.9 us, 20 000 rows of 100 at N = 1 15.4 -> 10.3 us; against nb_pr: 27-point stencil on 128^3 at
//   N = 1 / 4 122 / 137 -> 94 / 114 us, 776 379 rows of 22 over 27 098 columns at N = 1 79 -> 60 us, 187 500 Poisson rows of
//   8 at N = 4 17.7 -> 12.9 us; 262 144 rows of 64 at N = 1 85 -> 76 us.
//   Small matrices with uneven rows: the balanced kernels' start (searches, row marks, perhaps two launches) is most of
//   the call, and the longest row is `steps` rounds of loads for its lanes.  Lognormal rows of 8, row groups against the
//   better of nb_sr and nb_pr: 8192 rows at N = 1 / 4 / 16 / 33 4.0 / 4.1 / 5.4 / 6.4 against 6.9 / 6.6 / 7.0 / 9.5 us,
//   65 536 rows at N = 1 / 4 / 8 / 16 8.7 / 10.7 / 16 / 35 against 8.5 / 10.2 / 10.3 / 13.8 us; crossover near 500 000
//   entries at N <= 4 (150 000 rows of 8: 20 against 13.6 us).
//   Where row groups took the rules' kernel's place on 1276 drawn matrices, that kernel took 20 % longer on average; on 6 %
//   of them it would have been more than 10 % faster.
constexpr long long kSmallUnevenNnz = 600000, kTinyNnz = 130000;
inline bool row_groups_suit(const Problem& p) {
    if (p.switches != 0 || p.nnz <= 0 || p.M == 0 || p.cv_row < 0.0 || p.max_row < 0) return false;
    const double avg = (double)p.nnz / (double)p.M;
    if (p.cv_row <= kRowGroupCvMax && (double)p.max_row <= 8.0 * avg + 64.0) return p.N <= 4;
    if (p.nnz > kSmallUnevenNnz) return false;
    const int v = rs_sr_shape(p).v;
    const int lanes_log2 = rs_sr_split_log2(p, sr_columns(p.N, v, false).logG);
    // rounds of loads for the longest row, and the rounds of the LDS tile (six times as long) that it takes
    const double steps = (double)p.max_row / (double)(rs_sr_depth(v) << lanes_log2) + 6.0 * (double)(p.max_row / kRsSrTile);
    return steps <= (p.N <= 4 ? 16.0 : p.nnz <= kTinyNnz ? 12.0 : 8.0);
}

template <int V, bool RAGGED>
int launch_rs_sr_pick(const Problem& p) {
    const bool xb = x_fits_descriptor(p);
    // Rows of about equal length (what the selection rules send here) and N a multiple of 64: column blocks of 64
    // dense columns as in the balanced kernel, four rows per wave in step; 2-16 % faster at N >= 128 on such matrices.
    // With long rows among short ones the rows of a wave wait for the longest (+30 % measured), and without row
    // statistics nothing is known: then a group spans the whole width.
    const SrColumns cols = sr_columns(p.N, V, even_rows(p) && p.N >= 128);
    if (rows_in_step(p, cols)) return xb ? launch_rs_sr_v<V, true, 1, RAGGED>(p, cols, 0) : launch_rs_sr_v<V, false, 1, RAGGED>(p, cols, 0);
    const int logH = rs_sr_split_log2(p, cols.logG);
    constexpr int D = rs_sr_depth(V);
    return xb ? launch_rs_sr_v<V, true, D, RAGGED>(p, cols, logH) : launch_rs_sr_v<V, false, D, RAGGED>(p, cols, logH);
}

int launch_rs_sr(const Problem& p) {
    if (p.switches & DGSP_ABL_NO_SPARSE_STAGING) {
        switch (direct_kernel_vector_width(p)) {
            case 4: return launch_rs_sr_direct_v<4>(p);
            case 2: return launch_rs_sr_direct_v<2>(p);
            default: return launch_rs_sr_direct_v<1>(p);
        }
    }
    const SrShape shape = rs_sr_shape(p);
    switch (shape.v) {
        case 4: return shape.ragged ? launch_rs_sr_pick<4, true>(p) : launch_rs_sr_pick<4, false>(p);
        case 3: return launch_rs_sr_pick<3, false>(p);
        case 2: return launch_rs_sr_pick<2, false>(p);
        default: return launch_rs_sr_pick<1, false>(p);
    }
}

// ---------------------------------------------------------------- balanced launches
// Two rows a thread where chunks' first rows are wanted and there are enough rows: nearly every wave has a row at a chunk's start and
// goes through all of the kernel for it, and with 16 waves a SIMD that is what it takes (R-MAT 2^20 x 16 at N = 32 / 128, one / two
// / four rows a thread 9.5 / 6.8 / 9.1 and 11.8 / 11.2 / 14.0 us, with the zeros a dword at a time).  Fewer rows end later than they save
// (2^18 x 16 at N = 128 5.9 / 6.9 us, 2^19 x 16 6.1 / 6.1 us); without queues it is two to three trips to memory either way
// (2^20 x 16 at N = 1 4.9 / 4.8 us, and the product behind it 0.5 us later), and the scaled form's rows without entries want the waves.
constexpr long long kTwoRowsMin = 1 << 19;
// Zeroes (scaled form: multiplies by beta) the rows split by the `parts` chunks the main kernel derives
// (quanta of 2^quantum_log2 items), cut into tiles of 2^tile_log2 items (tile_log2 < 0: not cut further).
int launch_prepare(const Problem& p, unsigned parts, unsigned quantum_log2, int tile_log2, ChunkQueues queues = ChunkQueues{},
                   int empty_rows = 0) {
    const float beta = p.scaled ? p.beta : 0.0f;
    const auto launch = [&](auto with_queues, auto rows) -> int {
        constexpr int R = decltype(rows)::value;
        const dim3 grid((unsigned)(((long long)p.M + kBlock * R - 1) / (kBlock * R)));
        DGSP_LAUNCH((nb_prepare_kernel<decltype(with_queues)::value, R>), grid, p.M, p.N, p.ldy, p.rowptr, p.Y, parts, quantum_log2,
                    tile_log2, beta, queues, empty_rows);
        return DGSP_OK;
    };
    if (queues.starts && p.M >= kTwoRowsMin && !empty_rows) return launch(std::true_type{}, std::integral_constant<int, 2>{});
    return queues.starts ? launch(std::true_type{}, std::integral_constant<int, 1>{})
                         : launch(std::false_type{}, std::integral_constant<int, 1>{});
}

// How `waves` waves on each XCD share out the items (`lists` times: column blocks that are a grid dimension) with the help of
// memory of the caller's; nothing if it has none to give or where a wave's share is below `least` items.  About half of a share is its
// first piece, the rest goes by chunks of 512 items, 1024 from shares of 4096 on.  With 0.3 / 0.5 to 0.6 of the share R-MAT 2^20 x 16 at N = 32 / 64 / 128
// 227.7 / 440.1 / 872.4 and 225.9 / 440.2 / 868.7 us, 2^20 x 8 at N = 41 240.6 and 237.5 us, 2^19 x 16 at N = 100 397.4 and
// 390.4 us (0.8 of it at N = 128 1018 us, equal shares 1024 us); N = 32 with chunks of 256 / 512 / 768 / 1024 items 244 / 230 / 228.5 /
// 227 us (equal shares 248 us), and no better with chunks of 1024 first and smaller ones at the end (237 us and more): what a
// chunk costs beyond its entries, two shared rows and four trips to memory, is more than the ends lie apart.  Powers of two,
// so that the prepare launch knows rows within a chunk by a shift: 2^19 x 16 at N = 100, scaled, 475.5 -> 473 us, 2^20 x 16 at
// N = 32 228.7 -> 228.0 us.
constexpr double kFirstPiece = 0.55;
constexpr unsigned kQueueHelpers = 256;      // waves of an XCD that help others out: 0 / 32 / 128 of 512 at N = 128 1045 / 1018 / 969 us
ChunkQueues make_queues(const Problem& p, unsigned parts, unsigned waves, unsigned lists, long long least, unsigned fewest_a_row) {
    ChunkQueues q{};
    const long long items = p.size + (long long)p.M, share = items / parts / waves;
    if (share < least) return q;
    const unsigned size_log2 = share >= 4096 ? 10 : 9;
    const long long chunks = (items + (1ll << size_log2) - 1) >> size_log2;
    const unsigned run = (unsigned)((double)(chunks / parts) * kFirstPiece / waves);
    const size_t counters = (size_t)kXcd * lists;
    if (run == 0 || !p.more || !p.more->workspace || p.phase != DGSP_PHASE_ALL || p.switches != 0 ||
        (chunks << size_log2) > 0xffffffffll) return q;
    const size_t head = counters * kQueuePitch * sizeof(unsigned);
    char* mem = static_cast<char*>(p.more->workspace(p.more->context, head + (size_t)(chunks + 1) * sizeof(int)));
    if (!mem) return q;
    q.taken = reinterpret_cast<unsigned*>(mem);
    q.starts = reinterpret_cast<int*>(mem + head);
    q.chunks = (unsigned)chunks;
    q.size_log2 = size_log2;
    q.counters = (unsigned)counters;
    q.parts_log2 = (unsigned)__builtin_ctz(parts); q.waves = waves; q.run = run; q.helpers = kQueueHelpers;
    q.parts_per_chunk = (float)parts / (float)chunks;
    q.per_run = 1.0f / (float)run;
    q.fewest = (unsigned)(least * parts * waves); q.fewest_a_row = fewest_a_row;
    return q;
}

// Words by which the waves of `chunks` chunks (all column groups') agree on the rows they share, in memory of the call's; none if
// it has none to give or there would be more than `most` of them (the prepare launch clears these rows then).  Up to 1 MB in any
// case, what torch's allocator takes from its small blocks.
constexpr size_t kSharedWordsMax = 1 << 17;
inline bool may_share(const Problem& p) { return p.more && p.more->workspace && p.phase == DGSP_PHASE_ALL && p.switches == 0; }
RowSharing make_sharing(const Problem& p, size_t chunks, size_t most = kSharedWordsMax) {
    if (!may_share(p) || chunks > std::min(most, kSharedWordsMax)) return RowSharing{nullptr, 0};
    void* mem = p.more->workspace(p.more->context, chunks * sizeof(RowWord));
    return RowSharing{static_cast<RowWord*>(mem), mem ? next_call_number() : 0};
}

// Blocks of the grid that shares the nnz + M merge-path items of a balanced kernel, `tile` items per
// tile.  The gathers of a CU go through one L1 whose capacity for outstanding misses bounds them,
// whatever the number of waves, so CUs must finish together: the grid is a whole multiple of the CU
// count (544 blocks on 256 CUs ran 25 % slower than 512).  A matrix too small for one tile per wave
// on every CU gets one wave per tile.  Blocks per CU, at most what is resident:
//   sequential kernel: as many as there are tiles for (its dense-row loads want every wave they can get);
//   parallel kernel: one per 12 tiles per wave - a wave pays a start-up (a search in rowptr, loads
//     that nothing overlaps yet) and fewer waves leave more of the L1 to each - but two as soon as
//     that leaves a wave 6 tiles (measured on matrices of 1 M to 57 M entries).
constexpr long long kNbPrTilesPerWave = 12;
// quads of entries per lane and tile / block in the balanced parallel kernel for up to four columns per lane
// (four quads, 1024 items: 4-8 % faster on the stencil with item tiles, 2-12 % slower with entry blocks and on R-MAT)
constexpr int kNbPrKq = 2;

inline unsigned balanced_blocks(const Problem& p, long long tile, int blocks_per_cu, bool parallel,
                                long long col_blocks = 1, long long parallel_per_cu_max = 0) {
    const long long cus = device_info().cus;
    const long long cap = cus * blocks_per_cu;
    const long long tiles = p.size >= 0 ? (p.size + p.M + tile - 1) / tile : cap * kWavesPerBlock;
    // entry count unknown on the host and the matrix not known to be small: what serves large matrices best
    if (p.nnz < 0 && tiles > cus * kWavesPerBlock) return (unsigned)(parallel && blocks_per_cu > 2 ? cus * 2 : cap);
    const long long waves = cus * kWavesPerBlock;
    if (tiles <= waves) return clamp_blocks((tiles + kWavesPerBlock - 1) / kWavesPerBlock, cap);
    long long per_cu;
    if (parallel) {
        per_cu = tiles / (waves * kNbPrTilesPerWave);
        if (per_cu < 2) per_cu = tiles >= waves * kNbPrTilesPerWave ? 2 : 1;
        if (parallel_per_cu_max > 0 && per_cu > parallel_per_cu_max) per_cu = parallel_per_cu_max;
    } else {
        // the column blocks of a wide X (grid.y) are resident side by side: count them in
        const long long want = (tiles * col_blocks + waves - 1) / waves;
        if (col_blocks > 1 && want <= blocks_per_cu) return clamp_blocks(cus * want / col_blocks, cap);
        per_cu = (tiles + waves - 1) / waves;
    }
    if (per_cu > blocks_per_cu) per_cu = blocks_per_cu;
    return (unsigned)(cus * per_cu);
}

// Which pipeline the balanced parallel kernel runs.  Blocks of entries with the next block's gathers in flight
// during the row logic (nb_pr_kernel) for up to four dense columns per lane on matrices of six million entries
// and more: 2-6 % faster there on R-MAT matrices of every skew (2^20 vertices, degree 16, power law: 104 -> 98 us
// per call at N = 1, main launch 98 -> 90 us; N = 3: 122 -> 116 us, N = 4: 125 -> 120 us) and on random columns; not
// on banded matrices (see launch_nb_pr_v).  Smaller matrices give a wave only a few blocks, and the longer kernel's
// start-up costs what the overlap returns (10 % faster to 10 % slower on 18 matrices of 0.25 to 4 million entries), so they keep the
// tiles of merge-path items (nb_pr_tiled_kernel), as does a call that does not know its entry count.  With eight
// columns per lane the registers that hold a block's gathered values cost more occupancy than the overlap gives
// (R-MAT N = 8: 162 -> 178 us): tiles as well.  DGSP_ABL_ITEM_TILES / DGSP_ABL_ENTRY_BLOCKS force one or the other
// where both exist (the comparison for this choice).
template <int V>
constexpr bool kNbPrStreams = V <= 4;
constexpr long long kNbPrStreamNnzMin = 6000000;

// Do the chunks of a balanced kernel take whole rows?  That saves the atomics and the prepare launch (6 us with the gap
// behind it), and the wave with the longest row ends later: by up to `per_us` entries a microsecond, as it runs on when the
// others are through - behind a part of the time they take, as long as the call is short.  `lines`: lines of X per entry.
// 100 000 lognormal rows of 6 at N = 6 18.3 -> 11.7 us, 20 001 of 10 at N = 32 11.6 -> 8.6 us; not taken: 100 000 Zipf rows
// of 50 at N = 33 (139 against 186 us), 100 000 lognormal rows of 20 at N = 33 (65 against 78 us).  On 2036 drawn matrices the
// choice loses 1.6 % to the better of the two (never 8.8 %, always 20.7 %); 5 % of them lose more than 10 %.
inline bool snap_rows(const Problem& p, unsigned groups, double share_part, double per_us, double lines) {
    if (p.nnz < 0 || p.max_row < 0) return false;
    const double share = (double)(p.nnz + (long long)p.M) / ((double)groups * kWavesPerBlock);
    if ((double)p.max_row <= share_part * share) return true;
    const double x_bytes = (double)p.K * p.N * 4.0;
    const double missed = x_bytes > (double)kL2BytesPerXcd ? 1.0 - (double)kL2BytesPerXcd / x_bytes : 0.0;
    const double call_us = 5.0 + (double)p.nnz * lines * (6.5e-6 + 12.5e-6 * missed * missed);
    return (double)p.max_row / per_us <= 6.0 + (call_us < 100.0 ? 0.35 * call_us : 0.0);
}

// Runs of 2^shift columns that a table of hot runs counts a matrix of K columns by: 32, more where that would be more than
// 32768 runs; 0: too many columns.
inline int hot_shift(int64_t K) {
    int shift = kHotShiftMin;
    while (shift <= kHotShiftMax && (K - 1) >> shift >= 32ll * kHotWords) ++shift;
    return K >= 1 && shift <= kHotShiftMax ? shift : 0;
}
// Sampled where the column blocks of nb_sr_run_kernel want it, in the same launch: smaller matrices and shorter rows would gain
// 8 to 20 % of a product and pay 20 us for it when they are taken over.
// Reading hot runs from LDS pays where it saves the caches this many entries, as copying the runs costs every CU 4 to 5 us, and
// this share of them (hot_columns()): the others bound the product, all the more the more of them miss the L2.  66 matrices with 4
// to 32 million entries, share, general way -> hot runs:
//   R-MAT 2^20 x 16 at N = 1 / 2 / 3 / 4 (.31 .25 .19 .16) 90 / 100 / 109 / 111 -> 68 / 83 / 97 / 101 us, 2^20 x 32 (.31 .25
//   .19 .16) 168 / 181 / 194 / 196 -> 114 / 145 / 169 / 175 us, 2^18 x 32 (.40 .35 .28 .22) 40 / 43 / 46 / 48 ->
//   31 / 35 / 41 / 44 us, 2^21 x 8 (.27 .19 .16 .11) 108 / 119 / 127 / 136 -> 85 / 106 / 116 / 135 us;
//   N = 1, uniform columns: 16.8 M entries over 100 000 / 262 144 / 500 000 (.28 .11 .06) 94 / 97 / 98 -> 76 / 90 / 95 us, 4.7 M over
//   180 000 / 262 144 / 350 000 (.15 .10 .08; 0.73 / 0.49 / 0.37 M of them) 34.5 / 34.6 / 35.4 -> 32.9 / 34.1 / 35.4 us;
//   the lines, columns K u^p: N = 2 2^20 u^4 (.128) 123 -> 116 us, 1.5 M u^4 (.121) 46 -> 47 us, 3 M u^6 (.11) 141 -> 143 us;
//   N = 3 2^19 u^3 (.11) 131 -> 120 us, 2^20 u^4 (.10) 148 -> 149 us, 2^21 u^6 (.10) 150 -> 153 us; N = 4 2^18 u^4 (.12) 112 ->
//   99 us, 2^20 u^8 (.09) 115 -> 113 us, 2^20 u^4 (.08) 159 -> 161 us.  Columns as hot as 2^20 u^8 would gain below the lines
//   of N = 2 and 3, too (.12 101 -> 87, .10 111 -> 105 us).
constexpr double kHotEntriesMin = 0.45e6, kHotShareMin[kHotWidths] = {0.05, 0.123, 0.107, 0.1};
inline bool wants_hot_columns(const dgsp_internal_stats_t& s, int64_t N) {
    return N >= 1 && N <= kHotWidths && s.hot_share[N - 1] >= kHotShareMin[N - 1] &&
           (double)s.features.nnz * s.hot_share[N - 1] >= kHotEntriesMin;
}

// The hottest runs of X in LDS (nb_pr_kernel, HOT): one workgroup a CU.  Waves see to the rows that they share themselves wherever the call
// has memory for it, at all sizes that have a table.  With the prepare launch / without: R-MAT 2^20 x 16 at N = 1 / 2 / 3 / 4 68.2 / 85.3 / 97.5 /
// 101.6 -> 64.4 / 81.3 / 93.5 / 97.7 us, scaled at N = 1 / 4 74.2 / 106.8 -> 70.0 / 103.4 us, 2^20 x 32 114.1 -> 110.0 us, 2^18 x 32 32.6 ->
// 30.0 us, 2^19 x 16 with its gradient 75.6 -> 70.6 us; the smallest, 4.2 million entries and more: 2^19 x 8 at N = 1 / 2 / 4 26.5 / 30.4 / 36.3 ->
// 24.1 / 28.1 / 33.5 us, 2^19 x 12 at N = 1 / 4 32.5 / 45.8 -> 29.7 / 42.6 us, 2^18 x 20 24.9 / 34.8 -> 22.8 / 32.3 us, 2^19 x 10 scaled 32.4 / 43.4 ->
// 29.6 / 40.7 us, 2^18 x 18 with its gradient at N = 2 56.8 -> 52.7 us.
template <int V>
int launch_nb_pr_hot(const Problem& p) {
    constexpr int KQ = kNbPrKq;
    const HotColumns hot{p.hot_columns + (V - 1) * kHotTableInts, hot_shift(p.K)};
    const dim3 grid((unsigned)device_info().cus);
    constexpr int kGroups = kHotThreads / kBlock;                   // workgroups of the usual size in one of this kernel
    const bool snap = snap_rows(p, grid.x * kGroups, 0.1, 128.0, 1.0);
    const unsigned chunks = grid.x * kGroups * kWavesPerBlock;
    const RowSharing sharing = snap ? RowSharing{} : make_sharing(p, chunks);
    if (p.phase != DGSP_PHASE_MAIN && !snap && !sharing.words)
        if (int rc = launch_prepare(p, chunks, 6, -1)) return rc;
    if (p.phase == DGSP_PHASE_PREPARE) return DGSP_OK;
    const Scaling sc{p.alpha, p.beta};
    const auto launch = [&](auto whole, auto scaled, auto shares) -> int {
        DGSP_LAUNCH_THREADS((nb_pr_kernel<V, KQ, decltype(whole)::value, decltype(scaled)::value, decltype(shares)::value, false, true>), grid,
                            kHotThreads, p.M, p.K, p.N, p.ldx, p.ldy, p.rowptr, p.colidx, p.vals, p.X, p.Y, sc, sharing, hot);
        return DGSP_OK;
    };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    if (snap) return p.scaled ? launch(yes, yes, no) : launch(yes, no, no);
    if (sharing.words) return p.scaled ? launch(no, yes, yes) : launch(no, no, yes);
    return p.scaled ? launch(no, yes, no) : launch(no, no, no);
}

template <int V, int KQ>
int launch_nb_pr_v(const Problem& p) {
    constexpr unsigned tile = kWave * 4 * KQ;
    const unsigned col_groups = (unsigned)((p.N + V - 1) / V);      // V = 8 also takes N = 5, 6, 7: one group
    // the row store addresses a step's rows with 32-bit byte offsets: tile rows * N * 4 must fit
    if (col_groups > 65535u || p.ldy > kBalancedLdyMax) return DGSP_ERR_UNSUPPORTED;
    if constexpr (V <= kHotWidths) { if (p.N == V && p.ldx == V && p.hot_columns && p.switches == 0) return launch_nb_pr_hot<V>(p); }
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    const bool forced_blocks = (p.switches & (DGSP_ABL_ENTRY_BLOCKS | DGSP_ABL_SERIAL_SEGMENT_SCAN)) != 0;
    // A banded matrix (neighbouring rows share their columns: stencils, bands): its gathers hit the L1 and are bound
    // by the rate of the CU's address unit, not by latency, so gathers requested a block ahead gain nothing, and at up
    // to three columns per lane two workgroups per CU leave each wave more of the L1 than four do (27-point stencil on
    // 128^3 at N = 1: item tiles on 2 / 3 workgroups per CU 132 / 140 us, entry blocks on 2 / 3 / 4 155 / 139 / 143 us;
    // N = 2: 137 against 152 us; N = 3: 142 against 150 us; bands of 27 and 64: 116, 123 against 120, 134 us; with
    // four columns per lane the larger grid is as good: 153 / 148 / 149 us on 2 / 3 / 4).
    const bool banded_x = banded(p) && !forced_blocks;
    const bool tiled = !kNbPrStreams<V> || (p.switches & DGSP_ABL_ITEM_TILES) != 0 ||
                       (!forced_blocks && (p.nnz < kNbPrStreamNnzMin || banded_x));   // unknown entry count (-1): tiles
    // of the form that is launched (that of the plain one for the scaled one, which keeps two resident at four columns, was three: R-MAT
    // 2^20 x 32 249 / 200 us with three / two, lognormal rows of 30 492 / 456 us, Zipf rows of 50 741 / 751 us)
    const auto resident_of = [&](auto scaled, auto shares) -> int {
        if constexpr (kNbPrStreams<V>) {
            if (!tiled) return resident_blocks_per_cu(nb_pr_kernel<V, KQ, false, decltype(scaled)::value, decltype(shares)::value>);
        }
        return resident_blocks_per_cu(nb_pr_tiled_kernel<V, KQ, decltype(scaled)::value, decltype(shares)::value>);
    };
    const int resident = p.scaled ? may_share(p) ? resident_of(yes, yes) : resident_of(yes, no)
                                  : may_share(p) ? resident_of(no, yes) : resident_of(no, no);
    // Entry blocks at one and two columns, too: the gathers of two workgroups are as many as the L1 holds misses for, and more
    // would only be shorter shares (R-MAT 2^20 x 32 at N = 1 / 2 on 2 / 3 / 4 workgroups per CU 154.6 / 156.5 / 164.0 and
    // 171.0 / 173.2 / 179.5 us, Zipf rows of 50 317.8 / 321.0 / 332.7 and 515.6 / 515.7 / 519.7 us, in the scaled form at N = 2, which
    // keeps three resident, 521.9 / 521.7 / 560.0 us).
    const bool few_waves = (banded_x && V <= 3) || (!tiled && V <= 2);
    const dim3 grid(balanced_blocks(p, tile, resident, true, 1, few_waves ? 2 : 0), col_groups);
    // a wave alone takes 512 entries in about 4 us
    const bool snap = !(p.switches & DGSP_ABL_SERIAL_SEGMENT_SCAN) && snap_rows(p, grid.x, 0.1, 128.0, lines_per_row(V, p.ldx) * col_groups);
    // What a wave pays for its shared rows it pays in every round of resident waves, the prepare launch is paid once, and with many column
    // groups below eight columns a lane the launch is cheaper from the third round on.  Launch / shared on lognormal 20 000 x 16, Poisson
    // 50 000 x 12, Zipf 100 000 x 16, R-MAT 2^16 x 16: N = 21, three columns a lane, two rounds at most, 26.2 / 23.7, 48.6 / 45.9, 139.7 / 130.2,
    // 50.6 / 49.6 us; N = 63, five, Poisson 12 000 x 40 74.7 / 77.3, R-MAT in the scaled form 182.9 / 185.7 us; N = 150, twelve, scaled, 150.9 / 154.9,
    // 361.1 / 377.7, 1366.7 / 1363.4, 426.6 / 433.7 us; eight columns a lane: N = 16, one round, 14.1 / 12.1, 19.5 / 16.6, 43.5 / 40.2, 23.8 / 21.3 us; N = 48, two,
    // 30.4 / 26.8, 53.7 / 52.1, 153.1 / 153.1, 67.2 / 64.5 us; N = 128, four, scaled, 2 to 6 % faster.
    const size_t round = (size_t)device_info().cus * resident * kWavesPerBlock;
    const RowSharing sharing = snap ? RowSharing{} : make_sharing(p, (size_t)grid.x * kWavesPerBlock * col_groups, V == 8 ? kSharedWordsMax : 2 * round);
    if (p.phase != DGSP_PHASE_MAIN && !snap && !sharing.words)
        if (int rc = launch_prepare(p, grid.x * kWavesPerBlock, 6, -1)) return rc;
    if (p.phase != DGSP_PHASE_PREPARE) {
        const Scaling sc = p.scaled ? Scaling{p.alpha, p.beta} : Scaling{1.0f, 0.0f};
        if (tiled) {
            const auto launch = [&](auto scaled, auto shares) -> int {
                DGSP_LAUNCH((nb_pr_tiled_kernel<V, KQ, decltype(scaled)::value, decltype(shares)::value>), grid, p.M, p.K, p.N, p.ldx,
                            p.ldy, p.rowptr, p.colidx, p.vals, p.X, p.Y, snap, sc, sharing);
                return DGSP_OK;
            };
            if (sharing.words) return p.scaled ? launch(yes, yes) : launch(no, yes);
            return p.scaled ? launch(yes, no) : launch(no, no);
        } else if constexpr (kNbPrStreams<V>) {
            const auto launch = [&](auto whole, auto scaled, auto shares) -> int {
                DGSP_LAUNCH((nb_pr_kernel<V, KQ, decltype(whole)::value, decltype(scaled)::value, decltype(shares)::value>), grid, p.M, p.K,
                            p.N, p.ldx, p.ldy, p.rowptr, p.colidx, p.vals, p.X, p.Y, sc, sharing);
                return DGSP_OK;
            };
            if constexpr (V <= 2) {
                if (p.switches & DGSP_ABL_SERIAL_SEGMENT_SCAN) {
                    DGSP_LAUNCH((nb_pr_kernel<V, KQ, false, false, false, true>), grid, p.M, p.K, p.N, p.ldx, p.ldy, p.rowptr, p.colidx, p.vals,
                                p.X, p.Y, sc, sharing);
                    return DGSP_OK;
                }
            }
            if (snap) return p.scaled ? launch(yes, yes, no) : launch(yes, no, no);
            if (sharing.words) return p.scaled ? launch(no, yes, yes) : launch(no, no, yes);
            return p.scaled ? launch(no, yes, no) : launch(no, no, no);
        }
    }
    return DGSP_OK;
}

// One to three dense columns (one column per lane at any width when vector loads are switched off).
template <int V, bool XBUF, int DEPTH>
int launch_nb_sr_v(const Problem& p) {
    const SrColumns cols = sr_columns(p.N, V, p.N >= 128);
    if (cols.blocks > 65535u) return DGSP_ERR_INVALID_ARG;
    const int logU = kNbSrLogTile - 6 + cols.logG;   // items per lane-group run
    const dim3 grid(balanced_blocks(p, kNbSrTile, resident_blocks_per_cu(nb_sr_kernel<V, XBUF, DEPTH>), false, cols.blocks), cols.blocks);
    if (p.phase != DGSP_PHASE_MAIN)
        if (int rc = launch_prepare(p, grid.x * kWavesPerBlock, (unsigned)logU, kNbSrLogTile)) return rc;
    if (p.phase != DGSP_PHASE_PREPARE) {
        if (p.scaled)
            DGSP_LAUNCH((nb_sr_kernel<V, XBUF, DEPTH, true>), grid, p.M, p.K, p.N, p.ldx, p.ldy, p.rowptr, p.colidx,
                        p.vals, p.X, p.Y, cols.logG, cols.cols_per_block, Scaling{p.alpha, p.beta});
        else
            DGSP_LAUNCH((nb_sr_kernel<V, XBUF, DEPTH>), grid, p.M, p.K, p.N, p.ldx, p.ldy, p.rowptr, p.colidx, p.vals, p.X, p.Y,
                        cols.logG, cols.cols_per_block);
    }
    return DGSP_OK;
}

template <int V>
int launch_nb_sr_pick(const Problem& p) {
    const bool xb = x_fits_descriptor(p);
    if (banded(p)) return xb ? launch_nb_sr_v<V, true, 4>(p) : launch_nb_sr_v<V, false, 4>(p);
    constexpr int D = sr_depth_scattered<V>();
    return xb ? launch_nb_sr_v<V, true, D>(p) : launch_nb_sr_v<V, false, D>(p);
}

// Four columns and more.  Items a wave takes at least: fewer and the two searches that open a chunk outweigh it
// (4096 rows of 8 at N = 32: 6.2 / 6.8 / 8.3 us with 64 / 128 / 256; 20 001 uneven rows of 10: 9.6 / 8.7 / 9.6 us).
constexpr long long kRunItems = 128;

// N a multiple of 64 from 128 on: column blocks of 64, so that the rows of X that many matrix rows share compete for the L2
// with a quarter-kilobyte each instead of N * 4 bytes.
// At N = 64 and 128 blocks of 32 - two or four of them, every XCD on one, one 128-byte line of a row of X per entry and
// block - halve that once more, for one more pass over A.  They save the entries whose row of X an L2 keeps among its last
// 32768 lines but not among its last 16384 pairs of lines, a share that is measured on the columns (saved_share()).  Where it
// was 0.1 and more none of 24 matrices with four million entries and six a row was slower (blocks of 64 against 32, N = 64 / 128:
// R-MAT 2^20 x 16 612 / 1059 -> 522 / 1011 us, on another GPU 595 / 1073 -> 520 / 969 us, on two of eight at N = 128
// 988 -> 1012 us; 2^20 x 32, share 0.13, 15 / 13 %;
// 2^18 x 32, 0.15, 19 / 3 %; columns of that law in rows of another, 0.13, 11 / 10 %).  Below they mostly lose: the rows of
// R-MAT 2^20 x 16 with other columns, 0.02 to 0.06, 4-9 / 5-11 %, Zipf rows of 64 with uniform columns, 0.06, 0-3 / 0-3 %; and
// with short rows, whose ends are met once a block, or where the rest of a small X is in the L2 anyway (R-MAT 2^20 x 4 10 / -5 %,
// 2^16 x 64 8 / 20 %).  Eight blocks (N = 256) leave every XCD the whole matrix: 2081 -> 2302 us.
constexpr double kSavedShareMin = 0.1, kColumnsCvMin = 4.0, kColumnsAvgMin = 6.0;
constexpr long long kColumnsNnzMin = 4000000;
inline bool column_share_matters(const dgsp_features_t& f) {
    return f.nnz >= kColumnsNnzMin && f.cv_row >= kColumnsCvMin && f.avg_row >= kColumnsAvgMin;
}
inline SrColumns nb_sr_run_columns(int64_t N, double saved_share, int switches) {
    const bool wanted = saved_share >= kSavedShareMin && (N == 64 || N == 128);
    if (N % 32 == 0 && N >= 64 && (wanted || (switches & DGSP_ABL_COLUMN_BLOCKS_32))) return {3, 32, (unsigned)(N / 32)};
    return sr_columns(N, 4, N >= 128);
}

// Workgroups (all column blocks') where waves agree on shared rows among themselves: per CU as many as the square root of its items over
// this.  A wave pays for a start and two shared rows whatever its share, the others' gathers wait meanwhile, and what a wave
// alone cannot hide grows with the share.  1 / 2 / 3 / 4 workgroups a CU, us:
//   0.2 M items: R-MAT 2^14 x 20 at N = 72 21.1 / 17.6 / 18.6 / 19.9, 6001 rows of 40 at N = 95 18.6 / 17.1 / 20.0 / 22.0 (two are taken)
//   0.5 M: 12 001 rows of 40 at N = 95 30.5 / 24.2 / 26.9 / 27.5; 0.7 M: R-MAT 2^15 x 20 at N = 95 36.8 / 27.7 / 27.2 / 28.5 (two)
//   1.1 M: R-MAT 2^16 x 16 at N = 72 / 95 56.8 / 37.0 / 32.9 / 33.0 and 58.7 / 39.8 / 37.5 / 38.1 (three)
//   1.6 M: 27 705 rows of 56 over 17 795 columns at N = 72 / 95 77.8 / 48.3 / 43.4 / 41.7 and 82.6 / 54.7 / 56.9 / 55.8, R-MAT 2^16 x 24 at
//   N = 95 80.0 / 52.3 / 47.1 / 48.8 (three)
// From 17 lanes a row of X on rows that are alike would do with two at any size (up to 6 %; at N = 200 with one, 7 %), where power-law
// graphs lose up to 12 %.
constexpr double kSharedRunItems = 700.0;
inline unsigned shared_run_blocks(const Problem& p, int resident, unsigned col_blocks, int logG, unsigned others) {
    if (!may_share(p) || p.size < 0) return others;
    const double cus = device_info().cus, items = (double)(p.size + (long long)p.M) * col_blocks;
    const double per_cu = 1.0 + std::floor(std::sqrt(items / (cus * kSharedRunItems)));
    if (per_cu >= resident) return others;
    const double least = logG >= 3 ? 64.0 : (double)kRunItems;          // a batch of every lane group
    const double blocks = std::min(cus * per_cu, std::ceil(items / (least * kWavesPerBlock)));
    return (unsigned)std::max(1.0, blocks / col_blocks);
}

template <int LOGG, bool XBUF>
int launch_nb_sr_run_v(const Problem& p, const SrColumns& cols) {
    const unsigned col_blocks = cols.blocks;
    if (col_blocks > 65535u) return DGSP_ERR_INVALID_ARG;
    const int resident = p.scaled ? resident_blocks_per_cu(nb_sr_run_kernel<LOGG, XBUF, true>)
                                  : resident_blocks_per_cu(nb_sr_run_kernel<LOGG, XBUF, false>);
    // Two or four column blocks of a wide X: every XCD works on one block only, so that an L2 sees one block's slice of X
    // and the slices do not compete.  With eight blocks every XCD would walk the whole matrix alone (10-20 % slower): from
    // there on the blocks stay a second grid dimension.  DGSP_ABL_BLOCKS_OFF_XCDS: the comparison.
    unsigned pinned = 0;
    if (!(p.switches & DGSP_ABL_BLOCKS_OFF_XCDS) && p.N >= 64 &&
        (col_blocks == 2 || col_blocks == 4 || (col_blocks == 8 && (p.switches & DGSP_ABL_COLUMN_BLOCKS_32)))) pinned = col_blocks;
    const auto grid_of = [&](unsigned blocks) {
        // as many workgroups, in one dimension
        return pinned ? dim3((blocks * col_blocks + kXcd - 1) / kXcd * kXcd, 1) : dim3(blocks, col_blocks);
    };
    const auto groups_of = [&](const dim3& g) { return pinned ? g.x / pinned : g.x; };      // workgroups that share one chunk list
    const unsigned blocks = balanced_blocks(p, kRunItems, resident, false, col_blocks);
    dim3 grid = grid_of(blocks);
    // a wave alone takes one batch of its lane groups in about 1 us
    const int snap = snap_rows(p, groups_of(grid), 1.0, (double)((kWave >> LOGG) * kRunBatch), lines_per_row(cols.cols_per_block, p.ldx) * col_blocks);
    if (!snap && !p.scaled) grid = grid_of(shared_run_blocks(p, resident, col_blocks, LOGG, blocks));
    const unsigned chunk_groups = groups_of(grid);
    // Queues instead of equal shares where a chunk is long against what it costs to start one (5 us): from 2048 items a wave and
    // as many lanes to an entry that the share is 32 768 lane steps.  R-MAT 2^20 x 16 at
    // N = 32 / 41 / 64 / 128 256 / 422 / 507 / 1021 -> 240 / 405 / 443 / 880 us, 2^20 x 32 at N = 20 / 32 416 / 469 ->
    // 393 / 419 us, 2^20 x 8 at N = 41 257 -> 240 us, 2^18 x 16 at N = 128 201 -> 194 us, 2^19 x 16 at N = 100 405 -> 398 us;
    // not 2^20 x 16 at N = 16 (170 against 173 to 190 us), 2^19 x 16 at N = 32 (106 / 113 us), 2^18 x 32 at N = 48
    // (136 / 140 us), nor with few entries a row, whose workgroups are dealt to the XCDs one by one (2^20 x 6 at
    // N = 50 207 / 223 us).  Not from 1024 items and 16 384 lane steps on either, in chunks of 256: 2^18 x 16 at N = 64 103.1 / 108.4 us,
    // 2^18 x 32 at N = 48 126.6 / 140.2 us, 2^18 Zipf rows of 16 at N = 64 163.0 / 170.6 us, 2^18 rows of exactly 16 163.5 / 171.1 us.
    // A bound of the entry count (the length of colidx) will do, the kernels fit the chunks to the matrix: calls without statistics, R-MAT
    // 2^20 x 16 at N = 32 / 64 250 / 574 -> 228 / 497 us, 2^20 x 8 at N = 41 258 -> 231 us, 2^20 Zipf rows of 16 at N = 64
    // 662 -> 632 us, 635 441 Poisson rows of 13 at N = 60 434 -> 421 us; where the true share turns out to be below the line they
    // make the shares equal (ChunkQueues::fit()).
    ChunkQueues queues{};
    dim3 queue_grid = grid;
    if (XBUF && !snap && p.size > 0 && grid.x % kXcd == 0 && p.size / p.M >= run_dealt_below(LOGG)) {
        const unsigned parts = pinned ? kXcd / pinned : kXcd;
        // no more than are resident: what is started late finds the queues empty
        if (pinned) queue_grid.x = std::min<unsigned>(grid.x, (unsigned)(device_info().cus * resident) / kXcd * kXcd);
        const unsigned waves = queue_grid.x / kXcd * kWavesPerBlock;
        queues = make_queues(p, parts, waves, grid.y, std::max(2048, 32768 >> LOGG), run_dealt_below(LOGG));
    }
    const unsigned chunks = queues.starts ? queues.chunks : chunk_groups * kWavesPerBlock;
    RowSharing sharing{};
    if (!snap && !p.scaled && !queues.starts) sharing = make_sharing(p, (size_t)chunks * col_blocks);
    if (p.phase != DGSP_PHASE_MAIN && !snap && !sharing.words)
        if (int rc = launch_prepare(p, chunks, queues.starts ? queues.size_log2 : kRunQuantumLog2, -1, queues, p.scaled)) return rc;
    if (p.phase != DGSP_PHASE_PREPARE) {
        const Scaling sc = p.scaled ? Scaling{p.alpha, p.beta} : Scaling{1.0f, 0.0f};
        const auto launch = [&](auto scaled, auto queued, auto shares) -> int {
            DGSP_LAUNCH((nb_sr_run_kernel<LOGG, XBUF, decltype(scaled)::value, XBUF && decltype(queued)::value, decltype(shares)::value>),
                        queues.starts ? queue_grid : grid, p.M, p.K, p.N, p.ldx, p.ldy, p.rowptr, p.colidx, p.vals, p.X, p.Y,
                        cols.cols_per_block, snap, sc, pinned, queues, sharing);
            return DGSP_OK;
        };
        constexpr std::true_type yes{};
        constexpr std::false_type no{};
        if (queues.starts) return p.scaled ? launch(yes, yes, no) : launch(no, yes, no);
        if (sharing.words) return launch(no, no, yes);
        return p.scaled ? launch(yes, no, no) : launch(no, no, no);
    }
    return DGSP_OK;
}

template <bool XBUF>
int launch_nb_sr_run_x(const Problem& p) {
    const SrColumns cols = nb_sr_run_columns(p.N, p.saved_share, p.switches);
    switch (cols.logG) {
        case 0: return launch_nb_sr_run_v<0, XBUF>(p, cols);
        case 1: return launch_nb_sr_run_v<1, XBUF>(p, cols);
        case 2: return launch_nb_sr_run_v<2, XBUF>(p, cols);
        case 3: return launch_nb_sr_run_v<3, XBUF>(p, cols);
        case 4: return launch_nb_sr_run_v<4, XBUF>(p, cols);
        case 5: return launch_nb_sr_run_v<5, XBUF>(p, cols);
        default: return launch_nb_sr_run_v<6, XBUF>(p, cols);
    }
}

int launch_nb_sr_run(const Problem& p) {
    // the kernel spends the upper half of the offset range on switching lanes off
    return dense_bytes(p.K, p.ldx, p.N) <= 0x7fffffffull ? launch_nb_sr_run_x<true>(p) : launch_nb_sr_run_x<false>(p);
}

int launch_nb_sr(const Problem& p) {
    if (p.ldy > kBalancedLdyMax) return DGSP_ERR_UNSUPPORTED;
    if (p.N >= 4 && !(p.switches & DGSP_ABL_SCALAR_DENSE_LOADS)) return launch_nb_sr_run(p);
    return p.N == 2 && !(p.switches & DGSP_ABL_SCALAR_DENSE_LOADS) ? launch_nb_sr_pick<2>(p) : launch_nb_sr_pick<1>(p);
}

// Five to eight columns without a comparison switch: the same scheme - consecutive entries summed in a lane, one
// segmented scan over the lanes' open rows - with two lanes per entry (nb_sr_run_kernel), which reads a row of X in one
// access instead of two: R-MAT 2^20 x 16 at N = 5 / 8 158 / 157 -> 140 / 137 us, Zipf rows of 16 at N = 8 57 -> 52 us,
// lognormal rows of 64 at N = 5 / 8 174 / 189 -> 144 / 179 us.  On 349 drawn matrices the choice loses 1.0 % to the better of
// the two (always tiles 12.4 %, never 1.9 %).
// Not for a small matrix whose rows it cannot keep whole per wave, as some are long (R-MAT 2^14 x 24 at N = 6 12.4 against
// 13.6 us) or nothing is known of them: without statistics and with the entry count / a bound of it, drawn matrices of
// 0.1 to 1 million entries run 3-11 / 12-25 % faster on the tiles, from there on 2-12 / 0-9 % slower.
constexpr long long kRunNarrowNnzMin = 1000000, kRunNarrowRowMax = 1500;
int launch_nb_pr(const Problem& p) {
    const int v = nb_pr_lane_width(p.N, p.switches);
    const bool short_call = p.size >= 0 && p.size < kRunNarrowNnzMin && (p.max_row < 0 || p.max_row > kRunNarrowRowMax);
    if (v == 8 && p.N <= 8 && p.switches == 0 && p.ldy <= kBalancedLdyMax && !short_call) return launch_nb_sr_run(p);
    switch (v) {
        case 8: return launch_nb_pr_v<8, 1>(p);
        case 4: return launch_nb_pr_v<4, kNbPrKq>(p);
        case 3: return launch_nb_pr_v<3, kNbPrKq>(p);
        case 2: return launch_nb_pr_v<2, kNbPrKq>(p);
        default: return launch_nb_pr_v<1, kNbPrKq>(p);
    }
}

// ---------------------------------------------------------------- selector state
// Defaults fitted on MI355X on the 24-matrix synthetic sweep, pr_nnz_max on larger
// banded and random matrices (the paper prints no threshold values, Section 2.2).
std::mutex g_thresholds_mu;                 // guards g_thresholds: readers take a copy
dgsp_thresholds_t g_thresholds = {
    /* n_parallel_max  */ 4,
    /* pr_avg_row_min  */ 48.0,
    /* pr_cv_max       */ 0.05,
    /* sr_cv_min       */ 0.3,
    /* sr_stdv_min     */ 3.0,
    /* pr_nnz_max      */ 20000000,
    /* short_avg_row_max */ 20.0,
    /* short_max_row_max */ 64,
    /* wide_parallel_n   */ 8,
    /* big_x_bytes_min   */ 6000000,
    /* big_x_cv_max      */ 0.2,
    /* big_x_avg_row_max */ 64.0,
    /* short_min_waves   */ 2048,
    /* pr_small_nnz_max  */ 2000000,
    /* pr_small_cv_max   */ 0.6,
};

dgsp_thresholds_t thresholds_snapshot() {
    std::lock_guard<std::mutex> lock(g_thresholds_mu);
    return g_thresholds;
}

// The balanced kernels address the rows of a tile through 32-bit byte offsets and stop at a leading dimension
// of 2^20 floats (DGSP_ERR_UNSUPPORTED when asked for by name).  A choice the library makes itself moves to the
// row-split sequential kernel there, which has no such limit (so wide a Y means N or the stride is huge).
inline int library_choice(int algo, int64_t ldy) {
    return ((algo == DGSP_NB_SR || algo == DGSP_NB_PR) && ldy > kBalancedLdyMax) ? DGSP_RS_SR : algo;
}

// the kernel that runs where the rules name `algo`
inline int launched_algo(const Problem& p, int algo) { return algo != DGSP_RS_SR && row_groups_suit(p) ? DGSP_RS_SR : algo; }

int run(int64_t M, int64_t K, int64_t N, int64_t nnz, const int32_t* rowptr, const int32_t* colidx,
        const float* vals, const float* X, float* Y, int algo, void* stream, int phase = DGSP_PHASE_ALL,
        Hints hints = Hints(), int switches = 0, int64_t ldx = -1, int64_t ldy = -1, const Scaling* scaling = nullptr) {
    if (M < 0 || K < 0 || N < 0) return DGSP_ERR_INVALID_ARG;
    if (ldx < 0) ldx = N;            // packed rows unless the caller says otherwise
    if (ldy < 0) ldy = N;
    if (ldx < N || ldy < N) return DGSP_ERR_INVALID_ARG;
    if (algo < DGSP_AUTO || algo > DGSP_NB_PR) return DGSP_ERR_INVALID_ARG;
    if (M == 0 || N == 0) return DGSP_OK;
    // int32 index range; a little headroom keeps position arithmetic simple
    const int64_t lim = (int64_t)INT32_MAX - 4096;
    if (M > lim || K > lim || N > lim || nnz > lim || ldx > lim || ldy > lim) return DGSP_ERR_INVALID_ARG;
    if (!rowptr || !Y) return DGSP_ERR_INVALID_ARG;
    if (nnz > 0 && (!colidx || !vals || !X || K == 0)) return DGSP_ERR_INVALID_ARG;

    // no row statistics: the balanced kernels are safe for any row-length distribution; the parallel one while
    // it needs a single pass over the matrix (it was the faster of the two on 22 of 24 sweep matrices at N = 8)
    if (algo == DGSP_AUTO) {
        const dgsp_thresholds_t t = thresholds_snapshot();
        const int64_t one_pass = t.wide_parallel_n > t.n_parallel_max ? t.wide_parallel_n : t.n_parallel_max;
        algo = library_choice((N <= one_pass) ? DGSP_NB_PR : DGSP_NB_SR, ldy);
    }

    Problem p{(int)M, (int)N, (int)ldx, (int)ldy, K, nnz, rowptr, colidx, vals, X, Y, (hipStream_t)stream, phase, hints.col_span,
              hints.cv_row, hints.max_row, nnz >= 0 ? nnz : hints.size, hints.saved_share,
              hints.hot_K == K ? hints.hot_columns : nullptr, hints.more, switches};
    if (scaling) { p.scaled = true; p.alpha = scaling->alpha; p.beta = scaling->beta; }
    if (hints.chosen) algo = launched_algo(p, algo);
    switch (algo) {
        case DGSP_RS_SR: return phase == DGSP_PHASE_PREPARE ? DGSP_OK : launch_rs_sr(p);
        case DGSP_RS_PR: return phase == DGSP_PHASE_PREPARE ? DGSP_OK : launch_rs_pr(p);
        case DGSP_NB_SR: return launch_nb_sr(p);
        default: return launch_nb_pr(p);
    }
}

}  // namespace

// ==================================================================== C-ABI

extern "C" int dgsp_spmm_csr(int64_t M, int64_t K, int64_t N, const int32_t* rowptr, const int32_t* colidx,
                             const float* vals, const float* X, float* Y, int algo, void* stream) {
    return run(M, K, N, -1, rowptr, colidx, vals, X, Y, algo, stream);
}

extern "C" int dgsp_internal_spmm_csr(int64_t M, int64_t K, int64_t N, int64_t nnz, int64_t capacity, const int32_t* rowptr,
                                      const int32_t* colidx, const float* vals, const float* X, float* Y, int algo,
                                      const dgsp_internal_hints_t* more, void* stream) {
    Hints hints(nullptr, more);
    hints.size = capacity;
    return run(M, K, N, nnz < 0 ? -1 : nnz, rowptr, colidx, vals, X, Y, algo, stream, DGSP_PHASE_ALL, hints);
}

extern "C" int dgsp_spmm_csr_nnz(int64_t M, int64_t K, int64_t N, int64_t nnz, const int32_t* rowptr,
                                 const int32_t* colidx, const float* vals, const float* X, float* Y, int algo,
                                 void* stream) {
    return run(M, K, N, nnz < 0 ? -1 : nnz, rowptr, colidx, vals, X, Y, algo, stream);
}

extern "C" int dgsp_internal_spmm_phase(int64_t M, int64_t K, int64_t N, int64_t nnz, const int32_t* rowptr, const int32_t* colidx,
                                        const float* vals, const float* X, float* Y, int algo, int phase,
                                        const dgsp_features_t* features, const dgsp_internal_hints_t* more, void* stream) {
    if (algo < DGSP_RS_SR || algo > DGSP_NB_PR) return DGSP_ERR_INVALID_ARG;
    if (phase < DGSP_PHASE_ALL || phase > DGSP_PHASE_MAIN) return DGSP_ERR_INVALID_ARG;
    if (features && nnz < 0) nnz = features->nnz;
    return run(M, K, N, nnz < 0 ? -1 : nnz, rowptr, colidx, vals, X, Y, algo, stream, phase,
               Hints(features, more));
}

extern "C" int dgsp_spmm_csr_phase(int64_t M, int64_t K, int64_t N, int64_t nnz, const int32_t* rowptr,
                                   const int32_t* colidx, const float* vals, const float* X, float* Y, int algo,
                                   int phase, const dgsp_features_t* features, void* stream) {
    return dgsp_internal_spmm_phase(M, K, N, nnz, rowptr, colidx, vals, X, Y, algo, phase, features, nullptr, stream);
}

extern "C" int dgsp_internal_spmm_view(int64_t M, int64_t K, int64_t N, int64_t nnz, const int32_t* rowptr, const int32_t* colidx,
                                       const float* vals, const float* X, int64_t ldx, float* Y, int64_t ldy,
                                       const float* alpha_beta, int algo, const dgsp_features_t* features,
                                       const dgsp_internal_hints_t* more, void* stream) {
    if (ldx < N || ldy < N) return DGSP_ERR_INVALID_ARG;
    if (features && nnz < 0) nnz = features->nnz;
    Hints hints(features, more);
    if (algo == DGSP_AUTO && features && N >= 1) {
        algo = library_choice(dgsp_select_algo(features, N), ldy);
        hints.chosen = true;
    }
    const Scaling sc{alpha_beta ? alpha_beta[0] : 1.0f, alpha_beta ? alpha_beta[1] : 0.0f};
    return run(M, K, N, nnz < 0 ? -1 : nnz, rowptr, colidx, vals, X, Y, algo, stream, DGSP_PHASE_ALL,
               hints, 0, ldx, ldy, alpha_beta ? &sc : nullptr);
}

extern "C" int dgsp_spmm_csr_ld(int64_t M, int64_t K, int64_t N, int64_t nnz, const int32_t* rowptr,
                                const int32_t* colidx, const float* vals, const float* X, int64_t ldx, float* Y,
                                int64_t ldy, int algo, const dgsp_features_t* features, void* stream) {
    return dgsp_internal_spmm_view(M, K, N, nnz, rowptr, colidx, vals, X, ldx, Y, ldy, nullptr, algo, features, nullptr, stream);
}

extern "C" int dgsp_spmm_csr_axpby(int64_t M, int64_t K, int64_t N, int64_t nnz, const int32_t* rowptr,
                                   const int32_t* colidx, const float* vals, const float* X, int64_t ldx, float* Y,
                                   int64_t ldy, float alpha, float beta, int algo, const dgsp_features_t* features,
                                   void* stream) {
    const float factors[2] = {alpha, beta};
    return dgsp_internal_spmm_view(M, K, N, nnz, rowptr, colidx, vals, X, ldx, Y, ldy, factors, algo, features, nullptr, stream);
}

extern "C" int dgsp_spmm_csr_ablation(int64_t M, int64_t K, int64_t N, int64_t nnz, const int32_t* rowptr,
                                      const int32_t* colidx, const float* vals, const float* X, float* Y, int algo,
                                      int switches, const dgsp_features_t* features, void* stream) {
    if (algo < DGSP_RS_SR || algo > DGSP_NB_PR) return DGSP_ERR_INVALID_ARG;
    if (switches & ~(DGSP_ABL_SCALAR_DENSE_LOADS | DGSP_ABL_NO_SPARSE_STAGING | DGSP_ABL_ITEM_TILES | DGSP_ABL_SERIAL_SEGMENT_SCAN |
                     DGSP_ABL_COLUMN_BLOCKS_32 | DGSP_ABL_BLOCKS_OFF_XCDS | DGSP_ABL_ENTRY_BLOCKS))
        return DGSP_ERR_INVALID_ARG;
    if ((switches & DGSP_ABL_ENTRY_BLOCKS) &&
        (algo != DGSP_NB_PR || (switches & DGSP_ABL_ITEM_TILES) || nb_pr_lane_width(N, switches) > 4))
        return DGSP_ERR_UNSUPPORTED;
    if ((switches & (DGSP_ABL_COLUMN_BLOCKS_32 | DGSP_ABL_BLOCKS_OFF_XCDS)) && algo != DGSP_NB_SR) return DGSP_ERR_UNSUPPORTED;
    if ((switches & DGSP_ABL_NO_SPARSE_STAGING) && algo != DGSP_RS_SR) return DGSP_ERR_UNSUPPORTED;
    if ((switches & DGSP_ABL_ITEM_TILES) && algo != DGSP_NB_PR) return DGSP_ERR_UNSUPPORTED;
    if (switches & DGSP_ABL_SERIAL_SEGMENT_SCAN) {
        // offered at one or two dense columns per lane (on the entry-block pipeline)
        const bool narrow = nb_pr_lane_width(N, switches) <= 2;
        if (algo != DGSP_NB_PR || (switches & DGSP_ABL_ITEM_TILES) || !narrow) return DGSP_ERR_UNSUPPORTED;
    }
    if (features && nnz < 0) nnz = features->nnz;
    return run(M, K, N, nnz < 0 ? -1 : nnz, rowptr, colidx, vals, X, Y, algo, stream, DGSP_PHASE_ALL,
               Hints(features), switches);
}

extern "C" int dgsp_internal_spmm_auto(int64_t M, int64_t K, int64_t N, const dgsp_features_t* features, const dgsp_internal_hints_t* more,
                                       const int32_t* rowptr, const int32_t* colidx, const float* vals, const float* X,
                                       float* Y, int* chosen, void* stream) {
    if (!features) return DGSP_ERR_INVALID_ARG;
    if (features->M != M || features->nnz < 0) return DGSP_ERR_INVALID_ARG;
    int algo = (N >= 1) ? library_choice(dgsp_select_algo(features, N), N) : DGSP_NB_PR;
    if (algo < 0) return DGSP_ERR_INVALID_ARG;
    if (chosen) *chosen = algo;
    Hints hints(features, more);
    hints.chosen = true;
    return run(M, K, N, features->nnz, rowptr, colidx, vals, X, Y, algo, stream, DGSP_PHASE_ALL, hints);
}

extern "C" int dgsp_spmm_csr_auto(int64_t M, int64_t K, int64_t N, const dgsp_features_t* features,
                                  const int32_t* rowptr, const int32_t* colidx, const float* vals, const float* X,
                                  float* Y, int* chosen, void* stream) {
    return dgsp_internal_spmm_auto(M, K, N, features, nullptr, rowptr, colidx, vals, X, Y, chosen, stream);
}

// ---------------------------------------------------------------- 64-bit row pointers
namespace {
constexpr int64_t kSlabEntries = 1ll << 30;        // a slab holds this many entries plus at most one row more
inline int64_t slab_count(int64_t nnz) { return nnz <= 0 ? 1 : (nnz + kSlabEntries - 1) / kSlabEntries; }
inline int64_t round_up16(int64_t v) { return (v + 15) / 16 * 16; }
}  // namespace

extern "C" int64_t dgsp_spmm_csr_i64_workspace_bytes(int64_t M, int64_t nnz) {
    if (M < 0 || nnz < 0) return -1;
    return round_up16(4 * (M + 1)) + 16 * (slab_count(nnz) + 1);
}

extern "C" int dgsp_spmm_csr_i64(int64_t M, int64_t K, int64_t N, int64_t nnz, const int64_t* rowptr, const int32_t* colidx,
                                 const float* vals, const float* X, float* Y, int algo, void* workspace,
                                 int64_t workspace_bytes, void* stream) {
    if (M < 0 || K < 0 || N < 0 || nnz < 0) return DGSP_ERR_INVALID_ARG;
    if (algo < DGSP_AUTO || algo > DGSP_NB_PR) return DGSP_ERR_INVALID_ARG;
    if (M == 0 || N == 0) return DGSP_OK;
    const int64_t lim = (int64_t)INT32_MAX - 4096;
    if (M > lim || K > lim || N > lim) return DGSP_ERR_INVALID_ARG;
    if (!rowptr || !Y || (nnz > 0 && (!colidx || !vals || !X || K == 0))) return DGSP_ERR_INVALID_ARG;
    if (!workspace || !aligned(workspace, 16) || workspace_bytes < dgsp_spmm_csr_i64_workspace_bytes(M, nnz))
        return DGSP_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    const int nslabs = (int)slab_count(nnz);
    int* rowptr32 = static_cast<int*>(workspace);
    long long* cuts = reinterpret_cast<long long*>(static_cast<char*>(workspace) + round_up16(4 * (M + 1)));
    hipLaunchKernelGGL(i64_slab_bounds_kernel, dim3((unsigned)((nslabs + 1 + kWave - 1) / kWave)), dim3(kWave), 0, st,
                       (long long)M, reinterpret_cast<const long long*>(rowptr), nslabs, (long long)kSlabEntries, cuts);
    if (hipGetLastError() != hipSuccess) return DGSP_ERR_LAUNCH;
    // the cuts decide launch sizes, so the host has to see them: the one wait of this entry point
    long long h[2 * 16];
    if (nslabs + 1 > 16) return DGSP_ERR_UNSUPPORTED;                   // 15 * 2^30 entries and more
    if (hipMemcpyAsync(h, cuts, sizeof(long long) * 2 * (size_t)(nslabs + 1), hipMemcpyDeviceToHost, st) != hipSuccess)
        return DGSP_ERR_LAUNCH;
    if (hipStreamSynchronize(st) != hipSuccess) return DGSP_ERR_LAUNCH;
    if (h[1] != 0 || h[2 * nslabs + 1] != nnz) return DGSP_ERR_INVALID_ARG;      // rowptr[0] != 0 or rowptr[M] != nnz
    for (int k = 0; k < nslabs; ++k)
        if (h[2 * k + 3] - h[2 * k + 1] > lim || h[2 * k + 3] < h[2 * k + 1] || h[2 * k + 2] < h[2 * k]) return DGSP_ERR_UNSUPPORTED;
    for (int k = 0; k < nslabs; ++k) {
        const int64_t first = h[2 * k], rows = h[2 * k + 2] - first;
        const int64_t base = h[2 * k + 1], entries = h[2 * k + 3] - base;
        if (rows == 0) continue;
        const long long cap = (long long)device_info().cus * kBlocksPerCu * 4;
        hipLaunchKernelGGL(i64_slab_rowptr_kernel, dim3(clamp_blocks((rows + 1 + kBlock - 1) / kBlock, cap)), dim3(kBlock), 0, st,
                           (long long)rows, reinterpret_cast<const long long*>(rowptr) + first, (long long)base, rowptr32);
        if (hipGetLastError() != hipSuccess) return DGSP_ERR_LAUNCH;
        const int rc = run(rows, K, N, entries, rowptr32, colidx ? colidx + base : nullptr, vals ? vals + base : nullptr, X,
                           Y + (size_t)first * (size_t)N, algo, stream);
        if (rc != DGSP_OK) return rc;
    }
    return DGSP_OK;
}

// Section 2.2: N picks the reduction, row-length statistics pick the partition.
extern "C" int dgsp_select_algo(const dgsp_features_t* f, int64_t N) {
    if (!f || N < 1) return DGSP_AUTO;
    const dgsp_thresholds_t t = thresholds_snapshot();
    // all rows short: one lane group per row keeps a wave busy with no cross-lane step and no idle tail - provided
    // the rows fill the machine: the row-split sequential kernel runs M * (lanes per row) / 64 waves
    if (f->nnz > 0 && f->avg_row <= t.short_avg_row_max && f->max_row <= t.short_max_row_max) {
        const int lanes_log2 = N < 4 ? 0 : sr_lanes_log2(N, 4);
        if ((double)f->M * (double)(1 << lanes_log2) >= 64.0 * (double)t.short_min_waves) return DGSP_RS_SR;
    }
    if (N <= t.n_parallel_max) {
        // X beyond one L2, rows alike and spread over all columns: one row per lane sweeps X in step
        if (t.big_x_bytes_min > 0 && (double)f->K * (double)N * 4.0 >= (double)t.big_x_bytes_min &&
            f->cv_row <= t.big_x_cv_max && f->avg_row <= t.big_x_avg_row_max && f->col_span >= 0.5)
            return DGSP_RS_SR;
        // a small matrix of about equal rows: the balanced kernel's second launch (4-6 us) is a third of the call
        if (f->nnz > 0 && f->nnz <= t.pr_small_nnz_max && f->cv_row <= t.pr_small_cv_max) return DGSP_RS_PR;
        // parallel reduction: long rows keep a row's lanes busy, short rows idle them
        const bool row_split = f->avg_row >= t.pr_avg_row_min && f->cv_row <= t.pr_cv_max && f->nnz < t.pr_nnz_max;
        return row_split ? DGSP_RS_PR : DGSP_NB_PR;
    }
    // sequential reduction: balance only when stdv_row / avg_row says rows are uneven
    if (!(f->cv_row > t.sr_cv_min && f->stdv_row > t.sr_stdv_min)) return DGSP_RS_SR;
    // up to eight columns fit one lane of the balanced parallel kernel: still a single pass
    return (N <= t.wide_parallel_n) ? DGSP_NB_PR : DGSP_NB_SR;
}

extern "C" int dgsp_auto_algo(const dgsp_features_t* f, int64_t N) {
    const int algo = dgsp_select_algo(f, N);
    if (algo < 0) return algo;
    const int64_t lim = (int64_t)INT32_MAX - 4096;
    if (f->M < 0 || f->M > lim || f->K > lim || f->nnz > lim || N > lim) return algo;       // such calls are turned down
    const Hints hints(f);
    Problem p{(int)f->M, (int)N, (int)N, (int)N, f->K, f->nnz};
    p.col_span = hints.col_span; p.cv_row = hints.cv_row; p.max_row = hints.max_row; p.size = f->nnz;
    return launched_algo(p, library_choice(algo, N));
}

extern "C" void dgsp_get_thresholds(dgsp_thresholds_t* out) {
    if (out) *out = thresholds_snapshot();
}

extern "C" void dgsp_set_thresholds(const dgsp_thresholds_t* in) {
    if (!in) return;
    std::lock_guard<std::mutex> lock(g_thresholds_mu);
    g_thresholds = *in;
}

extern "C" int dgsp_features_from_rowptr_host(int64_t M, int64_t K, const int32_t* rowptr, dgsp_features_t* out) {
    if (M < 0 || K < 0 || !out || (!rowptr && M > 0)) return DGSP_ERR_INVALID_ARG;
    dgsp_features_t f{};
    f.M = M; f.K = K;
    if (M == 0) { *out = f; return DGSP_OK; }
    if (rowptr[0] != 0) return DGSP_ERR_INVALID_ARG;
    // one pass: sum and sum of squares in integers (exact), min and max
    unsigned __int128 sq = 0;
    int64_t mx = 0, mn = INT64_MAX;
    for (int64_t i = 0; i < M; ++i) {
        const int64_t len = (int64_t)rowptr[i + 1] - (int64_t)rowptr[i];
        if (len < 0) return DGSP_ERR_INVALID_ARG;
        sq += (unsigned __int128)((uint64_t)len * (uint64_t)len);
        mx = len > mx ? len : mx;
        mn = len < mn ? len : mn;
    }
    f.nnz = rowptr[M];
    f.max_row = mx; f.min_row = mn;
    f.avg_row = (double)f.nnz / (double)M;
    // population variance = E[len^2] - avg^2, formed from exact integers:
    // (M * sum len^2 - nnz^2) / M^2
    const unsigned __int128 num = sq * (unsigned __int128)M - (unsigned __int128)((uint64_t)f.nnz) * (uint64_t)f.nnz;
    const double var = (double)num / ((double)M * (double)M);
    f.stdv_row = std::sqrt(var);
    f.cv_row = f.avg_row > 0 ? f.stdv_row / f.avg_row : 0.0;
    f.col_span = 0.0;
    *out = f;
    return DGSP_OK;
}

constexpr int kGatherProbeBlocks = 4096;

extern "C" int64_t dgsp_gather_probe_out_len(void) { return (int64_t)kGatherProbeBlocks * kBlock; }

extern "C" int dgsp_gather_probe(float* out, const float* x, const int32_t* idx, int64_t n, void* stream) {
    if (n < 0 || !out || (n > 0 && (!x || !idx))) return DGSP_ERR_INVALID_ARG;
    hipLaunchKernelGGL(gather_probe_kernel, dim3(kGatherProbeBlocks), dim3(kBlock), 0, (hipStream_t)stream, out, x,
                       idx, (long long)n);
    return hipGetLastError() == hipSuccess ? DGSP_OK : DGSP_ERR_LAUNCH;
}

// ---------------------------------------------------------------- floor probes (measurement aids)
namespace {
// four workgroups per CU: what the lean pipeline ran best with (512 / 1024 / 1280 / 2048 workgroups on the R-MAT
// SpMV: 79 / 82 / 90 / 86 us; on the stencil: 118 / 110 / 152 / 114 us)
constexpr int kStreamProbeBlocks = 1024;

struct RowProbeShape { int logG; unsigned col_blocks; unsigned blocks; };
RowProbeShape row_probe_shape(int64_t N) {
    const int logG = sr_lanes_log2(N, 4, 4);                               // at most 16 lanes = 64 columns per group
    const unsigned col_blocks = (unsigned)((N + (4 << logG) - 1) / (4 << logG));
    const unsigned blocks = (unsigned)(device_info().cus * resident_blocks_per_cu(row_gather_probe_kernel));
    return {logG, col_blocks, blocks};
}
}  // namespace

extern "C" int64_t dgsp_floor_probe_out_len(int mode, int64_t N) {
    if (mode == DGSP_PROBE_GATHER) return dgsp_gather_probe_out_len();
    if (mode == DGSP_PROBE_STREAM_GATHER_FMA) return (N == 1 || N == 2 || N == 4) ? (int64_t)kStreamProbeBlocks * kBlock * N : -1;
    if (mode == DGSP_PROBE_ROW_GATHER) {
        if (N < 4 || N % 4 != 0) return -1;
        const RowProbeShape sh = row_probe_shape(N);
        return (int64_t)sh.blocks * sh.col_blocks * kBlock * 4;
    }
    return -1;
}

extern "C" int dgsp_floor_probe(int mode, int64_t nnz, int64_t K, int64_t N, const int32_t* colidx, const float* vals,
                                const float* X, float* out, void* stream) {
    if (nnz < 0 || K < 1 || N < 1 || !out || !X || (nnz > 0 && !colidx)) return DGSP_ERR_INVALID_ARG;
    const int64_t lim = (int64_t)INT32_MAX - 4096;
    if (nnz > lim || K > lim || N > (1 << 20)) return DGSP_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    if (mode == DGSP_PROBE_GATHER) {
        if (N != 1) return DGSP_ERR_UNSUPPORTED;
        return dgsp_gather_probe(out, X, colidx, nnz, stream);
    }
    if (nnz > 0 && !vals) return DGSP_ERR_INVALID_ARG;
    if (mode == DGSP_PROBE_STREAM_GATHER_FMA) {
        const dim3 grid(kStreamProbeBlocks);
        switch (N) {
            case 1: hipLaunchKernelGGL(stream_gather_fma_probe_kernel<1>, grid, dim3(kBlock), 0, st, out, X, (long long)K, 1, colidx, vals, (long long)nnz); break;
            case 2: hipLaunchKernelGGL(stream_gather_fma_probe_kernel<2>, grid, dim3(kBlock), 0, st, out, X, (long long)K, 2, colidx, vals, (long long)nnz); break;
            case 4: hipLaunchKernelGGL(stream_gather_fma_probe_kernel<4>, grid, dim3(kBlock), 0, st, out, X, (long long)K, 4, colidx, vals, (long long)nnz); break;
            default: return DGSP_ERR_UNSUPPORTED;
        }
        return hipGetLastError() == hipSuccess ? DGSP_OK : DGSP_ERR_LAUNCH;
    }
    if (mode == DGSP_PROBE_ROW_GATHER) {
        if (N < 4 || N % 4 != 0) return DGSP_ERR_UNSUPPORTED;
        const RowProbeShape sh = row_probe_shape(N);
        if (sh.col_blocks > 65535u) return DGSP_ERR_UNSUPPORTED;
        hipLaunchKernelGGL(row_gather_probe_kernel, dim3(sh.blocks, sh.col_blocks), dim3(kBlock), 0, st, out, X, (long long)K,
                           (int)N, (int)N, colidx, vals, (long long)nnz, sh.logG);
        return hipGetLastError() == hipSuccess ? DGSP_OK : DGSP_ERR_LAUNCH;
    }
    return DGSP_ERR_INVALID_ARG;
}

extern "C" int dgsp_features_from_csr_host(int64_t M, int64_t K, const int32_t* rowptr, const int32_t* colidx,
                                           dgsp_features_t* out) {
    const int rc = dgsp_features_from_rowptr_host(M, K, rowptr, out);
    if (rc != DGSP_OK) return rc;
    if (out->nnz > 0 && !colidx) return DGSP_ERR_INVALID_ARG;
    if (M == 0 || K == 0 || out->nnz == 0) return DGSP_OK;
    // mean over the non-empty rows of (largest - smallest column + 1) / K; the spans are summed as
    // integers so that the device version, which adds them in any order, gives the same bits
    uint64_t sum = 0;
    int64_t rows = 0;
    for (int64_t i = 0; i < M; ++i) {
        const int64_t s = rowptr[i], e = rowptr[i + 1];
        if (s == e) continue;
        int32_t lo = colidx[s], hi = colidx[s];
        if (colidx[e - 1] < lo || e - s <= 2) {
            for (int64_t p = s; p < e; ++p) { lo = colidx[p] < lo ? colidx[p] : lo; hi = colidx[p] > hi ? colidx[p] : hi; }
        } else {
            // sorted rows (the usual case) need only their two ends; verify cheaply, else scan
            bool sorted = true;
            for (int64_t p = s + 1; p < e; ++p) if (colidx[p] < colidx[p - 1]) { sorted = false; break; }
            if (sorted) hi = colidx[e - 1];
            else for (int64_t p = s; p < e; ++p) { lo = colidx[p] < lo ? colidx[p] : lo; hi = colidx[p] > hi ? colidx[p] : hi; }
        }
        sum += (uint64_t)((int64_t)hi - (int64_t)lo + 1);
        ++rows;
    }
    out->col_span = rows ? (double)sum / ((double)K * (double)rows) : 0.0;
    return DGSP_OK;
}

// ---------------------------------------------------------------- statistics of a matrix in device memory
// Scratch of the pass: static device arrays (every GPU holds its own copies, at addresses that hipGetSymbolAddress tells,
// asked once per device with that device current).  A call owns one of them from launch to result (stat_pool.hpp).
static __device__ __align__(256) StatScratch stat_scratch[kStatSlots];

namespace {

// the current device, as the pool asks about it
struct StatRuntime {
    static bool device(int& dev) { return hipGetDevice(&dev) == hipSuccess; }
    static StatScratch* scratch() {
        void* ptr = nullptr;
        return hipGetSymbolAddress(&ptr, HIP_SYMBOL(stat_scratch)) == hipSuccess ? static_cast<StatScratch*>(ptr) : nullptr;
    }
    static void* pinned(size_t bytes) {
        void* ptr = nullptr;
        if (hipHostMalloc(&ptr, bytes, hipHostMallocMapped | hipHostMallocCoherent) == hipSuccess) return ptr;
        (void)hipGetLastError();
        return nullptr;
    }
};
using StatisticsPool = StatPool<StatScratch, StatRuntime>;
StatisticsPool g_stat_pool;

// A stream that records a graph does not run what it is given, so no result would come - and a replay would write into a
// place of the pool that is another call's by then.
bool recording(hipStream_t st) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return false;
}

// Waits until the GPU has announced `ticket`: a look at host memory instead of a copy and an interrupt (15 us less).
template <typename Seen>
bool wait_until(Seen&& seen, hipStream_t st) {
    for (int i = 0; i < 20000; ++i) {
        if (seen()) return true;
        __builtin_ia32_pause();
    }
    // much work ahead of it in the stream, or an error
    return hipStreamSynchronize(st) == hipSuccess && seen();
}
bool wait_for_ticket(const unsigned long long* word, unsigned long long ticket, hipStream_t st) {
    return wait_until([&] { return __atomic_load_n(word, __ATOMIC_ACQUIRE) == ticket; }, st);
}

// what stands beside every piece of a call's statistics, and in no upper half that column_reuse_kernel leaves in these words
inline unsigned stat_tag(unsigned long long ticket) { return (unsigned)ticket | 0x80000000u; }

// the pieces that csr_statistics_kernel leaves
int fetch_statistics(const StatisticsPool::Slot& slot, unsigned long long* h, hipStream_t st) {
    if (slot.host) {
        int got = 0;
        const auto all = [&] {
            for (; got < kStatPieces; ++got) {
                h[got] = __atomic_load_n(slot.host + got, __ATOMIC_RELAXED);
                if (h[got] >> 32 != stat_tag(slot.ticket)) return false;
            }
            return true;
        };
        if (!wait_until(all, st)) return DGSP_ERR_LAUNCH;
    } else {
        if (hipMemcpyAsync(h, slot.scratch->result, sizeof(*h) * kStatPieces, hipMemcpyDeviceToHost, st) != hipSuccess) return DGSP_ERR_LAUNCH;
        if (hipStreamSynchronize(st) != hipSuccess) return DGSP_ERR_LAUNCH;
    }
    for (int i = 0; i < kStatPieces; ++i) h[i] &= 0xffffffffull;
    return DGSP_OK;
}

// the first `words` result words of a launch that announced itself in word kStatAnnounceWord, or, without pinned words, left
// them in the scratch
int fetch_result(const StatisticsPool::Slot& slot, unsigned long long* h, int words, hipStream_t st) {
    if (slot.host) {
        if (!wait_for_ticket(slot.host + kStatAnnounceWord, slot.ticket, st)) return DGSP_ERR_LAUNCH;
        for (int w = 0; w < words; ++w) h[w] = __atomic_load_n(slot.host + w, __ATOMIC_RELAXED);
        return DGSP_OK;
    }
    if (hipMemcpyAsync(h, slot.scratch->result, sizeof(*h) * (size_t)words, hipMemcpyDeviceToHost, st) != hipSuccess) return DGSP_ERR_LAUNCH;
    return hipStreamSynchronize(st) == hipSuccess ? DGSP_OK : DGSP_ERR_LAUNCH;
}

void finish_features(dgsp_features_t& f, unsigned long long sq, unsigned long long rows, unsigned long long span) {
    f.avg_row = (double)f.nnz / (double)f.M;
    const unsigned __int128 num = (unsigned __int128)sq * (unsigned __int128)f.M
                                  - (unsigned __int128)((uint64_t)f.nnz) * (uint64_t)f.nnz;
    f.stdv_row = std::sqrt((double)num / ((double)f.M * (double)f.M));
    f.cv_row = f.avg_row > 0 ? f.stdv_row / f.avg_row : 0.0;
    f.col_span = (f.K > 0 && rows > 0) ? (double)span / ((double)f.K * (double)rows) : 0.0;
}

// The pass over columns in any order; `ws`: kFeatureWords words of device scratch.
int features_of_unsorted_rows(int64_t M, int64_t K, const int32_t* rowptr, const int32_t* colidx, unsigned long long* ws,
                              dgsp_features_t* out, hipStream_t st) {
    hipLaunchKernelGGL(features_init_kernel, dim3(1), dim3(kWave), 0, st, ws);
    const long long waves = (M + kWave - 1) / kWave;
    const dim3 grid(clamp_blocks((waves + kWavesPerBlock - 1) / kWavesPerBlock, (long long)device_info().cus * kBlocksPerCu));
    hipLaunchKernelGGL(features_kernel, grid, dim3(kBlock), 0, st, (int)M, rowptr, colidx, ws);
    if (hipGetLastError() != hipSuccess) return DGSP_ERR_LAUNCH;
    unsigned long long h[kFeatureWords];
    if (hipMemcpyAsync(h, ws, sizeof(h), hipMemcpyDeviceToHost, st) != hipSuccess) return DGSP_ERR_LAUNCH;
    if (hipStreamSynchronize(st) != hipSuccess) return DGSP_ERR_LAUNCH;
    finish_features(*out, h[0], h[3], h[4]);
    return DGSP_OK;
}

// `entries`: length of colidx, -1: unknown.  I = int64_t: the 32-bit arrays are written too.
template <typename I>
int features_from_csr_device(int64_t M, int64_t K, int64_t entries, const I* rowptr, const I* colidx, int32_t* rowptr32,
                             int32_t* colidx32, bool may_allocate, dgsp_features_t* out, hipStream_t st) {
    using Word = std::conditional_t<sizeof(I) == 8, long long, int>;
    dgsp_features_t f{};
    f.M = M; f.K = K;
    if (recording(st)) return DGSP_ERR_LAUNCH;
    StatisticsPool::Slot slot;
    if (!g_stat_pool.take(slot, may_allocate)) return DGSP_ERR_LAUNCH;
    struct Return { const StatisticsPool::Slot& s; ~Return() { g_stat_pool.give_back(s); } } give_back{slot};
    // enough blocks for the pieces; with the entry count unknown, for rows of 16 and no fewer than one per CU
    const long long pieces = entries >= 0 ? std::max<long long>((entries + kStatChunk - 1) / kStatChunk, (M + kStatChunk - 1) / kStatChunk)
                                          : std::max<long long>(M / 128, device_info().cus);
    // A small matrix: workgroups of their own for the rows, a row a thread, as long as every workgroup has a CU (20 001 rows of 10, whole
    // call with one product 30.4 -> 29.3 us, 4096 rows of 8 24.3 -> 22.8 us; 60 000 rows of 8, 470 workgroups, 32.5 -> 33.0 us).
    const long long entry_blocks = entries > 0 && K > 0 && colidx ? (entries + kStatChunk - 1) / kStatChunk : 0;
    const long long row_blocks = entry_blocks > 0 ? (M + kBlock - 1) / kBlock : 0;
    const bool apart = row_blocks > 0 && entry_blocks + row_blocks <= std::min(device_info().cus, kStatBlocks);
    const dim3 grid(apart ? (unsigned)(entry_blocks + row_blocks) : clamp_blocks(pieces, kStatBlocks));
    hipLaunchKernelGGL((csr_statistics_kernel<Word>), grid, dim3(kBlock), 0, st, (int)M, (long long)entries,
                       reinterpret_cast<const Word*>(rowptr), K > 0 ? reinterpret_cast<const Word*>(colidx) : nullptr,
                       rowptr32, colidx32, slot.scratch, slot.host, stat_tag(slot.ticket), apart ? (unsigned)row_blocks : 0u);
    if (hipGetLastError() != hipSuccess) return DGSP_ERR_LAUNCH;
    unsigned long long h[kStatPieces];
    if (const int rc = fetch_statistics(slot, h, st)) return rc;
    if (h[5] != 0 || h[kStatWords] != 0) return DGSP_ERR_INVALID_ARG;       // decreasing row pointers, rowptr[0] != 0
    f.nnz = (int64_t)(int32_t)h[kStatWords + 1];
    f.max_row = (int64_t)h[1]; f.min_row = (int64_t)h[2];
    finish_features(f, h[0] | h[kStatWords + 2] << 32, h[3], h[4] | h[kStatWords + 3] << 32);
    if (h[6] != h[7]) {
        const int rc = features_of_unsorted_rows(M, K, sizeof(I) == 8 ? rowptr32 : reinterpret_cast<const int32_t*>(rowptr),
                                                 sizeof(I) == 8 ? colidx32 : reinterpret_cast<const int32_t*>(colidx),
                                                 slot.scratch->result, &f, st);
        if (rc != DGSP_OK) return rc;
    }
    *out = f;
    return DGSP_OK;
}

}  // namespace

extern "C" int dgsp_features_from_csr_device(int64_t M, int64_t K, const int32_t* rowptr, const int32_t* colidx,
                                             void* workspace, dgsp_features_t* out, void* stream) {
    if (M < 0 || K < 0 || !out || (!rowptr && M > 0)) return DGSP_ERR_INVALID_ARG;
    if (M > (int64_t)INT32_MAX - 4096) return DGSP_ERR_INVALID_ARG;
    if (M == 0) { dgsp_features_t f{}; f.K = K; *out = f; return DGSP_OK; }
    if (!workspace || !aligned(workspace, 8)) return DGSP_ERR_INVALID_ARG;
    return features_from_csr_device<int32_t>(M, K, -1, rowptr, colidx, nullptr, nullptr, true, out, (hipStream_t)stream);
}

// allocates nothing, not even the pinned words: the result comes back by a copy
extern "C" int dgsp_features_from_csr_device_noalloc(int64_t M, int64_t K, const int32_t* rowptr,
                                                     const int32_t* colidx, dgsp_features_t* out, void* stream) {
    if (M < 0 || K < 0 || !out || (!rowptr && M > 0)) return DGSP_ERR_INVALID_ARG;
    if (M > DGSP_FEATURES_NOALLOC_MAX_ROWS) return DGSP_ERR_INVALID_ARG;
    if (M == 0) { dgsp_features_t f{}; f.K = K; *out = f; return DGSP_OK; }
    return features_from_csr_device<int32_t>(M, K, -1, rowptr, colidx, nullptr, nullptr, false, out, (hipStream_t)stream);
}

extern "C" int dgsp_internal_take_csr(int64_t M, int64_t K, int64_t entries, int index_bytes, const void* rowptr,
                                      const void* colidx, int32_t* rowptr32, int32_t* colidx32, dgsp_features_t* out, void* stream) {
    const int64_t lim = (int64_t)INT32_MAX - 4096;
    if (M < 1 || M > lim || K < 0 || entries < 0 || entries > lim || !rowptr || !out) return DGSP_ERR_INVALID_ARG;
    if (K == 0 || entries == 0) colidx = nullptr;
    if (index_bytes == 4)
        return features_from_csr_device<int32_t>(M, K, entries, static_cast<const int32_t*>(rowptr), static_cast<const int32_t*>(colidx),
                                                 nullptr, nullptr, true, out, (hipStream_t)stream);
    if (index_bytes != 8 || !rowptr32 || (colidx && !colidx32)) return DGSP_ERR_INVALID_ARG;
    return features_from_csr_device<int64_t>(M, K, entries, static_cast<const int64_t*>(rowptr), static_cast<const int64_t*>(colidx),
                                             rowptr32, colidx32, true, out, (hipStream_t)stream);
}

// Good and Turing's estimate: among w entries the share that names a column met once is the share of further entries whose
// column is not among those met, D of them.  An L2 of D places misses as often; the sample gives the pairs (D, share) at
// three sizes, between which the share is taken as linear.
extern "C" double dgsp_internal_saved_share(const uint64_t* counts) {
    const double buckets = (double)(1 << kReuseBucketsLog2), rate = (double)(1 << kReuseRateLog2);
    double at[kReuseLevels + 1] = {0.0}, share[kReuseLevels + 1] = {1.0};
    for (int l = 0; l < kReuseLevels; ++l) {
        // columns that share a bucket count as one, and not as met once
        const double empty = std::fmax(1.0 - (double)counts[2 * l] / buckets, 1.0 / buckets);
        at[l + 1] = -buckets * std::log(empty) * rate;
        share[l + 1] = std::fmin((double)counts[2 * l + 1] / empty * rate / (double)((16 * kReuseThreads) << l), 1.0);
    }
    const auto missed = [&](double places) {
        for (int l = 0; l < kReuseLevels; ++l)
            if (at[l + 1] >= places && at[l + 1] > at[l]) return share[l] + (share[l + 1] - share[l]) * (places - at[l]) / (at[l + 1] - at[l]);
        return share[kReuseLevels];
    };
    return std::fmax(missed(16384.0) - missed(32768.0), 0.0);
}

namespace {
// counts[0 ... 5]: distinct columns and columns met once (column_reuse_kernel); counts[6 ... 9]: sampled entries in hot runs,
// where `hot_table` is given
int sample_columns(int64_t K, int64_t entries, const int32_t* colidx, uint32_t* hot_table, uint64_t* counts, hipStream_t st) {
    if (recording(st)) return DGSP_ERR_LAUNCH;
    StatisticsPool::Slot slot;
    if (!g_stat_pool.take(slot, true)) return DGSP_ERR_LAUNCH;
    struct Return { const StatisticsPool::Slot& s; ~Return() { g_stat_pool.give_back(s); } } give_back{slot};
    unsigned long long* out = slot.host ? slot.host : slot.scratch->result;
    hipLaunchKernelGGL(column_reuse_kernel, dim3(hot_table ? 1 + kHotWidths : 1), dim3(kReuseThreads), 0, st, (long long)entries,
                       colidx, hot_table, hot_table ? hot_shift(K) : 0, out, slot.host ? slot.host + kStatAnnounceWord : nullptr, slot.ticket);
    if (hipGetLastError() != hipSuccess) return DGSP_ERR_LAUNCH;
    // a place is given back when nothing is under way in it: all workgroups', whatever became of the first
    bool hot_done = true;
    for (int v = 1; hot_table && slot.host && v <= kHotWidths; ++v)
        hot_done = wait_for_ticket(slot.host + kStatAnnounceWord + v, slot.ticket, st) && hot_done;
    unsigned long long h[kReuseResultWords];
    if (const int rc = fetch_result(slot, h, kReuseResultWords, st)) return rc;
    if (!hot_done) return DGSP_ERR_LAUNCH;
    for (int i = 0; i < kReuseResultWords; ++i) counts[i] = h[i];
    return DGSP_OK;
}
}  // namespace

extern "C" int dgsp_internal_column_reuse(int64_t entries, const int32_t* colidx, uint64_t* counts, void* stream) {
    if (entries < kReuseEntriesMin || !colidx || !counts) return DGSP_ERR_INVALID_ARG;
    uint64_t h[kReuseResultWords];
    if (const int rc = sample_columns(0, entries, colidx, nullptr, h, (hipStream_t)stream)) return rc;
    for (int i = 0; i < 2 * kReuseLevels; ++i) counts[i] = h[i];
    return DGSP_OK;
}

extern "C" int64_t dgsp_internal_hot_columns_bytes(const dgsp_internal_stats_t* stats) {
    if (!stats) return 0;
    const dgsp_features_t& f = stats->features;
    return column_share_matters(f) && hot_shift(f.K) != 0 ? (int64_t)sizeof(int) * kHotTableInts * kHotWidths : 0;
}

extern "C" int dgsp_internal_wants_hot_columns(const dgsp_internal_stats_t* stats, int64_t N) {
    return stats && wants_hot_columns(*stats, N);
}

extern "C" int dgsp_internal_measure_columns(dgsp_internal_stats_t* stats, const int32_t* colidx, uint32_t* hot_columns, void* stream) {
    if (!stats) return DGSP_ERR_INVALID_ARG;
    stats->saved_share = 0.0;
    for (double& share : stats->hot_share) share = 0.0;
    if (!column_share_matters(stats->features)) return DGSP_OK;
    if (dgsp_internal_hot_columns_bytes(stats) == 0) hot_columns = nullptr;
    if (stats->features.nnz < kReuseEntriesMin || !colidx) return DGSP_ERR_INVALID_ARG;
    uint64_t counts[kReuseResultWords];
    if (const int rc = sample_columns(stats->features.K, stats->features.nnz, colidx, hot_columns, counts, (hipStream_t)stream)) return rc;
    stats->saved_share = dgsp_internal_saved_share(counts);
    for (int v = 0; hot_columns && v < kHotWidths; ++v) stats->hot_share[v] = (double)counts[2 * kReuseLevels + v] / (double)kHotSample;
    return DGSP_OK;
}

extern "C" int dgsp_internal_nb_sr_block(const dgsp_internal_stats_t* stats, int64_t N) {
    return N < 4 ? (int)N : nb_sr_run_columns(N, stats ? stats->saved_share : 0.0, 0).cols_per_block;
}

extern "C" int dgsp_autotune(int64_t M, int64_t K, int64_t N, int64_t nnz, const int32_t* rowptr,
                             const int32_t* colidx, const float* vals, const float* X, float* Y,
                             const dgsp_features_t* features, int reps, float* ms, int* best, void* stream) {
    if (!best) return DGSP_ERR_INVALID_ARG;
    if (reps < 1) reps = 1;
    if (reps > 100) reps = 100;
    if (features && nnz < 0) nnz = features->nnz;
    const Hints hints(features);
    hipStream_t st = (hipStream_t)stream;
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return DGSP_ERR_LAUNCH;
    if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return DGSP_ERR_LAUNCH; }
    float t[4];
    int rc = DGSP_OK;
    float best_ms = INFINITY;
    int best_algo = -1;
    for (int algo = DGSP_RS_SR; algo <= DGSP_NB_PR && rc == DGSP_OK; ++algo) {
        t[algo] = INFINITY;
        // one untimed call first (first-use costs, caches), then `reps` timed ones; keep the fastest
        for (int r = 0; r <= reps; ++r) {
            if (r > 0 && hipEventRecord(e0, st) != hipSuccess) { rc = DGSP_ERR_LAUNCH; break; }
            const int one = run(M, K, N, nnz < 0 ? -1 : nnz, rowptr, colidx, vals, X, Y, algo, stream, DGSP_PHASE_ALL,
                                hints);
            if (one == DGSP_ERR_UNSUPPORTED) break;            // this kernel does not take the shape: skip it
            if (one != DGSP_OK) { rc = one; break; }
            if (r == 0) continue;
            float dt = 0.0f;
            if (hipEventRecord(e1, st) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                hipEventElapsedTime(&dt, e0, e1) != hipSuccess) { rc = DGSP_ERR_LAUNCH; break; }
            t[algo] = dt < t[algo] ? dt : t[algo];
            if (dt > 20.0f * best_ms) break;                   // hopeless: do not repeat a kernel 20x off the pace
        }
        if (t[algo] < best_ms) { best_ms = t[algo]; best_algo = algo; }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc != DGSP_OK) return rc;
    if (hipStreamSynchronize(st) != hipSuccess) return DGSP_ERR_LAUNCH;
    if (ms) for (int a = 0; a < 4; ++a) ms[a] = t[a];
    if (best_algo < 0) {
        // nothing was timed (M == 0 or N == 0: every call returns at once): any kernel will do
        best_algo = (N <= thresholds_snapshot().n_parallel_max) ? DGSP_NB_PR : DGSP_NB_SR;
    }
    *best = best_algo;
    return DGSP_OK;
}

extern "C" int dgsp_copy_f32(float* dst, const float* src, int64_t n, void* stream) {
    if (n < 0 || (n > 0 && (!dst || !src))) return DGSP_ERR_INVALID_ARG;
    if (n == 0) return DGSP_OK;
    if (!aligned(dst, 16) || !aligned(src, 16)) return DGSP_ERR_INVALID_ARG;
    const long long cap = (long long)device_info().cus * kBlocksPerCu * 4;
    const dim3 grid(clamp_blocks((n / 4 + kBlock - 1) / kBlock, cap));
    hipLaunchKernelGGL(copy_kernel, grid, dim3(kBlock), 0, (hipStream_t)stream, dst, src, (long long)n);
    return hipGetLastError() == hipSuccess ? DGSP_OK : DGSP_ERR_LAUNCH;
}

extern "C" const char* dgsp_algo_name(int algo) {
    switch (algo) {
        case DGSP_RS_SR: return "rs_sr";
        case DGSP_RS_PR: return "rs_pr";
        case DGSP_NB_SR: return "nb_sr";
        case DGSP_NB_PR: return "nb_pr";
        case DGSP_AUTO: return "auto";
        default: return "unknown";
    }
}

extern "C" const char* dgsp_status_string(int status) {
    switch (status) {
        case DGSP_OK: return "ok";
        case DGSP_ERR_INVALID_ARG: return "invalid argument";
        case DGSP_ERR_UNSUPPORTED: return "unsupported";
        case DGSP_ERR_LAUNCH: return "kernel launch failed";
        default: return "unknown status";
    }
}
