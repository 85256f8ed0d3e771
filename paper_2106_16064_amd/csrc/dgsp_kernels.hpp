// The four CSR SpMV/SpMM kernels of the paper's design space (Section 2.1):
// {row-split, nnz-balanced} x {sequential, parallel reduction}, for gfx950.
//
// Common shape of all four
//   * 256-thread workgroups = 4 waves; every cooperative step is wave-local
//     (DPP moves or wave-private LDS), so there is no s_barrier anywhere.
//   * `V` is the vector width of dense-row accesses: one dword / dwordx2 /
//     dwordx3 / dwordx4 per lane, or two dwordx4 for V = 8 (vector-type
//     dense-row loading, Section 2.1.2).  The memory pipeline takes these at
//     any dword address, so the choice of V depends on N only, never on the
//     alignment of X and Y or on their leading dimensions.
//   * X and Y are row-major with leading dimensions ldx, ldy (floats per row,
//     >= N); only the N used columns of a row are touched.
//   * Grids are sized to the machine, not to the matrix: a wave walks a list
//     of row groups (row-split) or tiles (balanced).  That is what allows the
//     number of stored entries to be read on the device from rowptr[M].
#pragma once

#include "chunk_queues.hpp"
#include "dgsp_device.hpp"
#include "shared_rows.hpp"

#include <type_traits>

namespace dgsp {

// How the scheduler ranks the wave among those of its SIMD (the instruction takes a constant).  Left alone it issues for the
// oldest one that can go on, so a young wave waits with its searches and its staging while the others gather: of the four
// waves of a SIMD with equal shares the oldest ended at 13 us, the youngest at 18 of 24 (R-MAT 2^16 x 16 at N = 41), and the
// memory idled at both ends.  A wave that has no gather in flight yet needs few issue slots to get there, so it goes first.
__device__ __forceinline__ void set_wave_priority(unsigned level) {
    if (level >= 3u) __builtin_amdgcn_s_setprio(3);
    else if (level == 2u) __builtin_amdgcn_s_setprio(2);
    else if (level == 1u) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
}

// ===========================================================================
// Row-split, parallel reduction  (CSR-Vector lineage; Section 1, Fig. 2(c,d))
// ===========================================================================
//
// 2^logG lanes own a row: they load consecutive (colidx, val) pairs, each
// lane gathers V dense values with one vector load, multiplies, keeps V
// private partial sums, and the group is folded with the DPP scan (a plain
// merge tree is the special case of the segmented scan with fixed-width
// segments).  logG < 0 asks the kernel to derive it from rowptr[M] / M.
// A wave keeps kRsPrUnroll row groups in flight.  For N > V the columns are
// processed V at a time.

__host__ __device__ __forceinline__ int pr_lanes_log2(long long nnz, long long M) {
    // lanes per row ~ average row length, rounded up to a power of two in [2, 64]
    const double avg = M > 0 ? (double)nnz / (double)M : 0.0;
    int lg = 1;
    while (lg < 6 && (double)(1 << lg) < avg) ++lg;
    return lg;
}

constexpr int kRsPrUnroll = 4;   // row groups a wave keeps in flight

template <int V, bool XBUF, bool AXPBY = false>
__global__ __launch_bounds__(kBlock) void rs_pr_kernel(int M, long long K, int N, int ldx, int ldy, const int* __restrict__ rowptr,
                                                        const int* __restrict__ colidx,
                                                        const float* __restrict__ vals,
                                                        const float* __restrict__ X, float* __restrict__ Y,
                                                        int logG_in, Scaling sc = Scaling{1.0f, 0.0f}) {
    constexpr int U = kRsPrUnroll;
    const int lane = lane_id();
    const unsigned nnz = (unsigned)rowptr[M];
    const int logG = logG_in >= 0 ? logG_in : pr_lanes_log2(nnz, M);
    const int G = 1 << logG;
    const int gl = lane & (G - 1);              // lane inside the group
    const int g = lane >> logG;                 // group inside the wave
    const int rows_per_wave = kWave >> logG;    // at most 32: a row has at least two lanes
    const unsigned nwaves = gridDim.x * kWavesPerBlock;
    const unsigned gw = xcd_contiguous(blockIdx.x, gridDim.x) * kWavesPerBlock + wave_in_block();
    // a wave step covers U * rows_per_wave consecutive rows: U independent load -> gather -> reduce chains
    const unsigned rows_per_step = (unsigned)(U * rows_per_wave);
    const unsigned nsteps = ((unsigned)M + rows_per_step - 1) / rows_per_step;
    // XBUF: the dense operand is read through a descriptor (its byte offsets fit 32 bits)
    const __amdgpu_buffer_rsrc_t rx = make_buffer(X, XBUF ? dense_bytes(K, ldx, N) : 0ull);

    auto fetch_dense = [&](unsigned c, bool ok, int n0, float (&x)[V]) {
        if constexpr (XBUF) {
            buffer_load_vec<V>(rx, ok ? c * (unsigned)ldx * 4u + (unsigned)n0 * 4u : kOutOfRange, x);
        } else {
            load_vec_dword_aligned<V>(X + (size_t)c * ldx + n0, x);                      // c is 0 when switched off: a valid row
#pragma unroll
            for (int i = 0; i < V; ++i) x[i] = ok ? x[i] : 0.0f;
        }
    };

    for (int n0 = 0; n0 < N; n0 += V) {
        for (unsigned st = gw; st < nsteps; st += nwaves) {
            // Row bounds: lanes 0..rows_per_wave fetch consecutive rowptr entries with one coalesced
            // load per row group and every lane picks its row's pair from them (cross-lane read).
            // Letting all lanes of a group load the same two words costs the memory pipeline a
            // cycle per lane, as much as the gather itself.
            unsigned rs[U], re[U];
            const unsigned long long row0 = (unsigned long long)st * rows_per_step;
            const __amdgpu_buffer_rsrc_t rp = make_buffer(rowptr + row0, ((unsigned long long)M + 1 - row0) * 4ull);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const unsigned idx = (unsigned)(u * rows_per_wave + lane);
                const unsigned v = (unsigned)__builtin_amdgcn_raw_buffer_load_b32(
                    rp, lane <= rows_per_wave ? idx * 4u : kOutOfRange, 0, 0);     // past rowptr[M]: 0
                rs[u] = (unsigned)__shfl((int)v, g);
                re[u] = (unsigned)__shfl((int)v, g + 1);
                if (row0 + (unsigned)(u * rows_per_wave + g) >= (unsigned long long)M) re[u] = rs[u];   // no such row
            }
            // the step's entries start at its first row's start: offsets from there stay small
            const unsigned base = (unsigned)uniform((int)rs[0]);
            const unsigned long long bytes = (unsigned long long)(nnz - (base < nnz ? base : nnz)) * 4ull;
            const __amdgpu_buffer_rsrc_t rc = make_buffer(colidx + base, bytes);
            const __amdgpu_buffer_rsrc_t ra = make_buffer(vals + base, bytes);
            // column and value of the entry at position p (zeros when switched off)
            auto fetch_entry = [&](unsigned p, bool ok, unsigned& c, float& a) {
                const unsigned off = ok ? (p - base) * 4u : kOutOfRange;
                c = (unsigned)buffer_stream_i32(rc, off);
                a = buffer_stream_f32(ra, off);
            };
            float acc[U][V];
            // first entry of every lane: for rows no longer than the group this is all there is
            {
                unsigned c[U]; float a[U], x[U][V];
#pragma unroll
                for (int u = 0; u < U; ++u) fetch_entry(rs[u] + gl, rs[u] + gl < re[u], c[u], a[u]);
#pragma unroll
                for (int u = 0; u < U; ++u) fetch_dense(c[u], rs[u] + gl < re[u], n0, x[u]);
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int i = 0; i < V; ++i) acc[u][i] = a[u] * x[u][i];
            }
            // the rest of longer rows, two gathers in flight per lane
#pragma unroll
            for (int u = 0; u < U; ++u) {
                for (unsigned p = rs[u] + gl + G; p < re[u]; p += 2u * G) {
                    unsigned c0, c1; float a0, a1, x0[V], x1[V];
                    const bool ok1 = p + G < re[u];
                    fetch_entry(p, true, c0, a0);
                    fetch_entry(p + G, ok1, c1, a1);
                    fetch_dense(c0, true, n0, x0);
                    fetch_dense(c1, ok1, n0, x1);
#pragma unroll
                    for (int i = 0; i < V; ++i) acc[u][i] = fmaf(a1, x1[i], fmaf(a0, x0[i], acc[u][i]));
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                segmented_scan<V>(acc[u], gl, lane, G);   // all 64 lanes arrive here together
                const unsigned long long row = row0 + (unsigned)(u * rows_per_wave + g);
                if (row < (unsigned long long)M && gl == G - 1) {
                    float* y = Y + (size_t)row * ldy + n0;
                    if constexpr (AXPBY) scale_into<V, true>(acc[u], y, sc);
                    store_vec_dword_aligned<V>(y, acc[u]);
                }
            }
        }
    }
}

// ===========================================================================
// Row-split, sequential reduction with coalesced sparse-row caching
// (Section 2.1.3)
// ===========================================================================
//
// 2^logG lanes own a row and V*2^logG dense columns (lane gl owns columns
// [cb*G*V + gl*V, +V)); a wave owns the 64/G consecutive rows of its lane
// groups.  Those rows' (colidx, val) pairs are one contiguous stretch of the
// CSR arrays, so the whole wave stages it in LDS with coalesced loads, kRsSrTile
// pairs at a time (with few lanes per row a group-by-group load would fetch a
// handful of bytes per group).  Every group then walks the cached part of its
// own row and accumulates its own columns: the dense accesses of a group are
// one contiguous 4*V*G-byte piece of a row of X.
// blockIdx.y selects the column block when N > 64*V.
//
// When few lanes span the columns, 64 / G rows can be more than a round of the
// cache holds.  H = 2^logH lanes per column group then share a row's entries
// (lane h takes every H-th) and add their sums up at the end, so that a wave's
// 64 / (G H) rows fit one round and every lane walks in it.  Neighbouring lanes
// hold neighbouring rows: on a stencil or band their gathers fall into the same
// few lines of X, which costs the address unit a fraction of what one row's
// scattered columns cost.  27-point stencil on 128^3, one lane per row and column with its loads
// one after the other against H lanes with all of a round's loads at once: N = 1 154 -> 94 us (H = 4, 5.0 TB/s; through the
// balanced parallel kernel 122 us), N = 4 188 -> 114 us, N = 8 198 -> 145 us.
// Bound by: HBM streams on banded matrices; the lines gathered from X, out of
// the L1's and L2's misses, elsewhere.  There waves that fetch bounds and entries
// go before those that walk (`staging_first`, chosen by the host): they
// are few issue slots away from gathers of their own, and what the CU has in
// flight is what bounds the call: 262 144 rows of 64, N = 4, 103 -> 93 us.

constexpr int kRsSrTile = 512;   // cached pairs per wave and round
// DEPTH (template parameter of the sequential kernels) = dense-row loads a lane keeps in flight.
// More is not always better.  With ascending columns the lanes of a wave, and the waves that
// start together, sweep X from low to high rows in step; every load in flight widens the window
// of X they touch at one time, and once that window outgrows the L2 the hit rate drops (measured
// on 2^20 rows of 27 uniform columns, N = 4: 58 % L2 hits and 224 us at depth 1, 26 % and 373 us
// at depth 4).  Rows that hit in cache anyway want the latency hidden instead (27-point stencil,
// N = 8: 204 us at depth 4, 260 us at depth 1), and so do rows of uneven length.  The host picks.

// position of pair e of a round in the LDS tile: eight pairs of padding after every 64, so that rows of 32, 64, ... entries
// do not put all lane groups on the same banks
__device__ __forceinline__ unsigned padded(unsigned e) { return e + ((e >> 6) << 3); }

template <int V, bool XBUF, int DEPTH, bool AXPBY = false, bool RAGGED = false>
__global__ __launch_bounds__(kBlock) void rs_sr_kernel(int M, long long K, int N, int ldx, int ldy, const int* __restrict__ rowptr,
                                                        const int* __restrict__ colidx,
                                                        const float* __restrict__ vals,
                                                        const float* __restrict__ X, float* __restrict__ Y,
                                                        int logG, int logH, int cols_per_block, int staging_first,
                                                        Scaling sc = Scaling{1.0f, 0.0f}) {
    constexpr int T = kRsSrTile;
    __shared__ __align__(16) uint2 s_ent[kWavesPerBlock][T + T / 8];     // row of X (XBUF: its byte offset), value
    const int lane = lane_id();
    const int wib = wave_in_block();
    uint2* ent = s_ent[wib];
    const int G = 1 << logG;
    const int H = 1 << logH;                                     // lanes of a row that share its entries
    const int log_rows = 6 - logG - logH;
    const int rows_per_wave = 1 << log_rows;
    const int gl = lane & (G - 1);
    const int g = (lane >> logG) & (rows_per_wave - 1);
    const int h = lane >> (6 - logH);

    const LaneColumns mine = lane_columns<V, RAGGED>(blockIdx.y, cols_per_block, gl, N);
    const long long n = mine.first;                              // my first dense column
    const bool col_ok = mine.any;

    const unsigned nwaves = gridDim.x * kWavesPerBlock;
    const unsigned gw = xcd_contiguous(blockIdx.x, gridDim.x) * kWavesPerBlock + wib;
    const unsigned ngroups = (unsigned)(((long long)M + rows_per_wave - 1) >> log_rows);

    // XBUF: the dense operand is read through a descriptor (its byte offsets fit 32 bits)
    const unsigned long long x_bytes = dense_bytes(K, ldx, N);
    const __amdgpu_buffer_rsrc_t rx = make_buffer(X, XBUF ? x_bytes : 0ull);
    const unsigned n_bytes = (unsigned)n * 4u;
    const unsigned pitch = XBUF ? (unsigned)ldx * 4u : 1u;

    for (unsigned rg = gw; rg < ngroups; rg += nwaves) {
        if (staging_first) __builtin_amdgcn_s_setprio(3);
        const long long row0 = (long long)rg * rows_per_wave;
        const long long row = row0 + g;
        const bool live = row < M;
        unsigned rs = 0, re = 0;
        if (live) { rs = (unsigned)rowptr[row]; re = (unsigned)rowptr[row + 1]; }
        const long long row_end = row0 + rows_per_wave < M ? row0 + rows_per_wave : M;
        const unsigned ps = (unsigned)uniform((int)rs);                  // lane 0 holds row0
        const unsigned pe = (unsigned)uniform(rowptr[row_end]);          // the wave's rows span [ps, pe)
        float acc[V];
#pragma unroll
        for (int i = 0; i < V; ++i) acc[i] = 0.0f;
        float old[AXPBY ? V : 1];                            // scaled form: on its way while the row is summed
        if constexpr (AXPBY) {
#pragma unroll
            for (int i = 0; i < V; ++i) old[i] = 0.0f;
            if (live && col_ok && h == 0 && sc.beta != 0.0f) load_vec_dword_aligned<V>(Y + (size_t)row * ldy + n, old);
        }

        for (unsigned ws = ps; ws < pe; ws += (unsigned)T) {
            if (staging_first) __builtin_amdgcn_s_setprio(3);
            wave_lds_sync();                    // last round's readers are done
            const unsigned long long bytes = (unsigned long long)(pe - ws) * 4ull;
            const __amdgpu_buffer_rsrc_t rc = make_buffer(colidx + ws, bytes);
            const __amdgpu_buffer_rsrc_t ra = make_buffer(vals + ws, bytes);
            // C * 64 pairs from pair `from` on, all loads before the first wait (a branch around each one makes the compiler
            // wait inside it: up to eight round trips to memory in a row, 116 instead of 95 us on the stencil at N = 1);
            // past the stretch's end they read nothing
            auto stage = [&](unsigned from, auto count) {
                constexpr int C = decltype(count)::value;
                unsigned c[C]; float a[C];
#pragma unroll
                for (int k = 0; k < C; ++k) {
                    const unsigned off = (from + (unsigned)(k * kWave + lane)) * 4u;
                    c[k] = (unsigned)buffer_stream_i32(rc, off);
                    a[k] = buffer_stream_f32(ra, off);
                }
#pragma unroll
                for (int k = 0; k < C; ++k)
                    ent[(from >> 6) * (kWave + 8) + k * (kWave + 8) + lane] = make_uint2(c[k] * pitch, __builtin_bit_cast(unsigned, a[k]));
            };
            const unsigned left = pe - ws;                    // wave-uniform
            if constexpr (DEPTH == 1) {
                // rows in step: the L2 is to hold the band of X that all waves walk, and the streams in flight take room in
                // it, 4 KB a wave at eight loads per array (2^20 rows of 27, 16 MB of X: 228 -> 346 us)
                for (unsigned from = 0; from < (unsigned)T && from < left; from += 2u * kWave)
                    stage(from, std::integral_constant<int, 2>{});
            } else if (left <= 64u) {
                stage(0u, std::integral_constant<int, 1>{});
            } else if (left <= 128u) {
                stage(0u, std::integral_constant<int, 2>{});
            } else if (left <= 256u) {
                stage(0u, std::integral_constant<int, 4>{});
            } else {
                stage(0u, std::integral_constant<int, T / kWave>{});
            }
            wave_lds_sync();
            const unsigned we = pe - ws > (unsigned)T ? ws + T : pe;
            __builtin_amdgcn_s_setprio(0);
            const unsigned lo = (rs > ws ? rs : ws) - ws;
            const unsigned hi = (re < we ? re : we) - ws;         // may lie before lo: the row is not in this round
            if (col_ok) {
                for (unsigned p0 = lo + (unsigned)h; (int)p0 < (int)hi; p0 += (unsigned)(DEPTH * H)) {
                    float x[DEPTH][V]; float a[DEPTH];
#pragma unroll
                    for (int u = 0; u < DEPTH; ++u) {
                        const unsigned e = p0 + (unsigned)(u * H);
                        const bool ok = u == 0 || e < hi;
                        const uint2 t = ent[padded(ok ? e : p0)];
                        a[u] = ok ? __builtin_bit_cast(float, t.y) : 0.0f;
                        if constexpr (XBUF) {
                            buffer_load_vec<V>(rx, ok ? t.x + n_bytes : kOutOfRange, x[u]);
                        } else {
                            load_vec_dword_aligned<V>(X + (size_t)t.x * ldx + n, x[u]);      // switched off: the row of p0 once more
#pragma unroll
                            for (int i = 0; i < V; ++i) x[u][i] = ok ? x[u][i] : 0.0f;
                        }
                    }
#pragma unroll
                    for (int u = 0; u < DEPTH; ++u)
#pragma unroll
                        for (int i = 0; i < V; ++i) acc[i] = fmaf(a[u], x[u][i], acc[i]);
                }
            }
        }
        for (int m = kWave >> 1; m >= (G << log_rows); m >>= 1)           // the row's H partial sums
#pragma unroll
            for (int i = 0; i < V; ++i) acc[i] += __shfl_xor(acc[i], m);
        if (live && col_ok && h == 0) {
            float* y = Y + (size_t)row * ldy + n;
            if constexpr (AXPBY) {
#pragma unroll
                for (int i = 0; i < V; ++i) acc[i] = sc.beta != 0.0f ? fmaf(sc.alpha, acc[i], sc.beta * old[i]) : sc.alpha * acc[i];
            }
            if (AXPBY && RAGGED && mine.skip != 0) {
                // the scaled result depends on the old Y, which the neighbour (another column block, another time)
                // may have replaced: the shared columns are the neighbour's to write
#pragma unroll
                for (int i = 1; i < V; ++i)
                    if (i >= mine.skip) y[i] = acc[i];
            } else {
                store_vec_dword_aligned<V>(y, acc);      // plain product: shared columns hold the same bits in both lanes
            }
        }
    }
}

// Row-split sequential reduction WITHOUT the LDS tile (the kernel Section 2.1.3 compares its
// sparse-row caching against): same row and column mapping as rs_sr_kernel, but every lane of a
// group reads colidx[p] and vals[p] itself, straight from memory, one entry after the other.
// Kept for measurements only.
template <int V>
__global__ __launch_bounds__(kBlock) void rs_sr_direct_kernel(int M, int N, int ldx, int ldy, const int* __restrict__ rowptr,
                                                               const int* __restrict__ colidx,
                                                               const float* __restrict__ vals,
                                                               const float* __restrict__ X, float* __restrict__ Y,
                                                               int logG, int cols_per_block) {
    const int lane = lane_id();
    const int G = 1 << logG;
    const int gl = lane & (G - 1);
    const int g = lane >> logG;
    const int rows_per_wave = kWave >> logG;
    const LaneColumns mine = lane_columns<V, false>(blockIdx.y, cols_per_block, gl, N);
    const long long n = mine.first;
    const bool col_ok = mine.any;
    const unsigned nwaves = gridDim.x * kWavesPerBlock;
    const unsigned gw = xcd_contiguous(blockIdx.x, gridDim.x) * kWavesPerBlock + wave_in_block();
    const unsigned ngroups = ((unsigned)M + rows_per_wave - 1) / rows_per_wave;
    for (unsigned rg = gw; rg < ngroups; rg += nwaves) {
        const long long row = (long long)rg * rows_per_wave + g;
        if (row >= M || !col_ok) continue;
        const int rs = rowptr[row], re = rowptr[row + 1];
        float acc[V];
#pragma unroll
        for (int i = 0; i < V; ++i) acc[i] = 0.0f;
        for (int p = rs; p < re; ++p) {
            const int c = colidx[p];
            const float a = vals[p];
            float x[V];
            load_vec<V>(X + (size_t)c * ldx + n, x);
#pragma unroll
            for (int i = 0; i < V; ++i) acc[i] = fmaf(a, x[i], acc[i]);
        }
        store_vec<V>(Y + (size_t)row * ldy + n, acc);
    }
}

// ===========================================================================
// nnz-balanced kernels: common partition
// ===========================================================================
//
// The paper hands every warp the same count of stored entries (Section 2.1.1).
// Counting only stored entries leaves one hole: a stretch of (nearly) empty
// rows puts an unbounded number of row boundaries into one share.  So the
// unit of work here is the *item* of the merge path of Merrill & Garland, which the
// paper cites as the fine-grained way to balance (Section 1): the list
//     entries of row 0, end of row 0, entries of row 1, end of row 1, ...
// has nnz + M items; row r's entries sit at diagonals
// [r + rowptr[r], r + rowptr[r+1]) and its end marker at r + rowptr[r+1].
// Cutting that list into equal pieces bounds both the entries and the rows
// of a piece.  For matrices without empty stretches it is the paper's fixed
// share of non-zeros up to the few percent that row markers add.
//
// The list is cut into contiguous chunks, one a wave (waves of one XCD hold
// neighbouring chunks).  Chunks begin at multiples of a quantum of items and
// differ by at most one quantum: chunk c covers quanta [c*Q/parts, (c+1)*Q/parts)
// of the Q quanta, so no wave stays without work while another holds two quanta.
// A wave finds the first row of its chunk with a 64-way search and then walks.
// This split is static; where a wave's share is long and the call has memory for
// it, nb_sr_run_kernel cuts the list finer and the waves take most of the chunks
// from queues (ChunkQueues).
//
// Rows whose items straddle a chunk boundary (in the sequential kernel: the
// boundary of a lane group's run) are combined with fp32 atomic adds; the
// paper does not say how partial rows of different warps meet.  That needs
// zeros underneath.  Where the call has memory for it the waves see to them
// themselves (RowSharing); otherwise a small "prepare" kernel zeroes exactly
// those rows and no others (in the scaled form of nb_sr_run_kernel also the rows
// without entries).  Every other row is written once with a plain store by the
// chunk that holds its end marker.

// Zeroes the rows whose items do not all lie in one piece of the partition (beta != 0, the scaled
// variants: multiplies them by beta instead, so that the partial sums added later land on beta * Y).
// The pieces are the `parts` chunks of the even split with quanta of
// 2^quantum_log2 items, cut further into tiles of 2^tile_log2 items counted
// from the chunk's start when tile_log2 >= 0.
// R rows a thread for the test (split rows are few: at most two per piece); those with a multiple of the quantum among their items
// go on, one a thread and round.
// QUEUES: the chunks' first rows and the counters are written as well.
// Bound by the trips to memory (row bounds, zeros) and, with queues, by its instructions: at M = 2^20 nearly every wave has such a
// row and a row to clear.  R-MAT 2^20 x 16 at N = 32 / 128 12.2 / 11.8 -> 5.9 / 7.8 us with two rows a thread, the pieces told apart by
// one look at the second chunk in place of two searches and divisions, and zeros 16 bytes a lane in place of 4.
// `empty_rows`: rows without entries are treated alike and the main launch leaves them alone (nb_sr_run_kernel, scaled form).  Half of
// a power-law graph's rows are such; a wave at the sparse end has hundreds, and their old values were four or more trips to memory
// per 64 of them, one after the other.  R-MAT 2^17 x 16 at N = 8 / 16 / 40 / 100 29.5 / 41.6 / 74.2 / 153.4 ->
// 28.0 / 36.9 / 62.0 / 114.5 us, 2^20 x 12 at N = 20 305 -> 263 us.  Plain products write zeros without waiting and keep them
// where they are (by this launch 2^17 x 16 at N = 16 / 40 23.2 / 40.3 -> 23.9 / 43.1 us).
template <bool QUEUES, int R>
__global__ __launch_bounds__(kBlock) void nb_prepare_kernel(int M, int N, int ldy, const int* __restrict__ rowptr,
                                                             float* __restrict__ Y, unsigned parts, unsigned quantum_log2,
                                                             int tile_log2, float beta, ChunkQueues queues, int empty_rows) {
    const long long row0 = ((long long)blockIdx.x * kBlock + threadIdx.x) * R;
    const unsigned items = (unsigned)rowptr[M] + (unsigned)M;               // on its way with the rows' bounds
    if constexpr (QUEUES) { queues.fit(items, (unsigned)M); parts = queues.chunks; quantum_log2 = queues.size_log2; }
    unsigned bound[R + 1];
    if (R == 1 && row0 < M) {
        bound[0] = (unsigned)rowptr[row0];
        bound[1] = (unsigned)rowptr[row0 + 1];
    } else if (R > 1 && row0 + R <= M) {
        __builtin_memcpy(bound, rowptr + row0, sizeof(bound));
    } else {
#pragma unroll
        for (int k = 0; k <= R; ++k) bound[k] = (unsigned)rowptr[row0 + k < M ? row0 + k : M];
    }
    unsigned split = 0, look = 0;                                           // bit k: row row0 + k
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const long long row = row0 + k;
        const unsigned first = (unsigned)row + bound[k];                    // diagonal of the row's first item
        const unsigned last = (unsigned)row + bound[k + 1];                 // diagonal of its end marker
        const unsigned before = first - 1u;                                 // wraps for the list's first item: in no quantum of this row
        // An empty row is a single item.  Every chunk and tile starts at a multiple of the quantum, so a row
        // whose items lie inside one quantum cannot be split: most rows stop here, before the divisions.
        // Nor does a chunk start in a row that has no multiple of the quantum among its items.
        const bool across = first != last && (first >> quantum_log2) != (last >> quantum_log2);
        const bool starting = QUEUES && ((before >> quantum_log2) != (last >> quantum_log2) || row == M - 1);
        if (row < M) {
            if (empty_rows != 0 && first == last) split |= 1u << k;
            if (across || starting) look |= 1u << k;
        }
    }
    // The others, a row a lane and round: the first one of each lane's, and so on.  With one row a lane there is a single round, and
    // no lane waits for another's unless they write first rows together (R-MAT 2^20 x 16 at N = 1, whole calls 69.8 -> 69.0 us).
    const EvenSplit es(items, parts, quantum_log2);
    // Chunks of one quantum each, unless the caller's entry count was below the matrix's: no divisions
    const bool one_each = QUEUES && es.Q == parts;
    for (bool round = R == 1 ? QUEUES || look != 0u : __ballot(look != 0u) != 0ull; round; round = R > 1 && __ballot(look != 0u) != 0ull) {
        const bool any = look != 0u;
        const int k = any ? __builtin_ctz(look) : 0;
        look &= look - 1u;
        const long long row = row0 + k;
        unsigned first = bound[0], last = bound[1];
#pragma unroll
        for (int q = 1; q < R; ++q) { first = q == k ? bound[q] : first; last = q == k ? bound[q + 1] : last; }
        first += (unsigned)row; last += (unsigned)row;
        unsigned c_from = 0, c_to = 0;                                      // chunks that start within the row's items
        if (any) {
            const unsigned c1 = one_each ? first >> quantum_log2 : es.chunk_of(first);
            const unsigned c2 = one_each ? last >> quantum_log2 : es.chunk_of(last);
            if (first != last) {
                bool cut = c1 != c2;
                if constexpr (QUEUES) cut = cut && !queues.one_piece(c1, c2);
                if (!cut && tile_log2 >= 0) {
                    const unsigned start = es.start(c1);
                    cut = (first - start) >> tile_log2 != (last - start) >> tile_log2;
                }
                if (cut) split |= 1u << k;
            }
            if constexpr (QUEUES) {
                c_from = c1;
                if (one_each) {
                    c_from += first != c1 << quantum_log2;
                } else {
                    if (es.start(c1) < first) ++c_from;
                    while (c_from > 0u && es.start(c_from - 1u) >= first) --c_from;  // chunks without items start where the next one does
                }
                c_to = (c2 < parts ? c2 + 1u : parts);
            }
        }
        if constexpr (QUEUES) {
            // a few chunks each; a row of very many is written by the whole wave
            constexpr unsigned kOwn = 8;
            for (unsigned c = c_from; c < c_to && c < c_from + kOwn; ++c) queues.starts[c] = (int)row;
            unsigned long long wide = __ballot(c_to > c_from + kOwn);
            while (wide != 0ull) {                                          // wave-uniform
                const int src = __ffsll((long long)wide) - 1;
                wide &= wide - 1ull;
                const unsigned wide_from = (unsigned)read_lane((int)c_from, src) + kOwn, wide_to = (unsigned)read_lane((int)c_to, src);
                const int r = read_lane((int)row, src);
                for (unsigned c = wide_from + (unsigned)lane_id(); c < wide_to; c += (unsigned)kWave) queues.starts[c] = r;
            }
            // chunks past the last item, and the list's end
            if (any && row == M - 1)
                for (unsigned c = c_to; c <= parts; ++c) queues.starts[c] = M;
        }
    }
    if constexpr (QUEUES) {
        for (size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x; t < queues.counters; t += (size_t)gridDim.x * kBlock)
            queues.taken[t * kQueuePitch] = 0u;
    }
    if (N < 4 || (N <= 8 && !empty_rows)) {            // few and narrow: the thread clears its own
        for (; split != 0u; split &= split - 1u) {
            float* y = Y + (size_t)(row0 + __builtin_ctz(split)) * ldy;
            for (int n = 0; n < N; ++n) y[n] = beta != 0.0f ? beta * y[n] : 0.0f;
        }
        return;
    }
    // The workgroup treats its rows together: they are listed, 2^log_lanes lanes take one, eight of a lane's in flight at a time, so
    // that the loads of the scaled form overlap.  (The long rows of a graph are neighbours and all split: one row after the
    // other in one wave took R-MAT 2^18 x 13 at N = 58 100 of 206 us; with a wave to a row of 8 / 12 columns 2^18 x 6 / 2^17 x 16 in the
    // scaled form took 33 / 45 instead of 28 / 38 us, with one to a row of 12 / 20 columns plain products on 2^17 x 16
    // 28.3 / 31.6 instead of 26.5 / 30.6 us.)
    __shared__ int s_rows[kBlock * R];
    __shared__ int s_count[kWavesPerBlock];
    const int lane = lane_id(), wib = wave_in_block();
    unsigned long long mine[R];
    int own = 0;
#pragma unroll
    for (int k = 0; k < R; ++k) { mine[k] = __ballot((split >> k) & 1u); own += (int)__popcll(mine[k]); }
    if (lane == 0) s_count[wib] = own;
    __syncthreads();
    int before = 0, count = 0;
#pragma unroll
    for (int w = 0; w < kWavesPerBlock; ++w) { before += w < wib ? s_count[w] : 0; count += s_count[w]; }
#pragma unroll
    for (int k = 0; k < R; ++k) {
        if ((split >> k) & 1u) s_rows[before + (int)__popcll(mine[k] & ((1ull << lane) - 1ull))] = (int)(row0 + k);
        before += (int)__popcll(mine[k]);
    }
    __syncthreads();
    if (beta == 0.0f) {                                  // nothing to wait for: zeros, four columns a lane, the last four where N ends
        const int log_quads = N > 2 * kWave ? 6 : 32 - __builtin_clz((unsigned)(N + 3) / 4u - 1u | 1u);
        for (int r = (int)threadIdx.x >> log_quads; r < count; r += kBlock >> log_quads) {
            float* y = Y + (size_t)s_rows[r] * ldy;
            const float zero[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            for (int n = 4 * (int)(threadIdx.x & ((1u << log_quads) - 1u)); n < N; n += 4 << log_quads)
                store_vec_dword_aligned<4>(y + (n + 4 <= N ? n : N - 4), zero);
        }
        return;
    }
    constexpr int U = 8;
    const int log_lanes = N > kWave / 2 ? 6 : 32 - __builtin_clz((unsigned)N - 1u | 1u);
    const int lanes = 1 << log_lanes, step = kBlock >> log_lanes;                    // rows that the workgroup takes at once
    for (int r = log_lanes == 6 ? wib : (int)threadIdx.x >> log_lanes; r < count; r += step * U) {       // a wave's row is known to be one
        for (int n = lane & (lanes - 1); n < N; n += lanes) {
            float v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int at = r + u * step;
                v[u] = at < count ? Y[(size_t)s_rows[at] * ldy + n] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int at = r + u * step;
                if (at < count) Y[(size_t)s_rows[at] * ldy + n] = beta * v[u];
            }
        }
    }
}

// The chunk of the calling wave, number `wave` of `waves`.
struct ChunkPlan {
    unsigned nnz, items, wave;
    EvenSplit split;
    __device__ __forceinline__ ChunkPlan(unsigned nnz_, unsigned items_, unsigned waves, unsigned wave_, unsigned quantum_log2)
        : nnz(nnz_), items(items_), wave(wave_), split(items_, waves, quantum_log2) {}
    __device__ __forceinline__ bool range(unsigned& d0, unsigned& d1) const {
        d0 = split.start(wave);
        const unsigned e = split.start(wave + 1);
        d1 = e < items ? e : items;
        return d0 < d1;
    }
};

__device__ __forceinline__ ChunkPlan plan_chunks(const int* __restrict__ rowptr, int M, unsigned quantum_log2) {
    const unsigned nnz = (unsigned)rowptr[M];
    return ChunkPlan(nnz, nnz + (unsigned)M, gridDim.x * kWavesPerBlock,
                     xcd_contiguous(blockIdx.x, gridDim.x) * kWavesPerBlock + wave_in_block(), quantum_log2);
}

// What the first round of a search probes does not depend on what is searched for: asked for beside the entry count, from
// which the diagonals follow, it saves a chunk's start one round trip to memory.
__device__ __forceinline__ int first_probe(const int* __restrict__ rowptr, int M, int lane) {
    const long long r = (long long)lane * ((M + 63ll) >> 6);
    return r < M ? rowptr[r + 1] : 0;
}

// Number of rows whose end marker lies before diagonal d, i.e. rows r with
// r + rowptr[r+1] < d (that key is strictly increasing in r).  64-way search,
// wave-uniform result.
// `probe`: first_probe().
__device__ __forceinline__ int wave_merge_rows_before(const int* __restrict__ rowptr, int M, unsigned d, int lane, int probe) {
    int lo = 0, hi = M;   // rows < lo end before d; rows >= hi do not
    for (bool first = true; hi > lo; first = false) {
        const int step = (int)(((long long)hi - lo + 63) >> 6);
        const long long r = (long long)lo + (long long)lane * step;
        int v = probe;
        if (!first) v = r < hi ? rowptr[r + 1] : 0;
        const bool before = r < hi && (unsigned)r + (unsigned)v < d;
        const int cnt = __popcll(__ballot(before));   // probes are monotone: 1...10...0
        if (cnt == 0) {
            hi = lo;
        } else {
            const int nlo = lo + (cnt - 1) * step + 1;
            const int nhi = lo + cnt * step;
            lo = nlo;
            hi = nhi < hi ? nhi : hi;
        }
    }
    return uniform(lo);
}

// Rows that ended before diagonal da, and before db (both searches of wave_merge_rows_before in lock-step: their
// probes are in flight together, so the second costs no further round trips).  `probe`: first_probe().
__device__ __forceinline__ void wave_merge_rows_before2(const int* __restrict__ rowptr, int M, unsigned da, unsigned db,
                                                        int lane, int probe, int& ra, int& rb) {
    int lo[2] = {0, 0}, hi[2] = {M, M};
    const unsigned d[2] = {da, db};
    bool first = true;
    while (hi[0] > lo[0] || hi[1] > lo[1]) {
        int step[2], v[2];
        long long r[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            step[k] = (int)(((long long)hi[k] - lo[k] + 63) >> 6);
            r[k] = (long long)lo[k] + (long long)lane * step[k];
            v[k] = probe;
            if (!first) v[k] = (hi[k] > lo[k] && r[k] < hi[k]) ? rowptr[r[k] + 1] : 0;
        }
        first = false;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (hi[k] > lo[k]) {                                   // wave-uniform
                const bool before = r[k] < hi[k] && (unsigned)r[k] + (unsigned)v[k] < d[k];
                const int cnt = __popcll(__ballot(before));       // probes are monotone: 1...10...0
                if (cnt == 0) {
                    hi[k] = lo[k];
                } else {
                    const int nlo = lo[k] + (cnt - 1) * step[k] + 1;
                    const int nhi = lo[k] + cnt * step[k];
                    lo[k] = nlo;
                    hi[k] = nhi < hi[k] ? nhi : hi[k];
                }
            }
        }
    }
    ra = uniform(lo[0]);
    rb = uniform(lo[1]);
}

// SNAP: a row belongs wholly to the chunk that holds its first item (the host asks for it when the longest row is short
// against a wave's share).  Nothing is added to memory then, so the launch that clears the shared rows falls away (3-10 us)
// and the result is the same from run to run.  Turns the bounds of a chunk, [d0, d1) with `is` rows ended before d0 and `ie`
// before d1, into those of its rows.
__device__ __forceinline__ void snap_to_rows(const int* __restrict__ rowptr, int M, unsigned d0, unsigned d1, int& is, int& ie,
                                             unsigned& js, unsigned& je) {
    // Rows that started before a chunk's first item belong to the chunk before.  Asking for both rows' bounds at once saves a trip
    // to memory and costs more than it saves: 100 000 lognormal rows of 6 at N = 6 10.24 -> 10.40 us, of 20 at N = 1 16.1 -> 16.2 us.
    if (is < M && (unsigned)is + (unsigned)rowptr[is] < d0) ++is;
    if (ie < M && (unsigned)ie + (unsigned)rowptr[ie] < d1) ++ie;
    is = uniform(is); ie = uniform(ie);
    js = (unsigned)uniform(rowptr[is]);
    je = (unsigned)uniform(rowptr[ie]);
}

constexpr unsigned kNoRow = 0xffffffffu;

// Rows whose entries lie in several chunks, without a launch that clears them first (shared_rows.hpp).  `words`: one for each
// chunk and column group, for the row that starts in it and is open at its end; nullptr: the prepare launch has been there.
// The prepare launch is two to three dependent trips to memory, 4.8 us, whatever the size.  Here a wave claims its word in front of its
// searches, which take longer, and its zeros are under way beside its first entries; what is left of the cost is a trip to
// memory at a chunk's end (nb_sr_run_kernel: at its first row end, too).  Whole calls, with that launch / without: R-MAT 2^13 x 9 at N = 15 10.2 / 8.6 us, 2^18 x
// 10 at N = 6 32.0 / 29.5 us, 2^19 x 5 at N = 6, product and gradient 70.7 / 61.8 us, 2^16 x 16 at N = 41 57.1 / 49.6 us,
// 2^18 x 32 at N = 24 103.2 / 99.5 us.
struct RowSharing { RowWord* words; RowWord call; };

struct DeviceWords {
    static __device__ __forceinline__ RowWord load(RowWord* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    static __device__ __forceinline__ void store(RowWord* p, RowWord v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    static __device__ __forceinline__ RowWord exchange(RowWord* p, RowWord v) {
        return __hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    static __device__ __forceinline__ bool replace(RowWord* p, RowWord& seen, RowWord v) {
        return __hip_atomic_compare_exchange_strong(p, &seen, v, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    static __device__ __forceinline__ void pause() { __builtin_amdgcn_s_sleep(1); }
    // waves on all XCDs find it once stores_done() is past
    static __device__ __forceinline__ void put(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
};

// The wave's earlier stores have reached the place where they were sent.
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The rows at the two ends of a chunk whose first item is d0: rows [is, ie) end in it, entries [js, je) lie in it.
struct ChunkEnds {
    unsigned head = 0, tail = 0;    // words of row `is` and of row `ie`
    bool gives_head = false, starts = false, whole = false, gives_tail = false;
    // row `is` ends here, started in an earlier chunk and has entries here
    __device__ __forceinline__ bool shares_head() const { return gives_head; }
    // row `ie` has its first entries here, others in later chunks
    __device__ __forceinline__ bool starts_tail() const { return starts; }
    // row `ie` has all its entries here (its end marker is the next chunk's)
    __device__ __forceinline__ bool whole_tail() const { return whole; }
    // row `ie` has some of its entries here
    __device__ __forceinline__ bool shares_tail() const { return gives_tail; }
    __device__ __forceinline__ ChunkEnds() {}
    __device__ __forceinline__ ChunkEnds(const EvenSplit& split, const int* __restrict__ rowptr, int M, unsigned chunk, unsigned d0, int is,
                                         int ie, unsigned js, unsigned je) {
        const unsigned h0 = (unsigned)rowptr[is], h1 = (unsigned)rowptr[is < M ? is + 1 : M];
        const unsigned t0 = (unsigned)rowptr[ie], t1 = (unsigned)rowptr[ie < M ? ie + 1 : M];
        const bool here = ie < M && je > (t0 > js ? t0 : js), first = (unsigned)ie + t0 >= d0;
        gives_head = is < ie && (unsigned)is + h0 < d0 && h1 > js;
        starts = here && first && t1 > je;
        whole = here && first && t1 <= je;
        gives_tail = here && !whole;
        // whatever the row pointers hold, there is such a word
        const auto word_of = [&](unsigned item) {
            const unsigned c = split.chunk_of(item);
            return (unsigned)uniform((int)(c < split.parts ? c : split.parts - 1u));
        };
        head = gives_head ? word_of((unsigned)is + h0) : chunk;
        tail = gives_tail && !starts ? word_of((unsigned)ie + t0) : chunk;
    }
};

// The same in three registers, for kernels that keep them over a long walk: four booleans take a pair of scalar registers each
// (uniform(): the compiler takes the word apart again otherwise).  Spilled, four booleans -> one word: nb_pr_kernel at N = 1 / 2 0 / 8 ->
// 0 / 4 (scaled 7 / 18 -> 2 / 15), vector registers at N = 2 131 -> 127, four waves a SIMD in place of three; nb_sr_run_kernel 2 to 10 -> 0 to
// 6.  Their calls' times did not move by more than runs differ.  Not elsewhere, where it frees scalar registers alone: nb_pr_kernel at N = 3 and 4
// is slower with it (Zipf 165 040 x 44 at N = 3 / 4 47.4 / 47.5 -> 47.9 / 47.9 us, 0.3 % in the mean of 12 calls), and so are hot runs (R-MAT
// 2^20 x 16 scaled at N = 1 / 2 70.1 / 85.5 -> 70.5 / 86.3 us, at N = 4 103.9 -> 102.5 us) and the tiles, whose chunks are short (0.3 % in the mean of
// 18 calls, R-MAT 2^17 x 16 scaled at N = 1 16.8 -> 16.9 us, lognormal 100 003 x 30 at N = 4 without statistics 23.4 -> 23.6 us).
struct HeldEnds {
    unsigned head = 0, tail = 0, kinds = 0;
    __device__ __forceinline__ HeldEnds() {}
    __device__ __forceinline__ HeldEnds(const ChunkEnds& e)
        : head(e.head), tail(e.tail),
          kinds((unsigned)uniform((e.shares_head() ? 1 : 0) | (e.starts_tail() ? 2 : 0) | (e.whole_tail() ? 4 : 0) | (e.shares_tail() ? 8 : 0))) {}
    __device__ __forceinline__ bool shares_head() const { return (kinds & 1u) != 0u; }
    __device__ __forceinline__ bool starts_tail() const { return (kinds & 2u) != 0u; }
    __device__ __forceinline__ bool whole_tail() const { return (kinds & 4u) != 0u; }
    __device__ __forceinline__ bool shares_tail() const { return (kinds & 8u) != 0u; }
};

// The parallel kernels' shared rows of V columns: lane i treats column i, so that a row's columns are one access, and a chunk's two rows are
// given at its end, their words asked for together.  With the first one given in the loop, and every column an access of one lane:
// R-MAT 2^18 x 16 with statistics (four waves a CU) at N = 3 / 4 39.1 / 40.9 -> 32.9 / 35.8 us (with the prepare launch 34.6 / 37.7 us), 2^16 x 32
// 17.9 / 18.8 -> 16.0 / 17.6 us, 2^16 x 16 without statistics 10.6 / 11.2 -> 9.8 / 10.5 us, Zipf 100 000 x 20 so at N = 4 17.9 -> 18.7 us (19.5 us);
// named, eight columns a lane, N = 16 / 48 on Poisson 50 000 x 12 18.3 / 56.6 -> 16.6 / 52.1 us (19.4 / 53.9 us).  Which column is the
// lane's; none (-1) for the lanes behind them and, where the second four of eight start at `second` < 4, for those that they repeat.
template <int V>
__device__ __forceinline__ int shared_column(int lane, int second) {
    const int column = lane < 4 ? lane : second + lane - 4;
    return lane < V && (lane < 4 || column >= 4) ? column : -1;
}
// A wave's part of a row, `part` in the lane of its column; lane 0 has `seen` the row's word.
template <bool AXPBY>
__device__ __forceinline__ void give_part(RowWord* word, RowWord call, RowWord seen, float* y, float part, int column, float beta) {
    bool sum = false;
    if (lane_id() == 0) sum = row_has_sum<DeviceWords>(word, call, seen);
    if (uniform(sum ? 1 : 0) != 0) {
        if (column >= 0) unsafeAtomicAdd(y + column, part);
    } else {
        const float v[1] = {part};
        if (column >= 0) write_part<DeviceWords, 1, AXPBY>(y + column, v, beta);
        stores_done();
        if (lane_id() == 0) publish_part<DeviceWords>(word, call);
    }
}

// ===========================================================================
// nnz-balanced, parallel reduction: vectorized segment reduction (Section 2.1.1)
// ===========================================================================
//
// Tile = W = 64*E items (E = 4*KQ entries per lane).
//   1. Entry 64*e + l of the tile is loaded by lane l (coalesced dword loads),
//      which gathers V dense values for it with one vector load and
//      multiplies.  Consecutive lanes hold consecutive entries, so the gather
//      of a wave touches as few cache lines as the matrix allows.
//   2. The products go through LDS once to change hands: afterwards lane l
//      holds the products of the E consecutive entries E*l ... and reduces them
//      in order in registers.
//   3. Row ends are scattered into LDS as marks (row i ends after entry q), so
//      a lane sees its own boundaries with one 16-byte LDS read.  A lane
//      without a boundary contributes its whole sum to the row that is open
//      across lanes; a lane with boundaries closes that open row with its
//      leading part, finishes the rows that lie inside it, and opens a new
//      segment with its trailing part.
//   4. The open row's running sum across lanes is the paper's segment
//      reduction: the wave64 DPP scan that adds a partner lane's value only
//      when no row boundary lies in between (one scan per tile instead of
//      one per 64 entries).
//   5. The rows that end in a tile are consecutive, so finished sums are put
//      into LDS by row and written out together: lane l stores row is + l.
//      Rows without entries keep the zero the buffer was cleared to.  The
//      store of the first 64 rows is issued a tile later, behind that tile's
//      loads.
//   6. The sum still open at the end of a tile is handed to the chunk's next
//      tile in a register; only the two ends of a chunk can need an atomic add.
//
// Memory operations inside the tile loop are unconditional: loads and the row
// store go through buffer descriptors, and a lane that has nothing to load or
// write pushes its offset out of range (the buffer unit returns zero / drops
// the store and touches no memory).  With no branch around them the
// outstanding-operation counter can be waited on exactly, which is what lets
// the next tile's loads stay in flight while this tile is reduced.
// blockIdx.y selects the group of V dense columns (N > V: one pass each).

template <int V, int KQ, bool AXPBY, bool SHARES>
__global__ __launch_bounds__(kBlock) void nb_pr_tiled_kernel(int M, long long K, int N, int ldx, int ldy, const int* __restrict__ rowptr,
                                                        const int* __restrict__ colidx,
                                                        const float* __restrict__ vals,
                                                        const float* __restrict__ X, float* __restrict__ Y,
                                                        int snap, Scaling sc, RowSharing sharing) {
    constexpr int E = 4 * KQ;
    constexpr int W = kWave * E;
    // accessed 16 bytes at a time: every wave's part starts on a 16-byte boundary ((W + 4) * 4 and W * V * 4 are multiples of 16)
    __shared__ __align__(16) unsigned s_bnd[kWavesPerBlock][W + 4];   // [W]: rows that end before the tile's first entry
    __shared__ __align__(16) float s_buf[kWavesPerBlock][W * V];      // products, then the tile's row results
    __shared__ __align__(16) float s_first[SHARES ? kWavesPerBlock : 1][V];     // the sum of the first row to end in the chunk
    const int lane = lane_id();
    const int wib = wave_in_block();
    unsigned* bnd = s_bnd[wib];
    float* buf = s_buf[wib];
    const int n0 = blockIdx.y * V;

    // Until its gathers are out a wave goes before those that reduce (set_wave_priority): 100 001 Zipf rows of 12 without
    // statistics at N = 2 / 3 / 4 15.0 / 17.5 / 18.8 -> 14.7 / 17.0 / 18.4 us; at N = 1 300 001 lognormal rows of 30 59.3 -> 60.1 us.
    if constexpr (V >= 2) __builtin_amdgcn_s_setprio(3);
    const int probe = first_probe(rowptr, M, lane);
    const ChunkPlan plan = plan_chunks(rowptr, M, 6);        // quanta of one wave's width
    const unsigned nnz = plan.nnz;
    const unsigned long long y_elems = dense_bytes(M, ldy, N) / 4ull;
    // V = 8: the lane's second four columns start here.  N = 5, 6, 7 (one pass, n0 = 0): at N - 4, overlapping
    // the first four; the shared columns get the same sums twice and are added to memory once.
    const int second = (V == 8 && N - n0 < 8) ? N - n0 - 4 : 4;

    auto add_to_row = [&](float* y, const float (&v)[V]) {
        if constexpr (V == 8) atomic_add_halves(y, v, second); else atomic_add_vec<V>(y, v);
    };
    auto y_of = [&](int row) { return Y + (size_t)row * ldy + n0; };
    // Rows shared with other waves, where no launch has cleared them.  The sum of the first row to end in the chunk is kept until the end: in
    // the loop, the wait for its word held up the next entries and gathers in every turn.
    RowWord* const words = sharing.words + (size_t)blockIdx.y * plan.split.parts;
    constexpr bool shares = SHARES;
    float* const first_sum = s_first[SHARES ? wib : 0];
    const int my_column = shared_column<V>(lane, second);

    unsigned d0, d1;
    if (!plan.range(d0, d1)) return;

    if (nnz == 0) {
        // nothing stored: every item is a row end; my rows are [d0, d1)
        float zero[V];
#pragma unroll
        for (int i = 0; i < V; ++i) zero[i] = 0.0f;
        for (unsigned r = d0 + lane; r < d1; r += kWave) {
            float* y = Y + (size_t)r * ldy + n0;
            float out[V];
#pragma unroll
            for (int i = 0; i < V; ++i) out[i] = 0.0f;
            if constexpr (AXPBY) scale_into<V, true>(out, y, sc, second);
            store_vec_dword_aligned<V>(y, out, second);
        }
        return;
    }

    int is, ie1;                                            // rows that ended before my chunk, and in it
    unsigned js;                                            // entries consumed before my chunk
    // the first row to end in my chunk started before it?  then its sum is shared with another wave
    bool first_split = false;
    ChunkEnds ends;
    RowWord found = 0;
    if constexpr (shares) {
        if (lane == 0) found = claim_row<DeviceWords>(words + plan.wave, sharing.call);
        wave_merge_rows_before2(rowptr, M, d0, d1, lane, probe, is, ie1);
        js = d0 - (unsigned)is;
    } else if (snap) {
        unsigned je1;
        wave_merge_rows_before2(rowptr, M, d0, d1, lane, probe, is, ie1);
        snap_to_rows(rowptr, M, d0, d1, is, ie1, js, je1);
        if (is == ie1) return;
        d0 = (unsigned)is + js;
        d1 = (unsigned)ie1 + je1;
    } else {
        is = wave_merge_rows_before(rowptr, M, d0, lane, probe);
        js = d0 - (unsigned)is;
        first_split = is < M && (unsigned)is + (unsigned)rowptr[is] < d0;
    }
    const int r_first = is;

    // entries of a tile starting at entry `from`: at most W.  The descriptor ends at the arrays' end,
    // so lanes past it load nothing; `on` = false switches the whole load off.
    auto load_entries = [&](unsigned from, bool on, int (&c)[E], float (&a)[E]) {
        const unsigned long long bytes = on ? (unsigned long long)(nnz - from) * 4ull : 0ull;
        const __amdgpu_buffer_rsrc_t rc = make_buffer(colidx + from, bytes);
        const __amdgpu_buffer_rsrc_t ra = make_buffer(vals + from, bytes);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const unsigned off = (unsigned)(e * kWave + lane) * 4u;
            c[e] = (int)__builtin_amdgcn_raw_buffer_load_b32(rc, off, 0, 2);
            a[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(ra, off, 0, 2));
        }
    };
    // start and end offset of row `first + lane`; rows past the last one read as 0, 0
    auto load_row_bounds = [&](int first, bool on, unsigned& start, unsigned& end) {
        const unsigned long long bytes = (on && first < M) ? (unsigned long long)(M + 1 - first) * 4ull : 0ull;
        const __amdgpu_buffer_rsrc_t rr = make_buffer(rowptr + first, bytes);
        typedef unsigned u2 __attribute__((ext_vector_type(2)));
        const u2 t = __builtin_amdgcn_raw_buffer_load_b64(rr, (unsigned)lane * 4u, 0, 0);
        start = t.x; end = t.y;
    };
    // the dense operand: byte offsets of X rows fit 32 bits unless X is 4 GB or more
    const unsigned long long x_bytes = dense_bytes(K, ldx, N);
    const bool x_small = x_bytes <= 0xffffffffull;
    const __amdgpu_buffer_rsrc_t rx = make_buffer(X + n0, x_small ? x_bytes - (unsigned)n0 * 4ull : 0ull);

    float carry[V];      // running sum of the row that is open at the tile boundary (wave-uniform)
#pragma unroll
    for (int i = 0; i < V; ++i) carry[i] = 0.0f;

    // two register sets take turns: while one tile is reduced the other set receives the next tile
    int cA[E], cB[E]; float aA[E], aB[E]; unsigned wA, wB, w_unused;
    load_row_bounds(is, true, w_unused, wA);
    load_entries(js, true, cA, aA);
    unsigned ds = d0;
    // Behind the entries, which otherwise wait for the two rows' bounds: R-MAT 2^16 x 16 at N = 1 / 4 10.1 / 12.0 -> 9.9 / 11.8 us, at N = 8 without
    // statistics 13.7 -> 13.5 us, in nb_pr_kernel 2^20 x 8 at N = 2 without statistics 62.6 -> 62.2 us.
    if constexpr (shares) {
        first_split = is < M && (unsigned)is + (unsigned)rowptr[is] < d0;
        ends = ChunkEnds(plan.split, rowptr, M, plan.wave, d0, is, ie1, js, d1 - (unsigned)ie1);
        if (ends.starts_tail() && uniform(mine_to_clear(found, sharing.call) ? 1 : 0) != 0 && my_column >= 0)         // as lane 0 found it
            clear_row<DeviceWords, 1, AXPBY>(y_of(ie1) + my_column, sc.beta);
        stores_done();
        if (lane == 0) publish_start<DeviceWords>(words + plan.wave, sharing.call, found);
    }

    // The first 64 row results of a tile are stored one tile later, after the next tile's loads have been issued:
    // the memory pipeline retires loads and stores in issue order, so a store in front of the gathers would put
    // its own round trip into their wait.
    float pending_val[V];
    unsigned pending_off = kOutOfRange;
    unsigned long long pending_first = 0ull;             // first element of the rows the pending store addresses
#pragma unroll
    for (int i = 0; i < V; ++i) pending_val[i] = 0.0f;
    auto rows_descriptor = [&](unsigned long long first_elem) {
        const unsigned long long left = first_elem < y_elems ? (y_elems - first_elem) * 4ull : 0ull;
        return __builtin_amdgcn_make_buffer_rsrc((void*)(Y + first_elem), 0, left > 0xffffffffull ? 0xffffffffu : (unsigned)left,
                                                 kBufferFlags);
    };
    auto store_pending = [&]() {
        buffer_store_vec<V>(rows_descriptor(pending_first), pending_off, pending_val, second);
        pending_off = kOutOfRange;
    };

    // one tile: consumes (c, a, w_end), leaves the next tile's loads in flight in (c2, a2, w_end2)
    auto do_tile = [&](int (&c)[E], float (&a)[E], unsigned w_end, int (&c2)[E], float (&a2)[E], unsigned& w_end2) {
        if constexpr (V >= 2) __builtin_amdgcn_s_setprio(3);
        const unsigned de = (d1 - ds > (unsigned)W) ? ds + W : d1;

        // ---- row ends of this tile -> LDS marks
        wave_lds_sync();                                   // the previous tile's readers are done
#pragma unroll
        for (int k = 0; k < KQ; ++k)
            *reinterpret_cast<uint4*>(bnd + E * lane + 4 * k) = make_uint4(kNoRow, kNoRow, kNoRow, kNoRow);
        if (lane == 0) bnd[W] = kNoRow;
        wave_lds_sync();
        int ie = is;
        // marks the rows of one batch of 64 candidates that end in the tile; returns how many did
        auto mark_row_ends = [&](int m, unsigned end) {
            const long long r = (long long)is + m * kWave + lane;
            const bool ends = r < M && (unsigned)r + end < de;     // the row's end marker is inside the tile
            if (ends) {
                const unsigned q = end - js;               // it ends after entry q-1 of the tile
                atomicMin(bnd + (q ? q - 1 : (unsigned)W), (unsigned)(r - is));
            }
            return (int)__popcll(__ballot(ends));
        };
        int cnt = mark_row_ends(0, w_end);                 // the first 64 candidates were loaded a tile ago
        ie += cnt;
        if (cnt == kWave) {
            // a tile crowded with row ends (at most W of them): fetch all remaining candidates at once
            unsigned ms[E - 1], me[E - 1];
#pragma unroll
            for (int m = 1; m < E; ++m) load_row_bounds(is + m * kWave, true, ms[m - 1], me[m - 1]);
#pragma unroll
            for (int m = 1; m < E; ++m) {
                if (cnt == kWave) { cnt = mark_row_ends(m, me[m - 1]); ie += cnt; }
            }
        }
        const unsigned je = de - (unsigned)ie;             // entries [js, je) belong to the tile
        const int nE = (int)(je - js);
        const int nrows = ie - is;                         // rows [is, ie) end in the tile
        wave_lds_sync();

        // ---- gather for this tile, then the next tile's loads (they stay in flight during the reduction)
        float x[E][V];
        if (x_small) {
#pragma unroll
            for (int e = 0; e < E; ++e)
                buffer_load_vec<V>(rx, e * kWave + lane < nE ? (unsigned)c[e] * (unsigned)ldx * 4u : kOutOfRange, x[e], second);
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e) load_vec_dword_aligned<V>(X + (size_t)(e * kWave + lane < nE ? c[e] : 0) * ldx + n0, x[e], second);
        }
        {
            const bool more = d1 - ds > (unsigned)W;       // past the chunk's last tile the loads are switched off
            load_row_bounds(ie, more, w_unused, w_end2);
            load_entries(je, more, c2, a2);
        }
        store_pending();                                   // the previous tile's rows
        if constexpr (V >= 2) __builtin_amdgcn_s_setprio(0);

        // ---- products change hands through LDS: entry 64e+l -> lane (64e+l)/E
#pragma unroll
        for (int e = 0; e < E; ++e) {
            float p[V];
            const bool mine = e * kWave + lane < nE;
#pragma unroll
            for (int i = 0; i < V; ++i) p[i] = mine ? a[e] * x[e][i] : 0.0f;
            store_vec<V>(buf + (size_t)(e * kWave + lane) * V, p);
        }
        wave_lds_sync();
        const unsigned b_in = bnd[W];
        unsigned b[E];
#pragma unroll
        for (int k = 0; k < KQ; ++k) {
            const uint4 t = *reinterpret_cast<const uint4*>(bnd + E * lane + 4 * k);
            b[4 * k] = t.x; b[4 * k + 1] = t.y; b[4 * k + 2] = t.z; b[4 * k + 3] = t.w;
        }
        float pr[E][V];
#pragma unroll
        for (int e = 0; e < E; ++e) load_vec<V>(buf + (size_t)(E * lane + e) * V, pr[e]);
        wave_lds_sync();                                   // products are in registers: the buffer is free

        // ---- the tile's row results: cleared, so rows without entries come out as zeros
        for (int k = 0; k * kWave < nrows; ++k) {
            float zero[V];
#pragma unroll
            for (int i = 0; i < V; ++i) zero[i] = 0.0f;
            store_vec<V>(buf + (size_t)(k * kWave + lane) * V, zero);
        }
        wave_lds_sync();
        // rows that end before the tile's first entry take the sum carried in
        if (b_in != kNoRow) {
            if (lane == 0) store_vec<V>(buf + (size_t)b_in * V, carry);
#pragma unroll
            for (int i = 0; i < V; ++i) carry[i] = 0.0f;
        }

        // ---- in-lane reduction over my E consecutive entries
        float s[V], head[V];
        unsigned head_row = kNoRow;                        // kNoRow: no boundary inside this lane
#pragma unroll
        for (int i = 0; i < V; ++i) { s[i] = lane == 0 ? carry[i] : 0.0f; head[i] = 0.0f; }
#pragma unroll
        for (int e = 0; e < E; ++e) {
#pragma unroll
            for (int i = 0; i < V; ++i) s[i] += pr[e][i];
            if (b[e] != kNoRow) {
                if (head_row == kNoRow) {
                    head_row = b[e];
#pragma unroll
                    for (int i = 0; i < V; ++i) head[i] = s[i];
                } else {
                    store_vec<V>(buf + (size_t)b[e] * V, s);   // a row that begins and ends inside this lane
                }
#pragma unroll
                for (int i = 0; i < V; ++i) s[i] = 0.0f;
            }
        }

        // ---- the open row across lanes: segments start at lanes that hold a boundary
        const bool flagged = head_row != kNoRow;
        const int head_lane = (int)wave_max_scan(flagged ? (unsigned)lane : 0u);
        segmented_scan<V>(s, lane - head_lane, lane);      // s: sum of the open row up to and including my lane
        {
            float closing[V];
#pragma unroll
            for (int i = 0; i < V; ++i) closing[i] = dpp_or_zero<kDppWaveShr1, 0xf>(s[i]) + head[i];
            if (flagged) store_vec<V>(buf + (size_t)head_row * V, closing);
        }
#pragma unroll
        for (int i = 0; i < V; ++i) carry[i] = read_lane(s[i], kWave - 1);
        wave_lds_sync();

        // ---- write the rows [is, ie) out, lane l row is + l: the first 64 with one unconditional
        //      buffer store, further batches (tiles crowded with short rows) in a loop
        {
            const unsigned long long first_elem = (unsigned long long)is * (unsigned)ldy + (unsigned)n0;
            __amdgpu_buffer_rsrc_t yrows = rows_descriptor(first_elem);
            auto write_rows = [&](int k) {
                const int t = k * kWave + lane;                     // local row
                float val[V];
                load_vec<V>(buf + (size_t)t * V, val);
                const bool live = t < nrows;
                const bool shared = first_split && is + t == r_first;   // finished by an atomic add instead
                const unsigned off = (live && !shared) ? (unsigned)t * (unsigned)ldy * 4u : kOutOfRange;
                if (k == 0) {
                    pending_first = first_elem; pending_off = off;
#pragma unroll
                    for (int i = 0; i < V; ++i) pending_val[i] = val[i];
                    if constexpr (AXPBY) scale_into<V>(pending_val, yrows, off, sc, second);
                } else {
                    buffer_store_vec<V>(yrows, off, val, second);            // plain form only
                }
                if constexpr (AXPBY) {
#pragma unroll
                    for (int i = 0; i < V; ++i) val[i] *= sc.alpha;          // an added sum lands on beta * Y (prepare)
                }
                if (live && shared) {
                    if (!shares) add_to_row(y_of(is + t), val);
                    else store_vec<V>(first_sum, val);
                }
            };
            write_rows(0);
            if constexpr (AXPBY) {
                // the old values of F batches in flight together (a row end every other entry: five round trips fewer a tile).
                // The first batch's are waited for above: most tiles of long rows have no other, and holding them to the
                // next tile's store made every wait of that tile's loads one for them (Zipf rows of 48 at N = 2 49 -> 55 us)
                constexpr int F = V <= 2 ? 4 : 2;
                for (int k = 1; k * kWave < nrows; k += F) {
                    float val[F][V], old[F][V]; unsigned off[F];
#pragma unroll
                    for (int u = 0; u < F; ++u) {
                        const int t = (k + u) * kWave + lane;
                        off[u] = t < nrows ? (unsigned)t * (unsigned)ldy * 4u : kOutOfRange;
                        if (sc.beta != 0.0f) buffer_load_vec<V>(yrows, off[u], old[u], second);
                        load_vec<V>(buf + (size_t)(t < W ? t : 0) * V, val[u]);
                    }
#pragma unroll
                    for (int u = 0; u < F; ++u) {
#pragma unroll
                        for (int i = 0; i < V; ++i) val[u][i] = sc.beta != 0.0f ? fmaf(sc.alpha, val[u][i], sc.beta * old[u][i]) : sc.alpha * val[u][i];
                        buffer_store_vec<V>(yrows, off[u], val[u], second);
                    }
                }
            } else {
                for (int k = 1; k * kWave < nrows; ++k) write_rows(k);
            }
        }

        is = ie;
        js = je;
        ds += W;
    };
    while (ds < d1) {
        do_tile(cA, aA, wA, cB, aB, wB);
        if (ds >= d1) break;
        do_tile(cB, aB, wB, cA, aA, wA);
    }

    RowWord seen_head = 0, seen_tail = 0;                  // both on their way together
    if (shares && lane == 0) {
        seen_head = DeviceWords::load(words + ends.head);
        seen_tail = DeviceWords::load(words + ends.tail);
    }
    store_pending();                                       // the last tile's rows
    // the row still open at the end of my chunk is finished by another wave
    if (shares) {
        if (ends.shares_head()) {
            wave_lds_sync();
            give_part<AXPBY>(words + ends.head, sharing.call, seen_head, y_of(r_first), lane < V ? first_sum[lane] : 0.0f, my_column, sc.beta);
        }
        if (ends.whole_tail()) {
            if (lane == 0) {
                if constexpr (AXPBY) scale_into<V, true>(carry, y_of(is), sc, second);
                store_vec_dword_aligned<V>(y_of(is), carry, second);
            }
        } else if (ends.shares_tail()) {
            float part = carry[0];
#pragma unroll
            for (int i = 1; i < V; ++i) part = lane == i ? carry[i] : part;
            give_part<AXPBY>(words + ends.tail, sharing.call, seen_tail, y_of(is), AXPBY ? sc.alpha * part : part, my_column, sc.beta);
        }
        return;
    }
    bool any = false;
#pragma unroll
    for (int i = 0; i < V; ++i) any |= carry[i] != 0.0f;
    if constexpr (AXPBY) {
#pragma unroll
        for (int i = 0; i < V; ++i) carry[i] *= sc.alpha;
    }
    if (any && lane == 0 && is < M) add_to_row(y_of(is), carry);
}

// ===========================================================================
// nnz-balanced, parallel reduction with the entry stream decoupled from the rows
// ===========================================================================
//
// The kernel above cuts a chunk into tiles of W merge-path items, so where the entries of tile t + 1 begin is
// known only when the row ends of tile t have been counted: its gathers cannot be requested before the row
// logic of tile t is through, and a wave spends that logic with no gather in flight.  Here the chunk (still an
// equal share of merge-path items, found by two 64-way searches in lock-step) is walked in BLOCKS of W consecutive
// ENTRIES counted from the chunk's first entry, so every block's address is known from the start:
//   * everything a block needs from memory is requested one block ahead: while the rows of block k are finished,
//     the gathers of block k + 1 and the entries of block k + 2 are in flight (the entries land in registers of
//     their own and are moved when they have arrived, so the loop needs no unrolling);
//   * the products of a block change hands through LDS as before (lane l ends up with E consecutive products)
//     and stay in registers while the rows that end inside the block are finished in STEPS: a step takes up to W
//     row ends (the LDS marks and the staged row results are sized for that) and the entries up to the end of the
//     last of them, or up to the block's end when fewer than W rows end in the block - the usual case, one step
//     per block.  A stretch of empty rows simply takes more steps; entries outside the step's range are masked;
//   * per step everything else is the scheme of the kernel above: row-end marks in LDS, in-lane sums of E
//     consecutive products, one segmented DPP scan over the lanes' open-row partials (Section 2.1.1), results
//     staged by row and stored 64 rows at a time, the open row's sum carried in a register.
// The row-bound window of the next step is requested before the next entries, so waiting for it does not wait
// for them (loads return in issue order).

// The hottest runs of a packed X of V columns (found when a matrix is taken over, hot_columns()): as many runs of 2^shift rows
// of X as kHotFloats hold.  `table`: kHotWords words (bitmap of 32 runs, hot runs before them) and the hot runs' numbers,
// ascending, kNoRow behind the last one; one such table for every V.
constexpr int kHotThreads = 512, kHotWords = 1024, kHotWidths = 4, kHotShiftMin = 5, kHotShiftMax = 7;
constexpr int kHotTableInts = 3 * kHotWords;
// what the products, marks and bitmap of eight waves leave of 160 KB
constexpr int hot_floats(int v) { return v == 1 ? 31 * 1024 : v == 2 ? 28 * 1024 : v == 3 ? 24 * 1024 : 20 * 1024; }
__host__ __device__ constexpr int hot_room(int v, int shift) { return hot_floats(v) / (v << shift); }
// runs that the L1 (32 KB, half of it left by everything else that passes through) holds without a table
__host__ __device__ constexpr int hot_cached(int v, int shift) { return (128 << 5) / (v << shift); }
struct HotColumns { const unsigned* table; int shift; };

// SERIAL_SCAN (a comparison kernel for Section 2.1.1, not used by the library's own choices): the lanes' open-row
// partial sums meet through a serial segmented prefix sum - they are put into LDS and one lane adds them up in
// lane order, starting afresh at every lane that holds a row boundary - instead of the DPP network.  Everything
// else, the balanced split included, is the same, so the difference in time is the vectorized reduction's.
//
// HOT (packed X, one to four columns): the runs of X that most entries name are read from LDS.  A gather of scattered columns fetches a
// 128-byte line from the L2 for four to sixteen bytes of it, and the rate of these lines is what bounds the product (R-MAT 2^20 x 16: 14
// million of them, 75 us for nothing but the gather).  Where few lines hold many of the entries' columns - the columns of a
// power-law graph: 55 % of that one's are on 992 of its 32768 lines - every CU copies these lines when it starts, and a bitmap of
// the lines with a running count per word says for a column whether it is among them and where.  One workgroup of eight
// waves per CU, so that its LDS holds one table; the lanes that found their column there switch their gather off.
// R-MAT 2^20 x 16, N = 1 / 2 / 4, whole calls: 92.6 / 103.6 / 113.7 -> 68.7 / 87.1 / 102.2 us (64.4 / 81.3 / 97.7 us where the waves see
// to the rows that they share themselves, SHARES); 4 / 6 / 12 / 16 waves instead of
// eight, with tables as large as they leave room for: 88.6 / 73.6 / 75.0 / 77.4 us at N = 1.  Bound by the lines that are left, 8.7
// million of 14.1 by the L2s' counters, streams included: streams and look-ups alone take 24 us, with the gathers 54 us; which lanes of a gather are
// switched off, and by offset or by execution mask, makes no difference, nor would packing the others into fewer instructions.
template <int V, int KQ, bool SNAP, bool AXPBY, bool SHARES = false, bool SERIAL_SCAN = false, bool HOT = false>
__global__ __launch_bounds__(HOT ? kHotThreads : kBlock) void nb_pr_kernel(int M, long long K, int N, int ldx, int ldy,
                                                        const int* __restrict__ rowptr,
                                                        const int* __restrict__ colidx,
                                                        const float* __restrict__ vals,
                                                        const float* __restrict__ X, float* __restrict__ Y,
                                                        Scaling sc, RowSharing sharing, HotColumns hot = HotColumns{nullptr, 0}) {
    constexpr int E = 4 * KQ;
    constexpr int W = kWave * E;
    constexpr int kWaves = HOT ? kHotThreads / kWave : kWavesPerBlock;
    __shared__ __align__(16) unsigned short s_bnd[kWaves][W];         // which row (of the step) ends with an entry of the block
    __shared__ __align__(16) float s_buf[kWaves][W * V];              // products, then a step's row results
    constexpr bool kFirstInLds = SHARES && !HOT;
    __shared__ __align__(16) float s_first[kFirstInLds ? kWaves : 1][V];        // the sum of the first row to end in the chunk
    __shared__ __align__(16) float s_scan[SERIAL_SCAN ? kWaves : 1][SERIAL_SCAN ? kWave * (V + 1) : 1];   // serial scan only
    __shared__ __align__(16) float s_hot[HOT ? hot_floats(V) : 1];    // the hot runs of X
    __shared__ __align__(16) uint2 s_word[HOT ? kHotWords : 1];       // 32 runs: which are hot, how many hot ones lie before
    const int lane = lane_id();
    const int wib = wave_in_block();
    unsigned short* bnd = s_bnd[wib];
    float* buf = s_buf[wib];
    const int n0 = blockIdx.y * V;

    const int probe = first_probe(rowptr, M, lane);
    const unsigned nnz = (unsigned)rowptr[M];
    const ChunkPlan plan(nnz, nnz + (unsigned)M, gridDim.x * kWaves, xcd_contiguous(blockIdx.x, gridDim.x) * kWaves + wib,
                         6);                              // quanta of one wave's width
    const unsigned long long y_elems = dense_bytes(M, ldy, N) / 4ull;
    // V = 8: the lane's second four columns start here (N = 5, 6, 7: at N - 4, overlapping the first four)
    const int second = (V == 8 && N - n0 < 8) ? N - n0 - 4 : 4;

    auto add_to_row = [&](float* y, const float (&v)[V]) {
        if constexpr (V == 8) atomic_add_halves(y, v, second); else atomic_add_vec<V>(y, v);
    };
    auto y_of = [&](int row) { return Y + (size_t)row * ldy + n0; };
    // Rows shared with other waves, where no launch has cleared them.  The sum of the first row to end in the chunk is kept until the end: in
    // the loop, the wait for its word held up the next entries and gathers in every turn.
    RowWord* const words = sharing.words + (size_t)blockIdx.y * plan.split.parts;
    constexpr bool shares = SHARES;
    // HOT: between a claim and its publication lies the workgroup's barrier, up to which no wave waits for another workgroup's.
    static_assert(!SHARES || (!SNAP && !SERIAL_SCAN), "no shared rows, or a prepare launch for them");
    float* const first_sum = s_first[kFirstInLds ? wib : 0];
    float first_held[SHARES && HOT ? V : 1];              // HOT: the same in lane 0, as all LDS is the hot runs'
#pragma unroll
    for (float& f : first_held) f = 0.0f;
    const int my_column = shared_column<V>(lane, second);

    unsigned d0, d1;
    const bool any_items = plan.range(d0, d1);
    // The hot runs, 16 bytes a load, and their bitmap: the bitmap and the runs' numbers are on their way while the chunk's bounds are
    // searched, the runs themselves behind the chunk's first entries (loads return in order: in front of the search they
    // held up its rounds, first gathers 9.8 us after the start; R-MAT 2^20 x 16 / 2^19 x 16 at N = 1 70.1 / 39.0 -> 68.7 / 37.9 us).
    constexpr int kPieces = HOT ? (hot_floats(V) / 4 + kHotThreads - 1) / kHotThreads : 1;
    constexpr int kWordPieces = HOT ? (kHotWords + kHotThreads - 1) / kHotThreads : 1;
    float piece[kPieces][4];
    uint2 word[kWordPieces];
    unsigned run[kPieces];
    // piece i: 16 bytes of hot run (i / pieces of a run)
    const auto run_of = [&](unsigned i) { return (i >> (hot.shift - 2)) / (unsigned)V; };
    const unsigned pieces = HOT ? (unsigned)(hot_room(V, hot.shift) * V) << (hot.shift - 2) : 0u;
    if constexpr (HOT) {
#pragma unroll
        for (int k = 0; k < kWordPieces; ++k) {
            const unsigned i = (unsigned)k * kHotThreads + threadIdx.x;
            word[k] = reinterpret_cast<const uint2*>(hot.table)[i < (unsigned)kHotWords ? i : 0u];
        }
#pragma unroll
        for (int k = 0; k < kPieces; ++k) {
            const unsigned i = (unsigned)k * kHotThreads + threadIdx.x;
            run[k] = hot.table[2 * kHotWords + run_of(i < pieces ? i : 0u)];
        }
    }
    const auto load_hot = [&] {
        const __amdgpu_buffer_rsrc_t rh = make_buffer(X, dense_bytes(K, V, V));
#pragma unroll
        for (int k = 0; k < kPieces; ++k) {
            const unsigned i = (unsigned)k * kHotThreads + threadIdx.x;
            const unsigned inside = i - ((run_of(i) * (unsigned)V) << (hot.shift - 2));
            const bool none = i >= pieces || run[k] == kNoRow;
            buffer_load_vec<4>(rh, none ? kOutOfRange : ((run[k] * (unsigned)V) << (hot.shift + 2)) + inside * 16u, piece[k]);
        }
    };
    // the only step that the workgroup's waves take together
    const auto fill_hot = [&] {
#pragma unroll
        for (int k = 0; k < kWordPieces; ++k) {
            const int i = k * kHotThreads + (int)threadIdx.x;
            if (i < kHotWords) s_word[i] = word[k];
        }
#pragma unroll
        for (int k = 0; k < kPieces; ++k) {
            const int i = k * kHotThreads + (int)threadIdx.x;
            if (i < hot_floats(V) / 4) store_vec<4>(s_hot + 4 * i, piece[k]);
        }
        __syncthreads();
    };

    // my chunk: rows [is, ie1) end in it, entries [js0, je1) lie in it
    int is = 0, ie1 = 0;
    bool idle = !any_items || nnz == 0;                  // HOT: such a wave has an empty chunk and goes along up to the barrier
    RowWord found = 0;
    if (shares && !idle && lane == 0) found = claim_row<DeviceWords>(words + plan.wave, sharing.call);
    if (!idle) wave_merge_rows_before2(rowptr, M, d0, d1, lane, probe, is, ie1);
    // nothing stored: every item is a row end; my rows are [d0, d1)
    const auto rows_without_entries = [&] {
        if (!any_items) return;
        for (unsigned r = d0 + lane; r < d1; r += kWave) {
            float* y = Y + (size_t)r * ldy + n0;
            float out[V];
#pragma unroll
            for (int i = 0; i < V; ++i) out[i] = 0.0f;
            if constexpr (AXPBY) scale_into<V, true>(out, y, sc, second);
            store_vec_dword_aligned<V>(y, out, second);
        }
    };
    if constexpr (!HOT) {
        if (idle) {
            rows_without_entries();
            return;
        }
    }
    unsigned js0 = d0 - (unsigned)is, je1 = d1 - (unsigned)ie1;
    if (HOT && idle) js0 = je1 = 0u;
    if constexpr (SNAP) {
        if (!idle) snap_to_rows(rowptr, M, d0, d1, is, ie1, js0, je1);
        idle |= is == ie1;
        if constexpr (!HOT) {
            if (idle) return;
        }
    }
    unsigned js = js0;
    // the first row to end in my chunk started before it?  then its sum is shared with another wave
    const int r_first = is;
    const bool first_split = !SNAP && is < M && (unsigned)is + (unsigned)rowptr[is] < d0;
    std::conditional_t<!HOT && V <= 2, HeldEnds, ChunkEnds> ends;

    // entries of block k of my chunk (lane l: entries 64 e + l of the block); nothing past the chunk's last entry
    // One descriptor pair for the whole chunk (a wave's share of a matrix the library takes stays far below the
    // 4 GB a descriptor spans); a block is a byte offset into it, kept in a VGPR and advanced by 4 W per block.
    const unsigned long long chunk_bytes = ((unsigned long long)je1 - js0) * 4ull;
    const __amdgpu_buffer_rsrc_t rc = make_buffer(colidx + js0, chunk_bytes);
    const __amdgpu_buffer_rsrc_t ra = make_buffer(vals + js0, chunk_bytes);
    auto load_entries = [&](unsigned k, int (&c)[E], float (&a)[E]) {
        // past the chunk's last block every offset is out of range: nothing is loaded (k * W * 4 cannot wrap: k <= nb + 1)
        const unsigned base = (unsigned long long)k * W * 4ull < chunk_bytes ? k * (unsigned)(W * 4) + (unsigned)lane * 4u : kOutOfRange;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const unsigned off = base == kOutOfRange ? kOutOfRange : base + (unsigned)(e * kWave) * 4u;
            c[e] = (int)__builtin_amdgcn_raw_buffer_load_b32(rc, off, 0, 2);
            a[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(ra, off, 0, 2));
        }
    };
    // the dense operand: byte offsets of X rows fit 32 bits unless X is 4 GB or more
    const unsigned long long x_bytes = dense_bytes(K, ldx, N);
    const bool x_small = x_bytes <= 0xffffffffull;
    const __amdgpu_buffer_rsrc_t rx = make_buffer(X + n0, x_small ? x_bytes - (unsigned)n0 * 4ull : 0ull);
    // one vector gather per entry of block k, from the columns that load_entries(k) brought
    // Entries past the chunk's end were loaded as column 0, value 0: their gathers read row 0 of X (in range: the
    // matrix has entries, so K >= 1) and their products are masked, so the gathers need no mask of their own.
    // Row offsets: a shift when the row pitch is a power of two (packed X at N = 1, 2: the 32-bit multiply runs at
    // a quarter of the rate of other vector instructions), checked once.
    const unsigned pitch = (unsigned)ldx * 4u;
    const int pitch_shift = (pitch & (pitch - 1u)) == 0u ? __builtin_ctz(pitch) : -1;
    float in_lds[HOT ? E : 1][V];                         // the values found among the hot runs, 0 for the others
    auto gather = [&](unsigned k, const int (&c)[E], float (&x)[E][V]) {
        if ((unsigned long long)k * W * 4ull >= chunk_bytes && chunk_bytes != 0ull) {
            // no such block: nothing to request (the loop's last iteration)
#pragma unroll
            for (int e = 0; e < E; ++e) {
#pragma unroll
                for (int i = 0; i < V; ++i) x[e][i] = 0.0f;
                if constexpr (HOT)
#pragma unroll
                    for (int i = 0; i < V; ++i) in_lds[e][i] = 0.0f;
            }
        } else if constexpr (HOT) {
            uint2 w[E];
#pragma unroll
            for (int e = 0; e < E; ++e) w[e] = s_word[(unsigned)c[e] >> (hot.shift + 5)];
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const unsigned bit = ((unsigned)c[e] >> hot.shift) & 31u;
                const bool found = ((w[e].x >> bit) & 1u) != 0u;
                const unsigned before = w[e].y + (unsigned)__popc(w[e].x & ((1u << bit) - 1u));
                const unsigned at = found ? (before << hot.shift) + ((unsigned)c[e] & ((1u << hot.shift) - 1u)) : 0u;
                load_vec<V>(s_hot + at * (unsigned)V, in_lds[e]);
#pragma unroll
                for (int i = 0; i < V; ++i) in_lds[e][i] = found ? in_lds[e][i] : 0.0f;
                buffer_load_vec<V>(rx, found ? kOutOfRange : (unsigned)c[e] * (unsigned)(4 * V), x[e]);
            }
        } else if (x_small) {
            if (pitch_shift >= 0) {
#pragma unroll
                for (int e = 0; e < E; ++e) buffer_load_vec<V>(rx, (unsigned)c[e] << pitch_shift, x[e], second);
            } else {
#pragma unroll
                for (int e = 0; e < E; ++e) buffer_load_vec<V>(rx, (unsigned)c[e] * pitch, x[e], second);
            }
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e)
                load_vec_dword_aligned<V>(X + (size_t)c[e] * ldx + n0, x[e], second);
        }
    };
    // end offset of row `first + lane` (rows past the last one read as 0)
    auto load_row_ends = [&](int first, bool on, unsigned& end) {
        const unsigned long long bytes = (on && first < M) ? (unsigned long long)(M + 1 - first) * 4ull : 0ull;
        const __amdgpu_buffer_rsrc_t rr = make_buffer(rowptr + (bytes ? first : 0), bytes);
        end = __builtin_amdgcn_raw_buffer_load_b32(rr, (unsigned)(lane + 1) * 4u, 0, 0);
    };

    float carry[V];      // running sum of the row that is open at the step boundary (wave-uniform)
#pragma unroll
    for (int i = 0; i < V; ++i) carry[i] = 0.0f;

    // The first 64 row results of a step are stored one step later, behind the loads issued meanwhile (the memory
    // pipeline retires loads and stores in issue order: a store in front of the gathers adds its round trip to their wait).
    float pending_val[V];
    unsigned pending_off = kOutOfRange;
    unsigned long long pending_first = 0ull;             // first element of the rows the pending store addresses
#pragma unroll
    for (int i = 0; i < V; ++i) pending_val[i] = 0.0f;
    auto rows_descriptor = [&](unsigned long long first_elem) {
        const unsigned long long left = first_elem < y_elems ? (y_elems - first_elem) * 4ull : 0ull;
        return __builtin_amdgcn_make_buffer_rsrc((void*)(Y + first_elem), 0, left > 0xffffffffull ? 0xffffffffu : (unsigned)left,
                                                 kBufferFlags);
    };
    auto store_pending = [&]() {
        buffer_store_vec<V>(rows_descriptor(pending_first), pending_off, pending_val, second);
        pending_off = kOutOfRange;
    };

    int c[E]; float a[E], x[E][V];                        // the block whose gathers are in flight
    int lc[E]; float la[E];                               // landing registers of the next block's entries
    unsigned w_end;                                       // end offsets of rows is .. is + 63 (lane l: row is + l)
    // the zeros; with hot runs behind the entries, as they are waited for together with the runs
    const auto start_shared_rows = [&] {
        if constexpr (SHARES) {
            if (idle) return;
            ends = ChunkEnds(plan.split, rowptr, M, plan.wave, d0, is, ie1, js0, je1);
            if (ends.starts_tail() && uniform(mine_to_clear(found, sharing.call) ? 1 : 0) != 0 && my_column >= 0)     // as lane 0 found it
                clear_row<DeviceWords, 1, AXPBY>(y_of(ie1) + my_column, sc.beta);
        }
    };
    load_entries(0, c, a);
    load_row_ends(is, is < ie1, w_end);
    start_shared_rows();
    if constexpr (HOT) load_hot();
    load_entries(1, lc, la);
    if constexpr (HOT) {
        fill_hot();
        if (idle) {
            if (nnz == 0) rows_without_entries();
            return;
        }
    }
    if (shares) {                                         // the zeros have been under way as long as the entries
        stores_done();
        if (lane == 0) publish_start<DeviceWords>(words + plan.wave, sharing.call, found);
    }
    gather(0, c, x);

    // state of the step in flight between its two halves
    int ie = is, nrows = 0;
    unsigned je = js, blk_start = js0, blk_end = js0;
    bool capped = false, closes_carry = false;

    // first half of a step: which rows end in it, their marks, the next step's row window
    auto step_rows = [&]() {
        wave_lds_sync();                                   // the previous step's readers are done
#pragma unroll
        for (int k = 0; k < KQ; k += 2) {
            if constexpr (KQ % 2 == 0) *reinterpret_cast<uint4*>(bnd + E * lane + 4 * k) = make_uint4(kNoRow, kNoRow, kNoRow, kNoRow);
            else *reinterpret_cast<uint2*>(bnd + E * lane + 4 * k) = make_uint2(kNoRow, kNoRow);
        }
        wave_lds_sync();
        ie = is;
        // marks the rows of one batch of 64 candidates that end in this block (and in my chunk); returns how many did.
        // `before`: where the row in front of the batch ended.  A row without entries leaves no mark: two rows never end
        // with the same entry.
        auto mark_row_ends = [&](int m, unsigned end, unsigned before) {
            const long long r = (long long)is + m * kWave + lane;
            const unsigned start = (unsigned)__builtin_amdgcn_update_dpp((int)before, (int)end, kDppWaveShr1, 0xf, 0xf, false);
            const bool ends = r < ie1 && end <= blk_end;
            if (ends && end > start) bnd[end - blk_start - 1u] = (unsigned short)(m * kWave + lane);      // it ends after that entry
            return (int)__popcll(__ballot(ends));
        };
        int cnt = mark_row_ends(0, w_end, js);             // the first 64 candidates were loaded a step ago
        closes_carry = cnt != 0 && (unsigned)uniform((int)w_end) == js;      // row `is` ends before the step's first entry
        ie += cnt;
        unsigned last_end = 0;
        if (cnt == kWave) {
            // crowded with row ends: fetch all remaining candidates of the step at once
            unsigned me[E - 1];
#pragma unroll
            for (int m = 1; m < E; ++m) load_row_ends(is + m * kWave, true, me[m - 1]);
#pragma unroll
            for (int m = 1; m < E; ++m) {
                if (cnt == kWave) {
                    cnt = mark_row_ends(m, me[m - 1], (unsigned)read_lane((int)(m == 1 ? w_end : me[m > 1 ? m - 2 : 0]), kWave - 1));
                    ie += cnt;
                }
            }
            last_end = (unsigned)read_lane((int)me[E - 2], kWave - 1);      // end of row is + W - 1
        }
        nrows = ie - is;
        capped = nrows == W;                               // more rows may end in this block: another step
        je = capped ? last_end : blk_end;                  // capped: up to the end of the last row taken
        load_row_ends(ie, ie < ie1, w_end);                // candidates of the next step
    };

    // second half: reduce the step's entries, finish its rows
    auto step_sums = [&](float (&pr)[E][V]) {
        store_pending();                                   // the previous step's rows
        wave_lds_sync();                                   // marks are in place
        unsigned b[E];                                     // 0xffff: no row ends with this entry
#pragma unroll
        for (int e = 0; e < E; e += 2) {
            const unsigned two = *reinterpret_cast<const unsigned*>(bnd + E * lane + e);
            b[e] = two & 0xffffu; b[e + 1] = two >> 16;
        }
        // ---- the step's row results: cleared, so rows without entries come out as zeros
        for (int k = 0; k * kWave < nrows; ++k) {
            float zero[V];
#pragma unroll
            for (int i = 0; i < V; ++i) zero[i] = 0.0f;
            store_vec<V>(buf + (size_t)(k * kWave + lane) * V, zero);
        }
        wave_lds_sync();
        // a row that ends before the step's first entry takes the sum carried in
        if (closes_carry) {
            if (lane == 0) store_vec<V>(buf, carry);
#pragma unroll
            for (int i = 0; i < V; ++i) carry[i] = 0.0f;
        }

        // ---- in-lane reduction over my E consecutive entries.  Those of earlier steps have been set to 0; those behind a
        //      capped step's last row end only reach the carry, which is dropped then
        constexpr unsigned kNone = 0xffffu;
        float s[V], head[V];
        unsigned head_row = kNone;                         // kNone: no boundary inside this lane
#pragma unroll
        for (int i = 0; i < V; ++i) { s[i] = lane == 0 ? carry[i] : 0.0f; head[i] = 0.0f; }
#pragma unroll
        for (int e = 0; e < E; ++e) {
#pragma unroll
            for (int i = 0; i < V; ++i) s[i] += pr[e][i];
            if (b[e] != kNone) {
                if (head_row == kNone) {
                    head_row = b[e];
#pragma unroll
                    for (int i = 0; i < V; ++i) head[i] = s[i];
                } else {
                    store_vec<V>(buf + (size_t)b[e] * V, s);   // a row that begins and ends inside this lane
                }
#pragma unroll
                for (int i = 0; i < V; ++i) s[i] = 0.0f;
            }
        }

        // ---- the open row across lanes: segments start at lanes that hold a boundary
        const bool flagged = head_row != kNone;
        if constexpr (SERIAL_SCAN) {
            float* sc_val = s_scan[wib];                   // 64 x V partial sums, then 64 flags
            float* sc_flag = sc_val + kWave * V;
#pragma unroll
            for (int i = 0; i < V; ++i) sc_val[lane * V + i] = s[i];
            sc_flag[lane] = flagged ? 1.0f : 0.0f;
            wave_lds_sync();
            if (lane == 0) {
                float run[V];
#pragma unroll
                for (int i = 0; i < V; ++i) run[i] = 0.0f;
                for (int l = 0; l < kWave; ++l) {          // one lane, lane order: a boundary starts a new sum
                    const bool start = sc_flag[l] != 0.0f;
#pragma unroll
                    for (int i = 0; i < V; ++i) {
                        run[i] = (start ? 0.0f : run[i]) + sc_val[l * V + i];
                        sc_val[l * V + i] = run[i];
                    }
                }
            }
            wave_lds_sync();
#pragma unroll
            for (int i = 0; i < V; ++i) s[i] = sc_val[lane * V + i];
        } else {
            const int head_lane = (int)wave_max_scan(flagged ? (unsigned)lane : 0u);
            segmented_scan<V>(s, lane - head_lane, lane);  // s: sum of the open row up to and including my lane
        }
        {
            float closing[V];
#pragma unroll
            for (int i = 0; i < V; ++i) closing[i] = dpp_or_zero<kDppWaveShr1, 0xf>(s[i]) + head[i];
            if (flagged) store_vec<V>(buf + (size_t)head_row * V, closing);
        }
#pragma unroll
        for (int i = 0; i < V; ++i) carry[i] = read_lane(s[i], kWave - 1);
        if (capped) {                                      // the next step has the block's remaining entries
            const int taken = (int)(je - blk_start);
#pragma unroll
            for (int i = 0; i < V; ++i) {
                carry[i] = 0.0f;
#pragma unroll
                for (int e = 0; e < E; ++e) pr[e][i] = E * lane + e < taken ? 0.0f : pr[e][i];
            }
        }
        wave_lds_sync();

        // ---- write the rows [is, ie) out, lane l row is + l: the first 64 with one unconditional
        //      buffer store (issued a step later), further batches in a loop
        {
            const unsigned long long first_elem = (unsigned long long)is * (unsigned)ldy + (unsigned)n0;
            __amdgpu_buffer_rsrc_t yrows = rows_descriptor(first_elem);
            auto write_rows = [&](int k) {
                const int t = k * kWave + lane;                     // local row
                float val[V];
                load_vec<V>(buf + (size_t)t * V, val);
                const bool live = t < nrows;
                const bool shared = first_split && is + t == r_first;   // finished by an atomic add instead
                const unsigned off = (live && !shared) ? (unsigned)t * (unsigned)ldy * 4u : kOutOfRange;
                if (k == 0) {
                    pending_first = first_elem; pending_off = off;
#pragma unroll
                    for (int i = 0; i < V; ++i) pending_val[i] = val[i];
                    if constexpr (AXPBY) scale_into<V>(pending_val, yrows, off, sc, second);
                } else {
                    buffer_store_vec<V>(yrows, off, val, second);            // plain form only
                }
                if constexpr (AXPBY) {
#pragma unroll
                    for (int i = 0; i < V; ++i) val[i] *= sc.alpha;          // an added sum lands on beta * Y (prepare)
                }
                if (live && shared) {
                    if constexpr (!shares) {
                        add_to_row(y_of(is + t), val);
                    } else if constexpr (HOT) {                      // t = 0 of the first 64
#pragma unroll
                        for (int i = 0; i < V; ++i) first_held[i] = val[i];
                    } else {
                        store_vec<V>(first_sum, val);
                    }
                }
            };
            write_rows(0);
            if constexpr (AXPBY) {
                // the old values of F batches in flight together (a row end every other entry: five round trips fewer a tile).
                // The first batch's are waited for above: most tiles of long rows have no other, and holding them to the
                // next tile's store made every wait of that tile's loads one for them (Zipf rows of 48 at N = 2 49 -> 55 us)
                constexpr int F = V <= 2 ? 4 : 2;
                for (int k = 1; k * kWave < nrows; k += F) {
                    float val[F][V], old[F][V]; unsigned off[F];
#pragma unroll
                    for (int u = 0; u < F; ++u) {
                        const int t = (k + u) * kWave + lane;
                        off[u] = t < nrows ? (unsigned)t * (unsigned)ldy * 4u : kOutOfRange;
                        if (sc.beta != 0.0f) buffer_load_vec<V>(yrows, off[u], old[u], second);
                        load_vec<V>(buf + (size_t)(t < W ? t : 0) * V, val[u]);
                    }
#pragma unroll
                    for (int u = 0; u < F; ++u) {
#pragma unroll
                        for (int i = 0; i < V; ++i) val[u][i] = sc.beta != 0.0f ? fmaf(sc.alpha, val[u][i], sc.beta * old[u][i]) : sc.alpha * val[u][i];
                        buffer_store_vec<V>(yrows, off[u], val[u], second);
                    }
                }
            } else {
                for (int k = 1; k * kWave < nrows; ++k) write_rows(k);
            }
        }
        is = ie;
        js = je;
    };

    const unsigned nblocks = (je1 - js0 + (unsigned)W - 1) / (unsigned)W;
    const unsigned nb = nblocks ? nblocks : 1u;            // a chunk without entries still has its row ends to finish
    // Waves that lag behind go first, by quarters of the chunk, so that those of a SIMD end together: R-MAT 2^20 x 16 at
    // N = 2 / 4 86.7 / 102.4 -> 85.1 / 101.1 us, 300 001 lognormal rows of 30 at N = 1 56.0 -> 54.8 us.  In chunks of a few
    // blocks there is nothing to make up (R-MAT 2^18 x 16 at N = 2, four blocks, 32.4 -> 32.9 us).
    unsigned pace = 4u;
    for (unsigned k = 0; k < nb; ++k) {
        const unsigned behind = nb < 8u ? 0u : 3u - 4u * k / nb;
        if (behind != pace) { pace = behind; set_wave_priority(pace); }
        blk_start = js0 + k * (unsigned)W;                 // == js: the previous block was consumed to its end
        blk_end = (je1 - blk_start > (unsigned)W) ? blk_start + (unsigned)W : je1;
        // ---- products of block k change hands through LDS: entry 64e+l of the block -> lane (64e+l)/E
        const int nE = (int)(blk_end - blk_start);
        wave_lds_sync();                                   // the previous step's readers of the buffer are done
#pragma unroll
        for (int e = 0; e < E; ++e) {
            float p[V];
            const bool mine = e * kWave + lane < nE;
#pragma unroll
            for (int i = 0; i < V; ++i) {
                const float xi = HOT ? x[e][i] + in_lds[HOT ? e : 0][i] : x[e][i];          // one of the two is 0
                p[i] = mine ? a[e] * xi : 0.0f;
            }
            store_vec<V>(buf + (size_t)(e * kWave + lane) * V, p);
        }
        wave_lds_sync();
        float pr[E][V];
#pragma unroll
        for (int e = 0; e < E; ++e) load_vec<V>(buf + (size_t)(E * lane + e) * V, pr[e]);
        // ---- block k + 1's entries have landed: request its gathers and block k + 2's entries; both stay in
        //      flight while the rows of block k are finished
#pragma unroll
        for (int e = 0; e < E; ++e) { c[e] = lc[e]; a[e] = la[e]; }
        load_entries(k + 2, lc, la);
        gather(k + 1, c, x);
        do {                                               // one step, unless more than W rows end in this block
            step_rows();
            step_sums(pr);                                 // (its first LDS fence also frees the product buffer)
        } while (capped);
    }

    RowWord seen_head = 0, seen_tail = 0;                  // both on their way together
    if (shares && lane == 0) {
        seen_head = DeviceWords::load(words + ends.head);
        seen_tail = DeviceWords::load(words + ends.tail);
    }
    store_pending();                                       // the last step's rows
    // the row still open at the end of my chunk is finished by another wave
    if (shares) {
        if (ends.shares_head()) {
            wave_lds_sync();
            float part = 0.0f;
            if constexpr (HOT) {
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    const float of_first = read_lane(first_held[i], 0);
                    part = lane == i ? of_first : part;
                }
            } else if (lane < V) {
                part = first_sum[lane];
            }
            give_part<AXPBY>(words + ends.head, sharing.call, seen_head, y_of(r_first), part, my_column, sc.beta);
        }
        if (ends.whole_tail()) {
            if (lane == 0) {
                if constexpr (AXPBY) scale_into<V, true>(carry, y_of(is), sc, second);
                store_vec_dword_aligned<V>(y_of(is), carry, second);
            }
        } else if (ends.shares_tail()) {
            float part = carry[0];
#pragma unroll
            for (int i = 1; i < V; ++i) part = lane == i ? carry[i] : part;
            give_part<AXPBY>(words + ends.tail, sharing.call, seen_tail, y_of(is), AXPBY ? sc.alpha * part : part, my_column, sc.beta);
        }
        return;
    }
    bool any = false;
#pragma unroll
    for (int i = 0; i < V; ++i) any |= carry[i] != 0.0f;
    if constexpr (AXPBY) {
#pragma unroll
        for (int i = 0; i < V; ++i) carry[i] *= sc.alpha;
    }
    if (any && lane == 0 && is < M) add_to_row(y_of(is), carry);
}

// ===========================================================================
// nnz-balanced, sequential reduction with LDS-staged tiles (Sections 2.1.3, 1)
// ===========================================================================
//
// A wave stages a tile of W = 512 merge-path items in LDS: its entries
// (colidx, val) with coalesced loads (coalesced sparse-row caching) and the
// end offsets of the rows that end in it.  Its 64/G lane groups then each walk
// one run of U = W*G/64 consecutive items in order; lane gl of a group owns V
// dense columns, so per entry a group reads one contiguous piece of a row of
// X.  At a row end the accumulator is flushed.  A row whose items all lie in
// the run is stored directly (empty rows flush a zero accumulator, which is
// how they get their zeros).  A row that crosses run boundaries inside the
// tile is summed in LDS: every run adds its part to the slot named after the
// run the row started in, and after the walk one group writes the slot out -
// with a plain store if the row also ended inside the tile.  Only rows that
// cross the tile's own ends go to memory with atomic adds (prepare kernel:
// rows split by a tile boundary).
// blockIdx.y selects the block of G*V dense columns.
// Used at one to three columns (and with one column per lane at any width, the comparison without vector loads):
// from four columns on nb_sr_run_kernel takes over.

constexpr int kNbSrTile = 512;
constexpr int kNbSrLogTile = 9;

template <int V, bool XBUF, int DEPTH, bool AXPBY = false>
__global__ __launch_bounds__(kBlock) void nb_sr_kernel(int M, long long K, int N, int ldx, int ldy, const int* __restrict__ rowptr,
                                                        const int* __restrict__ colidx,
                                                        const float* __restrict__ vals,
                                                        const float* __restrict__ X, float* __restrict__ Y,
                                                        int logG, int cols_per_block, Scaling sc = Scaling{1.0f, 0.0f}) {
    constexpr int W = kNbSrTile;
    constexpr int kSlotFloats = 2 * kWave * V;          // (64/G + 1) slots of G*V floats each, G <= 64
    __shared__ __align__(16) int s_col[kWavesPerBlock][W];
    __shared__ __align__(16) float s_val[kWavesPerBlock][W];
    __shared__ __align__(16) unsigned short s_end[kWavesPerBlock][W + 8];   // end offsets (minus js) of the rows ending in the tile
    __shared__ __align__(16) float s_slot[kWavesPerBlock][kSlotFloats];     // slots are read 4 * V bytes at a time
    __shared__ int s_slot_row[kWavesPerBlock][kWave + 4];   // row of each slot (-1: unused)
    __shared__ int s_slot_end[kWavesPerBlock][kWave + 4];   // 1: the slot's row ended inside the tile
    const int lane = lane_id();
    const int wib = wave_in_block();
    int* cc = s_col[wib];
    float* cv = s_val[wib];
    unsigned short* ends = s_end[wib];
    float* slot_acc = s_slot[wib];
    int* slot_row = s_slot_row[wib];
    int* slot_end = s_slot_end[wib];

    const int G = 1 << logG;
    const int gl = lane & (G - 1);
    const int g = lane >> logG;
    const int groups = kWave >> logG;
    const int logU = kNbSrLogTile - 6 + logG;
    const unsigned U = 1u << logU;
    const LaneColumns mine = lane_columns<V, false>(blockIdx.y, cols_per_block, gl, N);
    const long long n = mine.first;
    const bool col_ok = mine.any;

    const int probe = first_probe(rowptr, M, lane);
    // chunks start at multiples of U: runs stay aligned
    const ChunkPlan plan = plan_chunks(rowptr, M, (unsigned)logU);
    const unsigned nnz = plan.nnz;
    const unsigned long long y_elems = dense_bytes(M, ldy, N) / 4ull;
    // XBUF: the dense operand is read through a descriptor (its byte offsets fit 32 bits)
    const unsigned long long x_bytes = dense_bytes(K, ldx, N);
    const __amdgpu_buffer_rsrc_t rx = make_buffer(X, XBUF ? x_bytes : 0ull);
    const unsigned n_bytes = (unsigned)n * 4u;

    unsigned d0, d1;
    if (!plan.range(d0, d1)) return;
    int is = wave_merge_rows_before(rowptr, M, d0, lane, probe);
    unsigned js = d0 - (unsigned)is;
    for (unsigned ds = d0; ds < d1; ds += W) {
        const unsigned de = (d1 - ds > (unsigned)W) ? ds + W : d1;

        wave_lds_sync();                        // previous tile's readers are done
        // entries: at most W, the exact count follows from the row ends
        {
            const unsigned long long bytes = (unsigned long long)(nnz - js) * 4ull;
            const __amdgpu_buffer_rsrc_t rc = make_buffer(colidx + js, bytes);
            const __amdgpu_buffer_rsrc_t ra = make_buffer(vals + js, bytes);
#pragma unroll
            for (int k = 0; k < W / kWave; ++k) {
                const int e = k * kWave + lane;
                cc[e] = buffer_stream_i32(rc, (unsigned)e * 4u);
                cv[e] = buffer_stream_f32(ra, (unsigned)e * 4u);
            }
        }
        // slots for the rows that cross run boundaries inside the tile
#pragma unroll
        for (int k = 0; k < kSlotFloats / kWave; ++k) slot_acc[k * kWave + lane] = 0.0f;
        slot_row[lane] = -1; slot_end[lane] = 0;
        if (lane == 0) { slot_row[kWave] = -1; slot_end[kWave] = 0; }
        // end offsets of rows is, is+1, ... while their end marker is inside the tile: 64 candidates first,
        // and if all of them end here (a tile crowded with short or empty rows) the other 448 in one go
        int ie = is;
        {
            const unsigned long long rbytes = is < M ? (unsigned long long)(M + 1 - is) * 4ull : 0ull;
            const __amdgpu_buffer_rsrc_t rr = make_buffer(rowptr + is, rbytes);     // rows past the last read as 0
            auto take = [&](int m, unsigned e) {
                const long long r = (long long)is + m * kWave + lane;
                const bool in = r < M && (unsigned)r + e < de;
                if (in) ends[m * kWave + lane] = (unsigned short)(e - js);
                return (int)__popcll(__ballot(in));
            };
            int cnt = take(0, (unsigned)__builtin_amdgcn_raw_buffer_load_b32(rr, (unsigned)(lane + 1) * 4u, 0, 0));
            ie += cnt;
            if (cnt == kWave) {
                unsigned e[W / kWave - 1];
#pragma unroll
                for (int m = 1; m < W / kWave; ++m)
                    e[m - 1] = (unsigned)__builtin_amdgcn_raw_buffer_load_b32(rr, (unsigned)(m * kWave + lane + 1) * 4u, 0, 0);
#pragma unroll
                for (int m = 1; m < W / kWave; ++m) {
                    if (cnt == kWave) { cnt = take(m, e[m - 1]); ie += cnt; }
                }
            }
        }
        const int nrows = ie - is;              // rows ending in this tile
        const unsigned rs_first = is < M ? (unsigned)rowptr[is] : nnz;   // start offset of row `is`
        wave_lds_sync();

        // rows [is, ie) end in this tile; their results leave through one descriptor based at row `is`
        const unsigned long long first_elem = (unsigned long long)is * (unsigned)ldy;
        const unsigned long long left = first_elem < y_elems ? (y_elems - first_elem) * 4ull : 0ull;
        const __amdgpu_buffer_rsrc_t yrows = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(Y + first_elem), 0, left > 0xffffffffull ? 0xffffffffu : (unsigned)left, kBufferFlags);

        // rows without entries get their zeros here, all groups together (group g: local rows g, g + groups, ...),
        // so that the walk below meets a store only where a row with entries ends.
        {
            float zero[V];
#pragma unroll
            for (int i = 0; i < V; ++i) zero[i] = 0.0f;
            for (int t0 = 0; t0 < nrows; t0 += 4 * groups) {      // wave-uniform; four independent stores per round
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int tz = t0 + q * groups + g;
                    bool empty = false;
                    if (tz < nrows) {
                        const int end = (int)ends[tz];
                        const int start = tz == 0 ? (int)(rs_first - js) : (int)ends[tz - 1];   // negative: began before the tile
                        empty = end == start;
                    }
                    const unsigned off = (empty && col_ok) ? (unsigned)tz * (unsigned)ldy * 4u + n_bytes : kOutOfRange;
                    if constexpr (AXPBY) {
                        float out[V];
#pragma unroll
                        for (int i = 0; i < V; ++i) out[i] = 0.0f;
                        scale_into<V>(out, yrows, off, sc);               // beta * Y
                        buffer_store_vec<V>(yrows, off, out);
                    } else {
                        buffer_store_vec<V>(yrows, off, zero);
                    }
                }
            }
        }

        // first local row in [lo, hi) whose end offset lies beyond `off` (end offsets never decrease); hi if none
        auto first_row_ending_after = [&](int lo, int hi, unsigned off) {
            if (lo >= hi || js + ends[lo] > off) return lo;          // the usual case: the next row has entries
            ++lo;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (js + ends[mid] <= off) lo = mid + 1; else hi = mid;
            }
            return lo;
        };

        // ---- my run: diagonals [dg, dh) = entries [j, j_end) and the end markers of rows [t, t_end)
        const unsigned dg = ds + ((unsigned)g << logU);
        const bool has_run = dg < de && col_ok;
        int t = 0, t_end = 0;
        unsigned j = 0, j_end = 0, next_end = kNoRow, cur_first = 0;
        if (has_run) {
            const unsigned dh = (de - dg > U) ? dg + U : de;
            // rows (local index t, row is+t) whose end marker lies before a diagonal d: is+t + ends[t] < d
            auto rows_before = [&](unsigned d) {
                int lo = 0, hi = nrows;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if ((unsigned)(is + mid) + js + ends[mid] < d) lo = mid + 1; else hi = mid;
                }
                return lo;
            };
            t = rows_before(dg);                             // first row (local) to end at or after dg
            t_end = rows_before(dh);                         // rows [t, t_end) end inside my run
            j = dg - (unsigned)(is + t);                     // first entry of my run
            j_end = dh - (unsigned)(is + t_end);
            // rows without entries at the head of the run are done already
            const unsigned start_off = t == 0 ? rs_first : js + ends[t - 1];   // where row t's entries begin
            t = first_row_ending_after(t, t_end, start_off);
            next_end = t < nrows ? js + ends[t] : kNoRow;    // end offset of the current row
            cur_first = (unsigned)(is + t) + start_off;      // first item of the current row
        }
        // lanes without a run keep j == j_end and t == t_end: they issue the same instructions, switched off

        float acc[V];
#pragma unroll
        for (int i = 0; i < V; ++i) acc[i] = 0.0f;

        // a partial sum of row is+t (it crosses my run's ends) goes to the slot of the run it started in
        auto to_slot = [&](bool ended) {
            const int s = cur_first < ds ? 0 : (int)((cur_first - ds) >> logU) + 1;
            float* dst = slot_acc + (size_t)(s * G + gl) * V;
#pragma unroll
            for (int i = 0; i < V; ++i) atomicAdd(dst + i, acc[i]);
            if (gl == 0) { slot_row[s] = is + t; if (ended) slot_end[s] = 1; }   // every writer of slot_row[s] writes the same row
        };
        // The current row ends here (closing: its end marker lies in my run).  A row that began inside my run is
        // stored, one that began earlier goes to its slot.  The store is issued by the whole wave whenever any
        // group closes a row - switched off where none does - so no memory operation sits in a divergent branch.
        auto close_row = [&](bool closing) {
            if (__ballot(closing) != 0ull) {                 // wave-uniform
                const bool direct = closing && cur_first >= dg;
                const unsigned off = direct ? (unsigned)t * (unsigned)ldy * 4u + n_bytes : kOutOfRange;
                if constexpr (AXPBY) {
                    float out[V];
#pragma unroll
                    for (int i = 0; i < V; ++i) out[i] = acc[i];
                    scale_into<V>(out, yrows, off, sc);
                    buffer_store_vec<V>(yrows, off, out);
                } else {
                    buffer_store_vec<V>(yrows, off, acc);
                }
                if (closing) {
                    if (!direct) to_slot(true);
#pragma unroll
                    for (int i = 0; i < V; ++i) acc[i] = 0.0f;
                    const unsigned off = next_end;           // the next row's entries begin where this one's end
                    t = first_row_ending_after(t + 1, t_end, off);   // rows without entries: zeros written above
                    cur_first = (unsigned)(is + t) + off;
                    next_end = t < nrows ? js + ends[t] : kNoRow;
                }
            }
        };
        // the dense-row load of entry p into register set u; switched off past the run's last entry
        float x[DEPTH][V]; float a[DEPTH];
        auto issue = [&](int u, unsigned p) {
            const bool ok = p < j_end;
            const int e = ok ? (int)(p - js) : 0;
            a[u] = ok ? cv[e] : 0.0f;
            const unsigned c = (unsigned)cc[e];
            if constexpr (XBUF) {
                buffer_load_vec<V>(rx, ok ? c * (unsigned)ldx * 4u + n_bytes : kOutOfRange, x[u]);
            } else {
                load_vec_dword_aligned<V>(X + (size_t)(ok ? c : 0u) * ldx + (col_ok ? n : 0), x[u]);
#pragma unroll
                for (int i = 0; i < V; ++i) x[u][i] = ok ? x[u][i] : 0.0f;
            }
        };
        // DEPTH loads stay in flight: entry p is consumed while entry p + DEPTH is requested
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) issue(u, j + u);
        for (unsigned p0 = j; __ballot(p0 < j_end) != 0ull; p0 += DEPTH) {     // the same trip count for every lane
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
                const unsigned p = p0 + u;
                close_row(p < j_end && next_end == p);       // the row before entry p is complete
#pragma unroll
                for (int i = 0; i < V; ++i) acc[i] = fmaf(a[u], x[u][i], acc[i]);   // a is 0 past the end
                issue(u, p + DEPTH);
            }
        }
        close_row(t < t_end);                                // the row whose end marker follows my last entry
        // what is left belongs to a row that goes on after my run (if the run held entries of it)
        if (has_run && (unsigned)(is + t) + j_end > cur_first) to_slot(false);
        wave_lds_sync();                                     // every run has added its parts

        // one group per slot writes the rows that crossed run boundaries: slot g+1 by group g, slot 0 by group 0 too
        if (col_ok) {
            for (int s = (g == 0 ? 0 : g + 1); s <= g + 1 && s <= groups; ++s) {
                const int row = slot_row[s];
                if (row >= 0) {
                    float val[V];
                    load_vec<V>(slot_acc + (size_t)(s * G + gl) * V, val);
                    float* y = Y + (size_t)row * ldy + n;
                    // started inside the tile (s > 0) and ended inside it: nobody else has a part of this row
                    const bool whole = s > 0 && slot_end[s];
                    if constexpr (AXPBY) {
                        if (whole) {
                            scale_into<V, true>(val, y, sc);
                        } else {
#pragma unroll
                            for (int i = 0; i < V; ++i) val[i] *= sc.alpha;          // lands on beta * Y (prepare)
                        }
                    }
                    if (whole) {
                        store_vec_dword_aligned<V>(y, val);
                    } else {
                        atomic_add_vec<V>(y, val);
                    }
                }
            }
        }

        js = de - (unsigned)ie;
        is = ie;
    }
}

// ===========================================================================
// nnz-balanced, sequential reduction on blocks of entries (four or more dense columns)
// ===========================================================================
//
// The wave's chunk (an equal share of merge-path items, as above) is walked in blocks of 512 consecutive entries:
//   1. the block's entries, loaded a block ahead, go to LDS as (byte offset of the row of X, value) pairs;
//   2. the rows that end in the block leave one bit each at their last entry and their numbers in a list; rows
//      without entries are zeroed on the way, all lane groups together;
//   3. the R = 64 / G lane groups (G lanes span the columns, four each) walk one run of U = 512 / R entries each, in
//      order, eight dense-row loads in flight.  What a step costs is one LDS read, one address addition, the load and
//      four multiply-adds: run bounds, row ends and row numbers are not looked at, because a batch's row-end bits of
//      all groups come as one scalar mask and only a step that has a bit there leaves this path.  At such a step the
//      groups concerned store their sum as the next row of the list and start afresh;
//   4. a row that crosses runs is what the first row end of a run finds unfinished: the runs' open sums meet in a
//      segmented scan over the R groups (the vectorized segment reduction of Section 2.1.1 with runs in place of
//      entries), the last one is carried to the next block.
// Bound by: what the L2s have to fetch of X (a probe that only gathers rows of X tops out at 7.5 TB/s of L2 misses),
// and for that the walk has to be short of vector instructions: a wave instruction occupies its SIMD for four cycles,
// and the walk with row state per lane group that this one replaces spent about 45 of them per step and waited for
// every single load.  Measured, that walk against this one, whole calls: R-MAT 2^20 x 16 at N = 8 / 16 / 32 / 128: 196 /
// 224 / 302 / 1024 us -> 137-142 / 174 / 237-269 / 985-1100 us (they differ between GPUs and processes); 20 001 uneven
// rows of 10 at N = 32: 25 -> 9 us; 65 536-vertex R-MAT at N = 41: 65 -> 31 us.
//
// SNAP (host: the longest row is short against a wave's share): a row belongs wholly to the chunk that holds its
// first item, so nothing is added to memory, the prepare launch falls away and the result is the same from run to
// run.  Otherwise rows that cross a chunk end are added with atomics to zeros (RowSharing) or to what the prepare launch left.
//
// When N is no multiple of four the last lane's window ends at N and overlaps its neighbour's: plain stores may repeat
// the shared columns (same bits); scaled stores, atomic adds and what they add to leave them to the neighbour, who may be another
// column block's (N = 16129: 63 blocks of 256 columns and one of a single column).
//
// pinned_blocks = nb (2 or 4; gridDim = (8 k, 1)): the workgroups of XCD x all take column block x % nb, so that an L2
// only ever sees one block's slice of X; the 8 / nb XCDs of a block share its chunk list, each a contiguous part.
// Otherwise blockIdx.y is the column block.
//
// QUEUED: equal shares do not end together.  What a row of X costs depends on how much of it the L2 holds, and the XCDs do not
// reach memory equally fast (R-MAT 2^20 x 16, us: N = 128 794 772 820 998 768 875 775 1002, column block 3 last; N = 32 184 to 226; Zipf
// rows of 16 at N = 64 138 to 146 on the even XCDs, 156 to 166 on the odd ones).  So a wave starts on a part of its share and takes the
// rest chunk by chunk from its XCD's queue, and some waves of an XCD that is done help the others (ChunkQueues).  A failed
// take is an add to a word that all waves of the XCD add to, 13 ns a time, which is why most waves stop at their first.
//
// Wave priorities (set_wave_priority): searches, staging, row marks and the sums across runs at the highest, so that a wave gets
// to its gathers; in the walk of a longer chunk the lower the further it has come, so that the waves of a SIMD end together.
// Without / walk at the lowest throughout / by thirds: R-MAT 2^17 x 16 at N = 9 / 16 / 40 / 64 / 100 30.2 / 27.1 / 44.1 / 48.5 / 82.2,
// 28.8 / 25.7 / 42.1 / 47.0 / 81.9, 27.9 / 25.2 / 40.2 / 48.0 / 80.9 us; 2^18 x 32 at N = 20 / 41 96 / 144, 95 / 143,
// 89.7 / 134.7 us.  Chunks of kPacedFrom entries or fewer have nothing to make up (2^13 x 16 at N = 100 20.0, 20.1, 20.4 us);
// without statistics on a 27-point stencil, 61^3 at N = 64, the walk's lines leave the L1 earlier (104.5, 105.6,
// 106.8 us).  Where a launch does not fill the SIMDs the priorities do not pay for themselves: without / with them R-MAT 2^12 x
// 4 at N = 120 15.1 / 15.6 us, 2^13 x 16 at N = 100 18.4 / 18.7 us, 20 001 lognormal rows of 10 at N = 32 8.8 / 9.05 us.
constexpr int kRunBlock = 512;       // entries per block
constexpr int kRunBatch = 8;          // dense-row loads a lane has in flight
constexpr unsigned kPacedFrom = 256;
// Equal shares differ by up to this many items: with small ones, 80 000 items over 1024 waves, half of the waves otherwise take twice what
// the rest does (64 / 32 / 16 items: R-MAT 2^13 x 10 at N = 54 11.1 / 10.2 / 10.2 us, 2^13 x 20 at N = 41 12.3 / 11.7 / 11.5 us, 2^14 x
// 20 at N = 64 17.4 / 16.8 / 16.5 us, lognormal 9000 x 20 at N = 96 16.8 / 17.1 / 17.3 us).
constexpr unsigned kRunQuantumLog2 = 5;

// the sum of the lanes' words under bitwise or, wave-uniform
__device__ __forceinline__ unsigned wave_or(unsigned v) {
    v |= dpp_or_zero_u<kDppRowShr1, 0xf>(v);
    v |= dpp_or_zero_u<kDppRowShr2, 0xf>(v);
    v |= dpp_or_zero_u<kDppRowShr4, 0xf>(v);
    v |= dpp_or_zero_u<kDppRowShr8, 0xf>(v);
    v |= dpp_or_zero_u<kDppRowBcast15, 0xa>(v);
    v |= dpp_or_zero_u<kDppRowBcast31, 0xc>(v);
    return (unsigned)read_lane((int)v, kWave - 1);
}

// entries per row below which neighbouring chunks go to different XCDs
__host__ __device__ constexpr int run_dealt_below(int log_lanes) { return log_lanes >= 5 ? 8 : 6; }

// Four workgroups a CU in all forms: without the bound the scaled ones of two and of four lanes take 130 and 132 vector registers, three waves a
// SIMD (three / four: lognormal 100 001 x 20 at N = 8 25.3 / 21.8 us, 2^16 x 16 at N = 16 24.6 / 23.4 us); the others fit anyway.
template <int LOGG, bool XBUF, bool AXPBY, bool QUEUED = false, bool SHARES = false>
__global__ __launch_bounds__(kBlock, 4) void nb_sr_run_kernel(int M, long long K, int N, int ldx, int ldy,
                                                           const int* __restrict__ rowptr, const int* __restrict__ colidx,
                                                           const float* __restrict__ vals, const float* __restrict__ X,
                                                           float* __restrict__ Y, int cols_per_block, int snap, Scaling sc,
                                                           unsigned pinned_blocks, ChunkQueues queues, RowSharing sharing) {
    constexpr int W = kRunBlock, E = W / kWave, B = kRunBatch;
    constexpr int G = 1 << LOGG, R = kWave / G;
    __shared__ __align__(16) uint2 s_ent[kWavesPerBlock][W];            // row offset in X, value
    __shared__ unsigned s_bits[kWavesPerBlock][W / 32 + 2];             // bit e: a row ends with entry e of the block
    __shared__ int s_rows[kWavesPerBlock][W + 1];                       // those rows, in order
    struct EmptyRows { unsigned long long which[E]; int from; };        // bit l of which[e]: row from + 64 e + l has no entries
    __shared__ EmptyRows s_empty[kWavesPerBlock];
    const int lane = lane_id();
    const int wib = wave_in_block();
    uint2* ent = s_ent[wib];
    unsigned* bits = s_bits[wib];
    int* rows = s_rows[wib];
    EmptyRows& remembered = s_empty[wib];
    const int gl = lane & (G - 1), g = lane >> LOGG;

    if constexpr (QUEUED) snap = 0;                      // queues are for rows that chunks share
    constexpr bool kZerosBehind = !QUEUED && !AXPBY;
    __builtin_amdgcn_s_setprio(3);
    int probe = 0;
    if constexpr (!QUEUED) probe = first_probe(rowptr, M, lane);
    const unsigned nnz = (unsigned)rowptr[M], items = nnz + (unsigned)M;
    // Neighbouring chunks on one XCD share lines of A and Y - but where rows have few entries what an item costs changes
    // along the list (row ends and empty rows at the sparse end of a graph), and an XCD with the dear part ends last
    // (R-MAT 2^20 x 6, contiguous against dealt out one by one: N = 32 112 or 128 / 113 us, N = 101 420 or 470 / 383 us, the
    // longer of the two on the hardware queue a process gets first; 2^20 x 8 at N = 32 138 / 143, at N = 101 503 / 478 us,
    // 2^20 x 16 at N = 32 252 / 260 us).
    unsigned col_block = blockIdx.y, wg, nwg;
    bool dealt = false;
    const unsigned xcd = blockIdx.x % kXcd;
    if (pinned_blocks) {
        const unsigned i = blockIdx.x / kXcd, per_xcd = gridDim.x / kXcd;
        col_block = xcd % pinned_blocks;
        wg = (xcd / pinned_blocks) * per_xcd + i;
        nwg = (kXcd / pinned_blocks) * per_xcd;
    } else {
        dealt = nnz / (unsigned)M < (unsigned)run_dealt_below(LOGG);
        wg = dealt ? blockIdx.x : xcd_contiguous(blockIdx.x, gridDim.x);
        nwg = gridDim.x;
    }
    if constexpr (QUEUED) queues.fit(items, (unsigned)M);
    const EvenSplit share(items, QUEUED ? queues.chunks : nwg * kWavesPerBlock, QUEUED ? queues.size_log2 : kRunQuantumLog2);
    // queue q: what the waves of XCD q leave of its part of the chunks
    const auto part_of = [&](unsigned q) { return pinned_blocks ? q / pinned_blocks : q; };
    const auto queue_size = [&](unsigned q) { return queues.part_from(part_of(q) + 1u) - queues.queue_from(part_of(q)); };
    unsigned* taken = queues.taken + (size_t)blockIdx.y * kXcd * kQueuePitch;
    unsigned queue = xcd;
    const unsigned own = blockIdx.x / kXcd * kWavesPerBlock + (unsigned)wib;         // of the XCD's waves
    bool first_piece = true;

    for (;;) {                                           // one piece, or one after the other
    unsigned chunk = wg * kWavesPerBlock + (unsigned)wib, chunk_end = chunk + 1u;
    if constexpr (QUEUED) {
        if (queues.run == 0u) {                          // equal shares: chunk `chunk`, nothing else
            if (!first_piece || chunk >= queues.chunks) return;
            first_piece = false;
        } else if (first_piece) {
            chunk = queues.part_from(part_of(xcd)) + own * queues.run;
            chunk_end = chunk + queues.run;
            first_piece = false;
        } else {
            bool found = false;
            while (!found) {
                unsigned n = 0;
                if (lane == 0) n = atomicAdd(taken + queue * kQueuePitch, 1u);
                n = (unsigned)uniform((int)n);
                const unsigned size = queue_size(queue);
                if (n < size) {
                    chunk = queues.queue_from(part_of(queue)) + n;
                    chunk_end = chunk + 1u;
                    if (pinned_blocks) col_block = queue % pinned_blocks;
                    found = true;
                    break;
                }
                // Empty.  The first waves to see it of their own queue help with the others, nearest first, the rest are done: a word
                // that all waves add to takes 13 ns a time.
                if (queue == xcd && n - size >= queues.helpers) break;
                queue = (queue + 1u) % kXcd;
                if (queue == xcd) break;
            }
            if (!found) return;
        }
    }
    const LaneColumns mine = lane_columns<4, true>(col_block, cols_per_block, gl, N);
    const bool col_ok = mine.any;
    const unsigned d0 = share.start(chunk), d_end = share.start(chunk_end), d1 = d_end < items ? d_end : items;
    if (d0 >= d1) {
        if constexpr (QUEUED) continue; else return;
    }
    int is, ie;
    // rows shared with other waves, where no launch has cleared them
    RowWord* const words = sharing.words + (size_t)col_block * share.parts;
    constexpr bool shares = SHARES;
    static_assert(!SHARES || (!QUEUED && !AXPBY), "queues and the scaled form have their prepare launch");
    RowWord found = 0;
    if (shares && lane == 0) found = claim_row<DeviceWords>(words + chunk, sharing.call);
    if constexpr (QUEUED) {
        is = queues.starts[chunk];
        ie = queues.starts[chunk_end];
    } else {
        wave_merge_rows_before2(rowptr, M, d0, d1, lane, probe, is, ie);
    }
    unsigned js, je;
    bool first_split = false;
    if (snap) {
        snap_to_rows(rowptr, M, d0, d1, is, ie, js, je);
    } else {
        js = d0 - (unsigned)is;
        je = d1 - (unsigned)ie;
        first_split = is < M && (unsigned)is + (unsigned)rowptr[is] < d0;
    }
    is = uniform(is); ie = uniform(ie);
    js = (unsigned)uniform((int)js); je = (unsigned)uniform((int)je);
    const int r_first = first_split ? is : -1;
    const unsigned n_ent = je - js;
    const unsigned long long chunk_bytes = (unsigned long long)n_ent * 4ull;
    const __amdgpu_buffer_rsrc_t rc = make_buffer(colidx + js, chunk_bytes);
    const __amdgpu_buffer_rsrc_t ra = make_buffer(vals + js, chunk_bytes);
    const __amdgpu_buffer_rsrc_t rx = make_buffer(X, XBUF ? dense_bytes(K, ldx, N) : 0ull);
    // XBUF: X spans less than 2 GB, so half of the offset range switches off a lane without columns, and an entry past
    // the chunk's end (a switched-off lane there wraps to the start of X: read, never used)
    constexpr unsigned kOff = 0x80000000u;
    const unsigned lane_bytes = col_ok ? (unsigned)mine.first * 4u : kOff;
    const float* lane_x = X + (col_ok ? mine.first : 0ll);
    const unsigned pitch = (unsigned)ldx * 4u, y_pitch = (unsigned)ldy * 4u;

    int lc[E]; float la[E];
    auto load_entries = [&](unsigned from) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const unsigned off = (from + (unsigned)(e * kWave + lane)) * 4u;
            lc[e] = buffer_stream_i32(rc, off);                 // past the chunk: column 0, value 0
            la[e] = buffer_stream_f32(ra, off);
        }
    };
    // start and end offsets of rows first .. first + 63 (lane l: row first + l; past the last one 0)
    auto load_window = [&](int first, unsigned& start, unsigned& end) {
        const unsigned long long bytes = first < ie ? (unsigned long long)(ie + 1 - first) * 4ull : 0ull;
        const __amdgpu_buffer_rsrc_t rr = make_buffer(rowptr + (bytes ? first : 0), bytes);
        typedef unsigned u2 __attribute__((ext_vector_type(2)));
        const u2 t = __builtin_amdgcn_raw_buffer_load_b64(rr, (unsigned)lane * 4u, 0, 0);
        start = t.x; end = t.y;
    };
    auto y_at = [&](int row) { return Y + (size_t)row * (size_t)ldy + mine.first; };
    auto store4 = [&](float* y, const float (&v)[4]) {
        typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
        f4u t = {v[0], v[1], v[2], v[3]};
        __builtin_nontemporal_store(t, reinterpret_cast<f4u*>(y));
    };
    // stores of the scaled form: the columns I share with my neighbour are the neighbour's
    auto store_own = [&](float* y, const float (&v)[4]) {
        if (mine.skip != 0) {
#pragma unroll
            for (int i = 1; i < 4; ++i) if (i >= mine.skip) y[i] = v[i];
        } else {
            store4(y, v);
        }
    };
    // a finished row's four columns of my lane
    auto write_row = [&](int row, const float (&v)[4]) {
        float* y = y_at(row);
        if constexpr (AXPBY) {
            float o[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            if (sc.beta != 0.0f) load_vec_dword_aligned<4>(y, o);
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = sc.beta != 0.0f ? fmaf(sc.alpha, v[i], sc.beta * o[i]) : sc.alpha * v[i];
            store_own(y, o);
        } else {
            store4(y, v);
        }
    };
    auto add_row = [&](int row, const float (&v)[4]) {
        float* y = y_at(row);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i >= mine.skip) unsafeAtomicAdd(y + i, AXPBY ? sc.alpha * v[i] : v[i]);
    };

    // all lanes that hold columns of a row shared with other waves
    auto give_to_row = [&](unsigned word, int row, bool lanes, const float (&v)[4]) {
        bool sum = false;
        if (lane == 0) sum = row_has_sum<DeviceWords>(words + word, sharing.call);
        if (uniform(sum ? 1 : 0) != 0) {
            if (lanes) add_row(row, v);
        } else {
            if (lanes) write_part<DeviceWords, 4, false>(y_at(row), v, 0.0f, mine.skip);
            stores_done();
            if (lane == 0) publish_part<DeviceWords>(words + word, sharing.call);
        }
    };

    unsigned w_start, w_end;
    load_window(is, w_start, w_end);
    load_entries(0);
    // Behind the first entries, which otherwise wait for the two rows' bounds, and published when these entries are in LDS: R-MAT 2^18 x 16 at N = 32
    // 45.8 -> 44.9 us, Poisson 50 000 x 12 at N = 12 without statistics 13.6 -> 13.2 us, Zipf rows of 16 at N = 32 85.4 -> 84.8 us.
    HeldEnds ends;
    if (shares) ends = ChunkEnds(share, rowptr, M, chunk, d0, is, ie, js, je);
    if (shares && ends.starts_tail()) {
        const bool clear = uniform(mine_to_clear(found, sharing.call) ? 1 : 0) != 0;       // as lane 0 found it
        if (clear && g == 0 && col_ok) clear_row<DeviceWords, 4, false>(y_at(ie), 0.0f, mine.skip);
    }
    float carry[4] = {0.0f, 0.0f, 0.0f, 0.0f};          // sum of the row that is open at the block's start (every group: its columns)
    unsigned done = 0;                                  // entries before the block
    const unsigned third = n_ent > kPacedFrom ? (n_ent + 2u) / 3u : 0u;
    do {
        const unsigned nE = n_ent - done < (unsigned)W ? n_ent - done : (unsigned)W;
        const unsigned to = done + nE;
        // steps per group, a multiple of the batch; a short last block is still shared by all groups
        const unsigned U = ((nE + R * B - 1) / (R * B)) * B;
        wave_lds_sync();
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const bool in = (unsigned)(e * kWave + lane) < nE;
            unsigned off;
            if constexpr (XBUF) off = in ? (unsigned)lc[e] * pitch : kOff; else off = in ? (unsigned)lc[e] : kNoRow;
            ent[e * kWave + lane] = make_uint2(off, __builtin_bit_cast(unsigned, la[e]));
        }
        if (lane < W / 32 + 2) bits[lane] = 0u;
        wave_lds_sync();
        // ---- rows that end in this block: a bit at their last entry, their numbers in order; which rows have no entries
        int listed = 0, windows = 0;                        // windows of 64 rows that are remembered
        unsigned any_zero = 0u;
        if constexpr (kZerosBehind) remembered.from = is;
        // 64 rows from `first` on, those without entries: all lane groups together
        auto write_zeros = [&](int first, unsigned long long m_zero) {
            const auto empty = [&](int q) { return ((m_zero >> (q * R + g)) & 1ull) != 0ull && col_ok; };          // R rows per round
            if constexpr (AXPBY) {
                constexpr int F = G < 4 ? G : 4;        // rounds whose old values are in flight together
#pragma unroll 1
                for (int q = 0; q < G; q += F) {
                    float v[F][4];
#pragma unroll
                    for (int u = 0; u < F; ++u) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[u][i] = 0.0f;
                        if (empty(q + u) && sc.beta != 0.0f) load_vec_dword_aligned<4>(y_at(first + (q + u) * R + g), v[u]);
                    }
#pragma unroll
                    for (int u = 0; u < F; ++u) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[u][i] = sc.beta != 0.0f ? sc.beta * v[u][i] : 0.0f;
                        if (empty(q + u)) store_own(y_at(first + (q + u) * R + g), v[u]);
                    }
                }
            } else if constexpr (QUEUED) {                                  // in fewer registers
                const float zero[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
                for (int q = 0; q < G; ++q)
                    if (empty(q)) write_row(first + q * R + g, zero);
            } else {
                const float zero[4] = {0.0f, 0.0f, 0.0f, 0.0f};
                const __amdgpu_buffer_rsrc_t ry = make_buffer(Y + (size_t)first * (size_t)ldy, (unsigned long long)kWave * y_pitch);
                const unsigned long long m_mine = col_ok ? m_zero >> g : 0ull;
                const unsigned y_mine = (unsigned)g * y_pitch + (unsigned)mine.first * 4u;
#pragma unroll 4
                for (int q = 0; q < G; ++q)
                    if (((m_zero >> (q * R)) & (~0ull >> (kWave - R))) != 0ull)
                        buffer_store_vec<4, 2>(ry, (m_mine >> (q * R)) & 1ull ? y_mine + (unsigned)(q * R) * y_pitch : kOutOfRange, zero);
            }
        };
        auto take_rows = [&](unsigned start, unsigned end) {
            const unsigned rel = end - js;
            const bool live = is + lane < ie && rel <= to;
            const bool has = live && end != start && rel > done;
            const unsigned long long m_has = __ballot(has);
            const unsigned long long m_zero = AXPBY && !snap ? 0ull : __ballot(live && end == start);      // the prepare launch's
            if constexpr (!kZerosBehind) {
                if (m_zero != 0ull) write_zeros(is, m_zero);
            } else {
                remembered.which[windows++] = m_zero;
                any_zero |= (unsigned)m_zero | (unsigned)(m_zero >> 32);
            }
            const int cnt = (int)__popcll(__ballot(live));
            if (has) {
                const unsigned q = rel - done - 1u;
                atomicOr(bits + (q >> 5), 1u << (q & 31u));
                rows[listed + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m_has >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m_has, 0u))] = is + lane;
            }
            listed += (int)__popcll(m_has);
            is += cnt;
            return cnt == kWave;
        };
        // Rows without entries, all lane groups together.  Nothing waits for these stores but what is loaded behind them, so they come
        // behind the walk, and behind the bounds of further rows: in front of either, a chunk at the sparse end of a graph, with
        // hundreds of such rows, had its first gathers at 25 us of 46 (R-MAT 2^18 x 16 at N = 32).  32-bit offsets, and rounds that
        // no row needs are passed by.  R-MAT 2^12 x 11 at N = 93 13.2 -> 12.1 us, 2^13 x 10 at N = 54 11.4 -> 10.8 us, 2^18 x 16 at N = 32
        // 46.1 -> 45.1 us (on another GPU 44.8 -> 43.9 us), 2^18 x 10 at N = 87 in a slice 134.6 -> 122.4 us.  Not where rows are dealt out with few entries each: there all
        // chunks have such rows, and their stores would all come at the end (2^18 x 6 at N = 35 36.6 us in front, 38.2 behind).  kZerosBehind: nor with
        // queues, whose waves have no registers left for it (2^20 x 16 at N = 32 222.1 us behind, 220.7 in front, Poisson rows of 13,
        // none of them empty, at N = 60 420.8 and 418.7 us), nor in the scaled form, where the prepare launch sees to these rows or few are
        // empty, and remembering them costs for nothing (behind / in front 2^12 x 16 at N = 8 10.2 / 10.1 us, Zipf 30 001 x 30 at N = 16 / 33 20.3 / 33.4 and
        // 20.1 / 33.0 us, lognormal 100 001 x 20 at N = 5 / 16 21.9 / 31.1 and 21.2 / 30.4 us).
        auto treat_empty_rows = [&]() {
            const int from = uniform(remembered.from);
#pragma unroll 1
            for (int e = 0; e < windows; ++e) {
                const unsigned long long m_lane = remembered.which[e];
                const unsigned long long m_zero = (unsigned long long)(unsigned)uniform((int)(m_lane >> 32)) << 32 | (unsigned)uniform((int)m_lane);
                if (m_zero != 0ull) write_zeros(from + e * kWave, m_zero);
            }
            windows = 0;
        };
        bool crowded = take_rows(w_start, w_end);
        while (crowded) {
            // the next seven windows at once, in front of the stores of the rows so far where these are too many to remember
            unsigned ms[E - 1], me[E - 1];
#pragma unroll
            for (int m = 0; m < E - 1; ++m) load_window(is + m * kWave, ms[m], me[m]);
            if (windows > 1) {
                treat_empty_rows();
                remembered.from = is;
            }
#pragma unroll
            for (int m = 0; m < E - 1; ++m)
                if (crowded) crowded = take_rows(ms[m], me[m]);
        }
        if (any_zero == 0u) windows = 0;
        wave_lds_sync();
        load_window(is, w_start, w_end);
        if (shares && done == 0u) {
            stores_done();
            if (lane == 0) publish_start<DeviceWords>(words + chunk, sharing.call, found);
        }
        if (to < n_ent) load_entries(to);
        if (dealt && windows > 0) treat_empty_rows();

        // ---- my group's run: entries [g * U, g * U + U) of the block; k: its next row end in `rows`
        const unsigned p0 = (unsigned)g * U;
        int k;
        {
            const unsigned word = lane < W / 32 ? bits[lane] : 0u;
            unsigned n = (unsigned)__popc(word);
            const unsigned own = n;
            n += dpp_or_zero_u<kDppRowShr1, 0xf>(n);
            n += dpp_or_zero_u<kDppRowShr2, 0xf>(n);
            n += dpp_or_zero_u<kDppRowShr4, 0xf>(n);
            n += dpp_or_zero_u<kDppRowShr8, 0xf>(n);        // lanes 0 ... 15: the block's 16 words
            const int wi = (int)(p0 >> 5) < W / 32 ? (int)(p0 >> 5) : W / 32 - 1;
            const unsigned before = (unsigned)__shfl((int)(n - own), wi);
            const unsigned here = (unsigned)__shfl((int)word, wi);
            k = p0 < (unsigned)W ? (int)(before + (unsigned)__popc(here & ((1u << (p0 & 31u)) - 1u))) : listed;
        }
        const int k0 = k;
        int next = rows[k < W ? k : W];
        float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f}, head[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        // a run that starts inside a row: the first row end it meets is finished after the walk
        bool pend = p0 == 0u ? true : ((bits[(p0 - 1u) >> 5] >> ((p0 - 1u) & 31u)) & 1u) == 0u;
        bool closed = false;
        unsigned until = 0u;                                // where the next priority begins
        for (unsigned s0 = 0; s0 < U; s0 += B) {
            const unsigned at = done + s0 * R;
            if (at >= until) {
                const unsigned behind = at < third ? 2u : at < 2u * third ? 1u : 0u;
                until = behind == 2u ? third : behind == 1u ? 2u * third : ~0u;
                set_wave_priority(behind);
            }
            const unsigned p = p0 + s0;
            float x[B][4], a[B];
#pragma unroll
            for (int s = 0; s < B; ++s) {
                const uint2 t = ent[p + s];
                a[s] = __builtin_bit_cast(float, t.y);
                if constexpr (XBUF) {
                    buffer_load_vec<4>(rx, t.x + lane_bytes, x[s]);
                } else {
                    const bool ok = t.x != kNoRow;
                    load_vec_dword_aligned<4>(lane_x + (size_t)(ok ? t.x : 0u) * (size_t)ldx, x[s]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) x[s][i] = ok ? x[s][i] : 0.0f;
                }
            }
            const unsigned m = (bits[p >> 5] >> (p & 31u)) & ((1u << B) - 1u);          // p is a multiple of B
            const unsigned any = wave_or(m);
#pragma unroll
            for (int s = 0; s < B; ++s) {
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[i] = fmaf(a[s], x[s][i], acc[i]);
                if ((any >> s) & 1u) {                                       // wave-uniform
                    if ((m >> s) & 1u) {
                        if (pend) {
#pragma unroll
                            for (int i = 0; i < 4; ++i) head[i] = acc[i];
                        } else if (col_ok) {
                            write_row(next, acc);
                        }
                        pend = false;
                        closed = true;
#pragma unroll
                        for (int i = 0; i < 4; ++i) acc[i] = 0.0f;
                        ++k;
                        next = rows[k];
                    }
                }
            }
        }
        __builtin_amdgcn_s_setprio(3);
        if constexpr (kZerosBehind) {
            if (windows > 0) treat_empty_rows();
        }
        // ---- the open row across the groups' runs: inclusive segmented sum of what each run leaves open, the block's
        //      carry in front; a run that met a row end starts a new segment
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = acc[i] + ((g == 0 && !closed) ? carry[i] : 0.0f);
        const unsigned long long m_closed = __ballot(closed);
        // groups directly below mine in my segment
        const unsigned long long below = m_closed & ((2ull << lane) - 1ull);
        const int seg = below != 0ull ? ((63 - __builtin_clzll(below)) >> LOGG) : 0;
        const int h = g - seg;
#pragma unroll
        for (int d = 1; d < R; d <<= 1) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float o = __shfl_up(v[i], (unsigned)(d * G));
                v[i] += h >= d ? o : 0.0f;
            }
        }
        float in[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float o = __shfl_up(v[i], (unsigned)G);
            in[i] = g == 0 ? carry[i] : o;
            carry[i] = __shfl(v[i], kWave - G + gl);
        }
        const bool starts_open = p0 == 0u ? true : ((bits[(p0 - 1u) >> 5] >> ((p0 - 1u) & 31u)) & 1u) == 0u;
        bool give = false;
        if (closed && starts_open && col_ok) {
            const int row = rows[k0];
#pragma unroll
            for (int i = 0; i < 4; ++i) in[i] += head[i];
            if (row != r_first) write_row(row, in); else if (shares) give = true; else add_row(row, in);
        }
        if (shares && __ballot(give) != 0ull) give_to_row(ends.head, r_first, give, in);
        done = to;
    } while (done < n_ent);
    // the row still open at the end of my chunk is finished by another wave
    if (shares) {
        if (ends.whole_tail()) {
            if (g == 0 && col_ok) write_row(ie, carry);
        } else if (ends.shares_tail()) {
            give_to_row(ends.tail, ie, g == 0 && col_ok, carry);
        }
    } else if (!snap && ie < M) {
        bool any = false;
#pragma unroll
        for (int i = 0; i < 4; ++i) any |= carry[i] != 0.0f;
        if (any && g == 0 && col_ok) add_row(ie, carry);
    }
    if constexpr (!QUEUED) return;
    }
}

// ===========================================================================
// row statistics of a matrix that lives in device memory (the selector's metrics, Section 2.2)
// ===========================================================================
// The span of a row whose columns ascend is that of its two ends, and whether all rows ascend is a matter of counting:
// the adjacent entries of the whole list that descend, less those where a row starts, lie inside rows.  So the columns
// are streamed once, in equal pieces whatever the rows are like (with int64 columns the 32-bit copy is written on the
// way), and a row costs a thread three of them.  A matrix with a descent inside a row is counted again by features_kernel.
// Blocks leave their sums in a scratch row each; the last one to finish adds these up and puts the result where the host
// looks for it.  All sums are integer sums, so the result does not depend on who comes when.
// The host goes on when it sees the result, before the kernel's end, so nothing here may wait in one XCD's L2 for that end:
// scratch rows, counters, result and the 32-bit arrays are accessed at device or system scope one by one, and a workgroup is
// counted in when the stores of all its waves are done.  A fence in their place would write back the whole L2 once per
// workgroup.  Against plain stores of the 32-bit arrays, whole calls: 20 001 rows of 10 18.5 -> 18.7 us, 200 001 rows of 10
// 27.1 -> 26.4 us, 27-point stencil on 128^3 186 us in both forms.
// Bound by the HBM stream on large matrices and by the launch and the host's wait on small ones.  Against two conversions, a
// clearing launch, a pass with one wave per 64 rows and a copy back, int64 columns: 20 001 rows of 10 66 -> 19 us, 27-point
// stencil on 128^3 966 -> 186 us (3.6 TB/s of indices read and written), R-MAT 2^20 x 16 1858 -> 56 us.
// On small ones the kernel is a chain of trips: two to the row's columns, the workgroup's sums, the counters, the last one's look at
// all sums, host memory.  No store of it waits that does not have to: the waves' stores are waited for behind their sums, the counters
// wrap to zero by themselves, every piece of the result carries the call's tag, so that no word has to come last, and a wave adds up by
// DPP.  20 001 rows of 10, int64: kernel 11.6 -> 8.5 us, with one product at N = 32 30.3 -> 27.1 us; 4096 rows of 8 at N = 4
// 25.0 -> 22.2 us, R-MAT 2^16 x 16 at N = 7 42.7 -> 37.9 us, 2^20 x 16 at N = 3 189.6 -> 186.6 us.
constexpr int kStatBlocks = 1024;
constexpr int kStatWords = 8;          // sum len^2, max len, min len, rows with a span, sum of spans, decreasing pointers, descents at row starts, descents
constexpr int kStatPieces = kStatWords + 4;            // their lower halves, rowptr[0], rowptr[M], the upper halves of the two sums
constexpr int kStatAnnounceWord = 10;                  // where column_reuse_kernel's result is announced, and behind
constexpr int kStatChunk = 2048;       // entries a block takes at a time
struct StatScratch {
    unsigned long long part[kStatBlocks][kStatWords];
    unsigned long long result[16];
    unsigned arrived[9][16];           // eight counters for blocks b % 8, one for those groups; zero between calls
};

__device__ __forceinline__ void stat_store(unsigned long long* p, unsigned long long v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Stores of the 32-bit arrays, one or two entries (8-byte aligned): written through the XCD's L2, so that kernels on other
// streams, on any XCD, find them once stores_done() is past.
__device__ __forceinline__ void stat_store(int* p, int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void stat_store_two(int* p, int v, int w) {
    stat_store(reinterpret_cast<unsigned long long*>(p), (unsigned)v | (unsigned long long)(unsigned)w << 32);
}

__device__ __forceinline__ unsigned long long shfl_xor_u64(unsigned long long v, int mask) {
    const unsigned lo = (unsigned)__shfl_xor((int)(unsigned)v, mask, kWave);
    const unsigned hi = (unsigned)__shfl_xor((int)(unsigned)(v >> 32), mask, kWave);
    return ((unsigned long long)hi << 32) | lo;
}

// word w of two partial results
__device__ __forceinline__ unsigned long long stat_join(int w, unsigned long long a, unsigned long long b) {
    return w == 1 ? (a > b ? a : b) : w == 2 ? (a < b ? a : b) : a + b;
}
// Joined with what the lane below (DPP control) has; a lane that has none below keeps its own.  Only the sums of squares and of spans
// need more than 32 bits.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ void stat_join_below(unsigned long long (&v)[kStatWords]) {
    const auto below = [](unsigned mine, unsigned none) {
        return (unsigned)__builtin_amdgcn_update_dpp((int)none, (int)mine, CTRL, ROW_MASK, 0xf, false);
    };
#pragma unroll
    for (int w = 0; w < kStatWords; ++w) {
        const unsigned long long none = w == 2 ? ~0ull : 0ull;
        const unsigned lo = below((unsigned)v[w], (unsigned)none);
        unsigned hi = 0;
        if (w == 0 || w == 4) hi = below((unsigned)(v[w] >> 32), 0u);
        v[w] = w == 0 || w == 4 ? stat_join(w, v[w], (unsigned long long)hi << 32 | lo)
                                : (unsigned long long)(unsigned)stat_join(w, (unsigned)v[w], lo);
    }
}
// The workgroup's partial results in thread 0; the stores of all its waves are done.
__device__ __forceinline__ void stat_reduce(unsigned long long (&v)[kStatWords], unsigned long long (*lds)[kStatWords]) {
    stat_join_below<kDppRowShr1, 0xf>(v);
    stat_join_below<kDppRowShr2, 0xf>(v);
    stat_join_below<kDppRowShr4, 0xf>(v);
    stat_join_below<kDppRowShr8, 0xf>(v);
    stat_join_below<kDppRowBcast15, 0xa>(v);
    stat_join_below<kDppRowBcast31, 0xc>(v);
    if (lane_id() == kWave - 1)
#pragma unroll
        for (int w = 0; w < kStatWords; ++w) lds[wave_in_block()][w] = v[w];
    stores_done();
    __syncthreads();
    if (threadIdx.x == 0)
#pragma unroll
        for (int w = 0; w < kStatWords; ++w) {
            v[w] = lds[0][w];
#pragma unroll
            for (int q = 1; q < kWavesPerBlock; ++q) v[w] = stat_join(w, v[w], lds[q][w]);
        }
    __syncthreads();
}

// I: int or long long.  `entries`: length of colidx, -1: rowptr[M].  colidx32 is written for 64-bit indices.  `host`: result
// in host memory, `tag` in the upper half of every word; nullptr: result in the scratch.
// row_blocks: so many workgroups at the end of the grid take the rows and the others the entries (small matrices: two chains of
// dependent loads side by side); 0: all take some of both.
template <typename I>
__global__ __launch_bounds__(kBlock) void csr_statistics_kernel(int M, long long entries, const I* __restrict__ rowptr,
                                                                const I* __restrict__ colidx, int* __restrict__ rowptr32,
                                                                int* __restrict__ colidx32, StatScratch* sc,
                                                                unsigned long long* host, unsigned tag, unsigned row_blocks) {
    constexpr bool kConvert = sizeof(I) == 8;
    __shared__ unsigned long long lds[kWavesPerBlock][kStatWords];
    __shared__ int s_last;
    const int t = (int)threadIdx.x;
    const int row_first = (int)rowptr[0], row_end = (int)rowptr[M];
    long long nnz = row_end < 0 ? 0 : row_end;                  // entries whose order counts
    if (entries >= 0 && nnz > entries) nnz = entries;
    const long long flat = colidx == nullptr ? 0 : kConvert ? entries : nnz;
    long long chunks = (flat + kStatChunk - 1) / kStatChunk;
    const long long by_rows = ((long long)M + kStatChunk - 1) / kStatChunk;
    if (chunks < by_rows && row_blocks == 0) chunks = by_rows;
    long long rows_per_chunk = ((long long)M + chunks - 1) / (chunks > 0 ? chunks : 1);
    const unsigned entry_blocks = gridDim.x - row_blocks;
    const bool takes_rows = row_blocks == 0 || blockIdx.x >= entry_blocks, takes_entries = blockIdx.x < entry_blocks;
    unsigned first = blockIdx.x, blocks = gridDim.x;
    if (row_blocks != 0) {
        if (takes_rows) {
            first -= entry_blocks;
            blocks = row_blocks;
            rows_per_chunk = ((long long)M + row_blocks - 1) / row_blocks;
            chunks = row_blocks;
        } else {
            blocks = entry_blocks;
        }
    }

    unsigned long long v[kStatWords] = {0, 0, ~0ull, 0, 0, 0, 0, 0};
    for (long long c = first; c < chunks; c += blocks) {
        if (takes_entries) {
        // ---- entries: two per thread and step
        constexpr int S = kStatChunk / (2 * kBlock);
        I x[S], y[S], z[S];                                      // entries p, p + 1 and p + 2
#pragma unroll
        for (int k = 0; k < S; ++k) {
            const long long p = c * kStatChunk + k * 2 * kBlock + 2 * t;
            x[k] = y[k] = z[k] = 0;
            if (p + 1 < flat) {
                I two[2];
                __builtin_memcpy(two, colidx + p, sizeof(two));
                x[k] = two[0]; y[k] = two[1];
            } else if (p < flat) {
                x[k] = colidx[p];
            }
            if (lane_id() == kWave - 1 && p + 2 < flat) z[k] = colidx[p + 2];
        }
        unsigned down = 0;
#pragma unroll
        for (int k = 0; k < S; ++k) {
            const long long p = c * kStatChunk + k * 2 * kBlock + 2 * t;
            const int a = (int)x[k], b = (int)y[k];
            const int next = __shfl_down(a, 1);
            const int d = lane_id() == kWave - 1 ? (int)z[k] : next;
            down += (p + 1 < nnz && a > b) ? 1u : 0u;
            down += (p + 2 < nnz && b > d) ? 1u : 0u;
            if constexpr (kConvert) {
                if (p + 1 < flat) stat_store_two(colidx32 + p, a, b);
                else if (p < flat) stat_store(colidx32 + p, a);
            }
        }
        v[7] += down;
        }
        if (!takes_rows) continue;
        // ---- rows
        const long long r1 = (c + 1) * rows_per_chunk < M ? (c + 1) * rows_per_chunk : M;
        for (long long r = c * rows_per_chunk + t; r < r1; r += kBlock) {
            const int s = (int)rowptr[r], e = (int)rowptr[r + 1];
            if constexpr (kConvert) {
                stat_store(rowptr32 + r, s);
                if (r == M - 1) stat_store(rowptr32 + M, e);
            }
            long long len = (long long)e - (long long)s;
            if (len < 0) { v[5] = 1; len = 0; }
            const unsigned long long l = (unsigned long long)len;
            v[0] += l * l;
            v[1] = l > v[1] ? l : v[1];
            v[2] = l < v[2] ? l : v[2];
            if (len > 0 && colidx != nullptr && s >= 0 && e <= nnz) {
                const int first = (int)colidx[s], last = (int)colidx[e - 1];
                const int before = s > 0 ? (int)colidx[s - 1] : first;
                v[3] += 1;
                v[4] += (unsigned long long)((long long)last - first + 1);
                v[6] += before > first ? 1ull : 0ull;
            }
        }
    }
    stat_reduce(v, lds);                                         // (every wave's stores, before its workgroup is counted in)
    if (t == 0) {
#pragma unroll
        for (int w = 0; w < kStatWords; ++w) stat_store(&sc->part[blockIdx.x][w], v[w]);
        stores_done();
        const unsigned group = blockIdx.x % 8, groups = gridDim.x < 8 ? gridDim.x : 8;
        const unsigned members = (gridDim.x - group + 7) / 8;
        // a counter is back at zero with the last one counted, for the place's next call, which may start before this one ends
        s_last = atomicInc(&sc->arrived[group][0], members - 1) == members - 1 && atomicInc(&sc->arrived[8][0], groups - 1) == groups - 1;
    }
    __syncthreads();
    if (s_last == 0) return;
    unsigned long long u[kStatWords] = {0, 0, ~0ull, 0, 0, 0, 0, 0};
    for (unsigned b = t; b < gridDim.x; b += kBlock)
#pragma unroll
        for (int w = 0; w < kStatWords; ++w)
            u[w] = stat_join(w, u[w], __hip_atomic_load(&sc->part[b][w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    stat_reduce(u, lds);
    // a piece of 32 bits a word, each beside the call's tag: the host takes the result when it has all of them, no store waits
    __shared__ unsigned s_piece[kStatPieces];
    if (t == 0) {
#pragma unroll
        for (int w = 0; w < kStatWords; ++w) s_piece[w] = (unsigned)u[w];
        s_piece[kStatWords] = (unsigned)row_first;
        s_piece[kStatWords + 1] = (unsigned)row_end;
        s_piece[kStatWords + 2] = (unsigned)(u[0] >> 32);
        s_piece[kStatWords + 3] = (unsigned)(u[4] >> 32);
    }
    __syncthreads();
    if (t < kStatPieces)
        __hip_atomic_store((host ? host : sc->result) + t, (unsigned long long)tag << 32 | s_piece[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ===========================================================================
// how popular the columns are (for the width of the column blocks of nb_sr_run_kernel and the hot runs of nb_pr_kernel)
// ===========================================================================
// Counts distinct columns, and those met once, among 16384, 32768 and 65536 sampled entries: the first 1024, 2048 and 4096 of
// 16 pieces, evenly spread.  Only columns whose hash falls into the lower half of its range are counted (saved_share(), host,
// doubles the counts and allows for the columns that share a bucket): counts of columns, so half of them tell the share to
// 0.003 to 0.008.  One workgroup, two bits per bucket in 64 KB of LDS, all loads at once: 10 us on R-MAT 2^20 x 16, 20 us
// with the launch and the host's wait; the loads of 64 pieces in four batches and a word of LDS that every thread added to
// had been 32 us.
constexpr int kReuseLevels = 3, kReusePieces = 16, kReuseThreads = 1024, kReuseBucketsLog2 = 18, kReuseRateLog2 = 1;
constexpr long long kReuseEntriesMin = 4 * kReuseThreads;              // a piece

constexpr int kReuseResultWords = 2 * kReuseLevels + kHotWidths;       // its counts, and the sampled entries in hot runs

// exclusive prefix sum over the threads of the workgroup; `total`: the sum of all
__device__ __forceinline__ unsigned reuse_prefix(unsigned v, unsigned* waves, unsigned& total) {
    unsigned sum = v;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const unsigned o = (unsigned)__shfl_up((int)sum, (unsigned)d);
        sum += lane_id() >= d ? o : 0u;
    }
    __syncthreads();                                             // the last call's readers are done
    if (lane_id() == kWave - 1) waves[threadIdx.x / kWave] = sum;
    __syncthreads();
    unsigned before = 0;
    total = 0;
    for (int w = 0; w < kReuseThreads / kWave; ++w) {
        before += w < (int)(threadIdx.x / kWave) ? waves[w] : 0u;
        total += waves[w];
    }
    return before + sum - v;
}

// The hot runs (HotColumns): 32768 entries, 512 pieces of 64 evenly spread, are counted by run of 2^shift columns, at most 32768
// runs, and the `room` fullest taken.  Thread t owns runs 32 t ... 32 t + 31, a word of the bitmap.  `bins`: 32768 words.
// Returns how many entries the table saves the caches, per kHotSample: those in hot runs, without those in the fullest `cached`
// ones, which an L1 holds anyway.  A run is among the fullest of a sample partly because the sample met it often, so the entries that
// made the choice overstate its share (uniform columns, 262 144 of them at N = 1: 23 % of the sample, 12 % of the matrix).  Every
// entry is therefore asked whether its run would have been taken by the others alone (12 % there; of 66 matrices the worst is 1.7 % of
// all entries away from the matrix's own count, without the question 11 %).
// A wave's 64 counters lie 32 words apart, on one bank, so the counters of a word are rotated by its number.
constexpr int kHotSamplePieces = 512, kHotSample = kHotSamplePieces * kWave, kHotLevels = kReuseThreads;

__device__ __forceinline__ unsigned hot_columns(long long entries, const int* __restrict__ colidx, unsigned* table, int shift,
                                                unsigned room, unsigned cached, unsigned* bins, unsigned* waves) {
    constexpr int kPerThread = kHotSample / kReuseThreads;
    // of the `room` and of the `cached` fullest runs: the count that all but the last have, how many have it and how many have one
    // less, the entries in runs with more than it and with just it
    __shared__ unsigned s_level[2], s_above[2], s_tied[2], s_sure[2], s_shared[2];
    const int t = (int)threadIdx.x;
    unsigned c[kPerThread];
#pragma unroll
    for (int q = 0; q < kPerThread; ++q)
        c[q] = (unsigned)colidx[(entries - kWave) / (kHotSamplePieces - 1) * (uniform(t / kWave) * kPerThread + q) + lane_id()];
    for (int i = 0; i < 8; ++i) reinterpret_cast<uint4*>(bins)[t + i * kReuseThreads] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    const auto place = [](unsigned word, unsigned bit) { return word * 32u + ((bit + word) & 31u); };
#pragma unroll
    for (int q = 0; q < kPerThread; ++q) {
        const unsigned run = c[q] >> shift < 32u * kHotWords ? c[q] >> shift : 32u * kHotWords - 1u;
        atomicAdd(&bins[place(run >> 5, run & 31u)], 1u);
    }
    __syncthreads();
    unsigned n[32];
#pragma unroll
    for (unsigned b = 0; b < 32; ++b) n[b] = bins[place((unsigned)t, b)];
    __syncthreads();
    // how many runs have each count (the last level: that and more, no more runs than there is room for).  Most have next to
    // none: these go a wave at a time.
    unsigned* levels = bins;
    levels[t] = 0u;
    __syncthreads();
    unsigned few = 0;                                            // a byte each for 0, 1, 2, 3
#pragma unroll
    for (unsigned b = 0; b < 32; ++b) {
        if (n[b] < 4u) few += 1u << (8u * n[b]);
        else atomicAdd(&levels[n[b] < (unsigned)kHotLevels ? n[b] : kHotLevels - 1], 1u);
    }
    unsigned even = few & 0x00ff00ffu, odd = (few >> 8) & 0x00ff00ffu;
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
        even += (unsigned)__shfl_xor((int)even, m);
        odd += (unsigned)__shfl_xor((int)odd, m);
    }
    if (lane_id() == 0) {
        atomicAdd(&levels[1], odd & 0xffffu);
        atomicAdd(&levels[2], even >> 16);
        atomicAdd(&levels[3], odd >> 16);
    }
    __syncthreads();
    // the lowest level that no more than `room` runs reach
    unsigned total;
    {
        const unsigned level = (unsigned)(kHotLevels - 1 - t), here = levels[level];
        // runs, and their entries in the upper half (the last level's as if they had just that count; neither sum goes beyond kHotSample)
        const unsigned before = reuse_prefix(here | (level * here) << 16, waves, total);
        const unsigned reach = (before & 0xffffu) + here, more = before >> 16;
        const unsigned up_to = (total >> 16) - more;                 // entries at this level and below
        const bool last = t == 0;                                    // all entries that are not below it are at the last level
        const unsigned in_last = kHotSample - (up_to - level * here);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const unsigned places = k == 0 ? room : cached;
            const unsigned below = level > 0u ? levels[level - 1u] : 0u;
            if (level >= 1u && reach <= places && (level == 1u || reach + below > places)) {
                s_level[k] = level;
                s_above[k] = reach;
                s_tied[k] = below;
                s_sure[k] = last ? in_last : kHotSample - up_to;
                s_shared[k] = last ? 0u : level * here;
            } else if (last && reach > places) {                     // even the last level has too many: `places` of them
                s_level[k] = (unsigned)kHotLevels;
                s_above[k] = 1u;
                s_tied[k] = here - 1u;
                s_sure[k] = 0u;
                s_shared[k] = in_last;
            }
        }
    }
    __syncthreads();
    // its runs, and of those one below the first ones, as many as there are places left
    const unsigned lowest = s_level[0], left = lowest > 1u ? room - s_above[0] : 0u;
    unsigned mask = 0, below = 0;
#pragma unroll
    for (unsigned b = 0; b < 32; ++b) {
        mask |= n[b] >= lowest ? 1u << b : 0u;
        below |= n[b] + 1u == lowest ? 1u << b : 0u;
    }
    const unsigned before = reuse_prefix((unsigned)__popc(mask) | (unsigned)__popc(below) << 16, waves, total);
    unsigned rank = before >> 16, at = (before & 0xffffu) + (rank < left ? rank : left);
    for (; below != 0u && rank < left; below &= below - 1u, ++rank) mask |= below & -below;
    const unsigned tied = total >> 16, hot = (total & 0xffffu) + (tied < left ? tied : left);
    stat_store_two(reinterpret_cast<int*>(table) + 2 * t, (int)mask, (int)at);
    unsigned* list = bins + kHotLevels;
#pragma unroll
    for (unsigned b = 0; b < 32; ++b)
        if ((mask >> b) & 1u) list[at++] = 32u * (unsigned)t + b;
    __syncthreads();
    stat_store(reinterpret_cast<int*>(table) + 2 * kHotWords + t, (int)((unsigned)t < hot ? list[t] : kNoRow));
    stores_done();
    __syncthreads();
    // Without one of its entries a run still has the count that was asked for, or it shares the places that are left with those
    // one below.
    const auto would_be_met = [&](int k, unsigned places) {
        const float share = s_level[k] == 1u ? 0.0f : (float)(places - s_above[k] + 1u) / (float)(s_tied[k] + 1u);
        return (float)s_sure[k] + share * (float)s_shared[k];
    };
    const float saved = would_be_met(0, room) - would_be_met(1, cached);
    return saved > 0.0f ? (unsigned)(saved + 0.5f) : 0u;
}
static_assert(kHotSample / kHotLevels <= hot_room(4, kHotShiftMax) && kHotSample / kHotLevels <= hot_room(3, kHotShiftMax),
              "the runs of the last level fit");
static_assert(kHotWords == kReuseThreads && hot_floats(1) >> kHotShiftMin <= kReuseThreads, "a thread a word of the bitmap and a hot run");

// Workgroup 0 counts distinct columns; workgroup v, where there is one, finds the hot runs for products with v columns, of a
// matrix whose columns fall into at most 32768 runs of 2^hot_shift.  Each announces itself in a word of its own.
__global__ __launch_bounds__(kReuseThreads) void column_reuse_kernel(long long entries, const int* __restrict__ colidx,
                                                                    unsigned* hot_table, int hot_shift,
                                                                    unsigned long long* out, unsigned long long* announce,
                                                                    unsigned long long ticket) {
    constexpr int kWords = (1 << kReuseBucketsLog2) / 16;
    constexpr int kOwn = kWords / kReuseThreads;
    __shared__ __align__(16) unsigned table[32 * kHotWords];     // kWords, and words behind for the columns that are not counted
    __shared__ unsigned sums[kReuseLevels][2];
    __shared__ unsigned waves[kReuseThreads / kWave];
    static_assert(kWords + kWave <= 32 * kHotWords, "the table holds both");
    const int t = (int)threadIdx.x;
    if (blockIdx.x != 0) {
        const int v = (int)blockIdx.x;
        const unsigned met = hot_columns(entries, colidx, hot_table + (v - 1) * kHotTableInts, hot_shift, (unsigned)hot_room(v, hot_shift),
                                         (unsigned)hot_cached(v, hot_shift), table, waves);
        if (t == 0) {
            __hip_atomic_store(out + 2 * kReuseLevels + v - 1, (unsigned long long)met, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            stores_done();
            if (announce) __hip_atomic_store(announce + v, ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        return;
    }
    unsigned c[4][kReusePieces];
#pragma unroll
    for (int part = 0; part < 4; ++part)
#pragma unroll
        for (int q = 0; q < kReusePieces; ++q)
            c[part][q] = (unsigned)colidx[(entries - kReuseEntriesMin) * q / (kReusePieces - 1) + part * kReuseThreads + t];
    for (int i = 0; i < kOwn; ++i) table[t + i * kReuseThreads] = 0u;
    if (t < kReuseLevels * 2) sums[t / 2][t % 2] = 0u;
    __syncthreads();
#pragma unroll
    for (int level = 0; level < kReuseLevels; ++level) {
#pragma unroll
        for (int part = level == 0 ? 0 : 1 << (level - 1); part < 1 << level; ++part) {
            unsigned at[kReusePieces], seen[kReusePieces], old[kReusePieces];
#pragma unroll
            for (int q = 0; q < kReusePieces; ++q) {
                unsigned key = c[part][q] * 2654435761u;         // one product alone spreads neighbours too evenly
                key = (key ^ (key >> 15)) * 2654435761u;
                const bool counted = (key >> (32 - kReuseRateLog2)) == 0u;
                const unsigned b = key >> (32 - kReuseRateLog2 - kReuseBucketsLog2);
                at[q] = counted ? b >> 4 : (unsigned)(kWords + lane_id());
                seen[q] = counted ? 1u << (2u * (b & 15u)) : 0u;
                old[q] = atomicOr(&table[at[q]], seen[q]);
            }
#pragma unroll
            for (int q = 0; q < kReusePieces; ++q)
                if (old[q] & seen[q]) atomicOr(&table[at[q]], seen[q] << 1);
        }
        __syncthreads();
        unsigned distinct = 0, once = 0;
        for (int i = 0; i < kOwn; ++i) {
            const unsigned w = table[t + i * kReuseThreads];
            distinct += (unsigned)__popc(w & 0x55555555u);
            once += (unsigned)__popc(w & 0x55555555u & ~(w >> 1));
        }
        unsigned both = distinct | once << 16;                   // at most 2^16 together in a wave's share of the table
#pragma unroll
        for (int m = 1; m < kWave; m <<= 1) both += (unsigned)__shfl_xor((int)both, m);
        if (lane_id() == 0) {                                    // one a wave: 1024 adds to one word take 4 us
            atomicAdd(&sums[level][0], both & 0xffffu);
            atomicAdd(&sums[level][1], both >> 16);
        }
        __syncthreads();
    }
    if (t == 0) {
        for (int i = 0; i < kReuseLevels * 2; ++i)
            __hip_atomic_store(out + i, (unsigned long long)sums[i / 2][i % 2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        stores_done();
        if (announce) __hip_atomic_store(announce, ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// The same metrics with every row's columns looked at (rows whose columns are not ascending).
// ws[0] sum of len^2, [1] max len, [2] min len, [3] non-empty rows whose span was taken,
// [4] sum of (largest - smallest column + 1), [5] a row pointer decreased, [6] rowptr[0], [7] rowptr[M].
constexpr int kFeatureWords = 8;
constexpr int kFeatureLongRow = 128;   // longer rows are scanned by the whole wave

__global__ void features_init_kernel(unsigned long long* __restrict__ ws) {
    if (blockIdx.x == 0 && threadIdx.x < kFeatureWords) ws[threadIdx.x] = threadIdx.x == 2 ? ~0ull : 0ull;
}

__global__ __launch_bounds__(kBlock) void features_kernel(int M, const int* __restrict__ rowptr,
                                                           const int* __restrict__ colidx,
                                                           unsigned long long* __restrict__ ws) {
    const int lane = lane_id();
    const long long nwaves = (long long)gridDim.x * kWavesPerBlock;
    const long long gw = (long long)blockIdx.x * kWavesPerBlock + wave_in_block();
    unsigned long long sq = 0, mx = 0, mn = ~0ull, rows = 0, span = 0, bad = 0;
    for (long long r0 = gw * kWave; r0 < M; r0 += nwaves * kWave) {
        const long long row = r0 + lane;
        const bool live = row < M;
        int s = 0, e = 0;
        if (live) { s = rowptr[row]; e = rowptr[row + 1]; }
        long long len = (long long)e - (long long)s;
        if (len < 0) { bad = 1; len = 0; }
        if (live) {
            const unsigned long long l = (unsigned long long)len;
            sq += l * l;
            mx = l > mx ? l : mx;
            mn = l < mn ? l : mn;
        }
        if (colidx != nullptr) {
            const bool long_row = live && len > kFeatureLongRow;
            if (live && len > 0 && !long_row) {
                int lo = colidx[s], hi = lo;
                for (int p = s + 1; p < e; ++p) {
                    const int c = colidx[p];
                    lo = c < lo ? c : lo;
                    hi = c > hi ? c : hi;
                }
                span += (unsigned long long)((long long)hi - lo + 1);
                rows += 1;
            }
            unsigned long long todo = __ballot(long_row);
            while (todo) {                                   // wave-uniform
                const int src = __ffsll((long long)todo) - 1;
                todo &= todo - 1;
                const int ss = __shfl(s, src, kWave), ee = __shfl(e, src, kWave);
                int lo = 0x7fffffff, hi = -0x7fffffff - 1;
                for (int p = ss + lane; p < ee; p += kWave) {
                    const int c = colidx[p];
                    lo = c < lo ? c : lo;
                    hi = c > hi ? c : hi;
                }
#pragma unroll
                for (int m = 1; m < kWave; m <<= 1) {
                    const int ol = __shfl_xor(lo, m, kWave), oh = __shfl_xor(hi, m, kWave);
                    lo = ol < lo ? ol : lo;
                    hi = oh > hi ? oh : hi;
                }
                if (lane == src) {
                    span += (unsigned long long)((long long)hi - lo + 1);
                    rows += 1;
                }
            }
        }
    }
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
        sq += shfl_xor_u64(sq, m);
        rows += shfl_xor_u64(rows, m);
        span += shfl_xor_u64(span, m);
        bad |= shfl_xor_u64(bad, m);
        const unsigned long long omx = shfl_xor_u64(mx, m), omn = shfl_xor_u64(mn, m);
        mx = omx > mx ? omx : mx;
        mn = omn < mn ? omn : mn;
    }
    if (lane == 0) {
        atomicAdd(&ws[0], sq);
        atomicMax(&ws[1], mx);
        atomicMin(&ws[2], mn);
        if (rows) atomicAdd(&ws[3], rows);
        if (span) atomicAdd(&ws[4], span);
        if (bad) atomicMax(&ws[5], 1ull);
        if (gw == 0) {
            ws[6] = (unsigned long long)(long long)rowptr[0];
            ws[7] = (unsigned long long)(long long)rowptr[M];
        }
    }
}

// ===========================================================================
// 64-bit row pointers: slabs of rows whose entry positions fit 32 bits
// ===========================================================================
// The kernels address entries with 32-bit positions.  A matrix with more than 2^31 stored entries is cut into
// slabs of consecutive rows: slab k starts at the first row whose pointer reaches k * slab_entries.  One thread
// per cut: out[2k] = the row, out[2k+1] = its pointer (the slab's base); cut nslabs is (M, rowptr[M]).
__global__ void i64_slab_bounds_kernel(long long M, const long long* __restrict__ rowptr, int nslabs, long long slab_entries,
                                       long long* __restrict__ out) {
    const int k = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (k > nslabs) return;
    long long r = M;
    if (k < nslabs) {
        const long long target = (long long)k * slab_entries;
        long long lo = 0, hi = M;                       // first r in [0, M] with rowptr[r] >= target
        while (lo < hi) {
            const long long mid = lo + (hi - lo) / 2;
            if (rowptr[mid] < target) lo = mid + 1; else hi = mid;
        }
        r = lo;
    }
    out[2 * k] = r;
    out[2 * k + 1] = rowptr[r];
}

// The 32-bit row pointers of one slab: out[i] = rowptr[first + i] - base for i in [0, rows].
__global__ __launch_bounds__(kBlock) void i64_slab_rowptr_kernel(long long rows, const long long* __restrict__ rowptr_first,
                                                                  long long base, int* __restrict__ out) {
    const long long nthreads = (long long)gridDim.x * kBlock;
    for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i <= rows; i += nthreads)
        out[i] = (int)(rowptr_first[i] - base);
}

// ===========================================================================
// measurement aids: pure gather, the memory side of the parallel and of the sequential kernels, plain streaming copy
// ===========================================================================

// Streams idx and gathers x[idx[i]], four independent gathers in flight per
// lane; nothing else.  One partial sum per thread keeps the loads alive.
__global__ __launch_bounds__(kBlock) void gather_probe_kernel(float* __restrict__ out, const float* __restrict__ x,
                                                               const int* __restrict__ idx, long long n) {
    const long long nthreads = (long long)gridDim.x * kBlock;
    const long long t = (long long)blockIdx.x * kBlock + threadIdx.x;
    float acc = 0.0f;
    for (long long base = t; base < n; base += nthreads * 4) {
        int c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const long long i = base + u * nthreads;
            c[u] = i < n ? stream_load(idx + i) : -1;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) acc += c[u] >= 0 ? x[c[u]] : 0.0f;
    }
    out[t] = acc;
}

// Floor of the parallel-reduction kernels: what they do to memory and nothing else.  A wave takes blocks of
// 512 consecutive entries; lane l loads entries 64 e + l (coalesced, non-temporal), gathers V dense values for
// each with one vector load and multiplies-adds them into V private sums.  The pipeline is the entry-block
// kernel's: while block b is multiplied, the gathers of block b + 1 and the entries of block b + 2 are in
// flight; arriving entries wait in a second register set and are moved over once block b is done.  No row
// bounds, no reduction across lanes, no result rows: the per-lane sums go to out[thread * V + i] so that the
// loads stay alive (and so that a test can check their total).
template <int V>
__global__ __launch_bounds__(kBlock) void stream_gather_fma_probe_kernel(float* __restrict__ out, const float* __restrict__ X,
                                                                         long long K, int ldx, const int* __restrict__ colidx,
                                                                         const float* __restrict__ vals, long long nnz) {
    constexpr int E = 8;
    constexpr long long W = kWave * E;
    const int lane = lane_id();
    const long long nwaves = (long long)gridDim.x * kWavesPerBlock;
    const long long gw = (long long)xcd_contiguous(blockIdx.x, gridDim.x) * kWavesPerBlock + wave_in_block();
    const long long nblocks = (nnz + W - 1) / W;
    const long long b0 = nblocks * gw / nwaves, b1 = nblocks * (gw + 1) / nwaves;      // my contiguous share
    const unsigned long long x_bytes = dense_bytes(K, ldx, V);
    const bool x_small = x_bytes <= 0xffffffffull;
    const __amdgpu_buffer_rsrc_t rx = make_buffer(X, x_small ? x_bytes : 0ull);
    float acc[V];
#pragma unroll
    for (int i = 0; i < V; ++i) acc[i] = 0.0f;
    int c[E], lc[E];
    float a[E], la[E], x[E][V];
    // entries of block b into the arriving set (nothing past my share or past the arrays' end: zeros, which add nothing)
    auto load_entries = [&](long long b) {
        const long long from = b * W;
        const unsigned long long bytes = (b < b1 && from < nnz) ? (unsigned long long)(nnz - from) * 4ull : 0ull;
        const __amdgpu_buffer_rsrc_t rc = make_buffer(colidx + (bytes ? from : 0), bytes);
        const __amdgpu_buffer_rsrc_t ra = make_buffer(vals + (bytes ? from : 0), bytes);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const unsigned off = (unsigned)(e * kWave + lane) * 4u;
            lc[e] = buffer_stream_i32(rc, off);
            la[e] = buffer_stream_f32(ra, off);
        }
    };
    auto take_entries = [&]() {
#pragma unroll
        for (int e = 0; e < E; ++e) { c[e] = lc[e]; a[e] = la[e]; }
    };
    // dense values for the entries in c (those of block b)
    auto gather = [&](long long b) {
        const long long left = b < b1 ? nnz - b * W : 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const bool ok = e * kWave + lane < left;
            if (x_small) {
                buffer_load_vec<V>(rx, ok ? (unsigned)c[e] * (unsigned)ldx * 4u : kOutOfRange, x[e]);
            } else {
                load_vec_dword_aligned<V>(X + (size_t)(ok ? c[e] : 0) * ldx, x[e]);
            }
        }
    };
    load_entries(b0);
    take_entries();
    load_entries(b0 + 1);
    gather(b0);
    for (long long b = b0; b < b1; ++b) {
#pragma unroll
        for (int e = 0; e < E; ++e)
#pragma unroll
            for (int i = 0; i < V; ++i) acc[i] = fmaf(a[e], x[e][i], acc[i]);
        take_entries();
        load_entries(b + 2);
        gather(b + 1);
    }
    const long long t = (long long)blockIdx.x * kBlock + threadIdx.x;
#pragma unroll
    for (int i = 0; i < V; ++i) out[t * V + i] = acc[i];
}

// Floor of the sequential-reduction kernels at width N: a wave stages 512 consecutive entries in LDS with
// coalesced loads, then each of its 64 / G lane groups walks 512 G / 64 of them in order, one dwordx4 load of the
// entry's row of X per lane and step (lane gl owns columns [block * 4 G + 4 gl, + 4)), multiply-add into four private
// sums.  No rows, no stores inside the walk.  blockIdx.y selects the block of 4 G columns.  N must be a multiple of 4.
__global__ __launch_bounds__(kBlock) void row_gather_probe_kernel(float* __restrict__ out, const float* __restrict__ X,
                                                                  long long K, int N, int ldx, const int* __restrict__ colidx,
                                                                  const float* __restrict__ vals, long long nnz, int logG) {
    constexpr int W = 512;
    __shared__ __align__(16) int s_col[kWavesPerBlock][W];
    __shared__ __align__(16) float s_val[kWavesPerBlock][W];
    const int lane = lane_id();
    const int wib = wave_in_block();
    int* cc = s_col[wib];
    float* cv = s_val[wib];
    const int G = 1 << logG;
    const int gl = lane & (G - 1), g = lane >> logG;
    const int U = W >> (6 - logG);                                   // entries per group and tile
    const long long n = (long long)blockIdx.y * 4 * G + 4 * gl;      // my first column
    const bool col_ok = n + 4 <= N;
    const long long nwaves = (long long)gridDim.x * kWavesPerBlock;
    const long long gw = (long long)xcd_contiguous(blockIdx.x, gridDim.x) * kWavesPerBlock + wib;
    const long long ntiles = (nnz + W - 1) / W;
    const long long t0 = ntiles * gw / nwaves, t1 = ntiles * (gw + 1) / nwaves;
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (long long t = t0; t < t1; ++t) {
        const long long from = t * W;
        const __amdgpu_buffer_rsrc_t rc = make_buffer(colidx + from, (unsigned long long)(nnz - from) * 4ull);
        const __amdgpu_buffer_rsrc_t ra = make_buffer(vals + from, (unsigned long long)(nnz - from) * 4ull);
        wave_lds_sync();
#pragma unroll
        for (int k = 0; k < W / kWave; ++k) {
            const int e = k * kWave + lane;
            cc[e] = buffer_stream_i32(rc, (unsigned)e * 4u);      // past the end: column 0, value 0
            cv[e] = buffer_stream_f32(ra, (unsigned)e * 4u);
        }
        wave_lds_sync();
        if (col_ok) {
            for (int e = g * U; e < (g + 1) * U; ++e) {
                float x[4];
                load_vec_dword_aligned<4>(X + (size_t)cc[e] * ldx + n, x);
                const float a = cv[e];
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[i] = fmaf(a, x[i], acc[i]);
            }
        }
    }
    const long long th = ((long long)blockIdx.y * gridDim.x + blockIdx.x) * kBlock + threadIdx.x;
#pragma unroll
    for (int i = 0; i < 4; ++i) out[th * 4 + i] = acc[i];
}

__global__ __launch_bounds__(kBlock) void copy_kernel(float* __restrict__ dst, const float* __restrict__ src,
                                                       long long n) {
    const long long nthreads = (long long)gridDim.x * kBlock;
    const long long t = (long long)blockIdx.x * kBlock + threadIdx.x;
    const long long n4 = n / 4;
    const float4* s4 = reinterpret_cast<const float4*>(src);
    float4* d4 = reinterpret_cast<float4*>(dst);
    for (long long i = t; i < n4; i += nthreads) d4[i] = s4[i];
    for (long long i = n4 * 4 + t; i < n; i += nthreads) dst[i] = src[i];
}

}  // namespace dgsp
