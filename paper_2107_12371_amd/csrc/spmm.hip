// Y = A X for a scalar CSR handle with k right-hand sides, X and Y row-major
// (the k values of one row contiguous), so one gather of X's row c brings
// all the columns a lane works on.
//
// One workgroup per tile of up to 1,024 or 2,048 stored entries (the rows
// outside the handle's long rows, whatever kernel its plan gives the
// single-vector product).  The tile's values, column indices and row bounds are
// staged in LDS with coalesced loads; then the lanes take (row, column group)
// tasks: a lane walks its row's entries in ascending order, U entries per round
// with all their gathers of KC adjacent values of X issued before any is used,
// and adds
// the rounded products one by one starting from zero, exactly as the
// single-vector product sums a row, so column j of Y equals the
// single-vector product of column j of X bit for bit.  A row longer than a
// tile is summed as the single-vector product sums it (pieces of 16,384
// entries): one workgroup per (piece, column) with the pieces' sums in Y's
// rows of the longest run without a long row, or, without room there, one
// workgroup per (row, column) walking the pieces.
// The values are read once for all k columns, which is what the batched
// requests of a serving workload need.  One column goes to the
// single-vector product.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "device.h"
#include "launch.h"
#include "spmm.h"
#include "tile.h"

namespace spmvlib {

__device__ __forceinline__ double add_rounded_product(double sum, double a, double b) {
#pragma clang fp contract(off)
    const double p = a * b;
    return sum + p;
}

// KC adjacent columns j0.. of row c of X (clamped into the row: columns at
// or beyond k read a valid word and are discarded by the caller); VEC: k is
// even and X 16-byte aligned, so pairs of columns move in 16-byte pieces.
template <int KC, bool VEC>
__device__ __forceinline__ void load_cols(const double *__restrict__ xr, int j0, int k, double (&o)[KC]) {
    if constexpr (VEC && KC >= 2) {
        typedef double d2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int p = 0; p < KC / 2; ++p) {
            const d2 v = *reinterpret_cast<const d2 *>(xr + min(j0 + 2 * p, k - 2));
            o[2 * p] = v[0];
            o[2 * p + 1] = v[1];
        }
    } else {
#pragma unroll
        for (int j = 0; j < KC; ++j) o[j] = xr[min(j0 + j, k - 1)];
    }
}

// KC adjacent columns of entries q .. q + U - 1 of a row that ends at z,
// gathered together, then added in ascending order.  TAIL: entries past z
// re-read the last one and are discarded by a select.  OFF32: sc holds byte
// offsets of X's rows (X under 4 GB), else column numbers.
template <int KC, int U, bool VEC, bool OFF32, bool TAIL>
__device__ __forceinline__ void add_entries(const double *sv, const uint32_t *sc, int q, int z,
                                            const double *__restrict__ X, int j0, int k, double (&acc)[KC]) {
    double v[U], xv[U][KC];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int qq = TAIL ? min(q + u, z - 1) : q + u;
        v[u] = sv[qq];
        const double *xr = OFF32 ? reinterpret_cast<const double *>(reinterpret_cast<const char *>(X) + sc[qq])
                                 : X + (size_t)sc[qq] * k;
        load_cols<KC, VEC>(xr, j0, k, xv[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < KC; ++j) {
            const double s = add_rounded_product(acc[j], v[u], xv[u][j]);
            acc[j] = !TAIL || q + u < z ? s : acc[j];
        }
}

// How a pair of columns of Y leaves: word by word (k odd, or Y not 16-byte
// aligned), in one 16-byte store, or in one past L2.
enum YStore : int { Y_WORDS, Y_PIECES, Y_PIECES_NT };

// Tasks are (row, group of KC columns); a lane takes U entries of its row per
// round.  What bounds it: the L1s, whose gathers of adjacent rows wait for the
// same lines (16M rows, k = 8: a line looked up in 51% of the cycles, stalled on
// lines under way in 39%), and the rounds' latencies.  So a tile is about one task per lane,
// the row bounds are staged with the entries, the rounds but the last need
// neither clamps nor selects, and rows keep their order: sorted by length they
// take fewer rounds, but adjacent rows share lines (4M-row 27-point mesh, k = 8:
// 436 us).  A shorter last round (U / 2 where that is enough) costs more than
// the gathers it saves: 419 us.  Y leaves in non-temporal 16-byte stores, or it
// evicts X (416 us without), and so does a stream that no cache holds
// for the next product (`stream_nt`).  Measured, 4M-row 27-point mesh / 4M-row
// kNN mesh: k = 2 228 -> 222 / 159 -> 131, k = 8 414 -> 399 / 306 -> 247, k = 16
// 675 -> 624 / 489 -> 396 us; the least traffic of the first at k = 8 takes 189.
template <int KC, int U, bool VEC, bool OFF32, YStore YS>
__global__ __launch_bounds__(kBlock) void k_spmm_tiles(const TileDesc *__restrict__ desc, int n_list, int per_xcd,
                                                       int chunk_log2,
                                                       const int32_t *__restrict__ row_ptr,
                                                       const int32_t *__restrict__ col,
                                                       const double *__restrict__ val, const double *__restrict__ X,
                                                       double *__restrict__ Y, int k, int cap, int stream_nt) {
    extern __shared__ __align__(16) unsigned char smem[];
    double *sv = reinterpret_cast<double *>(smem);
    uint32_t *sc = reinterpret_cast<uint32_t *>(sv + cap);
    __shared__ int32_t srow[kSpmmRows + 1];
    const int li = xcd_tile(blockIdx.x, per_xcd, chunk_log2);
    if (li >= n_list) return;
    const TileDesc d = desc[li];
    const int n = min(d.e - d.s, cap);  // the host sizes cap to the largest tile
    const auto stage = [&](auto load) {
        for (int i = (int)threadIdx.x; i < n; i += kBlock) {
            sv[i] = load(val + d.s + i);
            const uint32_t c = (uint32_t)load(col + d.s + i);
            sc[i] = OFF32 ? c * (uint32_t)(sizeof(double) * k) : c;
        }
    };
    if (stream_nt) stage([](auto *q) { return __builtin_nontemporal_load(q); });
    else stage([](auto *q) { return *q; });
    for (int i = (int)threadIdx.x; i <= d.r1 - d.r0; i += kBlock) srow[i] = min(row_ptr[d.r0 + i] - d.s, n);
    __syncthreads();
    const int groups = (k + KC - 1) / KC;
    const int tasks = (d.r1 - d.r0) * groups;
    for (int t = (int)threadIdx.x; t < tasks; t += kBlock) {
        const int i = t / groups, j0 = (t - i * groups) * KC;
        const int z = srow[i + 1];
        int q = srow[i];
        double acc[KC];
#pragma unroll
        for (int j = 0; j < KC; ++j) acc[j] = 0.0;
        for (; q + U <= z; q += U) add_entries<KC, U, VEC, OFF32, false>(sv, sc, q, z, X, j0, k, acc);
        if (q < z) add_entries<KC, U, VEC, OFF32, true>(sv, sc, q, z, X, j0, k, acc);
        double *__restrict__ yr = Y + (size_t)(d.r0 + i) * k + j0;
        if constexpr (YS != Y_WORDS) {
            static_assert(KC == 2, "one 16-byte store");
            typedef double d2 __attribute__((ext_vector_type(2)));
            if constexpr (YS == Y_PIECES_NT) __builtin_nontemporal_store(d2{acc[0], acc[1]}, reinterpret_cast<d2 *>(yr));
            else *reinterpret_cast<d2 *>(yr) = d2{acc[0], acc[1]};
        } else {
#pragma unroll
            for (int j = 0; j < KC; ++j)
                if (j0 + j < k) yr[j] = acc[j];
        }
    }
}

// Row d.r0 (longer than a tile), column blockIdx.y: the single-vector
// long-row sum (its pieces in order) with x read from column j of X.
__global__ __launch_bounds__(kBlock) void k_spmm_long(const TileDesc *__restrict__ desc,
                                                      const int32_t *__restrict__ col,
                                                      const double *__restrict__ val, const double *__restrict__ X,
                                                      double *__restrict__ Y, int k) {
    __shared__ double sh[kBlock / kWave];
    const TileDesc d = desc[blockIdx.x];
    const int j = (int)blockIdx.y;
    const auto gx = [X, k, j](int c) { return X[(size_t)c * k + j]; };
    double tot = 0.0;
    for (int ps = d.s; ps < d.e; ps += kLongPiece) {
        const double t = long_piece_sum<double>(val, col, ps, min(d.e, ps + kLongPiece), gx, sh);
        tot = ps == d.s ? t : tot + t;
        __syncthreads();
    }
    if (threadIdx.x == 0) Y[(size_t)d.r0 * k + j] = tot;
}

// Several workgroups per long row: one per (piece, column), its sum to
// ws[piece * k + column] ...
__global__ __launch_bounds__(kBlock) void k_spmm_long_pieces(const TileDesc *__restrict__ desc,
                                                             const int32_t *__restrict__ piece_long,
                                                             const int32_t *__restrict__ piece_ptr,
                                                             const int32_t *__restrict__ col,
                                                             const double *__restrict__ val,
                                                             const double *__restrict__ X, double *__restrict__ ws,
                                                             int k) {
    __shared__ double sh[kBlock / kWave];
    const int pc = (int)blockIdx.x, j = (int)blockIdx.y;
    const int li = piece_long[pc];
    const TileDesc d = desc[li];
    const int ps = d.s + (pc - piece_ptr[li]) * kLongPiece;
    const auto gx = [X, k, j](int c) { return X[(size_t)c * k + j]; };
    const double t = long_piece_sum<double>(val, col, ps, min(d.e, ps + kLongPiece), gx, sh);
    if (threadIdx.x == 0) ws[(size_t)pc * k + j] = t;
}

// ... then one wavefront per (long row, column) adds them in piece order,
// 64 sums per load round trip, as the single-vector combine does.
__global__ __launch_bounds__(kBlock) void k_spmm_long_combine(const TileDesc *__restrict__ desc,
                                                              const int32_t *__restrict__ piece_ptr,
                                                              const double *__restrict__ ws, double *__restrict__ Y,
                                                              int n_long, int k) {
    const int li = (int)(blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave);
    if (li >= n_long) return;  // the same for every lane of the wavefront
    const int j = (int)blockIdx.y;
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int p0 = piece_ptr[li], p1 = piece_ptr[li + 1];
    double tot = 0.0;
    for (int b = p0; b < p1; b += kWave) {
        const int n = min(kWave, p1 - b);
        const double v = lane < n ? ws[(size_t)(b + lane) * k + j] : 0.0;
        for (int i = 0; i < n; ++i) {
            const double w = __shfl(v, i, kWave);
            tot = b == p0 && i == 0 ? w : tot + w;
        }
    }
    if (lane == 0) Y[(size_t)desc[li].r0 * k + j] = tot;
}

constexpr size_t kL2Bytes = (size_t)32 << 20;  // the eight XCDs' L2s together
static size_t matrix_bytes(const DevMatrix &M) { return (sizeof(double) + sizeof(int32_t)) * (size_t)M.nnz; }

template <int KC, int U>
static void launch_tiles(const DevMatrix &M, const double *X, double *Y, int k, hipStream_t st) {
    // the larger tiles where a mean small one has tasks for half the lanes at
    // most (4M-row 27-point mesh: k = 2 222 us, 228 with the small ones; k = 4
    // 282 / 292; one workgroup of half the lanes per small tile: 258 / 305)
    const int64_t tasks = (int64_t)M.n_rows / M.spmm[0].n * ((k + KC - 1) / KC);
    const SpmmTiles &T = M.spmm[tasks <= kBlock / 2 ? 1 : 0];
    const int per_xcd = M.xcd_remap && T.n >= 16 ? (T.n + 7) / 8 : 0;
    const int chunk_log2 = M.xcd_chunk_log2;
    const int grid = xcd_grid(T.n, per_xcd, chunk_log2);
    const size_t lds = (size_t)T.entries * (sizeof(double) + sizeof(uint32_t));
    // X's alignment alone decides how X is gathered: with Y one word off, 4M-row
    // 27-point mesh k = 8 takes 420 us, and 548 with X gathered word by word
    const bool vec = KC >= 2 && k % 2 == 0 && (reinterpret_cast<uintptr_t>(X) & 15) == 0;
    const bool pieces = vec && (reinterpret_cast<uintptr_t>(Y) & 15) == 0;
    const size_t x_bytes = sizeof(double) * (size_t)M.n_cols * (size_t)k;
    const bool off32 = x_bytes < ((size_t)1 << 32);
    // Y past L2, but for the smallest (49K-row tet mesh k = 2 3.16 us ordinary,
    // 3.31 non-temporal, k = 8 4.97 / 4.80; 125K-row kNN mesh k = 8 7.5 / 6.6; 1M-row
    // 27-point mesh k = 8 104 / 81)
    const size_t y_bytes = sizeof(double) * (size_t)M.n_rows * (size_t)k;
    const bool y_nt = pieces && y_bytes >= ((size_t)2 << 20);
    // The stream goes past the caches where they cannot keep it for the next
    // product on the handle: from 272 MB of matrix, X and a Y that passes
    // through them on, a little over the 256 MB memory-side cache (one matrix,
    // ordinary / non-temporal loads: 1M-row 27-point mesh k = 2 47 / 60 us, k = 8
    // (256 MB) 81 / 100, k = 12 (287 MB) 148 / 146; 2M-row kNN mesh k = 4 (226 MB) 51 / 72,
    // k = 5 (313 MB) 117 / 108, k = 8 (287 MB) 116 / 106; 4M-row 27-point mesh k = 8
    // 398 / 389).  And where an XCD's L2 would hold its share of X but
    // for its share of the matrix: where the L2s hold the matrix alone (262K-row
    // kNN mesh, 21 MB, k = 2 5.9 / 7.7, k = 8 13.9 / 12.0; 125K-row 27-point mesh, 25 MB,
    // k = 4 7.9 / 8.0, k = 8 12.3 / 11.5; 512K-row kNN mesh, 40 MB, k = 8 23.2 / 29.3), or
    // each XCD gathers from all of a small X (random order: 125K-row kNN mesh k = 2
    // 6.3 / 7.7, k = 3 10.5 / 9.7; 125K-row 27-point mesh k = 2 14.7 / 13.1; 512K rows k = 2,
    // X of 8 MB, 85 / 79, k = 3 120 / 120; 125K-row kNN mesh with 3 long rows k = 3
    // 26.6 / 18.5).
    const size_t matrix = matrix_bytes(M), share = matrix / 8 + (M.x_spread ? x_bytes : x_bytes / 8);
    const int stream_nt = matrix + x_bytes + (y_nt ? 0 : y_bytes) > ((size_t)272 << 20) ||
                          (share > kL2Bytes / 8 && (M.x_spread ? x_bytes <= ((size_t)12 << 20) : matrix <= kL2Bytes));
    const auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(kBlock), lds, st, T.desc, T.n, per_xcd, chunk_log2,
                           M.row_ptr, M.col, M.val64, X, Y, k, T.entries, stream_nt);
    };
    if (y_nt && off32) go(k_spmm_tiles<KC, U, true, true, Y_PIECES_NT>);
    else if (pieces && off32) go(k_spmm_tiles<KC, U, true, true, Y_PIECES>);
    else if (pieces) go(k_spmm_tiles<KC, U, true, false, Y_PIECES_NT>);  // X of 4 GB and more
    else if (vec && off32) go(k_spmm_tiles<KC, U, true, true, Y_WORDS>);
    else if (vec) go(k_spmm_tiles<KC, U, true, false, Y_WORDS>);
    else if (off32) go(k_spmm_tiles<KC, U, false, true, Y_WORDS>);
    else go(k_spmm_tiles<KC, U, false, false, Y_WORDS>);
}

hipError_t launch_spmm(const spmv_matrix *A, const double *X, double *Y, int k, hipStream_t st) {
    const DevMatrix &M = A->M;
    // one column: the single-vector product itself (compact windows where
    // the plan has them), which is the same sum
    if (k == 1) return launch_spmv<double, double, double, double>(M, M.val64, X, Y, EPI_PLAIN, nullptr, nullptr,
                                                                   nullptr, st);
    if (M.n_long > 0) {
        // first: the pieces' sums can live in Y's rows of the longest run
        // without a long row, which the row tiles below write afterwards
        if (M.piece_long && M.long_split && M.y_ws_rows >= M.n_long_pieces) {
            double *ws = Y + (size_t)M.y_ws_row * k;
            hipLaunchKernelGGL(k_spmm_long_pieces, dim3(M.n_long_pieces, k), dim3(kBlock), 0, st, M.long_desc,
                               M.piece_long, M.long_piece_ptr, M.col, M.val64, X, ws, k);
            constexpr int kRowsPerWg = kBlock / kWave;
            hipLaunchKernelGGL(k_spmm_long_combine, dim3((M.n_long + kRowsPerWg - 1) / kRowsPerWg, k), dim3(kBlock), 0,
                               st, M.long_desc, M.long_piece_ptr, ws, Y, M.n_long, k);
        } else {
            hipLaunchKernelGGL(k_spmm_long, dim3(M.n_long, k), dim3(kBlock), 0, st, M.long_desc, M.col, M.val64, X,
                               Y, k);
        }
    }
    if (M.spmm[0].n > 0) {
        // two columns per lane for every k: the lanes sharing a row gather
        // its X row in 16-byte pieces side by side, so one gather
        // instruction touches half as many cache lines as with four
        // columns per lane (16M-row mesh matrix, k = 4 / 8 / 16: 1.10 /
        // 1.65 / 2.69 ms against 1.32 / 1.87 / 2.86 ms)
        // Eight entries per round where the matrix is larger than the L2s, its
        // mean row has two such rounds and columns come in pairs, else four
        // (4M-row 27-point mesh k = 8 389 us with eight, 402 with four; 262K rows,
        // 56 MB, k = 2 16.4 / 17.7, k = 3 25.2 / 24.4, k = 8 22.4 / 22.9; 125K rows, 26 MB,
        // k = 2 7.0 / 5.9, k = 8 13.1 / 12.3; 4M-row kNN mesh, 7 entries per row, k = 8
        // 254 / 236); where each XCD gathers from all of x, only for matrices that
        // stream from HBM (512K-row 27-point mesh in random order k = 2 86 / 80).
        const bool large = M.x_spread ? M.xcd_chunk_log2 >= 0 : matrix_bytes(M) > kL2Bytes;
        if (k % 2 == 0 && large && M.nnz >= 16 * (int64_t)M.n_rows)
            launch_tiles<2, 8>(M, X, Y, k, st);
        else launch_tiles<2, 4>(M, X, Y, k, st);
    }
    return hipGetLastError();
}

}  // namespace spmvlib
