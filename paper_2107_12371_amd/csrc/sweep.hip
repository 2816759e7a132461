// Sweep tiles: products of matrices whose ordering scatters the columns.
//
// With columns spread over all of x (a mesh numbered as its generator left
// it) every gather touches a cache line of its own, and the row tiles fetch
// one 128-byte line from beyond L2 for nearly every stored entry: that
// traffic, 7 times the matrix, bounds them.  Here a workgroup works up to
// 20,480 entries of consecutive rows, its products filling one CU's LDS, in
// ascending order of column, so that all workgroups of an XCD, which start
// together and advance at one rate, sweep over x side by side and a line
// that one of them brings into the XCD's L2 serves the others before it is
// dropped.  Entries carry their place in the tile (16 bits); after a barrier
// the products are summed row by row in CSR order, each rounded before it is
// added: the row tiles' sums, same bits.  The tiles fill whole rounds of one
// workgroup per CU, so that no round is nearly empty.
// Measured, row tiles -> sweep tiles, FP64, random order, three matrices in
// turn: kNN mesh of 1M rows 71.3 -> 54.7 us, 2M rows 181 -> 112 us, 8M rows
// 907 -> 696 us; 27-point mesh of 1M rows 173 -> 120 us, 4M rows 1,106 -> 723
// us.  Tiles of 16,384 / 8,192 / 4,096 entries took 122 / 143 / 175 us on the 2M
// rows (fewer entries swept together); one persistent workgroup per CU,
// loading the next tile behind the row sums, was equal.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "device.h"
#include "sweep.h"
#include "tile.h"

namespace spmvlib {

constexpr int kSweepLanes = 1024;
constexpr int kSweepBatch = 4;  // entries a lane gathers at once (1, 2, 5: within 4% on up to 2M rows)

template <typename T> __device__ __forceinline__ T add_each(T sum, T p) { return sum + p; }

template <typename V, typename T>
__global__ __launch_bounds__(kSweepLanes) void k_sweep(const TileDesc *__restrict__ desc, int n_tiles, int per_xcd,
                                                       int chunk_log2, const int32_t *__restrict__ row_ptr,
                                                       const int32_t *__restrict__ col,
                                                       const uint16_t *__restrict__ place,
                                                       const V *__restrict__ val, const T *__restrict__ x,
                                                       T *__restrict__ y, const int *__restrict__ done) {
    extern __shared__ __align__(16) unsigned char smem[];
    T *prod = reinterpret_cast<T *>(smem);
    const int li = xcd_tile(blockIdx.x, per_xcd, chunk_log2);
    if (li >= n_tiles) return;
    const TileDesc d = desc[li];
    if (done && *done) return;
    constexpr int kBatches = kSweepTile / (kSweepLanes * kSweepBatch);
    static_assert(kBatches * kSweepLanes * kSweepBatch == kSweepTile, "whole batches");
    const int tid = (int)threadIdx.x, n = d.e - d.s;
    const int last = max(n - 1, 0);  // the arrays are padded, so an empty tile reads a valid word
    int32_t c[kSweepBatch];
    V v[kSweepBatch];
    unsigned at[kSweepBatch];
    // the stream is read once: non-temporal, so that it leaves L2 to x
    const auto load = [&](int b) {
#pragma unroll
        for (int u = 0; u < kSweepBatch; ++u)
            c[u] = __builtin_nontemporal_load(col + d.s + min((b * kSweepBatch + u) * kSweepLanes + tid, last));
#pragma unroll
        for (int u = 0; u < kSweepBatch; ++u) {
            const int i = d.s + min((b * kSweepBatch + u) * kSweepLanes + tid, last);
            v[u] = __builtin_nontemporal_load(val + i);
            at[u] = __builtin_nontemporal_load(place + i);
        }
    };
    load(0);
#pragma unroll
    for (int b = 0; b < kBatches; ++b) {
        if (b * kSweepBatch * kSweepLanes >= n) break;  // the same for every lane
        T xv[kSweepBatch], vv[kSweepBatch];
        unsigned to[kSweepBatch];
#pragma unroll
        for (int u = 0; u < kSweepBatch; ++u) xv[u] = x[c[u]];
#pragma unroll
        for (int u = 0; u < kSweepBatch; ++u) {
            vv[u] = to_acc<T>(v[u]);
            to[u] = at[u];
        }
        if (b + 1 < kBatches) load(b + 1);  // behind the gathers
#pragma unroll
        for (int u = 0; u < kSweepBatch; ++u)
            if ((b * kSweepBatch + u) * kSweepLanes + tid < n) prod[to[u]] = vv[u] * xv[u];
    }
    __syncthreads();
    for (int r = d.r0 + tid; r < d.r1; r += kSweepLanes) {
        const int a = row_ptr[r] - d.s, z = row_ptr[r + 1] - d.s;
        T sum = T(0);
        int k = a;
        // one lane's chain of LDS reads and adds: a row of 2,000 entries takes
        // 21 us read by fours and 9.5 by sixteens, with the CU waiting for it
        for (; k + 16 <= z; k += 16) {
            T q[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) q[u] = prod[k + u];
#pragma unroll
            for (int u = 0; u < 16; ++u) sum = add_each(sum, q[u]);
        }
        for (; k + 4 <= z; k += 4) {
            T q[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) q[u] = prod[k + u];
#pragma unroll
            for (int u = 0; u < 4; ++u) sum = add_each(sum, q[u]);
        }
        for (; k < z; ++k) sum = add_each(sum, prod[k]);
        __builtin_nontemporal_store(sum, y + r);
    }
}

// entry i of tile [s, e) in sweep order is CSR entry s + place[i]
__global__ __launch_bounds__(kBlock) void k_sweep_fill(const TileDesc *__restrict__ desc,
                                                       const uint16_t *__restrict__ place,
                                                       const int32_t *__restrict__ csr_col,
                                                       int32_t *__restrict__ col) {
    const TileDesc d = desc[blockIdx.x];
    for (int i = d.s + (int)threadIdx.x; i < d.e; i += kBlock) col[i] = csr_col[d.s + place[i]];
}

template <typename V>
__global__ __launch_bounds__(kBlock) void k_sweep_fill_val(const TileDesc *__restrict__ desc,
                                                           const uint16_t *__restrict__ place,
                                                           const V *__restrict__ csr_val, V *__restrict__ val) {
    const TileDesc d = desc[blockIdx.x];
    for (int i = d.s + (int)threadIdx.x; i < d.e; i += kBlock) val[i] = csr_val[d.s + place[i]];
}

template <typename V, typename T>
void launch_sweep(const DevMatrix &M, const V *val, const T *x, T *y, const int *done, hipStream_t st) {
    const int per_xcd = M.xcd_remap && M.n_sweep >= 16 ? (M.n_sweep + 7) / 8 : 0;
    const int grid = xcd_grid(M.n_sweep, per_xcd, -1);
    const size_t lds = sizeof(T) * (size_t)std::max(M.sweep_width, 1);
    hipLaunchKernelGGL((k_sweep<V, T>), dim3(grid), dim3(kSweepLanes), lds, st, M.sweep_desc, M.n_sweep, per_xcd, -1,
                       M.row_ptr, M.sweep_col, M.sweep_place, val, x, y, done);
}

void launch_sweep_fill(const DevMatrix &M, int32_t *col, hipStream_t st) {
    hipLaunchKernelGGL(k_sweep_fill, dim3(M.n_sweep), dim3(kBlock), 0, st, M.sweep_desc, M.sweep_place, M.col, col);
}

template <typename V> void launch_sweep_fill_val(const DevMatrix &M, const V *csr_val, V *val, hipStream_t st) {
    hipLaunchKernelGGL((k_sweep_fill_val<V>), dim3(M.n_sweep), dim3(kBlock), 0, st, M.sweep_desc, M.sweep_place,
                       csr_val, val);
}

template <typename V, typename T> static hipError_t opt_in() {
    return hipFuncSetAttribute(reinterpret_cast<const void *>(&k_sweep<V, T>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, kSweepTile * (int)sizeof(T));
}

hipError_t prepare_sweep_kernels() {
    hipError_t e = opt_in<double, double>();
    if (e == hipSuccess) e = opt_in<float, float>();
    if (e == hipSuccess) e = opt_in<float, double>();
    if (e == hipSuccess) e = opt_in<uint16_t, float>();
    return e;
}

template void launch_sweep<double, double>(const DevMatrix &, const double *, const double *, double *, const int *,
                                           hipStream_t);
template void launch_sweep<float, float>(const DevMatrix &, const float *, const float *, float *, const int *,
                                         hipStream_t);
template void launch_sweep<float, double>(const DevMatrix &, const float *, const double *, double *, const int *,
                                          hipStream_t);
template void launch_sweep<uint16_t, float>(const DevMatrix &, const uint16_t *, const float *, float *, const int *,
                                            hipStream_t);
template void launch_sweep_fill_val<double>(const DevMatrix &, const double *, double *, hipStream_t);
template void launch_sweep_fill_val<float>(const DevMatrix &, const float *, float *, hipStream_t);
template void launch_sweep_fill_val<uint16_t>(const DevMatrix &, const uint16_t *, uint16_t *, hipStream_t);

}  // namespace spmvlib
