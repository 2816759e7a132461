// Sweep tiles (products of scattered orderings): launchers (host + device).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.h"

namespace spmvlib {

// y = A x over the handle's sweep tiles; `done` as in SpmvArgs.
template <typename V, typename T>
void launch_sweep(const DevMatrix &M, const V *val, const T *x, T *y, const int *done, hipStream_t st);

// Column and value arrays in sweep order from the CSR ones (creation only).
void launch_sweep_fill(const DevMatrix &M, int32_t *col, hipStream_t st);
template <typename V> void launch_sweep_fill_val(const DevMatrix &M, const V *csr_val, V *val, hipStream_t st);

// Opts the kernels into 160 KB of dynamic LDS (creation only: no attribute
// call happens during a capture).
hipError_t prepare_sweep_kernels();

// The values of type V in sweep order (nullptr: products of that type take
// the row tiles).
template <typename V> inline const V *sweep_values(const DevMatrix &M);
template <> inline const double *sweep_values<double>(const DevMatrix &M) { return M.sweep64; }
template <> inline const float *sweep_values<float>(const DevMatrix &M) { return M.sweep32; }
template <> inline const uint16_t *sweep_values<uint16_t>(const DevMatrix &M) { return M.sweep16; }

// Sweep tiles pay where x, of elements of type X, is well beyond an XCD's
// 4 MB L2 (row tiles -> sweep tiles, random order: binary64 x of 4.1 MB 24.6 ->
// 26.7 us, 6.9 MB 57.6 -> 49.7, 8 MB 72.4 -> 58.3; FP32 x of 4 MB 39.8 -> 47.1,
// 8 MB 119.6 -> 93.7).
constexpr int64_t kSweepMinXBytes = int64_t(6) << 20;
template <typename X> inline bool sweep_pays(int32_t n_cols) { return (int64_t)sizeof(X) * n_cols >= kSweepMinXBytes; }

}  // namespace spmvlib
