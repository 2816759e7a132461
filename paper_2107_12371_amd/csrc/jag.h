// Jagged window tiles: argument block, launchers (host + device).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.h"
#include "launch.h"

namespace spmvlib {

template <typename V, typename T> struct JagArgs {
    const int32_t *hdr;    // kJagHdr ints per slice
    const uint16_t *slot;  // per tile and lane: row length << 8 | row in the tile
    const int32_t *sect;   // `stride` window sectors per tile
    const uint32_t *pos;   // 12-bit window positions, 8 per three words
    const V *val;
    const T *x;
    T *y;
    const T *b;            // EPI_RESID: right-hand side
    double *part;          // EPI_DOT / EPI_RESID: one partial per tile
    const int *done;       // optional: non-zero makes the launch a no-op (CG)
    int32_t n_tiles, per_xcd, chunk_log2, stride, n_cols;
};

// y = A x (or its epilogues) over the handle's jagged tiles; partial t of
// EPI_DOT / EPI_RESID belongs to tile t.
template <typename V, typename T>
void launch_jag(const DevMatrix &M, const V *val, const SpmvArgs<V, T, T> &g, int epi, hipStream_t st);

// Fills pos, and one value array, of a handle whose headers, slots and
// sectors are resident, from its CSR arrays (creation only).
void launch_jag_fill_pos(const DevMatrix &M, uint32_t *pos, hipStream_t st);
template <typename V> void launch_jag_fill_val(const DevMatrix &M, const V *csr_val, V *val, hipStream_t st);

// The jagged copy of the values of type V (nullptr: products of that type
// take the handle's row tiles).
template <typename V> inline const V *jag_values(const DevMatrix &M);
template <> inline const double *jag_values<double>(const DevMatrix &M) { return M.jag64; }
template <> inline const float *jag_values<float>(const DevMatrix &M) { return M.jag32; }
template <> inline const uint16_t *jag_values<uint16_t>(const DevMatrix &M) { return M.jag16; }

// Partials an EPI_DOT / EPI_RESID product with values of type V leaves.
template <typename V> inline int32_t n_partials(const DevMatrix &M) {
    return jag_values<V>(M) ? M.n_jag + M.n_jag_rest + M.n_long : M.n_seg;
}

}  // namespace spmvlib
