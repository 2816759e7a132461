// Jagged window tiles: the compact-window product laid out by rows.
//
// A tile is up to 256 consecutive rows, one per lane of a workgroup, sorted
// by length within the tile and cut into four slices of 64 (a wavefront
// each).  A slice stores its entries jagged: the first entries of its rows,
// then the second entries of the rows that have one, and so on, so lane l
// finds entry j of its row at (start of run j) + l, the loads of a wavefront
// are contiguous and nothing is padded.  The tile's x words are staged in
// LDS as the sectors of 8 words it touches (at most 512), and an entry
// carries its 12-bit position there.  A lane adds its row's products in
// ascending order in a register, each product rounded first, which is the
// sum the row tiles form: same bits.
//
// What bounds it: the stream (9.6 bytes per entry in FP64, 5.6 and 3.6 in
// FP32 and BF16) once enough of it is in flight, so the kernel is built
// around its chain of memory round trips.  A slice's header (scalar loads)
// carries the runs' lengths, and headers, slots and sectors lie at addresses
// known from the tile's number: one round trip.  Then the sectors' x words
// go straight to LDS (16 bytes per lane, no registers) and every position
// and value load of the slice goes out behind them: the second round trip.
// The rest is LDS reads and adds.  The row tiles (k_stream, k_cwin) need
// three round trips and move products through LDS: on the 16M-row 27-point
// mesh in FP32 k_cwin issues 26.5 vector instructions per entry and lane, this
// kernel 11.9 (on short rows it issues the more, 21.6 against k_stream's 13.7 on
// the kNN mesh in FP64, and is faster all the same).  A
// version that took the runs' lengths from the lanes (four round trips) was
// 8-10% slower.  The slices of a tile share a window because a wider tile
// needs fewer words per row: 128 rows per tile were 5-9% slower, 512 rows
// within 1.5% (and their windows pass 4,096 words on the 27-point mesh).
// Non-temporal value loads were slower (a run's ends share their cache lines
// with the next run), non-temporal y stores 2-4% faster, also where a solver's
// next kernel reads y: the BF16 polynomial's product, solves on 91K to 8M rows,
// within 1% either way (and so for the sweep tiles).
// Measured, row tiles -> jagged tiles, three matrices in turn: kNN mesh, 2M
// rows, FP64 42.1 -> 35.5 us; 27-point mesh, 4M rows, FP32 81.0 -> 77.7 us
// and BF16 73.2 -> 68.0 us; one matrix kept in cache, 1M rows of the 27-point
// mesh, FP64 / FP32 / BF16 33.9 / 30.1 / 26.2 -> 28.5 / 17.6 / 16.2 us.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "device.h"
#include "jag.h"
#include "launch.h"
#include "tile.h"

namespace spmvlib {

template <typename A> __device__ __forceinline__ A add_rounded(A sum, A a, A b) {
#pragma clang fp contract(off)
    const A p = a * b;
    return sum + p;
}

// Entries in run j of a slice: byte j of the header's eight count words.
__device__ __forceinline__ int run_len(const int32_t (&c)[8], int j) {
    return (int)(((uint32_t)c[j >> 2] >> (8 * (j & 3))) & 0xffu);
}

// Keeps a uniform value in a scalar register: the run addresses are then a
// scalar base plus the lane's offset (the compiler otherwise chains them
// through vector adds).
__device__ __forceinline__ int scalar(int v) {
    asm("" : "+s"(v));
    return v;
}

// 16 or 4 bytes of every lane from its own address straight to LDS, where the
// lanes' pieces follow each other from dst (the same for the wavefront) on.
typedef const __attribute__((address_space(1))) void GlobalPtr;
typedef __attribute__((address_space(3))) void LdsPtr;
__device__ __forceinline__ void to_lds16(const void *src, void *dst) {
    __builtin_amdgcn_global_load_lds((GlobalPtr *)src, (LdsPtr *)dst, 16, 0, 0);
}
__device__ __forceinline__ void to_lds4(const void *src, void *dst) {
    __builtin_amdgcn_global_load_lds((GlobalPtr *)src, (LdsPtr *)dst, 4, 0, 0);
}

// Position M (0..7) of the 8 packed in three words.
template <int M> __device__ __forceinline__ unsigned pos12(uint32_t w0, uint32_t w1, uint32_t w2) {
    if constexpr (M < 5) return (unsigned)(((uint64_t)w0 | ((uint64_t)w1 << 32)) >> (12 * M)) & 0xfffu;
    else return (unsigned)(((uint64_t)w1 | ((uint64_t)w2 << 32)) >> (12 * M - 32)) & 0xfffu;
}

// G: groups of 4 entries the longest row of the handle's tiles has (the
// registers a lane holds its row in).  X16: x is 16-byte aligned; any other x
// has a kernel of its own, which the aligned one does not pay for (as a branch
// it did: FP32, 2M-row kNN mesh, 16.8 -> 17.7 us).  x one word off, staged word by
// word through registers -> in steps of 4 bytes straight to LDS: 4M-row 27-point
// mesh FP32 / BF16 / binary64 with FP32 values 101 / 103 / 131 -> 79 / 67 / 97 us (the
// row tiles 82 / 74 / 99).
template <typename V, typename T, int G, int EPI, bool X16>
__global__ __launch_bounds__(kJagRows) void k_jag(JagArgs<V, T> g) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double sh[kJagRows / kWave];
    T *win = reinterpret_cast<T *>(smem);
    const int li = xcd_tile(blockIdx.x, g.per_xcd, g.chunk_log2);
    if (li >= g.n_tiles) return;
    const int tid = (int)threadIdx.x, lane = tid & (kWave - 1);
    const unsigned ul = threadIdx.x & (kWave - 1);  // unsigned: scalar base + lane offset addresses
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    constexpr int kWaves = kJagRows / kWave;
    constexpr int kPiece = 16 / (int)sizeof(T);        // words a lane stages at once
    constexpr int kLanes = kJagSector / kPiece;        // lanes per sector
    constexpr int kSpp = kWave / kLanes;               // sectors a wavefront stages per pass
    constexpr int kPpr = kWave / kSpp;                 // passes per register of sector numbers
    constexpr int kRegs = kJagMaxSectors / kWaves / kWave;
    // first round trip: sectors and slot (vector loads), header (scalar)
    int sr[kRegs];
    const int32_t *__restrict__ sect = g.sect + (size_t)li * g.stride;
#pragma unroll
    for (int k = 0; k < kRegs; ++k)
        sr[k] = sect[min(((k * kPpr + lane / kSpp) * kWaves + wave) * kSpp + lane % kSpp, g.stride - 1)];
    const unsigned slot = g.slot[(size_t)li * kJagRows + tid];
    const int32_t *__restrict__ h = g.hdr + ((size_t)li * kWaves + wave) * kJagHdr;
    int vb = h[0], pb = h[1];
    const int ns = h[2], r0 = h[3], nr = h[4];
    const bool whole = h[5] == 0;
    int32_t cnt[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) cnt[i] = h[8 + i];
    if (g.done && *g.done) return;
    // second round trip: x to LDS, then the slice's stream
    if (whole) {
#pragma unroll
        for (int i = 0; i < kRegs * kPpr; ++i) {
            const int base = (i * kWaves + wave) * kSpp;
            if (base < ns) {
                if constexpr (X16) {
                    const int s = __shfl(sr[i / kPpr], (i % kPpr) * kSpp + lane / kLanes, kWave);
                    const T *src = g.x + (size_t)s * kJagSector + (lane % kLanes) * kPiece;
                    to_lds16(src, win + base * kJagSector);
                } else {  // the same pass in four steps of 4 bytes per lane
                    constexpr int kBytes = kJagSector * (int)sizeof(T), kStep = 4 * kWave / kBytes;  // sectors a step
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int at = (i % kPpr) * kSpp + j * kStep + lane / (kBytes / 4);
                        const int s = __shfl(sr[i / kPpr], at, kWave);
                        to_lds4(reinterpret_cast<const char *>(g.x) + (size_t)s * kBytes + lane % (kBytes / 4) * 4,
                                win + (base + j * kStep) * kJagSector);
                    }
                }
            }
        }
    } else {
        // a sector that reaches past x's end: one word at a time, columns
        // clamped into x
        for (int w = tid; w < ns * kJagSector; w += kJagRows)
            win[w] = g.x[min(sect[w / kJagSector] * kJagSector + w % kJagSector, g.n_cols - 1)];
    }
    // A group of 4 runs that are all full (the common one, the rows being
    // sorted) takes fixed offsets and no selects.  Lanes past a shorter run
    // read on into the next one (the arrays carry a wavefront of padding)
    // and drop what they read.
    V v[4 * G];
    uint32_t w[3 * ((G + 1) / 2)];
#pragma unroll
    for (int q = 0; q < G; ++q) {
        if (run_len(cnt, 4 * q + 3) == kWave) {
            const uint32_t *p = g.pos + pb;
            if ((q & 1) == 0) {
                w[3 * (q / 2)] = p[ul];
                w[3 * (q / 2) + 1] = p[ul + kWave];
            } else {
                w[3 * (q / 2) + 2] = p[ul];
            }
            pb = scalar(pb + ((q & 1) ? kWave : 2 * kWave));
            const V *e = g.val + vb;
#pragma unroll
            for (int u = 0; u < 4; ++u) v[4 * q + u] = e[ul + u * kWave];
            vb = scalar(vb + 4 * kWave);
        } else if (run_len(cnt, 4 * q) > 0) {
            if ((q & 1) == 0) {
                w[3 * (q / 2)] = (g.pos + pb)[ul];
                pb = scalar(pb + run_len(cnt, 4 * q));
                w[3 * (q / 2) + 1] = (g.pos + pb)[ul];
                pb = scalar(pb + run_len(cnt, 4 * q + 2));
            } else {
                w[3 * (q / 2) + 2] = (g.pos + pb)[ul];
                pb = scalar(pb + run_len(cnt, 4 * q + 1));
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                v[4 * q + u] = (g.val + vb)[ul];
                vb = scalar(vb + run_len(cnt, 4 * q + u));
            }
        }
    }
    const int r = r0 + min(tid, nr - 1);
    T op = T(0);
    if (EPI == EPI_DOT) op = g.x[r];
    else if (EPI == EPI_RESID) op = g.b[r];
    // the direct-to-LDS loads of every wave are complete before the barrier
    // (a workgroup barrier alone does not wait for them): vmcnt 0
    __builtin_amdgcn_s_waitcnt(0x0f70);
    __syncthreads();
    const int len = (int)(slot >> 8);
    T sum = T(0);
#pragma unroll
    for (int q = 0; q < G; ++q) {
        const bool full = run_len(cnt, 4 * q + 3) == kWave;
        if (run_len(cnt, 4 * q) > 0) {
            const uint32_t w0 = w[3 * (q / 2)], w1 = w[3 * (q / 2) + 1], w2 = (q & 1) ? w[3 * (q / 2) + 2] : 0u;
            unsigned p[4];
            if (q & 1) {
                p[0] = pos12<4>(w0, w1, w2);
                p[1] = pos12<5>(w0, w1, w2);
                p[2] = pos12<6>(w0, w1, w2);
                p[3] = pos12<7>(w0, w1, w2);
            } else {
                p[0] = pos12<0>(w0, w1, w2);
                p[1] = pos12<1>(w0, w1, w2);
                p[2] = pos12<2>(w0, w1, w2);
                p[3] = pos12<3>(w0, w1, w2);
            }
            T xv[4];
            if (full) {
#pragma unroll
                for (int u = 0; u < 4; ++u) xv[u] = win[p[u]];
#pragma unroll
                for (int u = 0; u < 4; ++u) sum = add_rounded<T>(sum, to_acc<T>(v[4 * q + u]), xv[u]);
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) xv[u] = win[4 * q + u < len ? p[u] : 0u];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const T t = add_rounded<T>(sum, to_acc<T>(v[4 * q + u]), xv[u]);
                    sum = 4 * q + u < len ? t : sum;
                }
            }
        }
    }
    // back to row order through LDS, so y is stored contiguously
    __syncthreads();
    win[slot & 0xffu] = sum;
    __syncthreads();
    double dot = 0.0;
    if (tid < nr) {
        const T s = win[tid];
        if (EPI == EPI_RESID) {
            const T res = op - s;
            g.y[r] = res;
            dot = static_cast<double>(res) * static_cast<double>(res);
        } else if (EPI == EPI_DOT) {
            g.y[r] = s;
            dot = static_cast<double>(s) * static_cast<double>(op);
        } else {
            __builtin_nontemporal_store(s, g.y + r);
        }
    }
    if (EPI != EPI_PLAIN) {
        const double t = block_sum(dot, sh);
        if (tid == 0) g.part[li] = t;
    }
}

// ------------------------------------------------------- layout (creation)

// Positions: lane of a slice, its row's entries in ascending order, each
// found in the tile's sorted sector list.
__global__ __launch_bounds__(kJagRows) void k_jag_fill_pos(const int32_t *__restrict__ hdr,
                                                           const uint16_t *__restrict__ slots,
                                                           const int32_t *__restrict__ sects, int stride,
                                                           const int32_t *__restrict__ row_ptr,
                                                           const int32_t *__restrict__ col,
                                                           uint32_t *__restrict__ pos) {
    const int li = (int)blockIdx.x, tid = (int)threadIdx.x, lane = tid & (kWave - 1);
    const int32_t *h = hdr + ((size_t)li * (kJagRows / kWave) + tid / kWave) * kJagHdr;
    const unsigned slot = slots[(size_t)li * kJagRows + tid];
    const int len = (int)(slot >> 8), ns = h[2];
    const int32_t *sect = sects + (size_t)li * stride;
    int32_t cnt[8];
    for (int i = 0; i < 8; ++i) cnt[i] = h[8 + i];
    const int s = len > 0 ? row_ptr[h[3] + (int)(slot & 0xffu)] : 0;
    size_t pb = (size_t)h[1];
    for (int j0 = 0; j0 < len; j0 += 8) {
        uint64_t lo = 0;
        uint32_t hi = 0;  // bits 64..95
        for (int m = 0; m < 8 && j0 + m < len; ++m) {
            const int c = col[s + j0 + m], want = c / kJagSector;
            int a = 0, b = ns - 1;
            while (a < b) {
                const int mid = (a + b) >> 1;
                if (sect[mid] < want) a = mid + 1;
                else b = mid;
            }
            const uint64_t p = (uint64_t)(a * kJagSector + c % kJagSector);
            const int bit = 12 * m;
            if (bit < 64) lo |= p << bit;
            if (bit >= 64) hi |= (uint32_t)(p << (bit - 64));
            else if (bit + 12 > 64) hi |= (uint32_t)(p >> (64 - bit));
        }
        pos[pb + lane] = (uint32_t)lo;
        pb += run_len(cnt, j0);
        if (len > j0 + 2) pos[pb + lane] = (uint32_t)(lo >> 32);
        pb += run_len(cnt, j0 + 2);
        if (len > j0 + 5) pos[pb + lane] = hi;
        pb += run_len(cnt, j0 + 5);
    }
}

template <typename V>
__global__ __launch_bounds__(kJagRows) void k_jag_fill_val(const int32_t *__restrict__ hdr,
                                                           const uint16_t *__restrict__ slots,
                                                           const int32_t *__restrict__ row_ptr,
                                                           const V *__restrict__ csr_val, V *__restrict__ val) {
    const int li = (int)blockIdx.x, tid = (int)threadIdx.x, lane = tid & (kWave - 1);
    const int32_t *h = hdr + ((size_t)li * (kJagRows / kWave) + tid / kWave) * kJagHdr;
    const unsigned slot = slots[(size_t)li * kJagRows + tid];
    const int len = (int)(slot >> 8);
    int32_t cnt[8];
    for (int i = 0; i < 8; ++i) cnt[i] = h[8 + i];
    const int s = len > 0 ? row_ptr[h[3] + (int)(slot & 0xffu)] : 0;
    size_t vb = (size_t)h[0];
    for (int j = 0; j < len; ++j) {
        val[vb + lane] = csr_val[s + j];
        vb += run_len(cnt, j);
    }
}

// ------------------------------------------------------------------ launch

template <typename V, typename T, int G>
static void launch_groups(const JagArgs<V, T> &a, int epi, int grid, size_t lds, hipStream_t st) {
    const bool x16 = (reinterpret_cast<uintptr_t>(a.x) & 15) == 0;
    const auto go = [&](auto aligned, auto other) {
        hipLaunchKernelGGL(x16 ? aligned : other, dim3(grid), dim3(kJagRows), lds, st, a);
    };
    switch (epi) {
        case EPI_DOT: go(k_jag<V, T, G, EPI_DOT, true>, k_jag<V, T, G, EPI_DOT, false>); break;
        case EPI_RESID: go(k_jag<V, T, G, EPI_RESID, true>, k_jag<V, T, G, EPI_RESID, false>); break;
        default: go(k_jag<V, T, G, EPI_PLAIN, true>, k_jag<V, T, G, EPI_PLAIN, false>); break;
    }
}

template <typename V, typename T>
void launch_jag(const DevMatrix &M, const V *val, const SpmvArgs<V, T, T> &g, int epi, hipStream_t st) {
    JagArgs<V, T> a{};
    a.hdr = M.jag_hdr;
    a.slot = M.jag_slot;
    a.sect = M.jag_sect;
    a.pos = M.jag_pos;
    a.val = val;
    a.x = g.x;
    a.y = g.y;
    a.b = g.b;
    a.part = g.part;
    a.done = g.done;
    a.n_tiles = M.n_jag;
    a.per_xcd = M.xcd_remap && M.n_jag >= 16 ? (M.n_jag + 7) / 8 : 0;
    a.chunk_log2 = M.xcd_chunk_log2;
    a.stride = M.jag_stride;
    a.n_cols = M.n_cols;
    const int grid = xcd_grid(M.n_jag, a.per_xcd, a.chunk_log2);
    // LDS for the handle's widest window in whole staging passes (at most
    // 256 words each), and at least one word per row for the way back to
    // row order
    const size_t lds = sizeof(T) * (size_t)std::max((M.jag_width + 255) / 256 * 256, kJagRows);
    if (M.jag_groups <= 2) launch_groups<V, T, 2>(a, epi, grid, lds, st);
    else if (M.jag_groups <= 4) launch_groups<V, T, 4>(a, epi, grid, lds, st);
    else launch_groups<V, T, kJagMaxLen / 4>(a, epi, grid, lds, st);
}

void launch_jag_fill_pos(const DevMatrix &M, uint32_t *pos, hipStream_t st) {
    hipLaunchKernelGGL(k_jag_fill_pos, dim3(M.n_jag), dim3(kJagRows), 0, st, M.jag_hdr, M.jag_slot, M.jag_sect,
                       M.jag_stride, M.row_ptr, M.col, pos);
}

template <typename V> void launch_jag_fill_val(const DevMatrix &M, const V *csr_val, V *val, hipStream_t st) {
    hipLaunchKernelGGL((k_jag_fill_val<V>), dim3(M.n_jag), dim3(kJagRows), 0, st, M.jag_hdr, M.jag_slot, M.row_ptr,
                       csr_val, val);
}

template void launch_jag<double, double>(const DevMatrix &, const double *, const SpmvArgs<double, double, double> &,
                                         int, hipStream_t);
template void launch_jag<float, float>(const DevMatrix &, const float *, const SpmvArgs<float, float, float> &, int,
                                       hipStream_t);
template void launch_jag<float, double>(const DevMatrix &, const float *, const SpmvArgs<float, double, double> &,
                                        int, hipStream_t);
template void launch_jag<uint16_t, float>(const DevMatrix &, const uint16_t *,
                                          const SpmvArgs<uint16_t, float, float> &, int, hipStream_t);
template void launch_jag_fill_val<double>(const DevMatrix &, const double *, double *, hipStream_t);
template void launch_jag_fill_val<float>(const DevMatrix &, const float *, float *, hipStream_t);
template void launch_jag_fill_val<uint16_t>(const DevMatrix &, const uint16_t *, uint16_t *, hipStream_t);

}  // namespace spmvlib
