// Limits of the jagged window tiles and of the sweep tiles (host and device).
#pragma once

namespace spmvlib {
constexpr int kJagRows = 256;        // rows per tile, one per lane of a workgroup
constexpr int kJagMaxLen = 28;       // entries per row
constexpr int kJagSector = 8;        // x words per window sector
constexpr int kJagMaxSectors = 512;  // sectors per window: 4,096 words, 12-bit positions
constexpr int kJagHdr = 16;          // header ints per slice
constexpr int kSweepTile = 20480;    // entries per sweep tile: their FP64 products fill 160 KB of LDS
}  // namespace spmvlib
