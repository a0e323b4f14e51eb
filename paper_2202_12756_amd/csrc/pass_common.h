// Addressing and launch helpers shared by the pass kernels.
#pragma once

#include "cx.h"
#include "kernels.h"

namespace gfft {

constexpr int ilog2_c(int v) { return v <= 1 ? 0 : 1 + ilog2_c(v / 2); }

// Largest radix per FFT stage.  The FP32 vector kernels take radix-32
// stages, one LDS exchange fewer for 512- and 1024-point transforms (FP32 is
// bound by instruction issue), and radix 64 where a thread holds 64 elements;
// FP64 and the matrix-core stage keep radix 16.
template <typename T, int MF = 0, int E = 0>
constexpr int radix_cap() { return sizeof(T) == 4 && MF == 0 ? (E >= 64 ? 64 : 32) : 16; }

__device__ __forceinline__ int64_t map_row(int64_t r, row_map m) {
    const int64_t bx = r >> m.lg_n;
    const int64_t y = r & ((int64_t(1) << m.lg_n) - 1);
    const int64_t b = bx >> m.lg_x;
    const int64_t xl = bx & ((int64_t(1) << m.lg_x) - 1);
    if (m.paper) return (b << (m.lg_x + m.lg_n)) + (y << m.lg_x) + xl;
    const int64_t j = y >> m.lg_y;
    const int64_t yl = y & ((int64_t(1) << m.lg_y) - 1);
    return (b << (m.lg_x + m.lg_n)) + ((((j << m.lg_x) + xl)) << m.lg_y) + yl;
}

// Offset (in complex values) of bin k of row r in a pencil plan's
// first-exchange order (row_map::pencil).
__device__ __forceinline__ int64_t pencil_bin(int64_t r, int k, int K, const row_map& m) {
    const int64_t item = r >> m.lg_rows;
    const int64_t rl = r & ((int64_t(1) << m.lg_rows) - 1);
    const int c = (k >> m.lg_w) < m.pc_last ? (k >> m.lg_w) : m.pc_last;
    const int64_t wc = (int64_t(1) << m.lg_w) + (c == m.pc_last ? 1 : 0);
    return ((item * K + (int64_t(c) << m.lg_w)) << m.lg_rows) + rl * wc + (k - (c << m.lg_w));
}

// Tile order.  Consecutive workgroup ids are dealt round-robin to the 8 XCDs,
// each with its own L2.  Neighbouring tiles share cache lines at their edges
// and should meet in one L2; the XCDs together should work on one region of
// memory.  ord >= 0 deals groups of 2^ord neighbouring tiles to the XCDs in
// turn (0: launch order); kContig gives every XCD one contiguous eighth of the
// tiles.  Groups of 16 (kGrouped) are within 2% of the best order for almost
// every pass over a large array: FP64 1024-point z rows R2C 5.89 TB/s (contiguous
// 5.56), C2R 5.95 (5.63); N = 2048 z 5.66 (5.30).  The long y lines of FP64 and
// the x lines measured below keep orders of their own.
constexpr int kContig = -1;
constexpr int kGrouped = 4;
__device__ __forceinline__ int64_t xcd_tile(int ord, uint32_t g, uint32_t G) {
    constexpr uint32_t kXcd = 8;
    if (ord == 0) return g;
    uint32_t base = 0, o = g;
    if (ord > 0) {
        const uint32_t span = kXcd << ord;
        base = g & ~(span - 1);
        o = g - base;
        if (G - base >= span) return base + ((o % kXcd) << ord) + o / kXcd;
        // the tiles left over (all of a small grid): contiguous eighths
    }
    const uint32_t per = (G - base) / kXcd;
    return o >= per * kXcd ? g : base + (o % kXcd) * per + o / kXcd;
}

// The order of a pass over a complex array of `bytes`: `large`, but contiguous
// eighths where the array is of the size of the eight L2s (32 MB) or less.  There
// a pass finds what the one before it left in its own XCD's L2 only if both deal
// the array out alike: pairs of 16 MB of reals in place, FP64 256 slabs 32 us
// against 47 with groups, 512 37 against 55; over all N and layouts 9% less at
// 8 MB, 10% at 16, 2% at 32, nothing at 64.
inline int tile_order(int64_t bytes, int large) {
    return bytes <= int64_t(40) << 20 ? kContig : large;
}

// Grids are one-dimensional, and a dispatch carries its size in work-items
// as a 32-bit count: refuse grids beyond either limit.
inline bool grid_fits(int64_t blocks, int64_t threads) {
    return blocks <= 0x7fffffff && blocks * threads <= int64_t(0xffffffff);
}

// Rows of up to 128 reals take 2 to 8 threads each, so the most rows that fit
// in memory (2^31 of 16 reals in 154 GB, in place) need more than one grid:
// such passes run in slices of 2^28 rows, whole entries of the batch (an entry
// has a power of two of at most N^2 rows), each at the same offset in rows of
// both arrays.  launch(r0, rows of the slice).
constexpr int64_t kSliceRows = int64_t(1) << 28;
template <typename F>
inline hipError_t in_slices(int64_t rows, F launch) {
    for (int64_t r0 = 0; r0 < rows; r0 += kSliceRows) {
        const hipError_t e = launch(r0, rows - r0 < kSliceRows ? rows - r0 : kSliceRows);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace gfft
