// HIP kernels of the slab 3D real FFT for gfx950 (MI355X).
//
// Three pass kinds cover the whole path (section 3 steps 1 and 5 and their
// inverse; steps 2-4 are row permutations folded into addressing):
//   z pass  : contiguous rows.  A row of N reals is read as N/2 complex
//             values z[n] = x[2n] + i x[2n+1], transformed with an N/2-point
//             complex FFT, and split into the K = N/2+1 bins of the real
//             transform (and the reverse for C2R).
//   y/x pass: strided lines.  A workgroup owns TC adjacent columns of a
//             batch of lines; lanes of consecutive columns read consecutive
//             addresses, so every load and store is a contiguous run of
//             TC complex values per line position.
//   pack    : the send-order permutation as a plain copy of contiguous runs.
// Pencil plans (section 2, pencil decomposition) reuse the same passes: the
// z pass scatters each row's bins to the first exchange's chunks, and the
// y/x passes address the received pencils through their line maps.
// Memory bound: each pass reads and writes its array once.  fused.h holds the
// kernels that take several axes, or part of one beside another, in a pass:
// full transforms and step 1 run those where they apply, the passes here run
// the rest, the single-pass entry points and the lines the others leave.
#include "cx.h"
#include "engine.h"
#include "fused.h"
#include "kernels.h"
#include "mfma_dft16.h"
#include "pass_common.h"

namespace gfft {

constexpr int kThreads = 256;

// A workgroup-uniform value in scalar registers that the optimiser cannot
// see through: expressions of it are formed where they are used.
__device__ __forceinline__ int opaque_uniform(int v) {
    int r = __builtin_amdgcn_readfirstlane(v);
    asm volatile("" : "+s"(r));
    return r;
}
__device__ __forceinline__ int64_t opaque_uniform(int64_t v) {
    const uint64_t u = uint64_t(v);
    const uint32_t lo = uint32_t(opaque_uniform(int(uint32_t(u)))),
                   hi = uint32_t(opaque_uniform(int(uint32_t(u >> 32))));
    return int64_t((uint64_t(hi) << 32) | lo);
}

template <int M, int EMAX = 16, int THREADS = kThreads>
struct zshape {
    static constexpr int E = M < EMAX ? M : EMAX;  // elements per thread
    static constexpr int TPT = M / E;              // threads per row
    static constexpr int NT = THREADS > TPT ? THREADS : TPT;
    static constexpr int RPB = NT / TPT;           // rows per workgroup
};

// Workgroup shape of the z passes up to N = 1024 (longer rows: k_rows_*),
// chosen by measurement (2^18 and 2^20 rows): FP64 R2C 8 elements per thread
// in 256-thread workgroups up to N = 512, 16 per thread in 128-thread ones for
// N = 1024 (7-8% faster there); FP64 C2R 16 per thread in 64-thread
// workgroups; FP32 32 per thread, in 256-thread workgroups for the R2C of
// N = 1024 (4-10% faster with the radix-32 stages) and 64-thread ones
// otherwise, except at N = 256 and 512: 16 per thread in 256-thread workgroups
// (the C2R of N = 512 in 128-thread ones), 5-13% faster there.
// Workgroups are dealt to the XCDs in groups of 16: TB/s against contiguous
// eighths, R2C / C2R, FP64 N = 1024 5.89 / 5.95 (5.56 / 5.63), 512 5.76 / 6.09
// (5.39 / 5.75), FP32 1024 5.32 / 5.35 (4.96 / 5.07), 512 5.19 / 5.25 (4.93 /
// 5.08).  The C2R also stores its line-aligned real rows non-temporally (they are
// not read again soon); the R2C's complex rows are not line-aligned and gain
// nothing from it.  Up to N = 128: 8 values per thread (N = 16: 4) in 256-thread
// workgroups, both types and directions (FP32 64 C2R 3.7 times, R2C 1.7 times as
// fast as the 64-thread shape; FP64 4-15% C2R, 3-8% R2C).
template <typename T, bool FWD, int N>
struct zcfg {
    static constexpr bool F64 = sizeof(T) == 8;
    static constexpr bool MID32 = !F64 && (N == 256 || N == 512);
    static constexpr int EMAX = N <= 16 ? 4
                                : N <= 128 ? 8
                                : F64 ? (FWD ? (N >= 1024 ? 16 : 8) : 16) : (MID32 ? 16 : 32);
    static constexpr int THREADS =
        N <= 128 ? 256
        : F64 ? (FWD ? (N >= 1024 ? 128 : 256) : 64)
              : MID32 ? (FWD || N == 256 ? 256 : 128) : (FWD && N >= 1024 ? 256 : 64);
};

// ---------------------------------------------------------------- z R2C
// ALIAS: `in` and `out` are the same buffer (in-place plans).  Each row is
// read completely before the first barrier and written after the last one,
// so a row is never overwritten before all of it has been loaded.
template <typename T, int N, int EMAX, int THREADS, bool ALIAS, bool PENCIL = false>
__device__ __forceinline__ void z_r2c_body(
    const T* in, cx<T>* out, const cx<T>* __restrict__ tw,
    int64_t rows, row_map map, T mul_edge, T mul_int, int ord) {
    constexpr int M = N / 2, K = M + 1;
    using Z = zshape<M, EMAX, THREADS>;
    constexpr int E = Z::E, TPT = Z::TPT, RPB = Z::RPB;
    constexpr int RM = radix_cap<T>();
    constexpr int PS = first_radix_shift<E, RM>::value, MP = padded_len<M, PS>::value;
    __shared__ cx<T> lds[RPB * MP];

    const int rl = threadIdx.x / TPT;
    const int t = threadIdx.x % TPT;
    const int64_t blk = xcd_tile(ord, blockIdx.x, gridDim.x);
    const int64_t row = blk * RPB + rl;
    const bool valid = row < rows;

    // Rows past the end (last workgroup) load the last row and discard it.
    const cx<T>* src = reinterpret_cast<const cx<T>*>(in + (valid ? row : rows - 1) * map.rs);
    cx<T> a[E];
#pragma unroll
    for (int m = 0; m < E; ++m) a[m] = src[t + m * TPT];

    const idx_rows<PS> ix{rl * MP};
    fft_regs<T, M, E, -1, RM>(a, t, tw, 2, xch_full<T, idx_rows<PS>>{lds, ix});

    // Split Z = FFT_M(z) into the real transform:
    //   X[k] = (Z[k] + conj Z[M-k])/2 - (i/2) W_N^k (Z[k] - conj Z[M-k]),
    //   X[M] = Re Z[0] - Im Z[0].
#pragma unroll
    for (int m = 0; m < E; ++m) lds[ix.at(xgeom<M, E, 1, 1>::template in_pad<PS>(t, m))] = a[m];
    __syncthreads();
    if (!valid) return;
    // FIRST: all bins are formed in registers before the first store, as a
    // twiddle load behind a store waits for it (FP32 N = 64 374 -> 261 us over
    // 537 MB, 256 224 -> 212; from 512 up the loads are hoisted anyway and
    // FP32 loses 2-3%).  With ALIAS nothing can be hoisted.
    constexpr bool FIRST = ALIAS || N <= 256;
    const cx<T> x_m{(a[0].x - a[0].y) * mul_edge, T(0)};
    cx<T>* dst = out + (PENCIL ? 0 : map_row(row, map) * K);
    auto put = [&](int k, cx<T> v) {
        if constexpr (PENCIL) out[pencil_bin(row, k, K, map)] = v;
        else dst[k] = v;
    };
#pragma unroll
    for (int m = 0; m < E; ++m) {
        const int k = t + m * TPT;
        const cx<T> zk = a[m];
        const cx<T> zc = conjg(lds[ix((M - k) & (M - 1))]);
        const cx<T> A = scal(zk + zc, T(0.5));
        const cx<T> B = scal(zk - zc, T(0.5));
        const cx<T> wb = cmul(tw[k], B);
        const T f = k == 0 ? mul_edge : mul_int;
        const cx<T> v{(A.x + wb.y) * f, (A.y - wb.x) * f};
        if constexpr (FIRST) a[m] = v;
        else put(k, v);
    }
    if constexpr (FIRST) {
#pragma unroll
        for (int m = 0; m < E; ++m) put(t + m * TPT, a[m]);
    }
    if (t == 0) put(M, x_m);
}

template <typename T, int N, int EMAX, int THREADS>
__global__ __launch_bounds__((zshape<N / 2, EMAX, THREADS>::NT)) void k_z_r2c(
    const T* __restrict__ in, cx<T>* __restrict__ out, const cx<T>* __restrict__ tw,
    int64_t rows, row_map map, T mul_edge, T mul_int, int ord) {
    z_r2c_body<T, N, EMAX, THREADS, false>(in, out, tw, rows, map, mul_edge, mul_int, ord);
}

template <typename T, int N, int EMAX, int THREADS>
__global__ __launch_bounds__((zshape<N / 2, EMAX, THREADS>::NT)) void k_z_r2c_inplace(
    const T* in, cx<T>* out, const cx<T>* __restrict__ tw,
    int64_t rows, row_map map, T mul_edge, T mul_int, int ord) {
    z_r2c_body<T, N, EMAX, THREADS, true>(in, out, tw, rows, map, mul_edge, mul_int, ord);
}

// Pencil plans: bins scattered to the first exchange's chunks.
template <typename T, int N, int EMAX, int THREADS>
__global__ __launch_bounds__((zshape<N / 2, EMAX, THREADS>::NT)) void k_z_r2c_pencil(
    const T* __restrict__ in, cx<T>* __restrict__ out, const cx<T>* __restrict__ tw,
    int64_t rows, row_map map, T mul_edge, T mul_int, int ord) {
    z_r2c_body<T, N, EMAX, THREADS, false, true>(in, out, tw, rows, map, mul_edge, mul_int, ord);
}

// ---------------------------------------------------------------- z C2R
template <typename T, int N, int EMAX, int THREADS, bool PENCIL = false>
__device__ __forceinline__ void z_c2r_body(
    const cx<T>* in, T* out, const cx<T>* __restrict__ tw,
    int64_t rows, row_map map, T mul_edge, T mul_int, int ord) {
    constexpr int M = N / 2, K = M + 1;
    using Z = zshape<M, EMAX, THREADS>;
    constexpr int E = Z::E, TPT = Z::TPT, RPB = Z::RPB;
    constexpr int RM = radix_cap<T>();
    constexpr int PS = first_radix_shift<E, RM>::value, MP = padded_len<M, PS>::value;
    __shared__ cx<T> lds[RPB * MP];

    const int rl = threadIdx.x / TPT;
    const int t = threadIdx.x % TPT;
    const int64_t blk = xcd_tile(ord, blockIdx.x, gridDim.x);
    const int64_t row = blk * RPB + rl;
    const bool valid = row < rows;
    const idx_rows<PS> ix{rl * MP};

    // Load G[0..M-1] (registers and LDS) and G[M] (thread t = 0), dropping
    // the imaginary parts of kz = 0 and kz = N/2 and applying the bin
    // multipliers (scale, and 1/w for the adjoint).
    // Rows past the end (last workgroup) load the last row and discard it.
    cx<T> g[E];
    cx<T> g_m;
    const int64_t lrow = valid ? row : rows - 1;
    if constexpr (PENCIL) {
#pragma unroll
        for (int m = 0; m < E; ++m) g[m] = in[pencil_bin(lrow, t + m * TPT, K, map)];
        g_m = t == 0 ? in[pencil_bin(lrow, M, K, map)] : cx<T>{T(0), T(0)};
    } else {
        const cx<T>* src = in + map_row(lrow, map) * K;
#pragma unroll
        for (int m = 0; m < E; ++m) g[m] = src[t + m * TPT];
        g_m = t == 0 ? src[M] : cx<T>{T(0), T(0)};
    }
#pragma unroll
    for (int m = 0; m < E; ++m) {
        const int k = t + m * TPT;
        if (k == 0) g[m] = cx<T>{g[m].x * mul_edge, T(0)};
        else g[m] = scal(g[m], mul_int);
        lds[ix.at(xgeom<M, E, 1, 1>::template in_pad<PS>(t, m))] = g[m];
    }
    g_m = cx<T>{g_m.x * mul_edge, T(0)};
    __syncthreads();

    // Z'[k] = (G[k] + conj G[M-k]) + i conj(W_N^k) (G[k] - conj G[M-k]);
    // its inverse M-point FFT interleaves the even and odd outputs.
    cx<T> a[E];
#pragma unroll
    for (int m = 0; m < E; ++m) {
        const int k = t + m * TPT;
        const cx<T> gc = conjg(k == 0 ? g_m : lds[ix(M - k)]);
        const cx<T> s = g[m] + gc;
        const cx<T> d = cmulc(g[m] - gc, tw[k]);
        a[m] = cx<T>{s.x - d.y, s.y + d.x};
    }
    __syncthreads();
    fft_regs<T, M, E, +1, RM>(a, t, tw, 2, xch_full<T, idx_rows<PS>>{lds, ix});
    if (!valid) return;
    cx<T>* dst = reinterpret_cast<cx<T>*>(out + row * map.rs);
#pragma unroll
    for (int m = 0; m < E; ++m) {
        __builtin_nontemporal_store(a[m].x, &dst[t + m * TPT].x);
        __builtin_nontemporal_store(a[m].y, &dst[t + m * TPT].y);
    }
}

template <typename T, int N, int EMAX, int THREADS>
__global__ __launch_bounds__((zshape<N / 2, EMAX, THREADS>::NT)) void k_z_c2r(
    const cx<T>* __restrict__ in, T* __restrict__ out, const cx<T>* __restrict__ tw,
    int64_t rows, row_map map, T mul_edge, T mul_int, int ord) {
    z_c2r_body<T, N, EMAX, THREADS>(in, out, tw, rows, map, mul_edge, mul_int, ord);
}

// In place: every load of a row precedes the barrier after the LDS fill, and
// every store follows the last barrier of the FFT.
template <typename T, int N, int EMAX, int THREADS>
__global__ __launch_bounds__((zshape<N / 2, EMAX, THREADS>::NT)) void k_z_c2r_inplace(
    const cx<T>* in, T* out, const cx<T>* __restrict__ tw,
    int64_t rows, row_map map, T mul_edge, T mul_int, int ord) {
    z_c2r_body<T, N, EMAX, THREADS>(in, out, tw, rows, map, mul_edge, mul_int, ord);
}

// Pencil plans: bins gathered from the first exchange's chunks.
template <typename T, int N, int EMAX, int THREADS>
__global__ __launch_bounds__((zshape<N / 2, EMAX, THREADS>::NT)) void k_z_c2r_pencil(
    const cx<T>* __restrict__ in, T* __restrict__ out, const cx<T>* __restrict__ tw,
    int64_t rows, row_map map, T mul_edge, T mul_int, int ord) {
    z_c2r_body<T, N, EMAX, THREADS, true>(in, out, tw, rows, map, mul_edge, mul_int, ord);
}

// ---------------------------------------------------------------- y / x C2C
// Tile shape of the strided pass: TC columns of length N per workgroup, E
// elements per thread (TPT = N/E threads per column), exchanges through LDS
// either as whole complex values or split into real and imaginary halves
// (half the LDS per tile, twice the barriers).  Chosen by measurement at
// 1024^3 (FP64: y 16 columns, 512 threads, 128 KiB; x 8 columns, 256
// threads, 64 KiB; FP32: 16 columns, 512 threads, 64 KiB, both axes):
//   AX = 0 (y lines, rows K apart) and any N >= 2048 get the wide budget,
//   AX = 1 (x lines, rows megabytes apart) keeps two tiles per CU in FP64.
// TC is at most 16 columns unless the lines are so short that 256 threads
// need more.
template <typename T, int N, int AX, bool MFMA = false>
struct sshape {
    static constexpr bool F64 = sizeof(T) == 8;
    static constexpr bool WIDE = AX == 0 || N >= 2048;
    // FP32 lines of N = 256 and x lines of N = 512: 32 columns (256-byte
    // runs), 4% faster than 16 (at N = 256 the x tile with 32 elements per
    // thread, the y tile with 16)
    static constexpr bool C32 = !F64 && !MFMA && (N == 256 || (N == 512 && AX == 1));
    // FP32 lines of 2048 and x lines of 4096: 64 elements per thread, two
    // stages and one exchange (64 x 32, 64 x 64) instead of three and two; an x
    // tile of 128 KiB fills the LDS, so its FFT phase overlaps nothing (a y tile
    // of 2048 takes half, two per CU).  The 4096 tile needs all 256 VGPRs and
    // spills 19 to 25 of them; it is the faster one all the same.  TB/s
    // against 32 per thread: 2048 x 4.29 / 3.82 (slab of 64 planes), 3.78 / 2.97
    // (8 x 8 pencil), y 3.55 / 3.40 and 4.56 / 4.38; 4096 x 3.16 / 3.00.  y lines
    // of 4096 gain in some layouts and lose in others (natural 3.10 / 3.22, 8 x
    // 16 pencil 3.74 / 3.49), and FP64 (256 registers of data) loses 2-35%.
    static constexpr bool E64 = !F64 && !MFMA && (N == 2048 || (N == 4096 && AX == 1));
    static constexpr int E = MFMA ? 16 : E64 ? 64 : (N >= 512 || (C32 && AX == 1)) ? 32 : 16;
    static constexpr int TPT = N / E;
    // FP32 y lines of N = 2048: two 8-column tiles per CU (9% faster than
    // one 16-column tile); FP64 y lines of N = 512: two 16-column tiles with
    // the split exchange (8% faster than one with whole values)
    static constexpr bool Y2048 = !F64 && !MFMA && AX == 0 && N == 2048;
    static constexpr bool Y512 = F64 && AX == 0 && N == 512;
    static constexpr bool BIG32 = N >= 2048 && !Y2048;
    static constexpr int MAXT = F64 ? (WIDE ? 512 : 256) : (BIG32 || MFMA ? 1024 : 512);
    static constexpr int LDS = (F64 ? WIDE && !Y512 : BIG32) ? 131072 : 65536;
    static constexpr int TC_T = MAXT / TPT;
    // FP64 x lines of N = 64: 32 columns, 5.85 against 5.33 TB/s with 64
    static constexpr int CAP = C32 || (F64 && !MFMA && AX == 1 && N == 64) ? 32
                               : (256 / TPT) > 16 ? (256 / TPT) : 16;
    static constexpr int FULL = LDS / (N * int(sizeof(cx<T>)));
    static constexpr int A0 = TC_T < CAP ? TC_T : CAP;
    static constexpr int A1 = A0 < 2 * FULL ? A0 : 2 * FULL;
    static constexpr int TC = A1 < 1 ? 1 : A1;
    static constexpr int XP = TC > FULL ? 2 : 1;
};

// XP: LDS rounds per exchange.  1 = whole complex values, 2 = real then
// imaginary parts; the LDS tile is N*TC/XP complex values (padded).
// NT: non-temporal loads and stores of the lines (no reuse), for tilings in
// which every 128-byte line belongs to one tile (the host checks this).
// MF: 0 vector stages; 2 or 3 the first radix-16 stage on the matrix cores;
// -1 no transform (each element replaced by its conjugate): the same loads
// and stores as the pass, a yardstick for its memory-access ceiling.
// ord: tile order (xcd_tile).
// FLAT: sets of fewer columns than a tile; tiles take TC columns of all sets
// numbered through (tiles_m: the number of all columns).  Otherwise tiles_m is
// below 2^31, as the grid is.
// TWS: tw is the table of a transform TWS times as long.
// src may be data itself (in place) or a distinct buffer of the same layout:
// every load of a tile precedes its stores, and tiles own their elements.
template <typename T, int N, int TC, int XP, int S, int E = 16, int MF = 0, bool NT = false,
          int TWS = 1, bool FLAT = false>
__global__ __launch_bounds__(TC * N / E) void k_strided(
    const cx<T>* src, cx<T>* data, const cx<T>* __restrict__ tw, int64_t m_cols,
    int64_t tiles_m, line_map lm, int ord) {
    constexpr int TPT = N / E;
    constexpr bool SPLIT = XP == 2;
    static_assert(XP == 1 || XP == 2, "XP: whole values (1) or real/imaginary halves (2)");
    constexpr int RM = radix_cap<T, MF, E>();
    constexpr int PS = first_radix_shift<E, RM>::value;
    constexpr int NP = padded_len<N, PS>::value;
    __shared__ cx<T> lds[(NP * TC + XP - 1) / XP];
    using IX = idx_cols<TC, PS>;

    const int c = threadIdx.x % TC;
    const int t = threadIdx.x / TC;
    const int64_t tile = xcd_tile(ord, blockIdx.x, gridDim.x);
    int64_t b, m0, m;
    bool valid;
    if constexpr (FLAT) {
        // the tile's first column by a scalar division, the lane's by a short one
        const int64_t g0 = tile * TC, b0 = g0 / m_cols;
        valid = g0 + c < tiles_m;
        const uint32_t r = uint32_t(g0 - b0 * m_cols) + (valid ? c : uint32_t(tiles_m - 1 - g0));
        const uint32_t q = r / uint32_t(m_cols);
        b = b0 + q;
        m = r - q * uint32_t(m_cols);
        m0 = 0;
    } else {
        b = uint32_t(tile) / uint32_t(tiles_m);
        m0 = (tile - b * tiles_m) * TC;
        m = m0 + c;
        valid = m < m_cols;
    }
    const int64_t ymask = (int64_t(1) << lm.lg_y) - 1;
    const int64_t set = (b >> lm.lg_bx) * lm.b_hi + (b & ((int64_t(1) << lm.lg_bx) - 1)) * lm.b_lo;
    const cx<T>* from = src + set;
    cx<T>* plane = data + set;
    auto off = [&](int64_t n) { return (n >> lm.lg_y) * lm.s_hi + (n & ymask) * lm.s_lo; };
    // Element n = t + i*TPT of a line: t < TPT and i*TPT have disjoint bits
    // (TPT a power of two), and off() adds over disjoint bit fields, so
    // off(n) = off(t) + off(i*TPT): a per-lane pointer plus an offset that
    // is the same for the whole workgroup, written in closed form as
    // off(i*TPT) = (i >> d) H + (i mod 2^d) Lo.  Lanes of the ragged last
    // tile read the last column instead (in bounds); their results are
    // dropped.
    constexpr int LGT = ilog2_c(TPT), LGE = ilog2_c(E);
    int d = 0;
    int64_t H = (int64_t(TPT) >> (lm.lg_y < LGT ? lm.lg_y : LGT)) * lm.s_hi, Lo = 0;
    if (lm.lg_y >= LGT) {
        d = lm.lg_y - LGT < LGE ? lm.lg_y - LGT : LGE;
        H = lm.s_hi;
        Lo = int64_t(TPT) * lm.s_lo;
    }
    auto uoff = [](int i, int d, int64_t H, int64_t Lo) {
        return int64_t(i >> d) * H + int64_t(i & ((1 << d) - 1)) * Lo;
    };
    int64_t lane_off = (FLAT || valid ? m : m_cols - 1) + off(t);
    const cx<T>* lane = from + lane_off;

    cx<T> a[E];
    if constexpr (MF < 0) {
#pragma unroll
        for (int i = 0; i < E; ++i) {
            const cx<T>* p = lane + uoff(i, d, H, Lo);
            if constexpr (NT) {
                a[i].x = __builtin_nontemporal_load(&p->x);
                a[i].y = -__builtin_nontemporal_load(&p->y);
            } else {
                a[i] = conjg(*p);
            }
        }
        // all loads of the tile before any store, as in the transform
        __syncthreads();
    } else if constexpr (MF == 0) {
#pragma unroll
        for (int i = 0; i < E; ++i) {
            const cx<T>* p = lane + uoff(i, d, H, Lo);
            if constexpr (NT) {
                a[i].x = __builtin_nontemporal_load(&p->x);
                a[i].y = __builtin_nontemporal_load(&p->y);
            } else {
                a[i] = *p;
            }
        }
        if constexpr (SPLIT)
            fft_regs<T, N, E, S, RM>(a, t, tw, TWS,
                                     xch_split<T, IX>{reinterpret_cast<T*>(lds), IX{c}});
        else
            fft_regs<T, N, E, S, RM>(a, t, tw, TWS, xch_full<T, IX>{lds, IX{c}});
    } else {
        // First radix-16 stage on the matrix cores.  The wave's 64 butterflies
        // (those of its own threads, j = t for thread (c, t)) go in two groups
        // of 32; lane (h, n) loads inputs 8h..8h+7 of butterfly 32g + n.
        static_assert(sizeof(T) == 4 && E == 16 && N >= 32, "MFMA stage: FP32, radix-16 first stage");
        const int lane = threadIdx.x & 63, h = lane >> 5;
        const int wbase = threadIdx.x & ~63;
        dft16_mfma<S, MF> dft;
        dft.init(lane);
        cx<float> y[2][8];
        int bc[2], bt[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const int tid_b = wbase + 32 * g + (lane & 31);
            bc[g] = tid_b % TC;
            bt[g] = tid_b / TC;
            const bool vb = m0 + bc[g] < m_cols;
            cx<float> in[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int64_t n = bt[g] + (8 * h + j) * TPT;
                in[j] = vb ? from[m0 + bc[g] + off(n)] : cx<float>{0.f, 0.f};
            }
            dft.run(in, y[g]);
        }
        // exchange: output r of butterfly (c_b, t_b) goes to position 16 t_b + r
        const IX pos_c{c};
        if constexpr (SPLIT) {
            T* buf = reinterpret_cast<T*>(lds);
#pragma unroll
            for (int part = 0; part < 2; ++part) {
#pragma unroll
                for (int g = 0; g < 2; ++g)
#pragma unroll
                    for (int v = 0; v < 8; ++v)
                        buf[IX{bc[g]}.at(xgeom<N, E, 1, 16>::template out_pad<PS>(bt[g], dft16_out_index(h, v) * (E / 16)))] =
                            part ? y[g][v].y : y[g][v].x;
                __syncthreads();
#pragma unroll
                for (int i = 0; i < E; ++i) {
                    const T val = buf[pos_c.at(xgeom<N, E, 1, 16>::template in_pad<PS>(t, i))];
                    if (part) a[i].y = val; else a[i].x = val;
                }
                __syncthreads();
            }
        } else {
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int v = 0; v < 8; ++v)
                    lds[IX{bc[g]}.at(xgeom<N, E, 1, 16>::template out_pad<PS>(bt[g], dft16_out_index(h, v) * (E / 16)))] = y[g][v];
            __syncthreads();
#pragma unroll
            for (int i = 0; i < E; ++i) a[i] = lds[pos_c.at(xgeom<N, E, 1, 16>::template in_pad<PS>(t, i))];
            __syncthreads();
        }
        if constexpr (SPLIT)
            fft_from<T, N, E, S, 16>(a, t, tw, 1,
                                     xch_split<T, IX>{reinterpret_cast<T*>(lds), IX{c}});
        else
            fft_from<T, N, E, S, 16>(a, t, tw, 1, xch_full<T, IX>{lds, IX{c}});
    }
    if (!valid) return;
    // Opaque to the optimiser, so the store addresses are formed afresh
    // instead of keeping the E load addresses live through the transform.
    asm volatile("" : "+v"(lane_off));
    d = opaque_uniform(d);
    H = opaque_uniform(H);
    Lo = opaque_uniform(Lo);
    cx<T>* dst = plane + lane_off;
#pragma unroll
    for (int i = 0; i < E; ++i) {
        cx<T>* p = dst + uoff(i, d, H, Lo);
        if constexpr (NT) {
            __builtin_nontemporal_store(a[i].x, &p->x);
            __builtin_nontemporal_store(a[i].y, &p->y);
        } else {
            *p = a[i];
        }
    }
}

// ---------------------------------------------------------------- pack
// One run per chunk c = (bb, j, xl), elements of 16 bytes where the runs
// allow it (V: an FP64 value or two FP32 ones).  A thread moves U elements
// (launch_pack), and there are as many threads as that takes up to the
// dispatch limit: like the streaming copy, the pass lives on many short
// workgroups (1024^3/8, U = 1: FP32 179 us, FP64 360, 6.0 TB/s; 2, 4, 8: 192,
// 198, 204 and 390, 406, 401; 8-byte FP32 elements, four rounds per thread 197
// and 389).  A workgroup takes `per` whole runs where they are short (per > 0),
// a part of one otherwise; all extents are in elements of V, inv = 1 / len.
template <typename V, int U>
__global__ __launch_bounds__(kThreads) void k_pack(
    const V* __restrict__ src, V* __restrict__ dst, int64_t len, int64_t chunks,
    int64_t blocks_per_chunk, int per, float inv, int lg_x, int lg_p, int64_t x_step,
    bool to_send) {
    auto run = [&](int64_t chunk, int64_t& nat, int64_t& snd) {
        // chunk = (bb, j, xl) with xl fastest
        const int64_t xl = chunk & ((int64_t(1) << lg_x) - 1);
        const int64_t j = (chunk >> lg_x) & ((int64_t(1) << lg_p) - 1);
        const int64_t bb = chunk >> (lg_x + lg_p);
        const int64_t plane = (bb << lg_x) * x_step;
        nat = plane + xl * x_step + j * len;
        snd = plane + ((j << lg_x) + xl) * len;
    };
    int64_t nat, snd;
    if (per > 0) {
        const int64_t first = int64_t(blockIdx.x) * per;
        const int runs = int(chunks - first < per ? chunks - first : per), l = int(len);
        for (int e = threadIdx.x; e < runs * l; e += kThreads) {
            // exact where per > 1 (l < 2^10): e < 2^11, so e + 1/2 is at least
            // 2^-11 of a run away from a run's end
            const int c = per == 1 ? 0 : int((float(e) + 0.5f) * inv);
            run(first + c, nat, snd);
            const int o = e - c * l;
            dst[(to_send ? snd : nat) + o] = src[(to_send ? nat : snd) + o];
        }
        return;
    }
    const int64_t chunk = blockIdx.x / blocks_per_chunk;
    const int64_t part = blockIdx.x - chunk * blocks_per_chunk;
    run(chunk, nat, snd);
    const V* s = src + (to_send ? nat : snd);
    V* d = dst + (to_send ? snd : nat);
    const int64_t step = blocks_per_chunk * kThreads;
    int64_t e = part * kThreads + threadIdx.x;
    for (; e + (U - 1) * step < len; e += U * step) {
        V v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = s[e + u * step];
#pragma unroll
        for (int u = 0; u < U; ++u) d[e + u * step] = v[u];
    }
    for (; e < len; e += step) d[e] = s[e];
}

// Row permutation copy: workgroup copies kRows rows, k values each.
constexpr int kPackRows = 4;
template <typename T>
__global__ __launch_bounds__(kThreads) void k_pack_rows(
    const cx<T>* __restrict__ src, cx<T>* __restrict__ dst, int64_t rows, int64_t k,
    row_map map, bool to_send) {
#pragma unroll
    for (int i = 0; i < kPackRows; ++i) {
        const int64_t r = int64_t(blockIdx.x) * kPackRows + i;
        if (r >= rows) return;
        const int64_t q = map_row(r, map);
        const cx<T>* s = src + (to_send ? r : q) * k;
        cx<T>* d = dst + (to_send ? q : r) * k;
        for (int64_t e = threadIdx.x; e < k; e += kThreads) d[e] = s[e];
    }
}

// ---------------------------------------------------------------- copy
// Plain streaming copy, one 16-byte element per work-item and no reuse: the
// reference rate for what any pass can reach on contiguous memory.
__global__ __launch_bounds__(kThreads) void k_copy16(const uint4* __restrict__ src,
                                                     uint4* __restrict__ dst, int64_t n) {
    const int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

// ---------------------------------------------------------------- launchers
template <typename T, int N>
static hipError_t z_r2c_n(const void* in, void* out, const void* tw, int64_t rows,
                          row_map map, double me, double mi, hipStream_t s) {
    if constexpr (N <= 128) {
        if (rows > kSliceRows)
            return in_slices(rows, [&](int64_t r0, int64_t nr) {
                return z_r2c_n<T, N>(static_cast<const T*>(in) + r0 * map.rs,
                                     static_cast<cx<T>*>(out) + r0 * (N / 2 + 1), tw, nr, map, me,
                                     mi, s);
            });
    }
    using C = zcfg<T, true, N>;
    using Z = zshape<N / 2, C::EMAX, C::THREADS>;
    const int64_t blocks = (rows + Z::RPB - 1) / Z::RPB;
    // the paper's chunk order sets a plane's rows X apart, and FP64 256 writes them
    // best in launch order (512 MB 198 us, groups 208; 64 and 128 lose 10-20% by it)
    const bool spread = sizeof(T) == 8 && N == 256 && map.paper;
    const int ord = tile_order(rows * (N / 2 + 1) * int64_t(sizeof(cx<T>)), spread ? 0 : kGrouped);
    if constexpr (sizeof(T) == 4 && N <= 128) {
        // chunks of one bin, a block of rows each: as many rows as can be at a time
        // (512 MB, one plane's columns to a rank: N = 64 203 us, the 8-values shape
        // 261, 128 242 and 272)
        if (map.pencil && map.lg_w == 0 && map.lg_rows >= 6) {
            using ZW = zshape<N / 2, 32, 64>;
            const int64_t wide = (rows + ZW::RPB - 1) / ZW::RPB;
            if (!grid_fits(wide, ZW::NT)) return hipErrorInvalidValue;
            hipLaunchKernelGGL((k_z_r2c_pencil<T, N, 32, 64>), dim3(wide), dim3(ZW::NT), 0, s,
                               static_cast<const T*>(in), static_cast<cx<T>*>(out),
                               static_cast<const cx<T>*>(tw), rows, map, T(me), T(mi), ord);
            return hipGetLastError();
        }
    }
    if (blocks == 0) return hipSuccess;
    if (!grid_fits(blocks, Z::NT)) return hipErrorInvalidValue;
    if (map.pencil)
        hipLaunchKernelGGL((k_z_r2c_pencil<T, N, C::EMAX, C::THREADS>), dim3(blocks),
                           dim3(Z::NT), 0, s, static_cast<const T*>(in), static_cast<cx<T>*>(out),
                           static_cast<const cx<T>*>(tw), rows, map, T(me), T(mi), ord);
    else if (in == out)
        hipLaunchKernelGGL((k_z_r2c_inplace<T, N, C::EMAX, C::THREADS>),
                           dim3(blocks), dim3(Z::NT), 0, s, static_cast<const T*>(in),
                           static_cast<cx<T>*>(out), static_cast<const cx<T>*>(tw), rows, map,
                           T(me), T(mi), ord);
    else
        hipLaunchKernelGGL((k_z_r2c<T, N, C::EMAX, C::THREADS>), dim3(blocks),
                           dim3(Z::NT), 0, s, static_cast<const T*>(in), static_cast<cx<T>*>(out),
                           static_cast<const cx<T>*>(tw), rows, map, T(me), T(mi), ord);
    return hipGetLastError();
}

template <typename T, int N>
static hipError_t z_c2r_n(const void* in, void* out, const void* tw, int64_t rows,
                          row_map map, double me, double mi, hipStream_t s) {
    if constexpr (N <= 128) {
        if (rows > kSliceRows)
            return in_slices(rows, [&](int64_t r0, int64_t nr) {
                return z_c2r_n<T, N>(static_cast<const cx<T>*>(in) + r0 * (N / 2 + 1),
                                     static_cast<T*>(out) + r0 * map.rs, tw, nr, map, me, mi, s);
            });
    }
    using C = zcfg<T, false, N>;
    using Z = zshape<N / 2, C::EMAX, C::THREADS>;
    const int64_t blocks = (rows + Z::RPB - 1) / Z::RPB;
    const int ord = tile_order(rows * (N / 2 + 1) * int64_t(sizeof(cx<T>)), kGrouped);
    if (blocks == 0) return hipSuccess;
    if (!grid_fits(blocks, Z::NT)) return hipErrorInvalidValue;
    if (map.pencil)
        hipLaunchKernelGGL((k_z_c2r_pencil<T, N, C::EMAX, C::THREADS>),
                           dim3(blocks), dim3(Z::NT), 0, s, static_cast<const cx<T>*>(in),
                           static_cast<T*>(out), static_cast<const cx<T>*>(tw), rows, map,
                           T(me), T(mi), ord);
    else if (in == out)
        hipLaunchKernelGGL((k_z_c2r_inplace<T, N, C::EMAX, C::THREADS>),
                           dim3(blocks), dim3(Z::NT), 0, s, static_cast<const cx<T>*>(in),
                           static_cast<T*>(out), static_cast<const cx<T>*>(tw), rows, map,
                           T(me), T(mi), ord);
    else
        hipLaunchKernelGGL((k_z_c2r<T, N, C::EMAX, C::THREADS>), dim3(blocks),
                           dim3(Z::NT), 0, s, static_cast<const cx<T>*>(in), static_cast<T*>(out),
                           static_cast<const cx<T>*>(tw), rows, map, T(me), T(mi), ord);
    return hipGetLastError();
}

// True when each tile of a multiple of `la` columns covers whole lines of
// `la` elements: the base is 128-byte aligned and every offset of the
// layout, and the column count, are multiples of `la`.
static bool whole_lines(const void* data, int64_t m_cols, const line_map& lm, int64_t la) {
    return reinterpret_cast<uintptr_t>(data) % 128 == 0 && m_cols % la == 0 &&
           lm.b_hi % la == 0 && lm.b_lo % la == 0 && lm.s_hi % la == 0 && lm.s_lo % la == 0;
}

// More line sets than one grid takes go in several launches, each of whole
// b_hi groups of sets (sets of one group share b_lo offsets): the most short
// lines that fit in memory need it, as a tile's lanes past the last column count
// (N = 16 in place: 9 of 256, so 2^24 planes, 20 GB of FP32).
template <typename T, int N, int AX, int MF, bool NT, int TWS = 1>
static hipError_t strided_run(int large, int sign, const void* src, void* data, const void* tw,
                              int64_t m_cols, int64_t n_b, line_map lm, hipStream_t s) {
    using SH = sshape<T, N, AX, (MF > 0)>;
    constexpr int TC = SH::TC;
    const int64_t tiles_m = (m_cols + TC - 1) / TC;
    const dim3 threads(TC * SH::TPT);
    if (tiles_m * n_b == 0) return hipSuccess;
    // FP32 lines of 2048 and what a first y step leaves of them share so much at
    // their tiles' edges that groups win at every size (one plane in place 31 us
    // an inverse, contiguous 35)
    const int ord = sizeof(T) == 4 && N * TWS == 2048
                        ? large
                        : tile_order(m_cols * n_b * N * int64_t(sizeof(cx<T>)), large);
    const int64_t groups = (int64_t(1) << 31) / ((tiles_m * threads.x) << lm.lg_bx);
    const int64_t most = groups > 0 ? groups << lm.lg_bx : n_b;
    for (int64_t b0 = 0; b0 < n_b; b0 += most) {
        const int64_t blocks = tiles_m * (n_b - b0 < most ? n_b - b0 : most);
        if (!grid_fits(blocks, threads.x)) return hipErrorInvalidValue;
        const int64_t off = (b0 >> lm.lg_bx) * lm.b_hi;
        const cx<T>* from = static_cast<const cx<T>*>(src) + off;
        cx<T>* to = static_cast<cx<T>*>(data) + off;
        const cx<T>* t = static_cast<const cx<T>*>(tw);
        if (MF < 0 || sign < 0)
            hipLaunchKernelGGL((k_strided<T, N, TC, SH::XP, -1, SH::E, MF, NT, TWS>),
                               dim3(blocks), threads, 0, s, from, to, t, m_cols, tiles_m, lm, ord);
        else if constexpr (MF >= 0)
            hipLaunchKernelGGL((k_strided<T, N, TC, SH::XP, +1, SH::E, MF, NT, TWS>),
                               dim3(blocks), threads, 0, s, from, to, t, m_cols, tiles_m, lm, ord);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Lines of sets narrower than a tile, the columns of all sets numbered through:
// y lines of pencils with narrow kz chunks (FP32 2048 1 x 1024 ranks, one bin, z, y
// and x 171 -> 124 us, FP64 1024 1 x 256 96 -> 52, 4096 8 x 2048 81 -> 65) and the
// 9 or 17 columns of N = 16 and 32.
// MF: 0 or -1 (k_strided).
template <typename T, int N, int AX, int MF>
static hipError_t strided_flat(int sign, const void* src, void* data, const void* tw,
                               int64_t m_cols, int64_t n_b, line_map lm, hipStream_t s) {
    using SH = sshape<T, N, AX>;
    constexpr int TC = SH::TC;
    const int64_t cols = m_cols * n_b, blocks = (cols + TC - 1) / TC;
    const int ord = tile_order(cols * N * int64_t(sizeof(cx<T>)), kGrouped);
    if (!grid_fits(blocks, TC * SH::TPT)) return hipErrorInvalidValue;
    const dim3 threads(TC * SH::TPT);
    if (MF < 0 || sign < 0)
        hipLaunchKernelGGL((k_strided<T, N, TC, SH::XP, -1, SH::E, MF, false, 1, true>),
                           dim3(blocks), threads, 0, s, static_cast<const cx<T>*>(src),
                           static_cast<cx<T>*>(data), static_cast<const cx<T>*>(tw), m_cols, cols, lm, ord);
    else if constexpr (MF >= 0)
        hipLaunchKernelGGL((k_strided<T, N, TC, SH::XP, +1, SH::E, MF, false, 1, true>),
                           dim3(blocks), threads, 0, s, static_cast<const cx<T>*>(src),
                           static_cast<cx<T>*>(data), static_cast<const cx<T>*>(tw), m_cols, cols, lm, ord);
    return hipGetLastError();
}

// Tile order and hints of the strided passes.  x passes whose tiles own whole
// 128-byte lines stream through non-temporally: neighbouring tiles share
// nothing, and the eight XCDs are kept on one run of columns by dealing small
// groups of tiles (line_order gives log2 of the group).  TB/s over 0.5-1.1 GB
// of received pencils, groups / launch order / contiguous eighths:
//   FP64 N = 64 5.93 / 5.80 / 5.84, 128 5.86 / 5.65 / 5.28, 512 full grid 5.17 /
//        4.92 / 4.67 and p = 8 4.89 / 4.82 / 4.34, 1024 full grid 5.14 / 4.56 /
//        5.10, p = 4 5.15 / 4.68 / 4.93, p = 16 5.06 / 4.73 / 4.50
//   FP32 N = 64 6.00 / 6.00 / 5.61, 128 5.62 / 5.45 / 5.19, 256 4.92 / 4.52 /
//        4.66 (p = 1) and 5.6 / 5.7 / 5.2 (p = 8), 512 5.02 / 5.01 / 3.92, 1024
//        full grid 4.87 / 4.57 / 4.81, p = 8 4.96 / 4.59 / 4.22, 2048 p = 32
//        3.93 / 3.91 / 3.68
// FP64 256 gains from it up to 512 KB between a line's elements (p = 2 4.67 /
// 4.44 against a full grid's 3.73 / 4.31, launch order / contiguous without
// the hint).  Below 4 KB few columns remain: contiguous order, from N = 512
// (FP32 256) with the hint (FP32 512 at 1 KB 14.4 us against 17.2 grouped and
// plain), below without (FP32 128 at 2 KB 5.2 against 4.3); and
// FP64 2048 (one 512-thread workgroup per CU) is 5% slower with the hint:
// these, lines shared between tiles and the y passes take plain accesses.
// Where tiles share lines the hint makes them travel twice (15-50% slower).
// Plain accesses go in groups of 16 (FP32 4096 y 3.34 TB/s, 2.84 contiguous,
// pencil x 3.00 and 2.60; whole chains: FP64 512^3/4 in the paper's order 320
// us against 337, FP64 1024 4 x 4 pencil 626 against 642, FP32 2048 1 x 256
// 209 against 235), but contiguously for y lines of 512 (FP64 5.23 against
// 4.65), for those of natural order in FP64 (1024 4.88 against 4.76) and of FP32
// 1024 (128 planes 234 us against 243, with the matrix-core stage 330 and 340; its
// lines of 64 327 and 336), for FP32 4096 pencils whose tiles own their lines (16 x
// 32 315 and 352), and in FP64 from N = 2048 (4096 16 x 32 pencil 1539 us against
// 1632) and for x lines of 256 (4.46 against 3.7) and 512 (the paper's order, p = 8,
// 223 us against 243).
template <typename T, int N>
struct line_order {
    static constexpr bool F64 = sizeof(T) == 8;
    static constexpr int NT = N <= 128 ? 2 : N == 512 ? 1 : (!F64 && N == 1024) || (F64 && N == 256) ? 4 : 6;
};

template <typename T, int N, int AX, int MF>
static hipError_t strided_ax(int sign, const void* src, void* data, const void* tw, int64_t m_cols,
                             int64_t n_b, line_map lm, hipStream_t s) {
    constexpr bool F64 = sizeof(T) == 8;
    constexpr int ES = int(sizeof(cx<T>));
    using SH = sshape<T, N, AX, (MF > 0)>;
    using O = line_order<T, N>;
    if constexpr (AX == 1 && MF <= 0 && N >= 64 && (!F64 || N <= 1024) && (SH::TC * ES) % 128 == 0) {
        if (whole_lines(src, m_cols, lm, 128 / ES) && whole_lines(data, m_cols, lm, 128 / ES)) {
            // mean distance between neighbouring elements of a line
            constexpr int64_t HALF = N / 2;
            const int64_t step = ((HALF >> lm.lg_y) * lm.s_hi +
                                  (HALF & ((int64_t(1) << lm.lg_y) - 1)) * lm.s_lo) / HALF * ES;
            constexpr int64_t FAR = F64 && N == 256 ? int64_t(512) << 10 : int64_t(1) << 62;
            if (step >= 4096 && step < FAR)
                return strided_run<T, N, AX, MF, true>(O::NT, sign, src, data, tw, m_cols, n_b, lm, s);
            if constexpr (N >= 512 || (!F64 && N == 256)) {
                if (step < 4096)
                    return strided_run<T, N, AX, MF, true>(kContig, sign, src, data, tw, m_cols, n_b, lm,
                                                                    s);
            }
        }
    }
    if constexpr (MF <= 0 && (AX == 0 || N <= 32)) {
        // sets that would leave half (from N = 1024), three quarters or (N = 16)
        // 15 of 16 of a tile's lanes idle: 512 MB of N = 16 slabs 9 columns FP64 232
        // us, a tile per set 348, but 18 columns 228 and 209; N = 32 17 columns 210
        // and 500
        if ((N >= 1024 ? 2 : N == 16 ? 16 : 4) * m_cols <= SH::TC && m_cols > 0 && n_b > 1)
            return strided_flat<T, N, AX, MF>(sign, src, data, tw, m_cols, n_b, lm, s);
    }
    // FP64 x lines of 64 in tiles of 32 columns: the 33 of the paper's order would
    // take two (512 MB 240 us, numbered through 208, one tile of 64 204)
    if constexpr (MF <= 0 && AX == 1 && F64 && N == 64) {
        if (m_cols > SH::TC && m_cols < 2 * SH::TC && n_b > 1)
            return strided_flat<T, N, AX, MF>(sign, src, data, tw, m_cols, n_b, lm, s);
    }
    if constexpr (AX == 1 && N <= 256) {
        if (lm.s_lo * ES < 4096)
            return strided_run<T, N, AX, MF, false>(kContig, sign, src, data, tw, m_cols, n_b, lm, s);
    }
    if constexpr (F64 && (N >= 2048 || (AX == 1 && (N == 256 || N == 512))))
        return strided_run<T, N, AX, MF, false>(kContig, sign, src, data, tw, m_cols, n_b, lm, s);
    if constexpr (AX == 0 && (F64 || N == 512 || N == 1024 || (MF > 0 && N == 64))) {
        if ((lm.lg_y >= ilog2_c(N) || N == 512) && lm.s_lo == m_cols)
            return strided_run<T, N, AX, MF, false>(kContig, sign, src, data, tw, m_cols, n_b, lm, s);
    }
    if constexpr (AX == 0 && !F64 && N == 4096) {
        if (whole_lines(data, m_cols, lm, 128 / ES))
            return strided_run<T, N, AX, MF, false>(kContig, sign, src, data, tw, m_cols, n_b, lm, s);
    }
    return strided_run<T, N, AX, MF, false>(kGrouped, sign, src, data, tw, m_cols, n_b, lm, s);
}

template <typename T, int N>
static hipError_t strided_n(int axis, int mfma_terms, int sign, const void* src, void* data,
                            const void* tw, int64_t m_cols, int64_t n_b, line_map lm, hipStream_t s) {
    if (mfma_terms == -1)
        return axis == 0 ? strided_ax<T, N, 0, -1>(sign, src, data, tw, m_cols, n_b, lm, s)
                         : strided_ax<T, N, 1, -1>(sign, src, data, tw, m_cols, n_b, lm, s);
    if constexpr (sizeof(T) == 4 && N >= 32) {
        if (mfma_terms == 2)
            return axis == 0 ? strided_ax<T, N, 0, 2>(sign, src, data, tw, m_cols, n_b, lm, s)
                             : strided_ax<T, N, 1, 2>(sign, src, data, tw, m_cols, n_b, lm, s);
        if (mfma_terms == 3)
            return axis == 0 ? strided_ax<T, N, 0, 3>(sign, src, data, tw, m_cols, n_b, lm, s)
                             : strided_ax<T, N, 1, 3>(sign, src, data, tw, m_cols, n_b, lm, s);
    }
    if (mfma_terms != 0) return hipErrorInvalidValue;
    if (axis == 0) return strided_ax<T, N, 0, 0>(sign, src, data, tw, m_cols, n_b, lm, s);
    return strided_ax<T, N, 1, 0>(sign, src, data, tw, m_cols, n_b, lm, s);
}

#define GFFT_CASES_TO_1024(FN, T, ...)              \
    case 16: return FN<T, 16>(__VA_ARGS__);         \
    case 32: return FN<T, 32>(__VA_ARGS__);         \
    case 64: return FN<T, 64>(__VA_ARGS__);         \
    case 128: return FN<T, 128>(__VA_ARGS__);       \
    case 256: return FN<T, 256>(__VA_ARGS__);       \
    case 512: return FN<T, 512>(__VA_ARGS__);       \
    case 1024: return FN<T, 1024>(__VA_ARGS__);
#define GFFT_DISPATCH_TO_1024(FN, T, ...)           \
    switch (n) {                                    \
        GFFT_CASES_TO_1024(FN, T, __VA_ARGS__)      \
        default: return hipErrorInvalidValue;       \
    }
#define GFFT_DISPATCH_N(FN, T, ...)                 \
    switch (n) {                                    \
        GFFT_CASES_TO_1024(FN, T, __VA_ARGS__)      \
        case 2048: return FN<T, 2048>(__VA_ARGS__); \
        case 4096: return FN<T, 4096>(__VA_ARGS__); \
        default: return hipErrorInvalidValue;       \
    }

hipError_t launch_z_r2c(bool f64, int n, const void* in, void* out, const void* tw,
                        int64_t rows, row_map map, double me, double mi, hipStream_t s) {
    if (n >= 2048) return launch_rows(f64, true, n, 1, in, out, tw, rows, map, me, mi, s);
    if (f64) { GFFT_DISPATCH_TO_1024(z_r2c_n, double, in, out, tw, rows, map, me, mi, s) }
    GFFT_DISPATCH_TO_1024(z_r2c_n, float, in, out, tw, rows, map, me, mi, s)
}

hipError_t launch_z_c2r(bool f64, int n, const void* in, void* out, const void* tw,
                        int64_t rows, row_map map, double me, double mi, hipStream_t s) {
    // FP64 2048 rows in an array of the L2s' size: a row to a 64-thread workgroup
    // and whole-value exchanges (one plane 12.5 us, k_rows_c2r 16.3; 16 planes 227
    // and 196)
    if (f64 && n == 2048 && tile_order(rows * 1025 * 16, kGrouped) == kContig)
        return z_c2r_n<double, 2048>(in, out, tw, rows, map, me, mi, s);
    if (n >= 2048) return launch_rows(f64, false, n, 1, in, out, tw, rows, map, me, mi, s);
    if (f64) { GFFT_DISPATCH_TO_1024(z_c2r_n, double, in, out, tw, rows, map, me, mi, s) }
    GFFT_DISPATCH_TO_1024(z_c2r_n, float, in, out, tw, rows, map, me, mi, s)
}

hipError_t launch_strided(bool f64, int n, int axis, int mfma_terms, int sign, const void* src,
                          void* data, const void* tw, int64_t m_cols, int64_t n_b, line_map lm,
                          hipStream_t s) {
    if (f64) { GFFT_DISPATCH_N(strided_n, double, axis, mfma_terms, sign, src, data, tw, m_cols, n_b, lm, s) }
    GFFT_DISPATCH_N(strided_n, float, axis, mfma_terms, sign, src, data, tw, m_cols, n_b, lm, s)
}

// The y lines a z pass with a first y step leaves (rows_step), in the y tile
// shape of their length and, in TB/s, the faster of the two orders: FP64 128
// of 1024 5.49 grouped, 5.41 contiguous, 1024 of 4096 4.58, 4.68; FP32 32 of
// 512 5.58, 5.78, 64 of 1024 5.55, 5.25, 256 of 2048 5.27, 4.89, 1024 of 4096
// 4.71, 4.39.
hipError_t launch_strided_lines(bool f64, int n, int ny, int sign, const void* src, void* data,
                                const void* tw, int64_t m_cols, int64_t n_b, line_map lm,
                                hipStream_t s) {
#define GFFT_LINES(T, N, NY, ORD)                                                               \
    if (n == N && ny == NY)                                                                     \
        return strided_run<T, N / NY, 0, 0, false, NY>(ORD, sign, src, data, tw, m_cols, n_b, lm, s);
    if (f64) {
        GFFT_LINES(double, 1024, 8, kGrouped)
        GFFT_LINES(double, 2048, 4, kContig)
        GFFT_LINES(double, 4096, 4, kContig)
    } else {
        GFFT_LINES(float, 512, 16, kContig)
        GFFT_LINES(float, 1024, 16, kGrouped)
        GFFT_LINES(float, 2048, 8, kGrouped)
        GFFT_LINES(float, 4096, 4, kGrouped)
    }
#undef GFFT_LINES
    return hipErrorInvalidValue;
}

template <typename V, int U>
static hipError_t pack_u(const void* src, void* dst, int64_t chunks, int lg_x, int lg_p,
                         int64_t x_step, int64_t len, bool to_send, hipStream_t s) {
    if (chunks == 0 || len == 0) return hipSuccess;
    // Whole runs, as many as fill a round of the workgroup, where a run cut into
    // rounds would leave most of its last one idle: up to two rounds (512 MB of
    // FP64 64 16 x 4 pencil runs of 128 elements 171 us, four rounds' worth of
    // runs to a workgroup 193; slab 64/8, 264 elements, 180 and 197), four in
    // arrays of up to 64 MB (FP64 1024/1024, 513 elements, 9.8 us, parts 11.6, but
    // 183 and 176 over 512 MB).  8-byte elements (runs of an odd length, at most
    // N/2 + 1): always, short ones four rounds' worth (FP32 128/128, 65 elements,
    // 185 us, one round's 244; 1024/1024 186, parts 307; 4096/4096 190, 253).
    constexpr bool PAIR = sizeof(V) == 16;
    const int64_t whole = !PAIR ? 8 * kThreads + 1
                          : chunks * len * int64_t(sizeof(V)) <= int64_t(64) << 20 ? 4 * kThreads + 76
                                                                                    : 2 * kThreads;
    const int64_t fill = PAIR || len > 2 * kThreads ? kThreads : 4 * kThreads;
    const bool even = PAIR && len > kThreads && len % kThreads == 0;  // no idle lanes in parts
    const int per = len <= whole && !even ? int((fill + len - 1) / len) : 0;
    int64_t bpc = (len + U * kThreads - 1) / (U * kThreads);
    // k_pack strides over its chunk, so fewer blocks per chunk keep very
    // large grids within the dispatch's 32-bit work-item count
    const int64_t cap = int64_t(0xffffffff) / (chunks * kThreads);
    if (bpc > cap) bpc = cap;
    if (bpc < 1) bpc = 1;
    const int64_t blocks = per > 0 ? (chunks + per - 1) / per : chunks * bpc;
    if (!grid_fits(blocks, kThreads)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_pack<V, U>), dim3(blocks), dim3(kThreads), 0, s,
                       static_cast<const V*>(src), static_cast<V*>(dst), len, chunks, bpc, per,
                       1.0f / float(len), lg_x, lg_p, x_step, to_send);
    return hipGetLastError();
}

// One element per thread, but eight at an eighth of the run apart for runs of a
// power of two (pencils) whose planes are 4 MB or more apart: reads and writes
// then stay a large power of two apart for a whole run, and the spread avoids
// that (4096 64 x 4, planes 4 and 8 MB apart, FP32 396 us against 515, FP64 794
// against 1090; with planes 2 MB or less apart it loses 2-30%: FP64 2048 32 x 4
// 232 against 173).
template <typename V>
static hipError_t pack_v(const void* src, void* dst, int64_t chunks, int lg_x, int lg_p,
                         int64_t x_step, int64_t len, bool to_send, hipStream_t s) {
    if (x_step * int64_t(sizeof(V)) >= int64_t(4) << 20 && len >= 32 * kThreads && (len & (len - 1)) == 0)
        return pack_u<V, 8>(src, dst, chunks, lg_x, lg_p, x_step, len, to_send, s);
    return pack_u<V, 1>(src, dst, chunks, lg_x, lg_p, x_step, len, to_send, s);
}

hipError_t launch_pack(bool f64, const void* src, void* dst, int64_t chunks, int lg_x,
                       int lg_p, int64_t n, int64_t y, int64_t k, bool to_send,
                       hipStream_t s) {
    // every run starts at a multiple of y k values from the 16-byte aligned
    // buffers, so FP32 runs of an even length move as pairs
    const int64_t len = y * k, x_step = n * k;
    if (f64) return pack_v<uint4>(src, dst, chunks, lg_x, lg_p, x_step, len, to_send, s);
    if (len % 2 == 0)
        return pack_v<uint4>(src, dst, chunks, lg_x, lg_p, x_step / 2, len / 2, to_send, s);
    return pack_v<cx<float>>(src, dst, chunks, lg_x, lg_p, x_step, len, to_send, s);
}

hipError_t launch_pack_rows(bool f64, const void* src, void* dst, int64_t rows, int64_t k,
                            row_map map, bool to_send, hipStream_t s) {
    const int64_t blocks = (rows + kPackRows - 1) / kPackRows;
    if (blocks == 0 || k == 0) return hipSuccess;
    if (!grid_fits(blocks, kThreads)) return hipErrorInvalidValue;
    if (f64)
        hipLaunchKernelGGL((k_pack_rows<double>), dim3(blocks), dim3(kThreads), 0, s,
                           static_cast<const cx<double>*>(src), static_cast<cx<double>*>(dst),
                           rows, k, map, to_send);
    else
        hipLaunchKernelGGL((k_pack_rows<float>), dim3(blocks), dim3(kThreads), 0, s,
                           static_cast<const cx<float>*>(src), static_cast<cx<float>*>(dst),
                           rows, k, map, to_send);
    return hipGetLastError();
}

hipError_t launch_copy16(const void* src, void* dst, int64_t n16, hipStream_t s) {
    // at most 2^31 work-items per dispatch; longer copies take several
    constexpr int64_t kMax = int64_t(1) << 31;
    for (int64_t done = 0; done < n16; done += kMax) {
        const int64_t len = n16 - done < kMax ? n16 - done : kMax;
        const int64_t blocks = (len + kThreads - 1) / kThreads;
        hipLaunchKernelGGL(k_copy16, dim3(blocks), dim3(kThreads), 0, s,
                           static_cast<const uint4*>(src) + done, static_cast<uint4*>(dst) + done,
                           len);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace gfft
