// Kernels that run several axes of the transform in one memory pass, and
// their launchers (part of the kernels.hip translation unit).
#pragma once

#include "cx.h"
#include "engine.h"
#include "kernels.h"
#include "pass_common.h"

namespace gfft {

// p advanced by a 32-bit byte offset: a uniform pointer and one vector
// register address the element.
template <typename C>
__device__ __forceinline__ const C* at_bytes(const C* p, uint32_t off) {
    return reinterpret_cast<const C*>(reinterpret_cast<const char*>(p) + off);
}
template <typename C>
__device__ __forceinline__ C* at_bytes(C* p, uint32_t off) {
    return reinterpret_cast<C*>(reinterpret_cast<char*>(p) + off);
}

// Hermitian part of a pair of bins, v at k and u at -k.  A bin that is its own
// partner keeps its real part, whatever its imaginary part holds (infinities and
// NaN too): the transform of a real field has none there.
template <typename T>
__device__ __forceinline__ cx<T> hermitian(cx<T> v, cx<T> u, bool own) {
    return {T(0.5) * (v.x + u.x), own ? T(0) : T(0.5) * (v.y - u.y)};
}

// FFT stages of R transforms side by side per thread (a[y], y < R), sharing
// their twiddles and barriers; exchanges through LDS as real, then imaginary
// parts.  Column c of TC; transform y occupies its own padded N x TC block.
// gap0, gap1: other work for the first exchange, beside the reads of the real
// and of the imaginary parts.
struct no_gap {
    __device__ void operator()() const {}
};
template <typename T, int N, int E, int R, int S, int L, int RM, int TC, int PS, class G0 = no_gap,
          class G1 = no_gap>
__device__ __forceinline__ void fft_multi(cx<T> (&a)[R][E], int t, int c, const cx<T>* __restrict__ tw,
                                          int tws, T* lds, G0 gap0 = {}, G1 gap1 = {}) {
    constexpr int RX = stage_radix<N, E, L, RM>::value;
    constexpr int NB = E / RX, TPT = N / E;
    constexpr int NP = padded_len<N, PS>::value;
#pragma unroll
    for (int q = 0; q < NB; ++q) {
        const int j = t + q * TPT;
        const int k = j & (L - 1);
        cx<T> w[RX];
        if constexpr (L > 1) {
#pragma unroll
            for (int r = 1; r < RX; ++r) w[r] = tw[r * k * (N / (L * RX)) * tws];
        }
#pragma unroll
        for (int y = 0; y < R; ++y) {
            cx<T> b[RX];
#pragma unroll
            for (int r = 0; r < RX; ++r) b[r] = a[y][q + r * NB];
            if constexpr (L > 1) {
#pragma unroll
                for (int r = 1; r < RX; ++r) b[r] = twiddle<S>(b[r], w[r]);
            }
            dft<RX, S>(b);
#pragma unroll
            for (int r = 0; r < RX; ++r) a[y][q + r * NB] = b[r];
        }
    }
    if constexpr (L * RX < N) {
        using G = xgeom<N, E, L, RX>;
        using IX = idx_cols<TC, PS>;
        const IX ix{c};
#pragma unroll
        for (int part = 0; part < 2; ++part) {
#pragma unroll
            for (int y = 0; y < R; ++y)
#pragma unroll
                for (int s = 0; s < E; ++s)
                    lds[y * NP * TC + ix.at(G::template out_pad<PS>(t, s))] = part ? a[y][s].y : a[y][s].x;
            __syncthreads();
            if (part == 0) gap0();
            else gap1();
#pragma unroll
            for (int y = 0; y < R; ++y)
#pragma unroll
                for (int m = 0; m < E; ++m) {
                    const T v = lds[y * NP * TC + ix.at(G::template in_pad<PS>(t, m))];
                    if (part) a[y][m].y = v;
                    else a[y][m].x = v;
                }
            __syncthreads();
        }
        fft_multi<T, N, E, R, S, L * RX, RM, TC, PS>(a, t, c, tw, tws, lds);
    }
}

// The real column kz = M of a tile's N rows beside the tile's own work: stage I
// of its forward transform, run by threads t < N/4 between two of the tile's
// barriers.  keep() takes Re Z[0] of every row from the column exchange, stage 0
// X[M] = Re Z[0] - Im Z[0], stage I buf[I % 2]; each writes the other buffer, the
// last in natural order.  Four values a thread, as these come on top of the
// tile's own (8 or 16 would cost FP64 a wave per SIMD, or spill).
template <typename T, int N>
struct side_column {
    static constexpr int E = 4, THREADS = N / E;
    static constexpr int PS = first_radix_shift<E>::value, NP = padded_len<N, PS>::value;
    static constexpr int STAGES = (ilog2_c(N) + 1) / 2;

    cx<T> (*buf)[NP];
    // re, im: row 0's part in the exchange buffer, rows LD apart
    template <int LD>
    __device__ __forceinline__ void keep(int t, const T* re) const {
        if (t >= THREADS) return;
#pragma unroll
        for (int m = 0; m < E; ++m) buf[0][lds_pad<PS>(t + m * THREADS)].x = re[(t + m * THREADS) * LD];
    }
    template <int LD>
    __device__ __forceinline__ void first(int t, const T* im, T mul) const {
        if (t >= THREADS) return;
        cx<T> e[E];
#pragma unroll
        for (int m = 0; m < E; ++m) {
            const int n = t + m * THREADS;
            e[m] = cx<T>{(buf[0][lds_pad<PS>(n)].x - im[n * LD]) * mul, T(0)};
        }
        run<0>(e, t, nullptr, 0);
    }
    template <int I>
    __device__ __forceinline__ void stage(int t, const cx<T>* __restrict__ tw, int tws) const {
        if constexpr (I < STAGES) {
            if (t >= THREADS) return;
            cx<T> e[E];
#pragma unroll
            for (int m = 0; m < E; ++m) e[m] = buf[I % 2][lds_pad<PS>(t + m * THREADS)];
            run<I>(e, t, tw, tws);
        }
    }
    template <int I>
    __device__ __forceinline__ void run(cx<T> (&e)[E], int t, const cx<T>* __restrict__ tw,
                                        int tws) const {
        constexpr int L = 1 << (2 * I);
        using G = xgeom<N, E, L, stage_radix<N, E, L>::value>;
        fft_stage<T, N, E, -1, L, 16>(e, t, tw, tws);
#pragma unroll
        for (int m = 0; m < E; ++m) buf[(I + 1) % 2][G::template out_pad<PS>(t, m)] = e[m];
    }
    __device__ __forceinline__ cx<T> get(int k) const { return buf[STAGES % 2][lds_pad<PS>(k)]; }
};

// ---------------------------------------------------------------- plane 2D R2C / C2R
// z R2C and y C2C of one x-plane (section 3, step 1; R = 1), or of every R-th
// row of it, in one kernel with the rows held in registers.  With R > 1 the
// y transform is split as N = NY R (y = y0 + R j, ky = k1 + NY k0): a tile
// takes the NY rows of one y0, transforms them along z and j, and writes
// bin k1 to row y0 NY + k1; the strided pass that follows (k_strided_r)
// reads the R rows {y0 NY + k1} of one k1, applies the twiddles W_N^(y0 k1)
// and the R-point DFT over y0, and writes the rows {k1 + NY k0} -- the same
// rows, so that pass stays in place.  The inverse runs the same steps
// backwards.
//   z phase: thread (r, t), r < NY rows, t < TZ = M/E, holds z[t + TZ m] of
//            row r (z[n] = x[2n] + i x[2n+1]); M-point FFT;
//   y phase: thread (s, p), p < M/2, holds columns p and M - p at rows
//            s + TY m, m < E/2; two NY-point FFTs.
// Between the phases the tile moves through LDS, real parts then imaginary
// parts.  The column pair makes the real split (bin k from Z[k] and Z[M-k];
// the inverse's pre-process likewise) a register operation with one twiddle
// per thread.  Columns 0 and M/2, their own partners, share thread p = 0.
// The z half spectrum has M + 1 columns.  Forward, column M is a side_column
// of the first TY threads, in the gaps of the column exchange: as the
// imaginary part of column 0 (both are real for a real row) it would take on
// rounding errors of column 0's size, 1.4 to 2.4 times its own in FP32 on
// fields that vary slowly along z.  The inverse does pack the two, P = G0 + i GM
// of their Hermitian parts (the C2R keeps only the real part of those columns
// after the y inverse, which is the inverse of their Hermitian parts; this
// holds for the rows of one y0 by themselves, which are real sequences in j):
// there they are summed into the same real row right after.  Every load of a
// tile precedes the first barrier and
// every store follows the last, so with R = 1 a plane may be transformed in
// place.
// TWD: the tile applies the twiddles W_N^(y0 k1) itself, which leaves an
// ordinary R-point y pass (rows follow `map`, NY of them contiguous), as in
// k_rows_*.
template <typename T, int N, int R, int E>
struct plane_shape {
    static constexpr int M = N / 2, K = M + 1, NY = N / R, H = M / 2;
    static constexpr int EY = E / 2;
    static constexpr int TZ = M / E, TY = NY / EY;
    static constexpr int NT = NY * TZ;  // = H * TY
    static constexpr int RM = radix_cap<T>();
    static constexpr int PS = TZ > 1 ? first_radix_shift<E, RM>::value : 0;
    static constexpr int MP = padded_len<M, PS>::value;
    // column exchange: padded where a row of H values covers fewer than all
    // 64 banks, so that the rows a wave touches fall on different ones
    static constexpr int PY = H * int(sizeof(T)) / 4 >= 64 ? 0 : first_radix_shift<EY, RM>::value;
    static constexpr int NP = padded_len<NY, PY>::value;
    // row stride of the transpose buffer: a wave's lanes are TZ values of
    // 64/TZ rows, so rows are staggered by TZ banks
    static constexpr int LD = M + TZ;
    static constexpr int A = TZ > 1 ? NY * MP : 0, B = TY > 1 ? NP * M : 0, C = NY * LD,
                         D = 6 * NY;
    static constexpr int AB = A > B ? A : B, CD = C > D ? C : D;
    static constexpr int LDS = AB > CD ? AB : CD;  // values of type T
    using nyquist = side_column<T, NY>;
    static_assert(M % E == 0 && NY % EY == 0 && NY * TZ == H * TY, "plane shape");
    static_assert(nyquist::THREADS <= NT && nyquist::STAGES <= (TY > 1 ? 4 : 2),
                  "a barrier follows every stage of the side column");
};

template <typename T, int N, int R, int E, int W, bool TWD = false>
__global__ __launch_bounds__((plane_shape<T, N, R, E>::NT), W) void k_plane_r2c(
    const T* in, cx<T>* out, const cx<T>* __restrict__ tw, row_map map, T mul_edge, T mul_int, int ord) {
    using P = plane_shape<T, N, R, E>;
    constexpr int M = P::M, K = P::K, H = P::H, NY = P::NY, TZ = P::TZ, TY = P::TY, EY = P::EY,
                  RM = P::RM;
    __shared__ T lds[P::LDS];
    const int64_t tile = xcd_tile(ord, blockIdx.x, gridDim.x);
    const int64_t plane = tile / R;
    const int y0 = int(tile % R);
    const int tid = threadIdx.x;
    const int r = tid / TZ, t = tid % TZ;          // z phase
    const int p = tid % H, s = TY == 1 ? 0 : tid / H;  // y phase
    const int c1 = p == 0 ? H : M - p;             // columns p and c1

    // z phase: row y0 + R r of the plane, read as M complex values
    cx<T> a[E];
    const cx<T>* src = reinterpret_cast<const cx<T>*>(in + (plane * N + y0 + R * r) * map.rs);
#pragma unroll
    for (int m = 0; m < E; ++m) a[m] = src[t + TZ * m];
    using IR = idx_rows<P::PS>;
    fft_regs<T, M, E, -1, RM>(a, t, tw, 2, xch_split<T, IR>{lds, IR{r * P::MP}});

    // rows -> columns, and the side column's stages after the barriers
    __shared__ cx<T> nyq[2][P::nyquist::NP];
    const typename P::nyquist col_m{nyq};
    const cx<T> w = tw[p];
    cx<T> b[2][EY];
#pragma unroll
    for (int m = 0; m < E; ++m) lds[r * P::LD + t + TZ * m] = a[m].x;
    __syncthreads();
    col_m.template keep<P::LD>(tid, lds);
#pragma unroll
    for (int m = 0; m < EY; ++m) {
        b[0][m].x = lds[(s + TY * m) * P::LD + p];
        b[1][m].x = lds[(s + TY * m) * P::LD + c1];
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < E; ++m) lds[r * P::LD + t + TZ * m] = a[m].y;
    __syncthreads();
#pragma unroll
    for (int m = 0; m < EY; ++m) {
        b[0][m].y = lds[(s + TY * m) * P::LD + p];
        b[1][m].y = lds[(s + TY * m) * P::LD + c1];
    }
    col_m.template first<P::LD>(tid, lds, mul_edge);
    __syncthreads();
    col_m.template stage<1>(tid, tw, R);
    // real split, bin multipliers applied: with A = (Z[p] + conj Z[M-p])/2,
    // B = (Z[p] - conj Z[M-p])/2 and w = W_N^p,
    //   X[p] = A - i w B,  X[M-p] = conj(A + i w B);
    // p = 0: X[0] = Re Z[0] + Im Z[0], and column M/2 is its own conjugate.
    const bool edge = p == 0;
#pragma unroll
    for (int m = 0; m < EY; ++m) {
        const cx<T> z = b[0][m], v = b[1][m];
        const cx<T> A = scal(z + conjg(v), T(0.5)), B = cmul(w, scal(z - conjg(v), T(0.5)));
        b[0][m].x = edge ? (z.x + z.y) * mul_edge : (A.x + B.y) * mul_int;
        b[0][m].y = edge ? T(0) : (A.y - B.x) * mul_int;
        b[1][m].x = edge ? v.x * mul_int : (A.x - B.y) * mul_int;
        b[1][m].y = edge ? -v.y * mul_int : (-A.y - B.x) * mul_int;
    }

    // y phase: NY-point FFTs of columns p and c1
    fft_multi<T, NY, EY, 2, -1, 1, RM, H, P::PY>(
        b, s, p, tw, R, lds, [&] { col_m.template stage<2>(tid, tw, R); },
        [&] { col_m.template stage<3>(tid, tw, R); });
    if constexpr (TY == 1) __syncthreads();  // the side column's last stage

    // All of b before the first store: otherwise the last stage is spread over
    // the stores and FP32 N = 256 (E = 32) spills 24 registers.
#pragma unroll
    for (int m = 0; m < EY; ++m)
        asm volatile("" : "+v"(b[0][m].x), "+v"(b[0][m].y), "+v"(b[1][m].x), "+v"(b[1][m].y));
    // store rows of the half spectrum: wave lanes are consecutive columns
    auto row_of = [&](int k1) {
        const int64_t row = plane * N + y0 * NY + k1;
        return out + (R > 1 && !TWD ? row : map_row(row, map)) * K;
    };
    // twiddles first: a load behind the stores would wait for them
    cx<T> xm{};
    if (tid < NY) xm = col_m.get(tid);
    if constexpr (TWD) {
        if (tid < NY) xm = cmul(xm, tw[y0 * tid]);
#pragma unroll
        for (int m = 0; m < EY; ++m) {
            const cx<T> wm = tw[y0 * (s + TY * m)];
            b[0][m] = cmul(b[0][m], wm);
            b[1][m] = cmul(b[1][m], wm);
        }
    }
#pragma unroll
    for (int m = 0; m < EY; ++m) {
        cx<T>* dst = row_of(s + TY * m);
        dst[p] = b[0][m];
        dst[c1] = b[1][m];
    }
    if (tid < NY) row_of(tid)[M] = xm;
}

template <typename T, int N, int R, int E, int W, bool TWD = false>
__global__ __launch_bounds__((plane_shape<T, N, R, E>::NT), W) void k_plane_c2r(
    const cx<T>* in, T* out, const cx<T>* __restrict__ tw, row_map map, T mul_edge, T mul_int, int ord) {
    using P = plane_shape<T, N, R, E>;
    constexpr int M = P::M, K = P::K, H = P::H, NY = P::NY, TZ = P::TZ, TY = P::TY, EY = P::EY,
                  RM = P::RM;
    __shared__ T lds[P::LDS];
    const int64_t tile = xcd_tile(ord, blockIdx.x, gridDim.x);
    const int64_t plane = tile / R;
    const int y0 = int(tile % R);
    const int tid = threadIdx.x;
    const int r = tid / TZ, t = tid % TZ;
    const int p = tid % H, s = TY == 1 ? 0 : tid / H;
    const int c1 = p == 0 ? H : M - p;

    // y phase input: columns p and c1 of the half spectrum; column 0 is
    // replaced by the Hermitian parts of kz = 0 (real) and kz = M
    // (imaginary), formed through LDS by one thread per row
    auto row_of = [&](int k1) {
        const int64_t row = plane * N + y0 * NY + k1;
        return in + (R > 1 && !TWD ? row : map_row(row, map)) * K;
    };
    // k1 = 0 is left as it is: a product with 1 - 0i makes NaN of an infinite
    // imaginary part
    auto turn = [&](cx<T> v, int k1) { return TWD && k1 != 0 ? cmulc(v, tw[y0 * k1]) : v; };
    cx<T> b[2][EY];
    cx<T>* col0 = reinterpret_cast<cx<T>*>(lds);
#pragma unroll
    for (int m = 0; m < EY; ++m) {
        const cx<T>* g = row_of(s + TY * m);
        b[0][m] = g[p];
        b[1][m] = g[c1];
    }
    if constexpr (TWD) {
#pragma unroll
        for (int m = 0; m < EY; ++m) {
            b[0][m] = turn(b[0][m], s + TY * m);
            b[1][m] = turn(b[1][m], s + TY * m);
        }
    }
    if (tid < NY) {
        const cx<T>* g = row_of(tid);
        col0[tid] = turn(g[0], tid);
        col0[NY + tid] = turn(g[M], tid);
    }
    __syncthreads();
    if (tid < NY) {
        const int kn = (NY - tid) & (NY - 1);
        const cx<T> h0 = hermitian(col0[tid], col0[kn], tid == kn);
        const cx<T> hm = hermitian(col0[NY + tid], col0[NY + kn], tid == kn);
        col0[2 * NY + tid] = cx<T>{h0.x - hm.y, h0.y + hm.x};  // h0 + i hm
    }
    __syncthreads();
    if (p == 0) {
#pragma unroll
        for (int m = 0; m < EY; ++m) b[0][m] = col0[2 * NY + s + TY * m];
    }
    __syncthreads();
    fft_multi<T, NY, EY, 2, +1, 1, RM, H, P::PY>(b, s, p, tw, R, lds);

    // pre-process of the row C2R, bin multipliers applied: with
    // S = G[p] + conj G[M-p], D = G[p] - conj G[M-p], w = W_N^p,
    //   Z'[p] = S + i conj(w) D,  Z'[M-p] = conj(S - i conj(w) D);
    // p = 0: column 0 holds the real bins (G[0], G[M]) and becomes
    // Z'[0] = (G[0] + G[M], G[0] - G[M]); Z'[M/2] = 2 conj G[M/2].
    const cx<T> w = tw[p];
    const bool edge = p == 0;
#pragma unroll
    for (int m = 0; m < EY; ++m) {
        const cx<T> z = b[0][m], u = conjg(b[1][m]);
        const cx<T> S = scal(z + u, mul_int), D = cmulc(scal(z - u, mul_int), w);
        b[0][m].x = edge ? (z.x + z.y) * mul_edge : S.x - D.y;
        b[0][m].y = edge ? (z.x - z.y) * mul_edge : S.y + D.x;
        b[1][m].x = edge ? u.x * (T(2) * mul_int) : S.x + D.y;
        b[1][m].y = edge ? u.y * (T(2) * mul_int) : D.x - S.y;
    }

    // columns -> rows
    cx<T> g[E];
#pragma unroll
    for (int m = 0; m < EY; ++m) {
        lds[(s + TY * m) * P::LD + p] = b[0][m].x;
        lds[(s + TY * m) * P::LD + c1] = b[1][m].x;
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < E; ++m) g[m].x = lds[r * P::LD + t + TZ * m];
    __syncthreads();
#pragma unroll
    for (int m = 0; m < EY; ++m) {
        lds[(s + TY * m) * P::LD + p] = b[0][m].y;
        lds[(s + TY * m) * P::LD + c1] = b[1][m].y;
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < E; ++m) g[m].y = lds[r * P::LD + t + TZ * m];
    __syncthreads();
    using IR = idx_rows<P::PS>;
    fft_regs<T, M, E, +1, RM>(g, t, tw, 2, xch_split<T, IR>{lds, IR{r * P::MP}});
    cx<T>* dst = reinterpret_cast<cx<T>*>(out + (plane * N + y0 + R * r) * map.rs);
#pragma unroll
    for (int m = 0; m < E; ++m) {
        // real rows past a y step are long: not read again soon, they leave the
        // memory cache to the half spectrum (256 MB of reals, FP64 1024 207 -> 151
        // us an inverse, FP32 512 196 -> 152; pairs of 64 MB FP32 512 88 -> 91)
        if constexpr (TWD) {
            __builtin_nontemporal_store(g[m].x, &dst[t + TZ * m].x);
            __builtin_nontemporal_store(g[m].y, &dst[t + TZ * m].y);
        } else {
            dst[t + TZ * m] = g[m];
        }
    }
}

// ---------------------------------------------------------------- long rows: z with a short y step
// z R2C of long rows, NY rows at a time:
// with N = NY R, y = y0 + R j, ky = k1 + NY k0, a tile takes the NY rows of
// one y0 through z and the NY-point DFT over j, applies W_N^(y0 k1) and
// writes bin k1 to row y0 NY + k1; what is left of the y transform is an
// R-point strided pass over n = y0 (rows n NY + k1, in place), an ordinary
// k_strided of shorter lines.  NY = 1 is a plain z pass.  As in k_plane_*,
// thread (r, t) transforms row r, thread p then holds the columns p and M - p
// (p = lt + NT1 q, q < Q) of all NY rows, so the real split and the y step
// need no further exchange.  Thread 0 takes column M besides 0 and M/2; the
// inverse packs the Hermitian parts of 0 and M into one, as in k_plane_c2r.
// Exchanges are split into real and imaginary parts: whole values would
// leave 4 waves on a CU at N = 4096.  Out of place for NY > 1.
template <typename T, int N, int NY, int E, int G>
struct rows_shape {
    static constexpr int M = N / 2, K = M + 1, H = M / 2, R = N / NY;
    static constexpr int TZ = M / E, NT1 = NY * TZ, NT = G * NT1, Q = H / NT1;
    static constexpr int RM = radix_cap<T>();
    static constexpr int PS = first_radix_shift<E, RM>::value;
    static constexpr int MP = padded_len<M, PS>::value;
    static constexpr int LD = TZ < 64 ? M + TZ : M;
    static constexpr int SZ = NY * (MP > LD ? MP : LD);  // values of type T per tile
    static_assert(Q >= 1 && Q * NT1 == H, "rows shape");
};

template <typename T, int N, int NY, int E, int G, int W, bool PENCIL>
__global__ __launch_bounds__((rows_shape<T, N, NY, E, G>::NT), W) void k_rows_r2c(
    const T* in, cx<T>* out, const cx<T>* __restrict__ tw, int64_t tiles, row_map map, T mul_edge,
    T mul_int, int ord) {
    using P = rows_shape<T, N, NY, E, G>;
    constexpr int M = P::M, K = P::K, H = P::H, R = P::R, TZ = P::TZ, NT1 = P::NT1, Q = P::Q,
                  RM = P::RM, LD = P::LD;
    __shared__ T lds_all[G * P::SZ];
    // whole waves belong to one tile: its row addresses stay in scalar registers
    const int grp = NT1 % 64 == 0 ? __builtin_amdgcn_readfirstlane(int(threadIdx.x) / NT1)
                                  : int(threadIdx.x) / NT1;
    const int lt = threadIdx.x % NT1;
    T* lds = lds_all + grp * P::SZ;
    const int r = lt / TZ, t = lt % TZ;
    const int64_t blk = xcd_tile(ord, blockIdx.x, gridDim.x);
    const int64_t tile = blk * G + grp;
    const bool valid = tile < tiles;
    // tiles past the end (last workgroup) load the last tile and drop it
    const int64_t tl = valid ? tile : tiles - 1;
    const int64_t plane = NY > 1 ? tl / R : 0;
    const int y0 = NY > 1 ? int(tl % R) : 0;
    const int64_t row0 = NY > 1 ? plane * N + y0 : tl;

    cx<T> a[E];
    const cx<T>* src = reinterpret_cast<const cx<T>*>(in + (row0 + R * r) * map.rs);
#pragma unroll
    for (int m = 0; m < E; ++m) a[m] = src[t + TZ * m];
    using IR = idx_rows<P::PS>;
    fft_regs<T, M, E, -1, RM>(a, t, tw, 2, xch_split<T, IR>{lds, IR{r * P::MP}});

    cx<T> b[Q][2][NY];
#pragma unroll
    for (int part = 0; part < 2; ++part) {
#pragma unroll
        for (int m = 0; m < E; ++m) lds[r * LD + t + TZ * m] = part ? a[m].y : a[m].x;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int p = lt + NT1 * q, c1 = p == 0 ? H : M - p;
#pragma unroll
            for (int j = 0; j < NY; ++j) {
                const T u = lds[j * LD + p], v = lds[j * LD + c1];
                if (part) {
                    b[q][0][j].y = u;
                    b[q][1][j].y = v;
                } else {
                    b[q][0][j].x = u;
                    b[q][1][j].x = v;
                }
            }
        }
        if (part == 0) __syncthreads();
    }
    if (!valid) return;

    // all twiddles before the first store: a load behind it would wait for it
    // (FP64 with a y step has few columns and no registers to spare: 3.60 ms
    // without, 3.73 with at N = 4096)
    constexpr bool WQ = sizeof(T) == 4 || NY == 1;
    cx<T> wy[NY], wq[Q];
#pragma unroll
    for (int k1 = 1; k1 < NY; ++k1) wy[k1] = tw[y0 * k1];
#pragma unroll
    for (int q = 0; q < Q; ++q) wq[q] = WQ ? tw[lt + NT1 * q] : cx<T>{};
    auto row_of = [&](int k1) {
        return out + map_row(NY > 1 ? plane * N + y0 * NY + k1 : tl, map) * K;
    };
    auto put = [&](int k1, int k, cx<T> v) {
        if constexpr (PENCIL) out[pencil_bin(tl, k, K, map)] = v;
        else row_of(k1)[k] = v;
    };
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int p = lt + NT1 * q, c1 = p == 0 ? H : M - p;
        const cx<T> w = WQ ? wq[q] : tw[p];
        const bool edge = p == 0;
        if (q == 0 && edge) {
            // X[M] = Re Z[0] - Im Z[0], a real column; before the others, as FP64
            // with a y step has no registers to spare
            cx<T> xm[NY];
#pragma unroll
            for (int j = 0; j < NY; ++j)
                xm[j] = cx<T>{(b[0][0][j].x - b[0][0][j].y) * mul_edge, T(0)};
            dft<NY, -1>(xm);
#pragma unroll
            for (int k1 = 0; k1 < NY; ++k1) put(k1, M, k1 > 0 ? cmul(xm[k1], wy[k1]) : xm[k1]);
        }
        cx<T> u[NY], v[NY];
#pragma unroll
        for (int j = 0; j < NY; ++j) {
            const cx<T> z = b[q][0][j], y = b[q][1][j];
            const cx<T> A = scal(z + conjg(y), T(0.5)), B = cmul(w, scal(z - conjg(y), T(0.5)));
            u[j].x = edge ? (z.x + z.y) * mul_edge : (A.x + B.y) * mul_int;
            u[j].y = edge ? T(0) : (A.y - B.x) * mul_int;
            v[j].x = edge ? y.x * mul_int : (A.x - B.y) * mul_int;
            v[j].y = edge ? -y.y * mul_int : (-A.y - B.x) * mul_int;
        }
        dft<NY, -1>(u);
        dft<NY, -1>(v);
#pragma unroll
        for (int k1 = 0; k1 < NY; ++k1) {
            put(k1, p, k1 > 0 ? cmul(u[k1], wy[k1]) : u[k1]);
            put(k1, c1, k1 > 0 ? cmul(v[k1], wy[k1]) : v[k1]);
        }
    }
}

template <typename T, int N, int NY, int E, int G, int W, bool PENCIL>
__global__ __launch_bounds__((rows_shape<T, N, NY, E, G>::NT), W) void k_rows_c2r(
    const cx<T>* in, T* out, const cx<T>* __restrict__ tw, int64_t tiles, row_map map, T mul_edge,
    T mul_int, int ord) {
    using P = rows_shape<T, N, NY, E, G>;
    constexpr int M = P::M, K = P::K, H = P::H, R = P::R, TZ = P::TZ, NT1 = P::NT1, Q = P::Q,
                  RM = P::RM, LD = P::LD;
    __shared__ T lds_all[G * P::SZ];
    // whole waves belong to one tile: its row addresses stay in scalar registers
    const int grp = NT1 % 64 == 0 ? __builtin_amdgcn_readfirstlane(int(threadIdx.x) / NT1)
                                  : int(threadIdx.x) / NT1;
    const int lt = threadIdx.x % NT1;
    T* lds = lds_all + grp * P::SZ;
    const int r = lt / TZ, t = lt % TZ;
    const int64_t blk = xcd_tile(ord, blockIdx.x, gridDim.x);
    const int64_t tile = blk * G + grp;
    const bool valid = tile < tiles;
    const int64_t tl = valid ? tile : tiles - 1;
    const int64_t plane = NY > 1 ? tl / R : 0;
    const int y0 = NY > 1 ? int(tl % R) : 0;

    auto get = [&](int k1, int k) {
        if constexpr (PENCIL) return in[pencil_bin(tl, k, K, map)];
        else return in[map_row(NY > 1 ? plane * N + y0 * NY + k1 : tl, map) * K + k];
    };
    cx<T> b[Q][2][NY];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int p = lt + NT1 * q, c1 = p == 0 ? H : M - p;
#pragma unroll
        for (int k1 = 0; k1 < NY; ++k1) {
            b[q][0][k1] = get(k1, p);
            b[q][1][k1] = get(k1, c1);
        }
    }
    cx<T> wy[NY];
#pragma unroll
    for (int k1 = 1; k1 < NY; ++k1) wy[k1] = tw[y0 * k1];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int p = lt + NT1 * q;
        const cx<T> w = tw[p];
        const bool edge = p == 0;
#pragma unroll
        for (int k1 = 1; k1 < NY; ++k1) {
            b[q][0][k1] = cmulc(b[q][0][k1], wy[k1]);
            b[q][1][k1] = cmulc(b[q][1][k1], wy[k1]);
        }
        if (q == 0 && edge) {
            // column 0: Hermitian parts (over the NY values of k1) of kz = 0
            // (real) and kz = M (imaginary)
            cx<T> g[NY], h[NY];
#pragma unroll
            for (int k1 = 0; k1 < NY; ++k1) {
                h[k1] = get(k1, M);
                if (k1 > 0) h[k1] = cmulc(h[k1], wy[k1]);
            }
#pragma unroll
            for (int k1 = 0; k1 < NY; ++k1) {
                constexpr auto kn = [](int k) { return (NY - k) % NY; };
                const cx<T> h0 = hermitian(b[0][0][k1], b[0][0][kn(k1)], k1 == kn(k1));
                const cx<T> hm = hermitian(h[k1], h[kn(k1)], k1 == kn(k1));
                g[k1] = cx<T>{h0.x - hm.y, h0.y + hm.x};
            }
#pragma unroll
            for (int k1 = 0; k1 < NY; ++k1) b[0][0][k1] = g[k1];
        }
        dft<NY, +1>(b[q][0]);
        dft<NY, +1>(b[q][1]);
#pragma unroll
        for (int j = 0; j < NY; ++j) {
            const cx<T> z = b[q][0][j], u = conjg(b[q][1][j]);
            const cx<T> S = scal(z + u, mul_int), D = cmulc(scal(z - u, mul_int), w);
            b[q][0][j].x = edge ? (z.x + z.y) * mul_edge : S.x - D.y;
            b[q][0][j].y = edge ? (z.x - z.y) * mul_edge : S.y + D.x;
            b[q][1][j].x = edge ? u.x * (T(2) * mul_int) : S.x + D.y;
            b[q][1][j].y = edge ? u.y * (T(2) * mul_int) : D.x - S.y;
        }
    }
    cx<T> a[E];
#pragma unroll
    for (int part = 0; part < 2; ++part) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int p = lt + NT1 * q, c1 = p == 0 ? H : M - p;
#pragma unroll
            for (int j = 0; j < NY; ++j) {
                lds[j * LD + p] = part ? b[q][0][j].y : b[q][0][j].x;
                lds[j * LD + c1] = part ? b[q][1][j].y : b[q][1][j].x;
            }
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < E; ++m) {
            const T v = lds[r * LD + t + TZ * m];
            if (part) a[m].y = v;
            else a[m].x = v;
        }
        __syncthreads();
    }
    using IR = idx_rows<P::PS>;
    fft_regs<T, M, E, +1, RM>(a, t, tw, 2, xch_split<T, IR>{lds, IR{r * P::MP}});
    if (!valid) return;
    const int64_t row0 = NY > 1 ? plane * N + y0 : tl;
    cx<T>* dst = reinterpret_cast<cx<T>*>(out + (row0 + R * r) * map.rs);
#pragma unroll
    for (int m = 0; m < E; ++m) {
        __builtin_nontemporal_store(a[m].x, &dst[t + TZ * m].x);
        __builtin_nontemporal_store(a[m].y, &dst[t + TZ * m].y);
    }
}

// ---------------------------------------------------------------- whole grids of N = 16 and 32
// The whole 3D transform of one small grid per workgroup: one read, one
// write, one launch.  A grid is N N M complex values z (M = N/2, z[n] =
// x[2n] + i x[2n+1] along z), one line of N values (or two of M along z) per
// thread, so every axis is a register transform and the grid only moves
// through LDS between them:
//   thread tid = (y, z) = y M + z    holds the x line of (y, z),
//          tid = (x, z) = x M + z    the y line,
//          l = x N + y, l = tid and tid + NT, the two z lines.
// Forward, z comes first and its real split follows in the registers of the two
// lines, so that y and x act on every kz by itself, with rounding errors of its
// own size (y first, on the packed grid, spreads those of a strong kz = 0 over
// all kz: 500 times the error at kz = 1 in FP32 where kz = 0 is 1000 times
// larger).  kz = 0 and kz = M are real N x N images; each takes half of the
// slots of one column, pairs of its rows as real and imaginary parts:
// T(x', y) = X(2x', y) + i X(2x' + 1, y), kz = 0 in slots 2x', kz = M in
// 2x' + 1.  y runs on these as on any column, x as two N/2-point transforms, and
// with C = conj T(-kx, -ky), E = (T + C)/2, O = (T - C)/2i the image's transform
// is E + W_N^kx O at kx and E - W_N^kx O at kx + N/2.
// The inverse forms Z' = (G + P) + i conj(W_N^kz) (G - P), P = conj G(-kx, -ky,
// M - kz), with the Hermitian parts of kz = 0 and kz = M at kz = 0 (their
// anti-Hermitian parts do not reach the real field), and runs the 3D transform
// of the packed grid.  The forward reads its z lines as they lie (the caches
// gather them; through y lines and an exchange 333 grids of FP32 N = 32 take 30
// us instead of 28).  Exchanges go real parts first, then imaginary parts.  Row
// stride M + 1 and plane stride N (M + 1) + M keep the lanes of all three line
// orders on different LDS banks (and leave room for the M + 1 columns of a half
// spectrum).  All loads precede the first barrier and all stores follow the last:
// grids may be transformed in place.
template <typename T, int N>
struct box_shape {
    static constexpr int M = N / 2, K = M + 1, NT = N * M;
    static constexpr int SY = M + 1, SX = N * SY + M;
    static constexpr int LDS = N * SX;                     // values of type T
    static constexpr int W = sizeof(T) == 8 && N == 32 ? 2 : 4;  // waves per SIMD
    static_assert(LDS >= 6 * N * N, "room for the packed columns");
};

// LDS exchange of the grid between two line orders: value m of the thread
// goes to from(m) and value m of the new line is read at to(m).
template <int N, typename T, class F, class G>
__device__ __forceinline__ void box_exchange(T* lds, cx<T> (&a)[N], F&& from, G&& to) {
#pragma unroll
    for (int part = 0; part < 2; ++part) {
#pragma unroll
        for (int m = 0; m < N; ++m) lds[from(m)] = part ? a[m].y : a[m].x;
        __syncthreads();
#pragma unroll
        for (int m = 0; m < N; ++m) {
            const T v = lds[to(m)];
            if (part) a[m].y = v;
            else a[m].x = v;
        }
        __syncthreads();
    }
}

// N-point DFT as the two N/2-point DFTs of the even and odd inputs, joined, or
// left as they are in the halves of a.
template <int N, int S, typename T>
__device__ __forceinline__ void dft_halves(cx<T>* a, const cx<T>* __restrict__ tw, bool join) {
    cx<T> e[N / 2], o[N / 2];
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
        e[i] = a[2 * i];
        o[i] = a[2 * i + 1];
    }
    dft<N / 2, S>(e);
    dft<N / 2, S>(o);
    if (join) {
#pragma unroll
        for (int k = 0; k < N / 2; ++k) {
            const cx<T> u = e[k], v = k > 0 ? twiddle<S>(o[k], tw[k]) : o[0];
            e[k] = u + v;
            o[k] = u - v;
        }
    }
#pragma unroll
    for (int k = 0; k < N / 2; ++k) {
        a[k] = e[k];
        a[k + N / 2] = o[k];
    }
}

template <typename T, int N>
__global__ __launch_bounds__((box_shape<T, N>::NT), (box_shape<T, N>::W)) void k_box_r2c(
    const T* in, cx<T>* out, const cx<T>* __restrict__ tw, int64_t rs, T mul_edge, T mul_int) {
    using P = box_shape<T, N>;
    constexpr int M = P::M, K = P::K, NT = P::NT, SY = P::SY, SX = P::SX;
    __shared__ T lds[P::LDS];
    const int tid = threadIdx.x, hi = tid / M, z = tid % M;
    const int half = int(rs / 2);  // complex values between real rows
    const cx<T>* src = reinterpret_cast<const cx<T>*>(in) + int64_t(blockIdx.x) * N * N * half;
    auto xline = [&](int m) { return m * SX + hi * SY + z; };  // hi = y
    auto yline = [&](int m) { return hi * SX + m * SY + z; };  // hi = x
    auto zline = [&](int m) {
        const int l = tid + (m / M) * NT;
        return (l / N) * SX + (l % N) * SY + m % M;
    };
    cx<T> a[N];
#pragma unroll
    for (int m = 0; m < N; ++m) a[m] = src[(tid + (m / M) * NT) * half + m % M];

    // z and its real split (as in k_plane_r2c); X[0] and X[M] in slot 0
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        cx<T>* b = a + h * M;
        dft<M, -1>(b);
        b[0] = cx<T>{(b[0].x + b[0].y) * mul_edge, (b[0].x - b[0].y) * mul_edge};
#pragma unroll
        for (int k = 1; k < M / 2; ++k) {
            const cx<T> u = b[k], v = conjg(b[M - k]);
            const cx<T> A = scal(u + v, T(0.5)), B = cmul(tw[k], scal(u - v, T(0.5)));
            b[k] = cx<T>{(A.x + B.y) * mul_int, (A.y - B.x) * mul_int};
            b[M - k] = cx<T>{(A.x - B.y) * mul_int, (-A.y - B.x) * mul_int};
        }
        b[M / 2] = cx<T>{b[M / 2].x * mul_int, -b[M / 2].y * mul_int};
    }

    // z lines -> y lines; a line of even x fills the real parts of its pair's
    // two slots 0, one of odd x the imaginary parts: X[0] in the even slot,
    // X[M] in the odd one
    const T x0[2] = {a[0].x, a[M].x};
#pragma unroll
    for (int part = 0; part < 2; ++part) {
#pragma unroll
        for (int m = 0; m < N; ++m) {
            if (m % M != 0) {
                lds[zline(m)] = part ? a[m].y : a[m].x;
            } else if (((tid + (m / M) * NT) / N) % 2 == part) {
                lds[zline(m) - part * SX] = x0[m / M];
                lds[zline(m) - part * SX + SX] = a[m].y;
            }
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < N; ++m) {
            const T v = lds[yline(m)];
            if (part) a[m].y = v;
            else a[m].x = v;
        }
        __syncthreads();
    }
    dft<N, -1>(a);
    box_exchange<N>(lds, a, yline, xline);
    dft_halves<N, -1>(a, tw, z != 0);

    // the two images apart: (kx, ky) and (kx + N/2, ky) of both per thread
    cx<T>* mir = reinterpret_cast<cx<T>*>(lds);
    if (z == 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) mir[i * N + hi] = a[i];
    }
    __syncthreads();
    const int q = tid / N, ky = tid % N, qm = (N / 2 - q) & (N / 2 - 1), ym = (N - ky) & (N - 1);
    const cx<T> w = tw[q];
#pragma unroll
    for (int im = 0; im < 2; ++im) {  // kz = 0, kz = M
        const cx<T> u = mir[(q + im * (N / 2)) * N + ky], c = conjg(mir[(qm + im * (N / 2)) * N + ym]);
        const cx<T> E = scal(u + c, T(0.5)), D = scal(u - c, T(0.5));
        const cx<T> O = cmul(w, cx<T>{D.y, -D.x});
        mir[(im + 1) * N * N + q * N + ky] = E + O;
        mir[(im + 1) * N * N + (q + N / 2) * N + ky] = E - O;
    }
    __syncthreads();
    // both back to threads of the row: its K bins are complete within two stores
    // (kz = 0 and M stored by the threads that form them reach memory in
    // pieces: FP64 N = 32, 1000 grids 173 us against 152)
    cx<T>* dst = out + int64_t(blockIdx.x) * N * N * K + hi * K + z;
#pragma unroll
    for (int m = 0; m < N; ++m) {
        cx<T> u{};  // kz = 0 for the threads z = 0, kz = M for z = 1
        if (z < 2) u = mir[(1 + z) * N * N + m * N + hi];
        dst[m * N * K] = cx<T>{z == 0 ? u.x : a[m].x, z == 0 ? u.y : a[m].y};
        if (z == 1) dst[m * N * K + M - 1] = u;
    }
}

template <typename T, int N>
__global__ __launch_bounds__((box_shape<T, N>::NT), (box_shape<T, N>::W)) void k_box_c2r(
    const cx<T>* in, T* out, const cx<T>* __restrict__ tw, int64_t rs, T scale, T weight) {
    using P = box_shape<T, N>;
    constexpr int M = P::M, K = P::K, NT = P::NT, SY = P::SY, SX = P::SX;
    __shared__ T lds[P::LDS];
    const int tid = threadIdx.x, hi = tid / M, z = tid % M;
    const cx<T>* src = in + int64_t(blockIdx.x) * N * N * K;
    auto xline = [&](int m) { return m * SX + hi * SY + z; };  // hi = ky
    auto yline = [&](int m) { return hi * SX + m * SY + z; };  // hi = x
    auto zline = [&](int m) {
        const int l = tid + (m / M) * NT;
        return (l / N) * SX + (l % N) * SY + m % M;
    };
    cx<T> a[N];
#pragma unroll
    for (int m = 0; m < N; ++m) a[m] = src[(m * N + hi) * K + z];

    // kz = 0 and kz = M: with H0, HM their Hermitian parts,
    // Z'(kz = 0) = (H0 + HM) + i (H0 - HM); two (kx, ky) per thread
    cx<T>* col = reinterpret_cast<cx<T>*>(lds);
    cx<T> g0[2], gm[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        g0[i] = src[(tid + i * NT) * K];
        gm[i] = src[(tid + i * NT) * K + M];
        col[tid + i * NT] = g0[i];
        col[N * N + tid + i * NT] = gm[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int l = tid + i * NT;
        const int lm = ((N - l / N) & (N - 1)) * N + ((N - l % N) & (N - 1));
        const cx<T> h0 = hermitian(g0[i], col[lm], l == lm);
        const cx<T> hm = hermitian(gm[i], col[N * N + lm], l == lm);
        const cx<T> s = h0 + hm, d = h0 - hm;
        col[2 * N * N + l] = cx<T>{s.x - d.y, s.y + d.x};
    }
    __syncthreads();
    if (z == 0) {
#pragma unroll
        for (int m = 0; m < N; ++m) a[m] = col[2 * N * N + m * N + hi];
    }
    __syncthreads();

    // 0 < kz < M: the mirrored values through LDS
    const int ym = (N - hi) & (N - 1), zm = M - z;
    const cx<T> w = tw[z];
    T d[N];  // differences of the real parts; a[m].x becomes their sum
#pragma unroll
    for (int m = 0; m < N; ++m) lds[xline(m)] = a[m].x;
    __syncthreads();
#pragma unroll
    for (int m = 0; m < N; ++m) {
        const T c = lds[((N - m) & (N - 1)) * SX + ym * SY + zm];
        d[m] = a[m].x - c;
        a[m].x = z == 0 ? a[m].x : a[m].x + c;
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < N; ++m) lds[xline(m)] = a[m].y;
    __syncthreads();
#pragma unroll
    for (int m = 0; m < N; ++m) {
        const T c = lds[((N - m) & (N - 1)) * SX + ym * SY + zm];
        const cx<T> D = cmulc(cx<T>{d[m], a[m].y + c}, w);
        const cx<T> v{(a[m].x - D.y) * weight, (a[m].y - c + D.x) * weight};
        a[m].x = z == 0 ? a[m].x : v.x;
        a[m].y = z == 0 ? a[m].y : v.y;
    }
    __syncthreads();

    dft<N, +1>(a);
    box_exchange<N>(lds, a, xline, zline);
    dft<M, +1>(a);
    dft<M, +1>(a + M);
    // the scale between the sums, as in the separate passes: neither the
    // largest nor the smallest spectra leave the type's range on the way
#pragma unroll
    for (int m = 0; m < N; ++m) a[m] = scal(a[m], scale);
    box_exchange<N>(lds, a, zline, yline);
    dft<N, +1>(a);
    const int half = int(rs / 2);
    cx<T>* dst = reinterpret_cast<cx<T>*>(out) + int64_t(blockIdx.x) * N * N * half;
#pragma unroll
    for (int m = 0; m < N; ++m) dst[(hi * N + m) * half + z] = a[m];
}

// ---------------------------------------------------------------- x C2C with the y radix-R step
// Second half of a split y transform (k_plane_* with R > 1) and the x
// transform, in one strided pass over [b][x][y][kz] (y and kz flattened to
// one contiguous column index per x).  A workgroup owns TC adjacent columns
// of the first NY rows' range and the R - 1 column runs NY K further on each:
// thread (c, t) holds x = t + TPT i of all R rows, so the R-point DFT over y0
// needs no exchange.  src and dst may be the same buffer.
//   NT: non-temporal loads and stores (no reuse), where every 128-byte line
//       belongs to one tile;
//   ord: tile order (xcd_tile).
template <typename T, int N, int R, int TC, int EX>
struct xr_shape {
    static constexpr int K = N / 2 + 1, NY = N / R, TPT = N / EX, NT = TC * TPT;
    static constexpr int RM = radix_cap<T>();
    static constexpr int PS = first_radix_shift<EX, RM>::value;
    static constexpr int NP = padded_len<N, PS>::value;
    static constexpr int LDS = R * NP * TC;  // values of type T
    static constexpr int COLS = NY * K;
    static constexpr int TILES = COLS / TC;  // per grid
    static_assert(COLS % TC == 0, "tiles own whole columns");
};

template <typename T, int N, int R, int TC, int EX, int S, bool NT, int W>
__global__ __launch_bounds__((xr_shape<T, N, R, TC, EX>::NT), W) void k_strided_r(
    const cx<T>* src, cx<T>* dst, const cx<T>* __restrict__ tw, int ord) {
    using P = xr_shape<T, N, R, TC, EX>;
    constexpr int K = P::K, NY = P::NY, TPT = P::TPT;
    __shared__ T lds[P::LDS];
    const int c = threadIdx.x % TC, t = threadIdx.x / TC;
    const int64_t tile = xcd_tile(ord, blockIdx.x, gridDim.x);
    const int64_t b = tile / P::TILES;
    const int m = int(tile - b * P::TILES) * TC + c;
    const int k1 = m / K;
    // Element (x, y0) of this lane: a workgroup-uniform base plus the lane's
    // byte offset, which fits 32 bits (checked below), so that one vector
    // register addresses all of them.
    constexpr int64_t XS = int64_t(N) * K, YS = int64_t(NY) * K;
    static_assert((TPT * XS + NY * K) * int64_t(sizeof(cx<T>)) < (int64_t(1) << 32), "lane offset");
    const uint32_t lane = uint32_t((t * XS + m) * int64_t(sizeof(cx<T>)));
    src += b * N * XS;
    dst += b * N * XS;

    cx<T> a[R][EX];
#pragma unroll
    for (int i = 0; i < EX; ++i)
#pragma unroll
        for (int y = 0; y < R; ++y) {
            const cx<T>* p = at_bytes(src + (i * TPT) * XS + y * YS, lane);
            if constexpr (NT) {
                a[y][i].x = __builtin_nontemporal_load(&p->x);
                a[y][i].y = __builtin_nontemporal_load(&p->y);
            } else {
                a[y][i] = *p;
            }
        }
    cx<T> w[R];
#pragma unroll
    for (int y = 1; y < R; ++y) w[y] = tw[y * k1];
#pragma unroll
    for (int i = 0; i < EX; ++i) {
        cx<T> v[R];
#pragma unroll
        for (int y = 0; y < R; ++y) v[y] = a[y][i];
        if constexpr (S < 0) {
#pragma unroll
            for (int y = 1; y < R; ++y) v[y] = twiddle<S>(v[y], w[y]);
        }
        dft<R, S>(v);
        if constexpr (S > 0) {
            // k1 = 0 as it is: see `turn` in k_plane_c2r
            if (k1 != 0) {
#pragma unroll
                for (int y = 1; y < R; ++y) v[y] = twiddle<S>(v[y], w[y]);
            }
        }
#pragma unroll
        for (int y = 0; y < R; ++y) a[y][i] = v[y];
    }
    fft_multi<T, N, EX, R, S, 1, P::RM, TC, P::PS>(a, t, c, tw, 1, lds);
#pragma unroll
    for (int i = 0; i < EX; ++i)
#pragma unroll
        for (int y = 0; y < R; ++y) {
            cx<T>* p = at_bytes(dst + (i * TPT) * XS + y * YS, lane);
            if constexpr (NT) {
                __builtin_nontemporal_store(a[y][i].x, &p->x);
                __builtin_nontemporal_store(a[y][i].y, &p->y);
            } else {
                *p = a[y][i];
            }
        }
}

// Shape of the one-plane kernels: elements per thread and the minimum of
// waves per SIMD the register allocation keeps.  Measured over 537 MB of
// reals (forward / inverse step 1, us; in brackets the separate z and y
// passes): FP64 N = 64 197 / 179 (363 / 462), N = 128 224 / 210 (365 / 408);
// FP32 N = 64 209 / 214 (468 / 479), N = 128 208 / 215 (432 / 450), N = 256
// 309 / 331 (416 / 443): there one plane fills half a CU's registers and its
// phases do not overlap another's.  Chosen over (forward / inverse, against
// the form of its time): FP64 N = 64 16 per thread 201 / 231 against 199 /
// 200; N = 128 at 4 waves 238 / 212 and 8 per thread 227 / 308 against 215 /
// 209; FP32 N = 64 16 per thread 252 / 255 against 219 / 222; N = 128 8 per
// thread 247 / 261 against 228 / 220.  The streaming copy of the same bytes
// takes 173.  N = 32 (8 per thread, one wave a
// plane; 4 per thread the same within 5%): a whole transform of 333 grids with
// its x pass 59 (126) in FP64, 37 (81) in FP32.
template <typename T, int N>
struct plane_cfg {
    static constexpr bool F64 = sizeof(T) == 8;
    static constexpr int E = N <= 64 ? 8 : N == 128 ? 16 : 32;
    static constexpr int W = N == 128 ? (F64 ? 2 : 8) : 4;
};

template <typename T, int N>
static hipError_t plane_n(bool forward, const void* in, void* out, const void* tw, int64_t planes,
                          row_map map, double me, double mi, hipStream_t s) {
    if (N <= 128 && planes * N > kSliceRows)
        return in_slices(planes * N, [&](int64_t r0, int64_t nr) {
            const int64_t ro = r0 * map.rs, co = r0 * (N / 2 + 1);
            const void* src = forward ? static_cast<const void*>(static_cast<const T*>(in) + ro)
                                      : static_cast<const cx<T>*>(in) + co;
            void* dst = forward ? static_cast<void*>(static_cast<cx<T>*>(out) + co)
                                : static_cast<T*>(out) + ro;
            return plane_n<T, N>(forward, src, dst, tw, nr / N, map, me, mi, s);
        });
    using C = plane_cfg<T, N>;
    constexpr int NT = plane_shape<T, N, 1, C::E>::NT;
    const int ord = tile_order(planes * N * (N / 2 + 1) * int64_t(sizeof(cx<T>)), kGrouped);
    if (planes == 0) return hipSuccess;
    if (!grid_fits(planes, NT)) return hipErrorInvalidValue;
    if (forward)
        hipLaunchKernelGGL((k_plane_r2c<T, N, 1, C::E, C::W>), dim3(planes), dim3(NT), 0, s,
                           static_cast<const T*>(in), static_cast<cx<T>*>(out),
                           static_cast<const cx<T>*>(tw), map, T(me), T(mi), ord);
    else
        hipLaunchKernelGGL((k_plane_c2r<T, N, 1, C::E, C::W>), dim3(planes), dim3(NT), 0, s,
                           static_cast<const cx<T>*>(in), static_cast<T*>(out),
                           static_cast<const cx<T>*>(tw), map, T(me), T(mi), ord);
    return hipGetLastError();
}

// Where a plane fills at least a wave and fits on a CU with room for a second
// one (FP64 up to N = 128: 131 KB) or at least once (FP32 N = 256: 262 KB); an
// FP64 256 x 256 plane (524 KB) would take the whole register file.  From N =
// 128 up a plane is long for one workgroup, and few of them leave CUs idle: there
// z and y passes are faster.  Step 1 forward / inverse in us, in brackets those:
// FP64 128 16 planes 12.0 / 12.4 (9.1 / 9.0), 96 13.5 / 13.6 (13.7 / 12.8), 192
// 16.8 / 16.6 (23.1 / 17.6); FP32 128 64 9.4 / 9.6 (8.6 / 8.3), 96 9.6 / 10.0
// (10.8 / 10.7); FP32 256 32 24.5 / 28.4 (12.8 / 12.1), 128 28 / 32 (31 / 28), 192
// 30 / 35 (41 / 38).  N = 32 and 64: 5.2-6.2 (7.8-8.8) from one plane on.
bool plane_supported(bool f64, int n, int64_t planes, bool forward) {
    if (n == 128) return planes >= (f64 && !forward ? 160 : 96);
    if (!f64 && n == 256) return planes >= (forward ? 128 : 192);
    return n == 32 || n == 64;
}

hipError_t launch_plane(bool f64, bool forward, int n, const void* in, void* out, const void* tw,
                        int64_t planes, row_map map, double me, double mi, hipStream_t s) {
    if (f64) {
        switch (n) {
            case 32: return plane_n<double, 32>(forward, in, out, tw, planes, map, me, mi, s);
            case 64: return plane_n<double, 64>(forward, in, out, tw, planes, map, me, mi, s);
            case 128: return plane_n<double, 128>(forward, in, out, tw, planes, map, me, mi, s);
            default: return hipErrorInvalidValue;
        }
    }
    switch (n) {
        case 32: return plane_n<float, 32>(forward, in, out, tw, planes, map, me, mi, s);
        case 64: return plane_n<float, 64>(forward, in, out, tw, planes, map, me, mi, s);
        case 128: return plane_n<float, 128>(forward, in, out, tw, planes, map, me, mi, s);
        case 256: return plane_n<float, 256>(forward, in, out, tw, planes, map, me, mi, s);
        default: return hipErrorInvalidValue;
    }
}

// Split y transform: R (row tiles of 64 rows), the row tile's elements per
// thread, and the x pass's columns per tile, elements per row and thread,
// hints and tile order.  64 rows leave room for two or more row tiles on a CU
// and keep the x tile's runs at 64 bytes or more.  Measured over 537 MB of
// reals, row tiles forward / inverse and x pass, us (in brackets the step 1
// and x passes they replace):
//   FP64 N = 128, R = 2: 197 / 177 + 195 (224 / 210 + 217)
//        N = 256, R = 4: 206 / 215 + 200 to 228 (358 / 412 + 242)
//   FP32 N = 128, R = 2: 203 / 199 + 182 (208 / 215 + 218)
//        N = 256, R = 4: 200 / 218 + 207 to 222 (309 / 331 + 233)
//        N = 512, R = 8: 236 / 242 + 293 to 319 (419 / 445 + 214)
// and over 1.07 GB FP64 N = 512, R = 8: 446 / 481 + 568 to 614 (762 / 844 + 415).
// N = 64 planes have room as they are.  Tiles in groups (ORD) of 64 run the x
// pass at 4.73 TB/s for FP64 256 (contiguous 4.41), 4.93 for FP32 256 (4.43),
// and 3.46 / 3.60 for FP32 / FP64 512 (3.27 / 3.08), whose 64-byte runs share
// lines; N = 128 in launch order, non-temporally (FP32 5.96, contiguous 5.53,
// without the hint 5.1).  At N = 256 the hint gains nothing.
template <typename T, int N>
struct split_cfg {
    static constexpr bool F64 = sizeof(T) == 8;
    static constexpr int R = N / 64;
    static constexpr int E = !F64 && N == 128 ? 8 : 16;
    // FP32 512: two tiles of 16 waves on a CU need 64 registers or fewer (pair
    // 1084 us, 1125 with 74)
    static constexpr int W = F64 ? (N == 256 ? 4 : 2) : N == 512 ? 8 : 4;
    static constexpr int TC = N == 128 ? 32 : N == 256 ? (F64 ? 8 : 16) : (F64 ? 4 : 8);
    static constexpr int EX = F64 && N == 512 ? 4 : 8;
    static constexpr int WX = R * EX * int(sizeof(cx<T>)) > 256 ? 2 : 4;
    static constexpr bool NT = N == 128;
    static constexpr int ORD = N == 128 ? 0 : 6;
    // row tiles: groups of 16 (FP64 512 pair 2097 us, contiguous 2138), but
    // FP64 256 contiguous (three pairs 644 us, groups 665)
    static constexpr int ROWS_ORD = F64 && N == 256 ? kContig : kGrouped;
};

template <typename T, int N>
static hipError_t split_rows_n(bool forward, const void* in, void* out, const void* tw,
                               int64_t planes, row_map map, double me, double mi, hipStream_t s) {
    using C = split_cfg<T, N>;
    constexpr int NT = plane_shape<T, N, C::R, C::E>::NT;
    const int ord = tile_order(planes * N * (N / 2 + 1) * int64_t(sizeof(cx<T>)), C::ROWS_ORD);
    const int64_t blocks = planes * C::R;
    if (blocks == 0) return hipSuccess;
    if (!grid_fits(blocks, NT)) return hipErrorInvalidValue;
    if (forward)
        hipLaunchKernelGGL((k_plane_r2c<T, N, C::R, C::E, C::W>), dim3(blocks), dim3(NT), 0, s,
                           static_cast<const T*>(in), static_cast<cx<T>*>(out),
                           static_cast<const cx<T>*>(tw), map, T(me), T(mi), ord);
    else
        hipLaunchKernelGGL((k_plane_c2r<T, N, C::R, C::E, C::W>), dim3(blocks), dim3(NT), 0, s,
                           static_cast<const cx<T>*>(in), static_cast<T*>(out),
                           static_cast<const cx<T>*>(tw), map, T(me), T(mi), ord);
    return hipGetLastError();
}

template <typename T, int N, int S, bool NT>
static hipError_t split_x_run(const void* src, void* dst, const void* tw, int64_t batch,
                              hipStream_t s) {
    using C = split_cfg<T, N>;
    using P = xr_shape<T, N, C::R, C::TC, C::EX>;
    // N = 128 in launch order at every size (16 MB of FP64 forward 16 us, contiguous 18)
    const int large = NT == C::NT ? C::ORD : kGrouped;
    const int ord = N == 128 ? large
                             : tile_order(batch * N * N * (N / 2 + 1) * int64_t(sizeof(cx<T>)), large);
    const int64_t blocks = batch * P::TILES;
    if (blocks == 0) return hipSuccess;
    if (!grid_fits(blocks, P::NT)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_strided_r<T, N, C::R, C::TC, C::EX, S, NT, C::WX>), dim3(blocks),
                       dim3(P::NT), 0, s, static_cast<const cx<T>*>(src),
                       static_cast<cx<T>*>(dst), static_cast<const cx<T>*>(tw), ord);
    return hipGetLastError();
}

template <typename T, int N, int S>
static hipError_t split_x_n(const void* src, void* dst, const void* tw, int64_t batch,
                            hipStream_t s) {
    // the non-temporal hint is for tiles that own their lines: a buffer off
    // the 128-byte grid takes plain accesses
    if constexpr (split_cfg<T, N>::NT) {
        const uintptr_t both = reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst);
        if (both % 128 == 0) return split_x_run<T, N, S, true>(src, dst, tw, batch, s);
    }
    return split_x_run<T, N, S, false>(src, dst, tw, batch, s);
}

bool split_supported(int n) { return n == 128 || n == 256 || n == 512; }

hipError_t launch_split_rows(bool f64, bool forward, int n, const void* in, void* out,
                             const void* tw, int64_t planes, row_map map, double me, double mi,
                             hipStream_t s) {
    if (!split_supported(n)) return hipErrorInvalidValue;
    if (f64) {
        switch (n) {
            case 128: return split_rows_n<double, 128>(forward, in, out, tw, planes, map, me, mi, s);
            case 256: return split_rows_n<double, 256>(forward, in, out, tw, planes, map, me, mi, s);
            default: return split_rows_n<double, 512>(forward, in, out, tw, planes, map, me, mi, s);
        }
    }
    switch (n) {
        case 128: return split_rows_n<float, 128>(forward, in, out, tw, planes, map, me, mi, s);
        case 256: return split_rows_n<float, 256>(forward, in, out, tw, planes, map, me, mi, s);
        default: return split_rows_n<float, 512>(forward, in, out, tw, planes, map, me, mi, s);
    }
}

template <int S>
static hipError_t split_x_sign(bool f64, int n, const void* src, void* dst, const void* tw,
                               int64_t batch, hipStream_t s) {
    if (f64) {
        switch (n) {
            case 128: return split_x_n<double, 128, S>(src, dst, tw, batch, s);
            case 256: return split_x_n<double, 256, S>(src, dst, tw, batch, s);
            default: return split_x_n<double, 512, S>(src, dst, tw, batch, s);
        }
    }
    switch (n) {
        case 128: return split_x_n<float, 128, S>(src, dst, tw, batch, s);
        case 256: return split_x_n<float, 256, S>(src, dst, tw, batch, s);
        default: return split_x_n<float, 512, S>(src, dst, tw, batch, s);
    }
}

hipError_t launch_split_x(bool f64, int n, int sign, const void* src, void* dst, const void* tw,
                          int64_t batch, hipStream_t s) {
    if (!split_supported(n)) return hipErrorInvalidValue;
    return sign < 0 ? split_x_sign<-1>(f64, n, src, dst, tw, batch, s)
                    : split_x_sign<+1>(f64, n, src, dst, tw, batch, s);
}

// First y step of the z pass (rows_step): NY rows a tile, leaving y lines of
// L = N / NY for launch_strided_lines.  TB/s of the z passes with the step,
// forward / inverse, and of the lines, over 2.1 GB of FP64 and 1.07 GB of FP32
// reals (N = 4096 twice that); in brackets the plain z and y passes:
//   FP64 N = 1024, NY = 8   5.76 / 5.28 and 5.59 / 5.43 (6.05 / 5.68 and 4.92 / 4.87)
//        2048, 4            5.31 / 5.24 and 4.61 / 4.52 (5.62 / 5.77 and 4.05 / 4.06)
//        4096, 4            4.87 / 5.35 and 4.64 / 4.62 (5.26 / 5.71 and 3.49 / 3.48)
//   FP32 N = 512, NY = 16   5.82 / 5.10 and 5.85 / 5.72 (5.43 / 5.01 and 4.85 / 4.76)
//        1024, 16           5.79 / 5.16 and 5.75 / 5.56 (5.49 / 5.12 and 4.66 / 4.56)
//        2048, 8            5.16 / 4.66 and 5.20 / 5.01 (5.15 / 5.05 and 3.98 / 3.84)
//        4096, 4            4.63 / 4.91 and 4.71 / 4.65 (4.64 / 5.06 and 3.36 / 3.33)
// Shorter lines run faster, longer first steps slower (FP32 1024 with 32 rows
// 4.9, 4096 with 8 3.1 / 4.5; FP64 1024 with 16 5.2): NY is where the two
// together are fastest.  FP64 512 gains nothing (16 rows 5.42 / 5.48 and 5.70
// against 5.76 / 6.09 and 5.23).  k_plane_* takes the step up to N = 1024
// (k_rows_r2c 4.7 there: its packed column needs every row in one thread),
// k_rows_* longer rows.
int rows_step(bool f64, int n) {
    switch (n) {
        case 512: return f64 ? 1 : 16;
        case 1024: return f64 ? 8 : 16;
        case 2048: return f64 ? 4 : 8;
        case 4096: return 4;
        default: return 1;
    }
}

// Elements per thread and tiles per workgroup of k_rows_*, forward (F) and
// inverse (I).  TB/s over 2.1 / 4.3 GB of FP64 and half as much FP32 reals
// (N = 2048 / 4096, 64 / 32 planes) at NY = 1, the plain z passes, forward /
// inverse, in brackets passes with whole-value exchanges in contiguous order:
//   FP64 2048 5.62 / 5.77 (4.65 / 4.93), 4096 5.26 / 5.71 (4.84 / 4.98)
//   FP32 2048 5.15 / 5.05 (4.67 / 4.57), 4096 4.64 / 5.06 (4.25 / 4.13)
// One tile a workgroup at N = 4096, NY = 1 runs at 4.2: rows share a line at
// their ends, so tiles of neighbouring rows go together.
template <typename T, int N, int NY>
struct rows_cfg {
    static constexpr bool F64 = sizeof(T) == 8;
    static constexpr int EF = F64 && (N == 2048 || NY == 4) ? 16 : 32;
    static constexpr int EI = F64 && N == 2048 ? 16 : 32;
    static constexpr int GF = NY > 1 ? 1 : N == 4096 ? (F64 ? 2 : 4) : (F64 ? 4 : 8);
    static constexpr int GI = NY > 1 ? 1 : N == 4096 || F64 ? 4 : 8;
    static constexpr int WF = EF == 16 ? 4 : 2, WI = EI == 16 ? 4 : 2;
};

template <typename T, int N, int NY>
static hipError_t rows_n(bool forward, const void* in, void* out, const void* tw, int64_t rows,
                         row_map map, double me, double mi, hipStream_t s) {
    const int64_t tiles = rows / NY;
    if (tiles == 0) return hipSuccess;
    const cx<T>* t = static_cast<const cx<T>*>(tw);
    // FP32 2048: groups at every size, as for its y lines (strided_run)
    const int ord = sizeof(T) == 4 && N == 2048
                        ? kGrouped
                        : tile_order(rows * (N / 2 + 1) * int64_t(sizeof(cx<T>)), kGrouped);
    if constexpr (N <= 1024) {
        // k_plane_*: 2 NY elements per thread, two NY-point columns of it
        constexpr int E = 2 * NY, R = N / NY, W = 2;
        constexpr int NT = plane_shape<T, N, R, E>::NT;
        if (!grid_fits(tiles, NT)) return hipErrorInvalidValue;
        if (forward)
            hipLaunchKernelGGL((k_plane_r2c<T, N, R, E, W, true>), dim3(tiles), dim3(NT),
                               0, s, static_cast<const T*>(in), static_cast<cx<T>*>(out), t, map,
                               T(me), T(mi), ord);
        else
            hipLaunchKernelGGL((k_plane_c2r<T, N, R, E, W, true>), dim3(tiles), dim3(NT),
                               0, s, static_cast<const cx<T>*>(in), static_cast<T*>(out), t, map,
                               T(me), T(mi), ord);
        return hipGetLastError();
    } else {
        using C = rows_cfg<T, N, NY>;
        auto go = [&](auto kernel, int64_t g, int nt, auto pin, auto pout) {
            const int64_t blocks = (tiles + g - 1) / g;
            if (!grid_fits(blocks, nt)) return hipErrorInvalidValue;
            hipLaunchKernelGGL(kernel, dim3(blocks), dim3(nt), 0, s, pin, pout, t, tiles, map, T(me),
                               T(mi), ord);
            return hipGetLastError();
        };
        if (forward) {
            constexpr int NT = rows_shape<T, N, NY, C::EF, C::GF>::NT;
            const T* pi = static_cast<const T*>(in);
            cx<T>* po = static_cast<cx<T>*>(out);
            if constexpr (NY == 1) {
                if (map.pencil)
                    return go(k_rows_r2c<T, N, 1, C::EF, C::GF, C::WF, true>, C::GF, NT, pi, po);
            }
            return go(k_rows_r2c<T, N, NY, C::EF, C::GF, C::WF, false>, C::GF, NT, pi, po);
        }
        constexpr int NT = rows_shape<T, N, NY, C::EI, C::GI>::NT;
        const cx<T>* pi = static_cast<const cx<T>*>(in);
        T* po = static_cast<T*>(out);
        if constexpr (NY == 1) {
            if (map.pencil)
                return go(k_rows_c2r<T, N, 1, C::EI, C::GI, C::WI, true>, C::GI, NT, pi, po);
        }
        return go(k_rows_c2r<T, N, NY, C::EI, C::GI, C::WI, false>, C::GI, NT, pi, po);
    }
}

hipError_t launch_rows(bool f64, bool forward, int n, int ny, const void* in, void* out,
                       const void* tw, int64_t rows, row_map map, double me, double mi,
                       hipStream_t s) {
#define GFFT_ROWS(T, N, NY) \
    if (n == N && ny == NY) return rows_n<T, N, NY>(forward, in, out, tw, rows, map, me, mi, s);
    if (f64) {
        GFFT_ROWS(double, 1024, 8)
        GFFT_ROWS(double, 2048, 1)
        GFFT_ROWS(double, 2048, 4)
        GFFT_ROWS(double, 4096, 1)
        GFFT_ROWS(double, 4096, 4)
    } else {
        GFFT_ROWS(float, 512, 16)
        GFFT_ROWS(float, 1024, 16)
        GFFT_ROWS(float, 2048, 1)
        GFFT_ROWS(float, 2048, 8)
        GFFT_ROWS(float, 4096, 1)
        GFFT_ROWS(float, 4096, 4)
    }
#undef GFFT_ROWS
    return hipErrorInvalidValue;
}

template <typename T, int N>
static hipError_t box_n(bool forward, const void* in, void* out, const void* tw, int64_t grids,
                        int64_t rs, double scale, bool weighted, hipStream_t s) {
    constexpr int NT = box_shape<T, N>::NT;
    if (grids == 0) return hipSuccess;
    if (!grid_fits(grids, NT)) return hipErrorInvalidValue;
    if (forward)
        hipLaunchKernelGGL((k_box_r2c<T, N>), dim3(grids), dim3(NT), 0, s,
                           static_cast<const T*>(in), static_cast<cx<T>*>(out),
                           static_cast<const cx<T>*>(tw), rs, T(scale),
                           T(weighted ? 2.0 * scale : scale));
    else
        hipLaunchKernelGGL((k_box_c2r<T, N>), dim3(grids), dim3(NT), 0, s,
                           static_cast<const cx<T>*>(in), static_cast<T*>(out),
                           static_cast<const cx<T>*>(tw), rs, T(scale), T(weighted ? 0.5 : 1.0));
    return hipGetLastError();
}

// One workgroup per grid pays where a grid is tiny or where there are enough
// of them for the chip.  Box kernel against plane and x passes (three passes at
// N = 16), us, forward / inverse: FP64 N = 16, GPU time of a forward, 5.4 / 9.4
// for one grid, 18 / 53 for 1000; calls of N = 32 FP64 25 / 24 (23 / 24) for 64
// grids, 26.5 / 25.8 (27.2 / 25.0) for 96, 30 / 28 (33 / 32) for 128, 150 / 157
// (207 / 208) for 1000; FP32 17.7 / 15.8 (19.1 / 17.7) for 64, 61 / 62 (99 / 101)
// for 1000.
bool box_supported(bool f64, int n, int64_t grids) {
    return n == 16 || (n == 32 && grids >= (f64 ? 96 : 64));
}

hipError_t launch_box(bool f64, bool forward, int n, const void* in, void* out, const void* tw,
                      int64_t grids, int64_t rs, double scale, bool weighted, hipStream_t s) {
    if (n != 16 && n != 32) return hipErrorInvalidValue;
    if (f64)
        return n == 16 ? box_n<double, 16>(forward, in, out, tw, grids, rs, scale, weighted, s)
                       : box_n<double, 32>(forward, in, out, tw, grids, rs, scale, weighted, s);
    return n == 16 ? box_n<float, 16>(forward, in, out, tw, grids, rs, scale, weighted, s)
                   : box_n<float, 32>(forward, in, out, tw, grids, rs, scale, weighted, s);
}

}  // namespace gfft
