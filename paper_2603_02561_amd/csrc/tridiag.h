// Eigenpairs of a small dense symmetric matrix in double precision, one workgroup of 512 threads:
// Householder tridiagonalization, multisection on Sturm counts for the wanted eigenvalues, twisted
// factorizations for their eigenvectors, and the reflectors applied backwards.
//
// The phase is bound by instructions, not by arithmetic: a wave issues one in five cycles whatever it is, and one Householder
// step is some two hundred, of which the two wave-wide sums, the reciprocals and the exchange of partial sums between
// the waves are the part that all waves repeat.  Double precision costs nothing against float here (a v_fma_f64 issues like a v_fma_f32,
// 9 cycles dependent and 5 independent, measured) except in the wave sums, and it is what lets the
// eigenvectors be computed independently of each other: their mutual orthogonality is about
// 1e-15 / gap, where gap is the distance of neighbouring eigenvalues relative to the norm.
//
// The matrix lives in the registers of four waves, one per SIMD: wave w holds the rows i with
// (i / 4) % 4 == w, a lane one column, or two of more than 64, so the trailing block stays spread over
// the waves while it shrinks.  A step needs a single barrier: each of the four forms the reflector and the correction
// vector for itself, from the four partial products A u and the next pivot row (as it was before the
// step), which they exchange through a double buffer in LDS.  (Eight waves, two per SIMD, do that
// redundant part twice on every SIMD: 1880 cycles per step at 40 columns.)
#pragma once

#include "common.h"

namespace solar {

constexpr int kTriThreads = 512;
constexpr int kTriWaves = 4;   // waves that hold the matrix
// What a column's sum of squares starts at (1e-180 in each of 64 lanes), so that a column of zeros still gives a proper reflector:
// u^2 = kTriSeed, and with half of it taken off h = u^2 / 2.  The loop of the reduction and the pass behind it must agree in this.
constexpr double kTriSeed = 6.4e-179;

template <int CTRL>
__device__ __forceinline__ double dpp_mov64(double v) {
    union { double d; int i[2]; } x, y;
    x.d = v;
    y.i[0] = __builtin_amdgcn_mov_dpp(x.i[0], CTRL, 0xf, 0xf, true);   // every lane has a source
    y.i[1] = __builtin_amdgcn_mov_dpp(x.i[1], CTRL, 0xf, 0xf, true);
    return y.d;
}

__device__ __forceinline__ double readlane64(double v, int lane) {
    union { double d; int i[2]; } x, y;
    x.d = v;
    y.i[0] = __builtin_amdgcn_readlane(x.i[0], lane);
    y.i[1] = __builtin_amdgcn_readlane(x.i[1], lane);
    return y.d;
}

// a_k += x[lane I + k of the row of 16 lanes] * y: the broadcast is an operand of the multiply-add.  It may not read what
// the vector ALU wrote in the last two instructions, which the compiler does not see to in here: hence the wait in front, and
// one statement for four of them (whose results may therefore not share a register with an operand, "&").
#define SOLAR_FMAC_BCAST(A, X, Y, I) "v_fmac_f64_dpp %" #A ", %" #X ", %" #Y " row_newbcast:%" #I " row_mask:0xf bank_mask:0xf\n\t"
template <int I>
__device__ __forceinline__ void fmac_bcast64(double& a0, double x, double y) {
    asm("s_nop 1\n\t" SOLAR_FMAC_BCAST(0, 1, 2, 3) : "+v"(a0) : "v"(x), "v"(y), "n"(I));
}
template <int I>
__device__ __forceinline__ void fmac_bcast64(double& a0, double& a1, double& a2, double& a3, double x, double y) {
    asm("s_nop 1\n\t" SOLAR_FMAC_BCAST(0, 4, 5, 6) SOLAR_FMAC_BCAST(1, 4, 5, 7) SOLAR_FMAC_BCAST(2, 4, 5, 8) SOLAR_FMAC_BCAST(3, 4, 5, 9)
        : "+&v"(a0), "+&v"(a1), "+&v"(a2), "+&v"(a3)
        : "v"(x), "v"(y), "n"(I), "n"(I + 1), "n"(I + 2), "n"(I + 3));
}
// p += the sum of x[lane I + k of the row of 16 lanes] * y_k
template <int I>
__device__ __forceinline__ void fmac_bcast64_sum(double& p, double x, double y0, double y1, double y2, double y3) {
    asm("s_nop 1\n\t" SOLAR_FMAC_BCAST(0, 1, 2, 6) SOLAR_FMAC_BCAST(0, 1, 3, 7) SOLAR_FMAC_BCAST(0, 1, 4, 8) SOLAR_FMAC_BCAST(0, 1, 5, 9)
        : "+&v"(p)
        : "v"(x), "v"(y0), "v"(y1), "v"(y2), "v"(y3), "n"(I), "n"(I + 1), "n"(I + 2), "n"(I + 3));
}
#undef SOLAR_FMAC_BCAST

// v of the lane whose number is byte / 4
__device__ __forceinline__ double bpermute64(int byte, double v) {
    union { double d; int i[2]; } x, y;
    x.d = v;
    y.i[0] = __builtin_amdgcn_ds_bpermute(byte, x.i[0]);
    y.i[1] = __builtin_amdgcn_ds_bpermute(byte, x.i[1]);
    return y.d;
}

// Sum over the 64 lanes, the same bits in every lane.  Two 4x4x4 products with ones add the lanes that
// share (l / 4) % 4 (the first over l / 16, the second over l % 4: 20 cycles each, where a DPP stage on
// a double takes 28), two mirrors the remaining four groups, as (g0 + g1) + (g2 + g3): an exchange of
// lanes l <-> l ^ 4 w beforehand does not change a bit of the result.
__device__ __forceinline__ double wave_sum64_begin(double v) {
    return __builtin_amdgcn_mfma_f64_4x4x4f64(v, 1.0, 0.0, 0, 0, 0);
}
__device__ __forceinline__ double wave_sum64_end(double v) {
    v = __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, v, 0.0, 0, 0, 0);
    v += dpp_mov64<0x141>(v);   // row_half_mirror
    v += dpp_mov64<0x140>(v);   // row_mirror
    return v;
}

// Sum over teams of T = 8 or 16 consecutive lanes.
template <int T>
__device__ __forceinline__ double team_sum64(double v) {
    static_assert(T == 8 || T == 16, "teams inside a row of 16 lanes");
    v += dpp_mov64<0xB1>(v);
    v += dpp_mov64<0x4E>(v);
    v += dpp_mov64<0x141>(v);
    if constexpr (T == 16) v += dpp_mov64<0x140>(v);
    return v;
}

// 1 / x and 1 / sqrt(x): the hardware's estimate (2^-23 or better) and one Newton step, about 1e-14.
__device__ __forceinline__ double rcp64(double x) {
    const double r = __builtin_amdgcn_rcp(x);
    return fma(fma(-x, r, 1.0), r, r);
}
__device__ __forceinline__ double rsq64(double x) {
    const double r = __builtin_amdgcn_rsq(x);
    return fma(fma(-x * r, r, 1.0), 0.5 * r, r);
}

// LDS of one solve, in doubles.  `wa` and `wb` are two work arrays of WA and WB doubles; the exchange
// buffers of the reduction live in `wb`.
template <int N, int RB>
struct TriCfg {
    static constexpr int NC = (N + 63) / 64;           // columns per lane
    static constexpr int RS = 4 * ((N + 15) / 16);     // rows per wave, in chunks of four
    static constexpr int PS = 64 * NC;
    // pivot rows, later reflectors: row k holds entries k .. N-1, packed where whole rows would not fit LDS; a
    // whole-wave store of row k runs on into rows that are stored later, and behind the last one
    static constexpr int USZ = (N > 64 ? N * (N + 1) / 2 : N * N) + PS;
    // exchange buffers, twice: partial products [waves][PS] and the four rows next to the pivot [4][PS]
    static constexpr int EXB = (kTriWaves + 4) * PS, EX = 2 * EXB;
    static constexpr int WA = N * RB;
    static constexpr int GRID = 1024 + N;              // of tri_values
    static constexpr int WB0 = N * (RB + 2) > EX ? N * (RB + 2) : EX, WB = WB0 > GRID ? WB0 : GRID;
    static constexpr int VEC = 6 * N + 16 + 64;        // d, e, 1/h, scaled e, (d, e^2) and a chunk, lambda
    static_assert(N % 8 == 0 && N >= 16 && N <= 128, "multiples of eight");
};
template <int N>
using TriRows = double[4 * ((N + 15) / 16)][(N + 63) / 64];   // rows per wave x columns per lane
template <int N>
using TriCols = double[(N + 63) / 64];

// where entry j of row k would be in U if its entries started at 0 (they start at k)
__device__ __forceinline__ constexpr int tri_row(int n, int k) { return n > 64 ? k * (n - 1) - (k * (k - 1)) / 2 : k * n; }

// State of the reduction that a wave carries from step to step.
template <int N>
struct TriState {
    TriCols<N> x;                        // the pivot row, updated
    TriCols<N> uo, po;                   // reflector of the last step and A u / h, which its correction comes from
    TriCols<N> qo;                       // negative correction of the last step, not yet applied to the rows
    double inv, up;                      // of the last step: 1 / h, u^T A u
    // entries of uo and qo that belong to the wave's own rows: that of row m = 4 q + s in lanes m % 16, m % 16 + 16, ...
    // of register m / 16
    TriCols<N> ur, qr;
};

// What the last step leaves to the gaps of the next one: its correction,
template <int N, int C0>
__device__ __forceinline__ void tri_correction(TriState<N>& st, int own) {
    constexpr int NC = TriCfg<N, 8>::NC;
    const double w2 = -0.5 * (st.inv * st.up) * st.inv;
#pragma unroll
    for (int c = C0; c < NC; ++c) {
        st.qo[c] = -fma(w2, st.uo[c], st.po[c]);
        st.qr[c] = bpermute64(own, st.qo[c]);
    }
}
// and the pivot row of step k, as it is, to U: what it makes of it is worked out from there afterwards, by all waves at once.
template <int N, int C0>
__device__ __forceinline__ void tri_keep_row(const TriState<N>& st, double* U, int k, int col) {
    using T = TriCfg<N, 8>;
    double* uk = U + tri_row(N, k);
#pragma unroll
    for (int c = C0; c < T::NC; ++c) {
        if constexpr (N > 64) uk[k + ((col + 64 * c - k) & (T::PS - 1))] = st.x[c];
        else uk[col] = st.x[c];
    }
}

// The last step's update of the rows 4 A0 .. MN - 1 of a wave, a[m][c] += ur(row m) qo[c] + qr(row m) uo[c], as blocks of four
// multiply-adds with a broadcast operand: those of share G of GN.
template <int A0, int MN, int C0, int NC, int B0, int B1, int N>
__device__ __forceinline__ void tri_update_blocks(TriRows<N>& a, const TriState<N>& st) {
    if constexpr (B0 < B1) {
        constexpr int NQ = (MN / 4 - A0) * (NC - C0), R = B0 % NQ, M = 4 * (A0 + R / (NC - C0)), c = C0 + R % (NC - C0);
        if constexpr (B0 < NQ) fmac_bcast64<M % 16>(a[M][c], a[M + 1][c], a[M + 2][c], a[M + 3][c], st.ur[M / 16], st.qo[c]);
        else fmac_bcast64<M % 16>(a[M][c], a[M + 1][c], a[M + 2][c], a[M + 3][c], st.qr[M / 16], st.uo[c]);
        tri_update_blocks<A0, MN, C0, NC, B0 + 1, B1, N>(a, st);
    }
}
template <int A0, int MN, int C0, int NC, int G, int GN, int N>
__device__ __forceinline__ void tri_update_share(TriRows<N>& a, const TriState<N>& st) {
    constexpr int TOTAL = 2 * (MN / 4 - A0) * (NC - C0);
    __builtin_amdgcn_sched_barrier(0);
    tri_update_blocks<A0, MN, C0, NC, TOTAL * G / GN, TOTAL * (G + 1) / GN, N>(a, st);
    __builtin_amdgcn_sched_barrier(0);
}
// and their product with x: p[c] += x(row m) a[m][c] (an accumulator that the next instruction adds to costs it no wait)
template <int M, int MN, int C0, int NC, int RS>
__device__ __forceinline__ void tri_product(const double (&a)[RS][NC], const double (&x)[NC], double (&p)[NC]) {
    if constexpr (M < MN) {
#pragma unroll
        for (int c = C0; c < NC; ++c) fmac_bcast64_sum<M % 16>(p[c], x[M / 16], a[M][c], a[M + 1][c], a[M + 2][c], a[M + 3][c]);
        tri_product<M + 4, MN, C0, NC, RS>(a, x, p);
    }
}

// Steps of the reduction whose next pivot is in rows 16 A0 .. 16 A0 + 15, then those of A0 + 1 and so on:
// the chunks of rows that are still in the trailing block are a compile-time set, so a step has no branch.
// A wave alone on its SIMD issues one instruction, scalar ones included, per five cycles, and every access
// to LDS delays the exchange (removing both sums changes nothing, removing a store of all waves takes 60 to
// 100 cycles off a step): entries of u and q that a row needs are broadcasts inside the multiply-adds, which reach 16
// lanes, so the wave's own entries are first brought to every 16 lanes by one lane permutation.  Nothing that can be worked out
// afterwards is in the loop: a step keeps its pivot row, and diagonal, off-diagonal and reflector come from those
// rows, all at once.  Cycles a step, with scalar operands (two lane reads for every multiply-add or two) and the results
// taken in the loop against this: 1220 -> 1110 at 40 columns, 1250 -> 1170 at 64, 1980 -> 1660 at 128.
template <int N, int A0>
__device__ __forceinline__ void tri_steps(TriRows<N>& a, TriState<N>& st, double* ex, double* U, int wave,
                                          int col, int own) {
    using T = TriCfg<N, 8>;
    constexpr int NC = T::NC, PS = T::PS, W = kTriWaves, NA = (N + 15) / 16;
    constexpr int C0 = A0 >= 4 ? 1 : 0;                 // columns of earlier registers have left the block
    constexpr int K0 = A0 ? 16 * A0 - 1 : 0, K1 = 16 * A0 + 15 < N - 2 ? 16 * A0 + 15 : N - 2;
    constexpr int MN = 4 * NA;
    double* at = ex + (K0 & 1) * T::EXB + col;          // this step's exchange buffer
    // one and zero in double precision by their high words
    auto unit = [](bool on) __attribute__((always_inline)) { return __hiloint2double(on ? 0x3ff00000 : 0, 0); };
#define SOLAR_TRI_FENCE __builtin_amdgcn_sched_barrier(0)
#pragma unroll 1
    for (int k = K0; k < K1; ++k) {
        const int k1 = k + 1;
        double u[NC], s2 = kTriSeed / 64;
#pragma unroll
        for (int c = C0; c < NC; ++c) {
            u[c] = st.x[c] * unit(col + 64 * c > k);
            s2 = fma(u[c], u[c], s2);
        }
        double xk1 = st.x[NC - 1];
        if constexpr (NC - C0 == 2) xk1 = k1 >= 64 ? st.x[1] : st.x[0];
        // the sum and the reciprocal square root are a chain whose gaps what the last step has left, and the update of
        // the own rows, fill; in front of the chain or behind it, where the compiler puts them, they take as long again
        SOLAR_TRI_FENCE;
        s2 = wave_sum64_begin(s2);
        SOLAR_TRI_FENCE;
        tri_correction<N, C0>(st, own);
        SOLAR_TRI_FENCE;
        s2 = __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, s2, 0.0, 0, 0, 0);
        SOLAR_TRI_FENCE;
        // (the diagonal entry of row 63 is still in the first register of the columns)
        if (wave == (k & (W - 1))) tri_keep_row<N, (A0 > 4 ? 1 : 0)>(st, U, k, col);
        const double alpha = readlane64(xk1, (k1 ^ (4 * wave)) & 63);
        SOLAR_TRI_FENCE;
        s2 += dpp_mov64<0x141>(s2);
        tri_update_share<A0, MN, C0, NC, 0, 6>(a, st);
        s2 += dpp_mov64<0x140>(s2);
        tri_update_share<A0, MN, C0, NC, 1, 6>(a, st);
        const double r0 = __builtin_amdgcn_rsq(s2);
        tri_update_share<A0, MN, C0, NC, 2, 6>(a, st);
        const double r1 = fma(-s2 * r0, r0, 1.0);
        tri_update_share<A0, MN, C0, NC, 3, 6>(a, st);
        const double r2 = fma(r1, 0.5 * r0, r0);
        tri_update_share<A0, MN, C0, NC, 4, 6>(a, st);
        // the reflector I - u u^T / h maps the column to g e_(k+1)
        const double g = -copysign(s2 * r2, alpha);
        tri_update_share<A0, MN, C0, NC, 5, 6>(a, st);
#pragma unroll
        for (int c = C0; c < NC; ++c) {
            u[c] = fma(-g, unit(col + 64 * c == k1), u[c]);
            st.ur[c] = bpermute64(own, u[c]);
        }
        SOLAR_TRI_FENCE;
        const double inv = rcp64(fma(-alpha, g, s2) - kTriSeed / 2);
        if (wave == ((k1 >> 2) & (W - 1))) {            // the next pivot row is one of this wave's
#pragma unroll
            for (int c = C0; c < NC; ++c)
#pragma unroll
                for (int s = 0; s < 4; ++s) at[(W + s) * PS + 64 * c] = a[4 * A0 + s][c];
        }
        SOLAR_TRI_FENCE;
        double pp[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) pp[c] = 0.0;
        tri_product<4 * A0, MN, C0, NC>(a, st.ur, pp);   // the own rows with u
#pragma unroll
        for (int c = C0; c < NC; ++c) at[wave * PS + 64 * c] = pp[c];
        __syncthreads();
        double r[NC][W], y[NC];
#pragma unroll
        for (int c = C0; c < NC; ++c) {
#pragma unroll
            for (int w = 0; w < W; ++w) r[c][w] = at[w * PS + 64 * c];
        }
#pragma unroll
        for (int c = C0; c < NC; ++c) y[c] = at[(W + (k1 & 3)) * PS + 64 * c];
        at = ex + ((at - ex) ^ T::EXB);
        // with w = u^T A u, the correction is q = p - (w / 2 h^2) u for p = A u / h, and the new pivot row
        // is row - u_(k+1) q - q_(k+1) u; all of it but the multiple of w is ready before w is
        double p[NC], t[NC], up = 0.0;
#pragma unroll
        for (int c = C0; c < NC; ++c) {
            p[c] = (r[c][0] + r[c][1]) + (r[c][2] + r[c][3]);
            up = fma(u[c], p[c], up);
        }
        SOLAR_TRI_FENCE;
        up = wave_sum64_begin(up);
        SOLAR_TRI_FENCE;
#pragma unroll
        for (int c = C0; c < NC; ++c) p[c] *= inv;
        SOLAR_TRI_FENCE;
        up = __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, up, 0.0, 0, 0, 0);
        SOLAR_TRI_FENCE;
        double ps = p[NC - 1];
        if constexpr (NC - C0 == 2) ps = k1 >= 64 ? p[1] : p[0];
        const double uk1 = alpha - g, pk1 = readlane64(ps, (k1 ^ (4 * wave)) & 63);
        SOLAR_TRI_FENCE;
        up += dpp_mov64<0x141>(up);
        SOLAR_TRI_FENCE;
#pragma unroll
        for (int c = C0; c < NC; ++c) {
            y[c] = fma(-uk1, p[c], fma(-pk1, u[c], y[c]));
            t[c] = inv * uk1 * inv * u[c];
        }
        SOLAR_TRI_FENCE;
        up += dpp_mov64<0x140>(up);
#pragma unroll
        for (int c = C0; c < NC; ++c) {
            st.x[c] = fma(up, t[c], y[c]);
            st.uo[c] = u[c];
            st.po[c] = p[c];
        }
        st.inv = inv;
        st.up = up;
    }
    if constexpr (K1 < N - 2) {
        tri_steps<N, A0 + 1>(a, st, ex, U, wave, col, own);
    } else {
        tri_correction<N, C0>(st, own);
        if (wave == ((N - 2) & (W - 1))) tri_keep_row<N, C0>(st, U, N - 2, col);
    }
#undef SOLAR_TRI_FENCE
}

// Householder reduction of the matrix in `a` to tridiagonal form: diagonal dd[N], off-diagonal ee[N-1],
// reflector k in row k of U (entries k+1 .. N-1) with its 1/h in ih[k].  Waves 0 .. 3 hold the matrix:
// a[4 q + s][c] is entry (16 q + 4 wave + s, (lane ^ 4 wave) + 64 c), zero outside.  With the columns
// exchanged like that the lanes of a wave's own rows are the same for every wave.
template <int N>
__device__ __forceinline__ void tri_reduce(TriRows<N>& a, double* ex, double* U,
                                           double* dd, double* ee, double* ih) {
    using T = TriCfg<N, 8>;
    constexpr int NC = T::NC, PS = T::PS, W = kTriWaves;
    const int tid = fresh_tid(), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (wave >= W) {
#pragma unroll 1
        for (int k = 0; k < N - 1; ++k) __syncthreads();   // one for the first row, N - 2 steps
    } else {
        const int col = (tid & 63) ^ (4 * wave);
        double* row0 = ex + T::EXB;
        if (wave == 0) {
#pragma unroll
            for (int c = 0; c < NC; ++c) row0[col + 64 * c] = a[0][c];
        }
        __syncthreads();
        TriState<N> st;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            st.x[c] = row0[col + 64 * c];
            st.uo[c] = st.po[c] = st.qo[c] = st.ur[c] = st.qr[c] = 0.0;
        }
        st.inv = st.up = 0.0;
        // where a wave's own entries are: row 16 q + 4 wave + s in lane 16 q + s (the columns are exchanged)
        const int i16 = tid & 15;
        tri_steps<N, 0>(a, st, ex, U, wave, col, 4 * (16 * (i16 >> 2) + (i16 & 3)));
        // of row N-1 only the last diagonal entry is missing the last update
        if (wave == (((N - 1) >> 2) & 3) && col + 64 * (NC - 1) == N - 1)
            dd[N - 1] = fma(2.0 * st.uo[NC - 1], st.qo[NC - 1], a[4 * ((N - 1) >> 4) + 3][NC - 1]);
    }
    __syncthreads();
    // diagonal, off-diagonal and reflector from the pivot rows, eight lanes to a row
    const int u = tid & 7;
#pragma unroll 1
    for (int k = tid >> 3; k < N - 1; k += kTriThreads / 8) {
        double* uk = U + tri_row(N, k);
        double s2 = u == 0 ? kTriSeed : 0.0;
        for (int j = k + 1 + u; j < N; j += 8) s2 = fma(uk[j], uk[j], s2);
        s2 = team_sum64<8>(s2);
        const double alpha = uk[k + 1], g = k < N - 2 ? -copysign(s2 * rsq64(s2), alpha) : alpha;
        if (u == 0) {
            dd[k] = uk[k];
            ee[k] = g;
            ih[k] = rcp64(fma(-alpha, g, s2) - kTriSeed / 2);
            uk[k + 1] = alpha - g;
        }
    }
    __syncthreads();
}

// What the minors say at a point: the number of eigenvalues >= the point, and (DET) the determinant of T - point as m 2^e.
struct SturmPoint {
    int c, e;
    double m;
};

// The tridiagonal matrix (t[i].x = d_i, t[i].y = e_(i-1)^2, t[0].y = 0) at two points, from its leading minors and their
// signs.  Two points per lane share the reads of t, which
// four waves could not feed to one point each (a 16-byte read occupies the LDS port for 8 cycles per
// wave, even of one address).  The recurrences are rescaled every 16 steps: a minor shrinks by about
// |lambda| per step at most, and no wanted eigenvalue is below 1e-10 of the norm.
template <int N, bool DET>
__device__ __forceinline__ void sturm_points(const double2* t, double la, double lb, SturmPoint& a, SturmPoint& b) {
    double p = 1.0, pm = 0.0, r = 1.0, rm = 0.0;
    uint32_t bp = 0, br = 0;
    int np = 0, nr = 0;
    if constexpr (DET) a.e = b.e = 0;
    auto load = [&](double2 (&v)[8], int i0) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 8; ++s) v[s] = t[i0 + s];
    };
    auto steps = [&](const double2 (&v)[8]) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const double pn = fma(v[s].x - la, p, -(v[s].y * pm));
            const double rn = fma(v[s].x - lb, r, -(v[s].y * rm));
            pm = p; p = pn;
            rm = r; r = rn;
            bp = __builtin_amdgcn_alignbit(bp, (uint32_t)__double2hiint(pn), 31);
            br = __builtin_amdgcn_alignbit(br, (uint32_t)__double2hiint(rn), 31);
        }
    };
    double2 v0[8], v1[8];
    load(v0, 0);
    if constexpr (N % 16 == 8) {
        load(v1, 8);
        steps(v0);
        np = __popc((bp ^ (bp >> 1)) & 0xffu);
        nr = __popc((br ^ (br >> 1)) & 0xffu);
#pragma unroll
        for (int s = 0; s < 8; ++s) v0[s] = v1[s];
    }
#pragma unroll 1
    for (int i0 = N % 16; i0 < N; i0 += 16) {
        load(v1, i0 + 8);
        steps(v0);
        load(v0, i0 + 16);                               // the last one reads past the matrix
        steps(v1);
        np += __popc((bp ^ (bp >> 1)) & 0xffffu);
        nr += __popc((br ^ (br >> 1)) & 0xffffu);
        const int ep = -__builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(pm)));
        const int er = -__builtin_amdgcn_frexp_exp(fmax(fabs(r), fabs(rm)));
        p = __builtin_amdgcn_ldexp(p, ep);
        pm = __builtin_amdgcn_ldexp(pm, ep);
        r = __builtin_amdgcn_ldexp(r, er);
        rm = __builtin_amdgcn_ldexp(rm, er);
        if constexpr (DET) {
            a.e -= ep;
            b.e -= er;
        }
    }
    a.c = N - np;
    b.c = N - nr;
    if constexpr (DET) {
        a.m = p;
        b.m = r;
    }
}

// the largest (UP) or smallest v of a team of TP lanes
template <int TP, bool UP>
__device__ __forceinline__ double team_end64(double v) {
    auto step = [](double x, double y) __attribute__((always_inline)) { return UP ? fmax(x, y) : fmin(x, y); };
    v = step(v, dpp_mov64<0xB1>(v));
    v = step(v, dpp_mov64<0x4E>(v));
    if constexpr (TP == 8) v = step(v, dpp_mov64<0x141>(v));
    return v;
}

// What the minors say at the point x of a team, from the lane that has it among its own two; `f` if none has.
template <int TP>
__device__ __forceinline__ SturmPoint team_point(double x, bool is_a, bool is_b, const SturmPoint& a, const SturmPoint& b,
                                                 const SturmPoint& f, int lane) {
    SturmPoint o;
    const double m = is_a ? a.m : b.m;
    const int ec = is_a ? (a.e << 8) + a.c : (b.e << 8) + b.c;   // counts are at most 128
    const uint32_t team = (uint32_t)(__ballot(is_a || is_b) >> (lane & ~(TP - 1))) & ((1u << TP) - 1u);
    const int src = 4 * ((lane & ~(TP - 1)) + __builtin_ctz(team | (1u << TP)));
    const double mo = bpermute64(src, m);
    const int eco = __builtin_amdgcn_ds_bpermute(src, ec);
    o.m = team ? mo : f.m;
    o.e = team ? eco >> 8 : f.e;
    o.c = team ? eco & 255 : f.c;
    return o;
}

// Eigenvalues below kTriDead of the norm are not resolved: kDeadRel^2 of the largest, which the norm is at most four times
// of, is above it, and smaller ones are dropped by every caller.
constexpr double kTriDead = 3.637978807091713e-12;      // 2^-38
constexpr double kTriDone = 1.7763568394002505e-15;     // 2^-49
constexpr double kNear = 0.01;   // share of an interval where the first guess is trusted to be

// The matrix scaled by a power of two so that its norm is at most one, as t and es; the scale (0: the matrix is zero) in
// scal[0].  Wave 0; no barrier.
template <int N>
__device__ __forceinline__ void tri_scale(const double* dd, const double* ee, double* es, double2* t, double* scal) {
    const int tid = fresh_tid(), lane = tid & 63;
    if (tid < 64) {
        double bmax = 0.0;
        for (int i = lane; i < N; i += 64)
            bmax = fmax(bmax, fabs(dd[i]) + (i ? fabs(ee[i - 1]) : 0.0) + (i < N - 1 ? fabs(ee[i]) : 0.0));
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) bmax = fmax(bmax, __shfl_xor(bmax, m));
        const int ex = __builtin_amdgcn_frexp_exp(bmax);
        if (lane == 0) scal[0] = bmax > 0.0 ? __builtin_amdgcn_ldexp(1.0, ex) : 0.0;
        for (int i = lane; i < N; i += 64) {
            const double e1 = i ? __builtin_amdgcn_ldexp(ee[i - 1], -ex) : 0.0;
            t[i] = double2{__builtin_amdgcn_ldexp(dd[i], -ex), e1 * e1};
            if (i) es[i - 1] = e1;
        }
    }
}

// The R largest eigenvalues of the scaled matrix, lam[0..R-1] descending, to 2^-49 absolute.  256 threads (one wave per SIMD)
// first count at 512 points for all eigenvalues together; then TP lanes share an eigenvalue and cut its interval
// into 2 TP + 1 parts per round.  Returns the scale.
template <int N, int TP>
__device__ __forceinline__ double tri_values_even(const double* dd, const double* ee, double* es, double2* t, double* lam,
                                                  double* scal, int* cnt, int R) {
    static_assert(TP == 8, "32 eigenvalues at most");
    const int tid = fresh_tid(), lane = tid & 63;
    tri_scale<N>(dd, ee, es, t, scal);
    __syncthreads();
    const double bound = scal[0];
    // positive semidefinite up to rounding: [-2^-20, 1] holds every eigenvalue that matters
    constexpr double kLo = -9.5367431640625e-07, kStep = (1.0 - kLo) / 512;
    if (tid < 256) {
        SturmPoint a, b;
        sturm_points<N, false>(t, fma(kStep, (double)tid, kLo), fma(kStep, (double)(tid + 256), kLo), a, b);
        cnt[tid] = a.c;
        cnt[tid + 256] = b.c;
    }
    __syncthreads();
    if (tid < 256) {
        const int v = tid / TP, pt = tid % TP;
        const int k = v < R ? v : R - 1;
        int at = 0;                                      // last point whose count exceeds k
#pragma unroll
        for (int s = 256; s; s >>= 1) at += cnt[at + s] > k ? s : 0;
        double lo = fma(kStep, (double)at, kLo), w = kStep;
        constexpr int rounds = 10;                       // 17^10 > 2^40, after the first 2^9
#pragma unroll 1
        for (int it = 0; it < rounds; ++it) {
            w *= 1.0 / (2 * TP + 1);
            SturmPoint a, b;
            sturm_points<N, false>(t, fma(w, (double)(pt + 1), lo), fma(w, (double)(pt + 1 + TP), lo), a, b);
            const uint64_t m0 = __ballot(a.c > k), m1 = __ballot(b.c > k);
            constexpr uint32_t kTeam = (1u << TP) - 1u;
            const int sh = lane & ~(TP - 1);
            const int above = __popc((uint32_t)(m0 >> sh) & kTeam) + __popc((uint32_t)(m1 >> sh) & kTeam);
            lo = fma(w, (double)above, lo);
        }
        if (pt == 0 && v < R) lam[v] = fma(0.5, w, lo);
    }
    __syncthreads();
    return bound;
}

// The R largest eigenvalues of the tridiagonal matrix, scaled by a power of two so that its norm is at
// most one: lam[0..R-1] descending, to 2^-49 absolute.  256 threads (one wave per SIMD) first count
// at 512 points for all eigenvalues together, half of them spread evenly, half evenly in the logarithm below 2^-8 (a
// Gram matrix of iterated columns has its smallest eigenvalues there).  Then TP lanes share an eigenvalue and look at 2 TP
// points per round: as long as its interval holds others too, evenly spread; once it is alone, half of them so and
// half around the zero of the line through the determinants at the ends, at distances that the last round's miss
// suggests (the miss of that zero falls with the square of the width).  Counts decide what is kept, so a bad guess costs a
// round that cuts to a fifth or ninth.  Five to eight rounds, where cutting into 2 TP + 1 parts takes 10 or 13: 31 -> 25
// thousand cycles at 40 columns, 38 -> 28 at 64, 91 -> 60 at 128.  Up to 32 columns a round of counts is so short that what
// the guess costs (two hundred instructions) is not saved, and the parts stay even (24 columns: 14 thousand against 16).
// Returns the scale (0: the matrix is zero).
template <int N, int TP>
__device__ __forceinline__ double tri_values_guided(const double* dd, const double* ee, double* es, double2* t, double* lam,
                                                    double* scal, double* work, int R) {
    const int tid = fresh_tid(), lane = tid & 63;
    int* cnt = reinterpret_cast<int*>(work);             // [512], [512] and [512]: what the minors say on the grid
    int* ex2 = cnt + 512;
    double* det = work + 512;
    int* pos = reinterpret_cast<int*>(det + 512);        // [N] point of the grid below eigenvalue k
    static_assert(TriCfg<N, 8>::GRID >= 1024 + N / 2, "all of them in a work array");
    tri_scale<N>(dd, ee, es, t, scal);
    if (tid >= 64 && tid < 64 + N) pos[tid - 64] = 0;
    __syncthreads();
    const double bound = scal[0];
    // positive semidefinite up to rounding: [-2^-20, 1] holds every eigenvalue that matters
    constexpr double kLo = -9.5367431640625e-07;
    // 0: kLo; 1 .. 255: 2^(-38 + 30 (i - 1) / 254); 256 .. 511: evenly from 2^-8; 512: 1
    auto grid = [&](int i) __attribute__((always_inline)) {
        const float l = __builtin_amdgcn_exp2f(-38.f + (30.f / 254.f) * (float)(i - 1));
        return i == 0 ? kLo : i < 256 ? (double)l : i < 512 ? fma((double)(i - 256), (1.0 - 0.00390625) / 256, 0.00390625 + 1e-6) : 1.0;
    };
    if (tid < 256) {
        SturmPoint a, b;
        sturm_points<N, true>(t, grid(tid), grid(tid + 256), a, b);
        cnt[tid] = a.c;
        ex2[tid] = a.e;
        det[tid] = a.m;
        cnt[tid + 256] = b.c;
        ex2[tid + 256] = b.e;
        det[tid + 256] = b.m;
    }
    __syncthreads();
    static_assert(kTriThreads == 512, "a thread to a point");
    const int over = cnt[tid] < R ? cnt[tid] : R;
    for (int k = tid < 511 ? cnt[tid + 1] : 0; k < over; ++k) pos[k] = tid;
    __syncthreads();
    if (tid < 256) {
        const int v = tid / TP, pt = tid % TP;
        const int k = v < R ? v : R - 1;
        const int at = pos[k];
        double lo = grid(at), hi = grid(at + 1);
        SturmPoint fl = {cnt[at], ex2[at], det[at]}, fh = {-1, 0, 0.0};   // nothing is known at 1
        if (at < 511) fh = SturmPoint{cnt[at + 1], ex2[at + 1], det[at + 1]};
        double near = kNear * (hi - lo);                 // distance of the innermost points around the guess
        constexpr int H = TP / 2;
        const int ring = pt < H ? H - 1 - pt : pt - H;   // 0: innermost
        const double far = (pt < H ? -1.0 : 1.0) * (ring == 0 ? 1.0 : ring == 1 ? 64.0 : ring == 2 ? 512.0 : 4096.0);
        const double even_half = (pt + 1) * (1.0 / (TP + 1)), even_a = (pt + 1) * (1.0 / (2 * TP + 1)),
                     even_b = (pt + 1 + TP) * (1.0 / (2 * TP + 1));
#pragma unroll 1
        for (int it = 0; it < 20; ++it) {
            const double w = hi - lo;
            if (!__any(w > kTriDone && hi > kTriDead)) break;
            const bool alone = fl.c == k + 1 && fh.c == k;
            // zero of the line through the determinants at the ends
            const double ratio = fmax(__builtin_amdgcn_ldexp(fh.m, fh.e - fl.e) * rcp64(fl.m), -1.0e100);
            const double guess = fma(w, rcp64(1.0 - ratio), lo);
            const double xa = fma(w, alone ? even_half : even_a, lo);
            const double aim = fmin(fmax(fma(near, far, guess), lo), hi), xb = alone ? aim : fma(w, even_b, lo);
            SturmPoint a, b;
            sturm_points<N, true>(t, xa, xb, a, b);
            const bool ua = a.c > k, ub = b.c > k;
            const double l2 = team_end64<TP, true>(fmax(fmax(lo, ua ? xa : lo), ub ? xb : lo));
            const double h2 = team_end64<TP, false>(fmin(fmin(hi, ua ? hi : xa), ub ? hi : xb));
            fl = team_point<TP>(l2, ua && xa == l2, ub && xb == l2, a, b, fl, lane);
            fh = team_point<TP>(h2, !ua && xa == h2, !ub && xb == h2, a, b, fh, lane);
            // the miss of the guess was at most the distance to the further end; the next one's is smaller by the square
            // of the ratio of the widths
            const double w2 = h2 - l2, shrink = w2 * rcp64(w);
            const double miss = fmax(fabs(h2 - guess), fabs(guess - l2));
            near = fmin(alone ? fmax(miss * shrink * shrink, 0.25 * kTriDone) : w2, kNear * w2);
            lo = l2;
            hi = h2;
        }
        if (pt == 0 && v < R) lam[v] = fma(0.5, hi - lo, lo);
    }
    __syncthreads();
    return bound;
}

template <int N, int TP>
__device__ __forceinline__ double tri_values(const double* dd, const double* ee, double* es, double2* t, double* lam,
                                             double* scal, double* work, int R) {
    if constexpr (N <= 32) return tri_values_even<N, TP>(dd, ee, es, t, lam, scal, reinterpret_cast<int*>(work), R);
    else return tri_values_guided<N, TP>(dd, ee, es, t, lam, scal, work, R);
}

// multipliers of the factorization of T - l I from the top (DIR = 1) or the bottom (DIR = -1)
template <int N, int RB, int DIR>
__device__ __forceinline__ void tri_factor(const double2* t, const double* es, double l, double* w) {
    double dn = t[DIR > 0 ? 0 : N - 1].x - l;
#pragma unroll 8
    for (int s = 0; s < N - 1; ++s) {
        const int i = DIR > 0 ? s : N - 1 - s;
        const double e = es[DIR > 0 ? i : i - 1];
        const double m = -e * rcp64(dn + 1.0e-300);      // a zero pivot becomes a tiny one
        w[i * RB] = m;
        dn = fma(e, m, t[i + DIR].x - l);
    }
}

// Eigenvectors v0 .. v0 + nb - 1 of the scaled tridiagonal matrix, from twisted factorizations: the
// multipliers of the forward and backward factorizations (one wave each) in wa and wb [N][RB], the
// twist where the pivot is smallest, and the vector grown from it in both directions.  The
// unnormalized vector replaces wa.
template <int N, int RB>
__device__ __forceinline__ void tri_vectors(const double2* t, const double* es, const double* lam, double* wa,
                                            double* wb, int* twist, int v0, int nb) {
    const int tid = fresh_tid(), lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (wave == 0) {
        if (lane < nb) tri_factor<N, RB, 1>(t, es, lam[v0 + lane], wa + lane);
    } else if (wave == 1) {
        if (lane < nb) tri_factor<N, RB, -1>(t, es, lam[v0 + lane], wb + lane);
    }
    __syncthreads();
    {
        const int v = tid >> 3, s = tid & 7;
        if (v < nb) {
            const double l = lam[v0 + v];
            double best = 1.0e300;
            int bi = 0;
#pragma unroll 4
            for (int i = s; i < N; i += 8) {
                const int ip = i > 0 ? i - 1 : 0, in = i < N - 1 ? i : N - 2;
                double g = t[i].x - l;
                g = fma(i > 0 ? es[ip] : 0.0, wa[ip * RB + v], g);
                g = fma(i < N - 1 ? es[in] : 0.0, wb[(in + 1) * RB + v], g);
                g = fabs(g);
                if (g < best) { best = g; bi = i; }
            }
#pragma unroll
            for (int m = 1; m < 8; m <<= 1) {
                const double ob = __shfl_xor(best, m);
                const int oi = __shfl_xor(bi, m);
                if (ob < best || (ob == best && oi < bi)) { best = ob; bi = oi; }
            }
            if (s == 0) twist[v] = bi;
        }
    }
    __syncthreads();
    if (wave < 2 && lane < nb) {
        const int r = twist[lane];
        double z = 1.0;
        if (wave == 0) {
#pragma unroll 8
            for (int i = N - 2; i >= 0; --i) {
                const double m = wa[i * RB + lane];
                z *= i < r ? m : 1.0;
                if (i < r) wa[i * RB + lane] = z;
            }
            wa[r * RB + lane] = 1.0;
        } else {
#pragma unroll 8
            for (int i = 1; i < N; ++i) {
                const double m = wb[i * RB + lane];
                z *= i > r ? m : 1.0;
                if (i > r) wa[i * RB + lane] = z;
            }
        }
    }
    __syncthreads();
}

// Vector v of wa (a column of [N][RB]), normalized, in a team of TB lanes: entry TB*q + u in y[q] of lane u.
template <int N, int RB, int TB>
__device__ __forceinline__ void tri_load(const double* wa, int v, int u, double (&y)[N / TB]) {
    double nn = 0.0;
#pragma unroll
    for (int q = 0; q < N / TB; ++q) {
        y[q] = wa[(TB * q + u) * RB + v];
        nn = fma(y[q], y[q], nn);
    }
    const double sc = rsq64(team_sum64<TB>(nn));
#pragma unroll
    for (int q = 0; q < N / TB; ++q) y[q] *= sc;
}

// cross[k] = u_k . u_(k+1) of the reflectors in U, for k = 0 .. N - 4, one team of eight lanes each.
template <int N>
__device__ __forceinline__ void tri_cross(const double* U, double* cross) {
    const int tid = fresh_tid(), team = tid >> 3, s = tid & 7;
    for (int k = team; k < N - 3; k += kTriThreads / 8) {
        const double *uk = U + tri_row(N, k), *ul = U + tri_row(N, k + 1);
        double d = 0.0;
        for (int j = k + 2 + s; j < N; j += 8) d = fma(uk[j], ul[j], d);
        d = team_sum64<8>(d);
        if (s == 0) cross[k] = d;
    }
    __syncthreads();
}

// The reflectors applied to the vector in y, last one first and two at a time: with s1 = u1 . y and
// s0 = u0 . y taken together, the first one changes the second product by (u0 . u1) s1 / h1.  The block of
// TB rows that the pivots are in is a compile-time constant, so only one entry per lane needs a mask.
template <int N, int TB, int QK>
__device__ __forceinline__ void tri_back_block(const double* U, const double* ih, const double* cross, int u,
                                               double (&y)[N / TB]) {
    constexpr int QB = N / TB;
    constexpr int kTop = TB * QK + TB - 1 < N - 3 ? TB * QK + TB - 1 : N - 3;
    auto load = [&](int k, double (&w)[QB]) __attribute__((always_inline)) {
        const double* uk = U + tri_row(N, k) + u;
        w[QK] = TB * QK + u > k ? uk[TB * QK] : 0.0;
#pragma unroll
        for (int q = QK + 1; q < QB; ++q) w[q] = uk[TB * q];
    };
    int k = kTop;
    if constexpr ((kTop - TB * QK) % 2 == 0) {
        double w[QB], s = 0.0;
        load(k, w);
#pragma unroll
        for (int q = QK; q < QB; ++q) s = fma(w[q], y[q], s);
        s = team_sum64<TB>(s) * ih[k];
#pragma unroll
        for (int q = QK; q < QB; ++q) y[q] = fma(-s, w[q], y[q]);
        --k;
    }
#pragma unroll 1
    for (; k > TB * QK; k -= 2) {
        double w1[QB], w0[QB], s1 = 0.0, s0 = 0.0;
        load(k, w1);
        load(k - 1, w0);
        const double h1 = ih[k], h0 = ih[k - 1], cr = cross[k - 1];
#pragma unroll
        for (int q = QK; q < QB; ++q) {
            s1 = fma(w1[q], y[q], s1);
            s0 = fma(w0[q], y[q], s0);
        }
        s1 = team_sum64<TB>(s1) * h1;
        s0 = team_sum64<TB>(s0);
        s0 = fma(-cr, s1, s0) * h0;
#pragma unroll
        for (int q = QK; q < QB; ++q) y[q] = fma(-s0, w0[q], fma(-s1, w1[q], y[q]));
    }
    if constexpr (QK > 0) tri_back_block<N, TB, QK - 1>(U, ih, cross, u, y);
}

template <int N, int TB>
__device__ __forceinline__ void tri_back(const double* U, const double* ih, const double* cross, int u,
                                         double (&y)[N / TB]) {
    tri_back_block<N, TB, (N - 3) / TB>(U, ih, cross, u, y);
}

}  // namespace solar
