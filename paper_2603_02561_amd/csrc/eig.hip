// Top-r eigenpairs of each user's d x d Gram matrix G = X^T X, one workgroup per
// user, iterate blocks held in LDS.  S = sqrt(eigenvalues), V = eigenvectors are
// the s and R that Algorithm 1 ("Randomized SVD with Power Iteration") returns.
//
// Wide blocks (r near d) are solved directly, by the double-precision solver of tridiag.h applied to G.
//
// Otherwise the iteration is Algorithm 1 expressed on G: a Gaussian start block Omega
// (d x L, L = r + oversampling), power steps Omega <- X^T (X Omega) = G Omega, an
// orthonormal basis of the block, and a small decomposition of the projected
// problem.  On the first power steps only the span of the block matters, and the
// basis is taken panel by panel (basis_panels).  After those, basis and small
// decomposition are done together on the d x L block Z = G Q: making its columns mutually
// orthogonal diagonalizes Q^T G^2 Q, which is the Rayleigh-Ritz step for G^2 on span(Q), and
// the normalized columns are the next orthonormal basis.  ritz_rotate does it through the
// eigenvectors of Z^T Z in double precision; the narrowest blocks and those with coinciding
// eigenvalues take one-sided (Hestenes) Jacobi sweeps over the columns of Z, and so does d = 64, r = 9 .. 16 with more
// users than compute units.  Both are insensitive
// to the huge dynamic range of the block (G Omega is dominated by the leading
// eigenvectors) and to rank deficiency (columns that vanish are dropped).  The power
// step after a Jacobi phase yields the residuals |G q_i - theta_i q_i| of the Ritz
// pairs; the iteration ends when every wanted pair is below tol_res * theta_max, and a
// failed check doubles the number of such steps before the next Jacobi phase.
//
// The block stays in registers, a wave holding whole rows of it, which is how the products leave it and how the basis wants
// it; columns of floats in LDS exist only where a Ritz step or a sweep needs them.  What bounds the phase is latency:
// factorizations of the panels, the reduction of the dense solver and Jacobi sweeps are chains of dependent steps
// (d = 128, 40 columns, thousands of cycles: staging and start 9, four products 16, two bases 38, Ritz step 109,
// checks and output 10; with the block in LDS, products on the float instruction and a modified Gram-Schmidt pass over the
// columns 18, 30, 56, 118, 28; 64 users 109 -> 83 us, d = 256 178 -> 114).  A wave that has its SIMD to itself issues an
// instruction in five cycles, so the chains count their instructions; dozens of lane addresses that the compiler formed ahead
// of the loop and then kept in scratch cost as much as a Gram-Schmidt pass (fresh_tid).  The
// kernel runs eight waves (two per SIMD), gives every column pair of a sweep a team of up to 16
// lanes whose partial dot products are combined with DPP lane permutations, and keeps
// every trip count a compile-time constant.
#include "column_block.h"
#include "common.h"
#include "kernels.h"

namespace solar {

namespace {

__device__ __forceinline__ uint32_t mix32(uint32_t x) {
    x ^= x >> 16; x *= 0x7feb352du; x ^= x >> 15; x *= 0x846ca68bu; x ^= x >> 16;
    return x;
}

// Two standard normal draws for the start block, entries (i, j) and (i + 1, j) for even i: counter-based, Box-Muller.
__device__ __forceinline__ float2 omega_pair(int b, int j, int i) {
    const uint32_t c = mix32((uint32_t)b * 0x9e3779b9u + (uint32_t)j * 0x85ebca6bu + (uint32_t)i + 0x1234567u);
    const uint32_t c2 = mix32(c ^ 0x68bc21ebu);
    const float u1 = ((c >> 8) + 1u) * (1.0f / 16777217.0f);
    const float u2 = (c2 >> 8) * (1.0f / 16777216.0f);          // in turns
    const float m = __builtin_amdgcn_sqrtf(-1.38629436112f * __builtin_amdgcn_logf(u1));   // 2 ln 2 log2(u1)
    return float2{m * __builtin_amdgcn_cosf(u2), m * __builtin_amdgcn_sinf(u2)};
}

// Where G lies in LDS (d <= 128) column CPL*i + s of X, CPL = D/16, is row and column 16*s + i, and so it is in the
// iterate; otherwise the order is that of X.
template <int D>
__device__ __forceinline__ int eig_row(int p) { return D <= 128 ? (D / 16) * (p % 16) + p / 16 : p; }
template <int D>
__device__ __forceinline__ int eig_place(int i) { return D <= 128 ? 16 * (i % (D / 16)) + i / (D / 16) : i; }

// Orders entries v of a column by magnitude, the first in the order of X (index i) on ties; the lowest bit is the sign.
template <int D>
__device__ __forceinline__ uint64_t entry_key(float v, int i) {
    const uint32_t x = __float_as_uint(v);
    return (uint64_t)(x & 0x7fffffffu) << 32 | (uint32_t)((D - 1 - i) << 1) | x >> 31;
}

// most power steps that a slow convergence rate may add before the first Ritz step or Jacobi phase
constexpr int kExtraStepsCap = 4;

// three bf16 terms of eight consecutive values
__device__ __forceinline__ void split3_eight(v4f lo, v4f hi, v4u (&o)[3]) {
    float x[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const v2bf t = {(__bf16)x[2 * u], (__bf16)x[2 * u + 1]};
            o[q][u] = __builtin_bit_cast(uint32_t, t);
            x[2 * u] -= bf16_lo(o[q][u]);
            x[2 * u + 1] -= bf16_hi(o[q][u]);
        }
}

template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_rows(float v) {     // v where the rows of ROWS do not take part
    const int i = __float_as_int(v);
    return __int_as_float(__builtin_amdgcn_update_dpp(i, i, CTRL, ROWS, 0xf, false));
}
// In lane 63: the largest of the wave's values, none of them negative.
__device__ __forceinline__ float wave_top(float v) {
    v = fmaxf(v, dpp_mov<0xB1>(v));
    v = fmaxf(v, dpp_mov<0x4E>(v));
    v = fmaxf(v, dpp_mov<0x141>(v));
    v = fmaxf(v, dpp_mov<0x140>(v));
    v = fmaxf(v, dpp_rows<0x142, 0xa>(v));               // row_bcast15: rows 1 and 3 take over the row before
    return fmaxf(v, dpp_rows<0x143, 0xc>(v));            // row_bcast31
}

// The iteration runs on 2^-ge G, with ge even and the largest entry, which is on the diagonal, brought to about one: squares of
// columns of G Q, in the panels, the sweeps and the residuals, would leave the range of a float for s_1 above 4e9 or below
// 1e-10, and the factors would come out as those of a zero matrix, or as NaN.  A power of two changes no rounding.
__device__ __forceinline__ int gram_exponent(int top_bits) { return min(top_bits >> 23 & ~1, 252) - 126; }
__device__ __forceinline__ float gram_scale(int ge) { return __int_as_float((127 - ge) << 23); }

// G as the operand of G Q: the wave's rows, three bf16 terms per value (what is left after three is below 2^-26), lane
// (i, g) holding entries 32 k + 8 g .. + 7 of row i of a block in chunk k.  Up to d = 128 they stay in registers for the
// whole solve; at d = 256 that would take 192 of them, so the rows come from L2 for every product, three chunks ahead, and
// are split on the way.
template <int D>
struct GramRows {
    static constexpr bool kKept = D <= 128;
    static constexpr int NB = D > 128 ? D / 128 : 1, NK = D / 32, RING = kKept ? 1 : 4;
    v4u a[kKept ? NK : 1][3];
    v4f ring[RING][NB][2];
    const float* rows;                                   // of this lane, in memory (d = 256)

    __device__ __forceinline__ void keep(const float* Gs, int stride, float scale, int wave, int i16, int g) {
#pragma unroll
        for (int k = 0; k < NK; ++k) {
            const float* src = Gs + (16 * wave + i16) * stride + 32 * k + 8 * g;
            split3_eight(scale * *reinterpret_cast<const v4f*>(src), scale * *reinterpret_cast<const v4f*>(src + 4), a[k]);
        }
    }
    __device__ __forceinline__ void load(int k) {
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                ring[k % RING][n][h] = *reinterpret_cast<const v4f*>(rows + (size_t)n * 128 * D + 32 * k + 4 * h);
    }
    // ahead of a product, before the barrier it waits at
    __device__ __forceinline__ void prefetch() {
        if constexpr (!kKept) {
#pragma unroll
            for (int k = 0; k < RING - 1; ++k) load(k);
        }
    }
};

// Images of the iterate for the products: [term][column][row], three bf16 terms per value.
template <int D, int LP>
__device__ __forceinline__ void store_images(uint16_t* img, const typename Iterate<D, LP>::Regs& q, int wave) {
    const int lane = fresh_tid() & 63, i16 = lane & 15, g = lane >> 4;
    using I = Iterate<D, LP>;
    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int n = 0; n < I::NB; ++n)
#pragma unroll
        for (int c = 0; c < I::NC; ++c) {
            v4f x = q[n][c];
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                const v2bf lo = {(__bf16)x[0], (__bf16)x[1]}, hi = {(__bf16)x[2], (__bf16)x[3]};
                const uint2 w = {__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
                *reinterpret_cast<uint2*>(img + (e * LP + 16 * c + i16) * I::LDI + 16 * (wave + kEigWaves * n) + 4 * g) = w;
                x[0] -= bf16_lo(w.x); x[1] -= bf16_hi(w.x);
                x[2] -= bf16_lo(w.y); x[3] -= bf16_hi(w.y);
            }
        }
}

// z = (2^-ge G - shift I) q on the bf16 instruction: the six products of terms above 2^-25 of a product of two values, smallest
// first.  (Rows that stay in registers have the factor in them; otherwise it is applied behind the products, a twentieth of the
// multiplications that the rows would take on their way.)  Against the float instruction (256 cycles per 32 rows and 16 x 16 block instead of 96, and G from LDS) the four
// products of a solve at d = 128, 40 columns take 15 thousand cycles instead of 30, at d = 256 65
// instead of 140.
template <int D, int LP>
__device__ __forceinline__ void multiply(GramRows<D>& G, const uint16_t* img, const typename Iterate<D, LP>::Regs& q,
                                         float shift, int ge, typename Iterate<D, LP>::Regs& z) {
    const int lane = fresh_tid() & 63, i16 = lane & 15, g = lane >> 4;
    using I = Iterate<D, LP>;
    constexpr int NB = I::NB, NC = I::NC, NK = D / 32;
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
        for (int c = 0; c < NC; ++c) z[n][c] = -(GramRows<D>::kKept ? shift : __builtin_amdgcn_ldexpf(shift, ge)) * q[n][c];
    const uint16_t* base = img + i16 * I::LDI + 8 * g;
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        v4u a[NB][3];
        if constexpr (GramRows<D>::kKept) {
#pragma unroll
            for (int e = 0; e < 3; ++e) a[0][e] = G.a[k][e];
        } else {
            if (k + GramRows<D>::RING - 1 < NK) G.load(k + GramRows<D>::RING - 1);
#pragma unroll
            for (int n = 0; n < NB; ++n) split3_eight(G.ring[k % GramRows<D>::RING][n][0], G.ring[k % GramRows<D>::RING][n][1], a[n]);
        }
        v4u b[NC][3];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int e = 0; e < 3; ++e)
                b[c][e] = *reinterpret_cast<const v4u*>(base + (e * LP + 16 * c) * I::LDI + 32 * k);
        constexpr int kA[6] = {0, 2, 1, 0, 1, 0}, kB[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
        for (int p = 0; p < 6; ++p)
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int c = 0; c < NC; ++c) z[n][c] = mfma16x16x32bf16(a[n][kA[p]], b[c][kB[p]], z[n][c]);
    }
    if constexpr (!GramRows<D>::kKept) {
        const float scale = gram_scale(ge);
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int c = 0; c < NC; ++c) z[n][c] *= scale;
    }
}

// the iterate to and from columns of floats in LDS, column stride D + 4
template <int D, int LP>
__device__ __forceinline__ void store_columns(float* Cc, const typename Iterate<D, LP>::Regs& q, int wave) {
    const int lane = fresh_tid() & 63, i16 = lane & 15, g = lane >> 4;
    using I = Iterate<D, LP>;
#pragma unroll
    for (int n = 0; n < I::NB; ++n)
#pragma unroll
        for (int c = 0; c < I::NC; ++c)
            *reinterpret_cast<v4f*>(Cc + (16 * c + i16) * (D + 4) + 16 * (wave + kEigWaves * n) + 4 * g) = q[n][c];
}
template <int D, int LP>
__device__ __forceinline__ void load_columns(const float* Cc, typename Iterate<D, LP>::Regs& q, int wave) {
    const int lane = fresh_tid() & 63, i16 = lane & 15, g = lane >> 4;
    using I = Iterate<D, LP>;
#pragma unroll
    for (int n = 0; n < I::NB; ++n)
#pragma unroll
        for (int c = 0; c < I::NC; ++c)
            q[n][c] = *reinterpret_cast<const v4f*>(Cc + (16 * c + i16) * (D + 4) + 16 * (wave + kEigWaves * n) + 4 * g);
}

// lane ^ 1 or ^ 2
template <int X>
__device__ __forceinline__ float quad_xor(float v) { return dpp_mov<X == 1 ? 0xB1 : 0x4E>(v); }
template <int X>
__device__ __forceinline__ double quad_xor(double v) { return dpp_mov64<X == 1 ? 0xB1 : 0x4E>(v); }

// sums[c] = the sum of v over all rows of column c, in a fixed order.  `red` has 4 W rows of LP values.  Ends with a barrier.
template <int D, int LP, typename T>
__device__ __forceinline__ void column_sums(const T (&v)[LP / 16], T* red, float* sums, int wave) {
    const int tid = fresh_tid(), lane = tid & 63, i16 = lane & 15, g = lane >> 4;
    using I = Iterate<D, LP>;
    if (wave < I::W) {
#pragma unroll
        for (int c = 0; c < I::NC; ++c) red[(4 * wave + g) * LP + 16 * c + i16] = v[c];
    }
    __syncthreads();
    const int c = tid >> 2, u = tid & 3;
    if (c < LP) {
        T s = 0;
#pragma unroll
        for (int w = 0; w < I::W; ++w) s += red[(4 * w + u) * LP + c];
        s += quad_xor<1>(s);
        s += quad_xor<2>(s);
        if (u == 0) sums[c] = (float)s;
    }
    __syncthreads();
}

// Rank of v[e / 8] among v[0 .. L-1], largest first (the earlier one on ties), by the eight lanes with that e / 8; `top`
// receives the largest.  The rank means nothing from e = 8 L on.
template <int L>
__device__ __forceinline__ int rank_of(const float* v, int e, float& top) {
    const int k0 = e >> 3, u = e & 7;
    const float mine = v[k0 < L ? k0 : 0];
    int rk = 0;
    top = v[u];
#pragma unroll
    for (int k = 0; k < L; k += 8) {
        const float vk = v[k + u];
        top = fmaxf(top, vk);
        rk += (vk > mine || (vk == mine && k + u < k0)) ? 1 : 0;
    }
    top = fmaxf(top, dpp_mov<0xB1>(top));
    top = fmaxf(top, dpp_mov<0x4E>(top));
    top = fmaxf(top, dpp_mov<0x141>(top));
    return (int)team_sum<8>((float)rk);
}

// a += a[lane I of the row of 16 lanes] * y
template <int I>
__device__ __forceinline__ void fmac_own_bcast(float& a, float y) {
    a = fmaf(__int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(a), 0x150 + I, 0xf, 0xf, true)), y, a);
}

// Elimination on the leading KN x KN block of a 16 x 16 Gram matrix, by one wave: a[i] is row i, lane j (and j + 16, ...)
// column j.  m[k] receives the negative multipliers of pivot row k; afterwards lane k of a[k] is pivot k.  A
// pivot not above dead2 is passed over.  The wave has its SIMD to itself and issues an instruction in five cycles, so what
// counts is how few a step takes: entry (k, i) of the pivot row is a lane broadcast inside the multiply-add
// of row i (16 lanes are the widest it reaches).  A lane broadcast as an instruction of its own needs one for each
// half of a double; the rank-one update as a matrix instruction in double precision holds the unit, which
// the vector ALU's doubles share, for 64 cycles: 280 to 440 cycles a step, 150 this way.
template <int I, int KN, int K>
__device__ __forceinline__ void eliminate_rows(double (&a)[16], double nra) {
    if constexpr (I + 3 < KN) {
        fmac_bcast64<I>(a[I], a[I + 1], a[I + 2], a[I + 3], a[K], nra);
        eliminate_rows<I + 4, KN, K>(a, nra);
    } else if constexpr (I < KN) {
        fmac_bcast64<I>(a[I], a[K], nra);
        eliminate_rows<I + 1, KN, K>(a, nra);
    }
}
template <int K, int KN>
__device__ __forceinline__ void panel_steps(double (&a)[16], float (&m)[16], double dead2) {
    if constexpr (K + 1 < KN) {
        const double piv = readlane64(a[K], K);
        const double nra = a[K] * (piv > dead2 ? -rcp64(piv) : 0.0);
        eliminate_rows<K + 1, KN, K>(a, nra);
        m[K] = (float)nra;
        panel_steps<K + 1, KN>(a, m, dead2);
    }
}
// z <- z R^-1 up to the scale of its columns: the same eliminations on the columns of the wave's rows
template <int K, int KN, int NV>
__device__ __forceinline__ void panel_solve(float (&z)[NV], const float (&m)[16]) {
    if constexpr (K + 1 < KN) {
#pragma unroll
        for (int v = 0; v < NV; ++v) fmac_own_bcast<K>(z[v], m[K]);
        panel_solve<K + 1, KN, NV>(z, m);
    }
}

// A basis of span(z), orthonormal to about 2^-24 * cond(z), which is all a power step needs: panels of 16 columns.  The
// Gram matrix of a panel is formed and factored in double precision, Q_p = Z_p R^-1, and Q_p is projected out of the
// columns after it, both on the float instruction.  Only the factorization, 16 steps of one wave, is a
// chain; column by column (modified Gram-Schmidt, a team of lanes per column) a pass was one chain of all columns: 28
// thousand cycles at d = 128, 40 columns, and 45 at d = 256, now 17 and 28.  Columns that collapse below kBasisDead of the largest of the first panel are dropped (zero).
// pivot2[j] receives the squared norm that column j had when it was normalized (the squared diagonal of the
// triangular factor, which tends to the eigenvalues of G in decreasing order).  No barrier before the first
// and after the last access to LDS.
template <int D, int L, int LP, int P>
__device__ __forceinline__ void basis_panels(typename Iterate<D, LP>::Regs& z, typename Iterate<D, LP>::Regs& q,
                                             const BasisLds<D, LP>& w, float* pivot2, double dead2, int wave) {
    using I = Iterate<D, LP>;
    constexpr int NB = I::NB, NC = I::NC, W = I::W, kT = BasisLds<D, LP>::kT, NR = NC - 1 - P;
    const int tid = fresh_tid(), lane = tid & 63, i16 = lane & 15, g = lane >> 4;
    float* tr = w.tr + wave * (NB * 16 * kT);
    const bool holds = wave < W;
    constexpr int KN = L - 16 * P < 16 ? L - 16 * P : 16;   // columns of the panel that are not padding
    if (holds) {
        v4d ac = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const double x = (double)z[n][P][t];
                ac = mfma16x16x4f64(x, x, ac);
            }
#pragma unroll
        for (int t = 0; t < 4; ++t) w.gm[(wave * 16 + g + 4 * t) * 16 + i16] = ac[t];
    }
    __syncthreads();
    if (tid < 256) {
        double s = w.gm[tid];
#pragma unroll
        for (int v = 1; v < W; ++v) s += w.gm[v * 256 + tid];
        w.gs[tid] = s;
    }
    __syncthreads();
    if (wave == 0) {
        double a[16];
#pragma unroll
        for (int k = 0; k < KN; ++k) a[k] = w.gs[16 * k + i16];
        if constexpr (P == 0) {                          // the largest norm of the panel
            float top = i16 < KN ? (float)w.gs[17 * i16] : 0.f;
            top = fmaxf(top, dpp_mov<0xB1>(top));
            top = fmaxf(top, dpp_mov<0x4E>(top));
            top = fmaxf(top, dpp_mov<0x141>(top));
            top = fmaxf(top, dpp_mov<0x140>(top));
            dead2 = (double)kBasisDead * (double)kBasisDead * (double)top;
        }
        float m[16];
        panel_steps<0, KN>(a, m, dead2);
        double piv = 0.0;
#pragma unroll
        for (int k = 0; k < KN; ++k) piv = i16 == k ? a[k] : piv;
        if (lane < 16) {                                 // lane j: column j of the multipliers, zero up to the diagonal
#pragma unroll
            for (int k = 0; k < KN; k += 4) {
                v4f o;
#pragma unroll
                for (int u = 0; u < 4; ++u) o[u] = k + u + 1 < KN && i16 > k + u ? m[k + u] : 0.f;
                *reinterpret_cast<v4f*>(w.tm + i16 * kT + k) = o;
            }
            w.tm[i16 * kT + 16] = piv > dead2 ? (float)rsq64(piv) : 0.f;
            pivot2[16 * P + i16] = fmaxf((float)piv, 0.f);
        }
    }
    __syncthreads();
    v4f qt[NB];                                          // the wave's rows of Q_p, lane (i, g): row i, columns 4 g ..
    if (holds) {
        float m[16], x[4 * NB];
#pragma unroll
        for (int k = 0; k < KN; k += 4) {
            const v4f o = *reinterpret_cast<const v4f*>(w.tm + i16 * kT + k);
#pragma unroll
            for (int u = 0; u < 4; ++u) m[k + u] = o[u];
        }
        const float rs = w.tm[i16 * kT + 16];
#pragma unroll
        for (int v = 0; v < 4 * NB; ++v) x[v] = z[v / 4][P][v % 4];
        panel_solve<0, KN, 4 * NB>(x, m);
#pragma unroll
        for (int v = 0; v < 4 * NB; ++v) q[v / 4][P][v % 4] = x[v] * rs;
    }
    if constexpr (NR > 0) {
        if (holds) {
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int t = 0; t < 4; ++t) tr[n * 16 * kT + (4 * g + t) * kT + i16] = q[n][P][t];
            wave_order();
#pragma unroll
            for (int c = 0; c < NR; ++c) {
                v4f o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int n = 0; n < NB; ++n)
#pragma unroll
                    for (int t = 0; t < 4; ++t) o = mfma16x16x4(q[n][P][t], z[n][P + 1 + c][t], o);
                *reinterpret_cast<v4f*>(w.cp + (wave * NR + c) * 256 + 4 * lane) = o;
            }
#pragma unroll
            for (int n = 0; n < NB; ++n) qt[n] = *reinterpret_cast<const v4f*>(tr + n * 16 * kT + i16 * kT + 4 * g);
        }
        __syncthreads();
        for (int e = tid; e < NR * 256; e += kEigThreads) {
            float s = 0.f;
#pragma unroll
            for (int v = 0; v < W; ++v) s += w.cp[v * NR * 256 + e];
            w.cs[e] = s;
        }
        __syncthreads();
        if (holds) {
#pragma unroll
            for (int c = 0; c < NR; ++c) {
                const v4f cv = *reinterpret_cast<const v4f*>(w.cs + c * 256 + 4 * lane);
#pragma unroll
                for (int n = 0; n < NB; ++n)
#pragma unroll
                    for (int s = 0; s < 4; ++s) z[n][P + 1 + c] = mfma16x16x4(-qt[n][s], cv[s], z[n][P + 1 + c]);
            }
            wave_order();                                // tr is written again
        }
        basis_panels<D, L, LP, P + 1>(z, q, w, pivot2, dead2, wave);
    }
}

// The r leading eigenpairs straight from the D x D matrix in Gs (LDS, row stride GS), written to S and V.
// Takes all of the dynamic LDS; Gs may lie anywhere in it.  False (nothing written): two wanted
// eigenvalues are too close.
template <int D, int RMAX, int RB, int GS>
__device__ __forceinline__ bool eig_direct(const float* Gs, double* sm, double* scal, int* twist, int r, float* S,
                                           float* V) {
    constexpr int TB = RMAX <= 32 && D == 128 ? 16 : 8;
    using T = TriCfg<D, RB>;
    static_assert(RMAX * TB <= kEigThreads, "a team to a vector");
    const TriLds<D, RB> w(sm, nullptr);
    const int tid = fresh_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    TriRows<D> a;
    if (wave < kTriWaves) {
#pragma unroll
        for (int m = 0; m < T::RS; ++m)
#pragma unroll
            for (int c = 0; c < T::NC; ++c)
                a[m][c] = Gs[(16 * (m / 4) + 4 * wave + m % 4) * GS + (lane ^ (4 * wave)) + 64 * c];
    }
    __syncthreads();
    tri_reduce<D>(a, w.wb, w.U, w.dd, w.ee, w.ih);
    const double bound = tri_values<D, (RMAX <= 32 ? 8 : 4)>(w.dd, w.ee, w.es, w.t, w.lam, scal,
                                                             w.wb, r);
    const double l0 = w.lam[0], dead = (double)kDeadRel * l0;
    const bool any = bound > kTriZero && l0 > 0.0;
    const bool close = tid + 1 < r && w.lam[tid + 1] > dead && w.lam[tid] - w.lam[tid + 1] < kTriGap;
    if (__syncthreads_or(any && close)) return false;
    const int v = tid / TB, u = tid % TB;
    double y[D / TB];
#pragma unroll 1
    for (int v0 = 0; v0 < r; v0 += RB) {
        const int nb = r - v0 < RB ? r - v0 : RB;
        tri_vectors<D, RB>(w.t, w.es, w.lam, w.wa, w.wb, twist, v0, nb);
        if (v >= v0 && v < v0 + nb) tri_load<D, RB, TB>(w.wa, v - v0, u, y);
        __syncthreads();
    }
    tri_cross<D>(w.U, w.dd);
    float* out = reinterpret_cast<float*>(w.wb);         // [D][r + 1]
    static_assert(2 * T::WB >= D * (RMAX + 1), "V in a work array");
    if (v < r) {
        tri_back<D, TB>(w.U, w.ih, w.dd, u, y);
        const double l = w.lam[v];
        const bool live = any && l > dead;
        // sign fixed by the largest-magnitude entry
        uint64_t best = 0;
#pragma unroll
        for (int q = 0; q < D / TB; ++q) best = max(best, entry_key<D>((float)y[q], eig_row<D>(TB * q + u)));
#pragma unroll
        for (int m = 1; m < TB; m <<= 1) best = max(best, (uint64_t)__shfl_xor((unsigned long long)best, m));
        const float sgn = (best & 1) ? -1.f : 1.f;
#pragma unroll
        for (int q = 0; q < D / TB; ++q) out[eig_row<D>(TB * q + u) * (r + 1) + v] = live ? sgn * (float)y[q] : 0.f;
        if (u == 0) S[v] = live ? (float)(l * bound * rsq64(l * bound)) : 0.f;
    }
    // by way of LDS, a row of V to a wave (16 users, d = 64, r = 20: 1.5 us less than the lanes' own stores)
    __syncthreads();
    if (lane < r) {
#pragma unroll 4
        for (int i = wave; i < D; i += kEigWaves) V[(size_t)i * r + lane] = out[i * (r + 1) + lane];
    }
    return true;
}

template <int D, int L, bool MANY>
__global__ __launch_bounds__(kEigThreads, (EigCfg<D, L, MANY>::groups * kEigWaves / 4)) void eig_topr_kernel(
    const float* __restrict__ G, const float* __restrict__ partials, int nsplit,
    const int32_t* __restrict__ lengths, int N, int r,
    float* __restrict__ S, float* __restrict__ V, int32_t* __restrict__ info, EigParams prm) {
    using C = EigCfg<D, L, MANY>;
    using I = Iterate<D, C::LP>;
    constexpr int LP = C::LP, LD = C::LD, TC = C::TC, NC = I::NC;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    float* Zc = smem;                                    // columns of the block, where a step needs them
    float* Qc = Zc + LP * LD;
    uint16_t* img = reinterpret_cast<uint16_t*>(smem);   // images of the block, for the products: the same memory
    float* theta = smem + C::x_floats;                   // [LP]
    float* resid = theta + LP;                           // [LP] residuals, also column norms
    int* rankv = reinterpret_cast<int*>(resid + LP);     // [LP]
    int* order = rankv + LP;                             // [LP] column of rank k
    float* scratch = reinterpret_cast<float*>(order + LP);   // of the basis, the column sums and the dense solver, in turn
    float* Gs = smem;                                    // [D][GS] at the start, when C::GLDS
    __shared__ int sh_bits;
    __shared__ int sh_ge;
    __shared__ int sh_top[kEigWaves];                    // largest entry of G that a wave met, as bits
    __shared__ float sh_rate[2];
    __shared__ double sh_scal[1];
    __shared__ int sh_twist[64];
    const int tid = threadIdx.x, lane = tid & 63, i16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // known from d = 128 on: loads and products do not stand behind a branch (d = 256, r = 32, 16 users 119 -> 114 us)
    const bool holds = I::W == kEigWaves || wave < I::W;
    const int b = blockIdx.x;
    const float* Gb = G + (size_t)b * D * D;

    {
        const int raw = lengths ? lengths[b] : N;
        if (raw < r || raw > N) {  // uniform over the workgroup
            for (int e = tid; e < D * r; e += kEigThreads) V[(size_t)b * D * r + e] = 0.f;
            for (int e = tid; e < r; e += kEigThreads) S[(size_t)b * r + e] = 0.f;
            if (tid == 0 && info) info[b] = -1;
            return;
        }
    }
    if (tid == 0) sh_bits = 0;
    // G to LDS where it fits; true if this thread met an entry that is not finite.  One that is not finite shows on
    // the diagonal too (|G_ij|^2 <= G_ii G_jj), which is what is looked at where G stays in memory.
    // `meanwhile` runs while the loads are on their way.
    auto stage = [&](auto&& meanwhile) __attribute__((always_inline)) {
        v4f probe = v4f{0.f, 0.f, 0.f, 0.f};             // NaN where an entry was not finite
        float top = 0.f;
        if constexpr (C::GLDS) {
            // G from the split-N partial blocks of the Gram kernel: per chunk and fragment pair
            // (s1 <= s2 of CPL = D/16 column fragments) a 16 x 16 block in MFMA layout, lane
            // i2 + 16*(i1/4), component i1%4, holding G[CPL*i1 + s1][CPL*i2 + s2]; pairs with
            // s1 < s2 also supply the mirror image.  Chunks are summed in a fixed order.
            // In LDS column CPL*i + s of X is row and column 16*s + i (eig_row): a block stays a block there, and
            // neither it nor its mirror image meets a bank conflict.  In the order of X the mirror images had 32 lanes on a
            // bank, a third of the whole staging.
            constexpr int CPL = D / 16, NP = CPL * (CPL + 1) / 2;
            const float* pb = partials + (size_t)b * nsplit * (NP * 256);
            // all loads of four chunks are issued before the first is used: the blocks were
            // written by other compute units and come from beyond this XCD's L2
            constexpr int ITEMS = (NP * 64 + kEigThreads - 1) / kEigThreads;
            v4f acc[ITEMS];
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) acc[i] = v4f{0.f, 0.f, 0.f, 0.f};
            for (int sp0 = 0; sp0 < nsplit; sp0 += 4) {
                v4f part[4][ITEMS];
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int i = 0; i < ITEMS; ++i) {
                        const int e = tid + i * kEigThreads;
                        const bool on = e < NP * 64 && sp0 + q < nsplit;
                        part[q][i] = on ? *reinterpret_cast<const v4f*>(pb + (size_t)(sp0 + q) * (NP * 256) + e * 4)
                                        : v4f{0.f, 0.f, 0.f, 0.f};
                    }
                if (sp0 == 0) meanwhile();
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int i = 0; i < ITEMS; ++i) acc[i] += part[q][i];
            }
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {
                const int pair = wave + i * kEigWaves;   // uniform over the wave
                if (pair < NP) {
                    int s1 = 0, rest = pair;
                    while (rest >= CPL - s1) { rest -= CPL - s1; ++s1; }
                    const int s2 = s1 + rest;
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        probe[t] = fmaf(acc[i][t], 0.f, probe[t]);
                        top = fmaxf(top, acc[i][t]);
                    }
                    const int a = 16 * s1 + 4 * g, c = 16 * s2 + i16;
#pragma unroll
                    for (int t = 0; t < 4; ++t) Gs[(a + t) * C::GS + c] = acc[i][t];
                    if (s1 < s2) *reinterpret_cast<v4f*>(Gs + c * C::GS + a) = acc[i];
                }
            }
        } else {
            const float v = tid < D ? Gb[(size_t)tid * (D + 1)] : 0.f;
            static_assert(D <= kEigThreads, "a thread to an entry of the diagonal");
            meanwhile();
            probe[0] = v * 0.f;
            top = fmaxf(v, 0.f);
        }
        top = wave_top(top);
        if (lane == 63) sh_top[wave] = __float_as_int(top);
        return (probe[0] + probe[1]) + (probe[2] + probe[3]) != 0.f;
    };
    // A G with entries that are not finite has no factors.  Neither solver would say so: norms and maxima drop NaN,
    // so one takes G for zero and the other for converged.
    auto not_finite = [&]() __attribute__((always_inline)) {
        const float nan = __int_as_float(0x7fc00000);
        for (int e = tid; e < D * r; e += kEigThreads) V[(size_t)b * D * r + e] = nan;
        for (int e = tid; e < r; e += kEigThreads) S[(size_t)b * r + e] = nan;
        if (tid == 0 && info) info[b] = prm.max_iter;
    };
    // start block Omega (columns >= L stay zero)
    typename I::Regs q, z;
    auto draw = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < I::NB; ++n)
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int t = 0; t < 4; t += 2) {
                    const float2 o = omega_pair(b, 16 * c + i16, 16 * (wave + kEigWaves * n) + 4 * g + t);
                    const bool on = 16 * c + 15 < L || 16 * c + i16 < L;
                    q[n][c][t] = on ? o.x : 0.f;
                    q[n][c][t + 1] = on ? o.y : 0.f;
                }
    };
    const bool bad = stage([&]() __attribute__((always_inline)) { if constexpr (!C::direct) draw(); });
    if (__syncthreads_or(bad)) { not_finite(); return; }   // uniform
    // wide blocks; a test that caps the power steps wants to see the iteration
    bool by_ritz = true;
    if constexpr (C::direct) {
        if (prm.direct) {
            constexpr int RMAX = L == D ? D : L - 8;     // a block as wide as G serves every rank up to d
            if (eig_direct<D, RMAX, C::RB, C::GS>(Gs, reinterpret_cast<double*>(smem), sh_scal, sh_twist, r,
                                            S + (size_t)b * r, V + (size_t)b * D * r)) {
                if (tid == 0 && info) info[b] = 0;
                return;
            }
            __syncthreads();
            stage([]() {});
            __syncthreads();
        }
        by_ritz = false;
        draw();
    }
    GramRows<D> Gr;
    {
        int top = 0;
#pragma unroll
        for (int w = 0; w < kEigWaves; ++w) top = max(top, sh_top[w]);
        const int ge = gram_exponent(top);
        if (tid == 0) sh_ge = ge;                        // read where it is needed: a register less
        if constexpr (GramRows<D>::kKept) {
            if (holds) Gr.keep(Gs, C::GS, gram_scale(ge), wave, i16, g);
        } else {
            Gr.rows = Gb + (size_t)(16 * wave + i16) * D + 8 * g;
        }
    }
    __syncthreads();                                     // G is in registers

    const int col = tid / TC, cu = tid % TC;
    // The iteration alternates cheap and full steps.  After a power step Z = G Q the block is
    // re-orthonormalized either by panels (`mgs_steps` times in a row: only the
    // span matters then) or by the Ritz step or Jacobi phase, which also rotates the basis to Ritz vectors;
    // the step after such a phase checks the residuals of those Ritz pairs.
    bool orth_ok = false;
    float prev_res = 3.0e38f;
    int it = 0;
    int status = 0;
    bool have_ritz = false;
    int cheap_left = prm.mgs_steps;
    int cycle = 0;
    // the cheap steps that the convergence rate adds are filtered: step j of k applies G - t_j I
    // with t_j the roots of the Chebyshev polynomial of degree k on [0, cheb_b]
    float cheb_b = 0.f;
    int cheb_k = 0, cheb_j = 0;
    for (;; ++it) {
        if (holds) {
            Gr.prefetch();
            store_images<D, LP>(img, q, wave);
        }
        __syncthreads();
        float shift = 0.f;
        if (cheb_j < cheb_k) {
            shift = 0.5f * cheb_b * (1.f + __cosf((2 * cheb_j + 1) * 1.57079632679f / cheb_k));
            ++cheb_j;
        }
        if (holds) multiply<D, LP>(Gr, img, q, shift, GramRows<D>::kKept ? 0 : __builtin_amdgcn_readfirstlane(sh_ge), z);
        if (have_ritz) {
            // Rayleigh quotients and residuals of the pairs
            double qz[NC];                               // what S comes from: no rounding beside that of z
            float v[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                qz[c] = 0.0;
#pragma unroll
                for (int n = 0; n < I::NB; ++n)
#pragma unroll
                    for (int t = 0; t < 4; ++t) qz[c] = fma((double)q[n][c][t], (double)z[n][c][t], qz[c]);
            }
            column_sums<D, LP>(qz, reinterpret_cast<double*>(scratch), theta, wave);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const float th = theta[16 * c + i16];
                v[c] = 0.f;
#pragma unroll
                for (int n = 0; n < I::NB; ++n)
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const float e = z[n][c][t] - th * q[n][c][t];
                        v[c] = fmaf(e, e, v[c]);
                    }
            }
            column_sums<D, LP>(v, scratch, resid, wave);
            float thmax;
            for (int e = tid; e == tid || e < 8 * L; e += kEigThreads) {   // every thread wants thmax
                const int rk = rank_of<L>(theta, e, thmax);
                if (e < 8 * L && (e & 7) == 0) {
                    rankv[e >> 3] = rk;
                    if (rk < r) atomicMax(&sh_bits, __float_as_int(sqrtf(resid[e >> 3])));
                }
            }
            __syncthreads();
            const float maxres = __int_as_float(sh_bits);
            bool done = orth_ok && (maxres <= prm.tol_res * thmax);
            // stagnation at the rounding floor counts as converged
            if (orth_ok && it >= 3 && maxres > 0.5f * prev_res && maxres <= 1.0e-4f * thmax) done = true;
            prev_res = maxres;
            if (done) break;
            if (it >= prm.max_iter) { status = it; break; }
        }
        if (cheap_left > 0) {
            --cheap_left;
            have_ritz = false;
            basis_panels<D, L, LP, 0>(z, q, BasisLds<D, LP>(scratch), resid, 0.0, wave);
            if (tid == 0) sh_bits = 0;
            if (cycle == 0 && cheap_left == 0 && it > 0) {   // the last of the initial cheap steps
                // Convergence rate seen by this pass: the smallest diagonal entry of the triangular
                // factor over the r-th largest estimates lambda_(L+1) / lambda_r.  A slowly decaying
                // spectrum (ratio above 0.3) would fail the check after the usual two steps and pay
                // a whole Ritz step or Jacobi phase for it, so cheap steps are added up front instead (each costs
                // a sixth to a tenth of that phase), and these k steps apply G - t_j I with the t_j
                // at the roots of the Chebyshev polynomial of degree k on [0, lambda_L]: together
                // they are the polynomial of degree k that is smallest on the unwanted part of the
                // spectrum relative to its value at lambda_r (at a ratio of 0.6, 1/44 after three
                // steps where three plain power steps give 1/4.6); the basis taken between two
                // steps only changes the basis of the block, not its span.  Four filtered steps
                // leave the residuals of the first check ten times below the tolerance where five
                // plain ones left some users just above it, who then paid a second such phase.
                // (Ending the cheap steps after one when the
                // ratio is ~ 0, as for inputs of rank r, was tried: one user in eight then failed
                // the check by a small margin and took seven steps.)
                float top;
                for (int e = tid; e < 8 * L; e += kEigThreads) {
                    const int rk = rank_of<L>(resid, e, top);
                    if (rk == r - 1) sh_rate[0] = resid[e >> 3];
                    if (rk == L - 1) sh_rate[1] = resid[e >> 3];
                }
                __syncthreads();
                const float vr = sh_rate[0], vmin = sh_rate[1];
                const float rho = vr > 0.f ? sqrtf(fmaxf(vmin, 0.f) / vr) : 0.f;
                if (rho > 0.3f && rho < 1.f) {
                    const int want = (int)ceilf(-11.5f / __logf(rho)) - 3;   // ln(1e-5) = -11.5
                    cheap_left = want < 0 ? 0 : (want > kExtraStepsCap ? kExtraStepsCap : want);
                    cycle = -1;   // the rate is not looked at again
                    // the interval that the filter damps ends at the estimate of lambda_L and in any
                    // case well below that of lambda_r (a root next to a wanted eigenvalue would
                    // remove that direction from the block)
                    cheb_b = fminf(sqrtf(fmaxf(vmin, 0.f)), 0.85f * sqrtf(vr));
                    cheb_k = cheap_left;
                }
            }
            continue;
        }
        // a failed check means slow convergence: spend more cheap steps before the next one
        cycle = cycle < 0 ? 1 : cycle + 1;
        cheap_left = prm.mgs_steps << (cycle < 3 ? cycle : 3);
        have_ritz = true;
        __syncthreads();                                 // the images are done with
        if (holds) store_columns<D, LP>(Zc, z, wave);
        if (tid == 0) sh_bits = 0;
        __syncthreads();
        // orthogonalize the columns of Z (this also rotates them to Ritz vectors)
        bool rotated = false;
        if constexpr (C::ritz) {
            if (by_ritz) {
                const TriLds<L, L> w(reinterpret_cast<double*>(scratch), reinterpret_cast<double*>(Qc));
                rotated = ritz_rotate<D, L>(Zc, Qc, w, sh_scal, sh_twist, resid, r);
                by_ritz = rotated;                       // close eigenvalues: sweeps, from here on
                orth_ok = true;
            }
        }
        if (!rotated) {
            orth_ok = false;
            auto column_norms = [&]() __attribute__((always_inline)) {
                if (col < L) {
                    const float* zc = Zc + col * LD;
                    float nn = 0.f;
                    for (int i = cu; i < D; i += TC) nn += zc[i] * zc[i];
                    nn = team_sum<TC>(nn);
                    if (cu == 0) resid[col] = nn;
                }
                __syncthreads();
                float top = 0.f;
#pragma unroll
                for (int k = 0; k < L; ++k) top = fmaxf(top, resid[k]);
                return top;                              // the largest, squared
            };
            const float dead2 = kDeadRel * kDeadRel * column_norms();
            for (int sw = 0; sw < prm.sweeps; ++sw) {
                const float mine = jacobi_sweep<D, L>(Zc, dead2);
                const bool any = __syncthreads_or(mine > (C::ritz || C::direct ? prm.tol_orth_tied : prm.tol_orth));
                if (!any) { orth_ok = true; break; }
            }
            // normalize; drop columns that are numerically zero
            const float top = column_norms();
            if (col < LP) {
                const float nn = col < L ? resid[col] : 0.f;
                const float inv = nn > kDeadRel * kDeadRel * top && nn > 0.f ? 1.f / sqrtf(nn) : 0.f;
                const float* zc = Zc + col * LD;
                float* qc = Qc + col * LD;
                for (int i = cu; i < D; i += TC) qc[i] = zc[i] * inv;
            }
            __syncthreads();
        }
        if (holds) load_columns<D, LP>(Qc, q, wave);
        __syncthreads();                                 // the images take the place of the columns
    }

    // outputs: columns ranked by Ritz value, sign fixed by the largest-magnitude entry (the first in the order of X)
    __syncthreads();
    uint64_t* keys = reinterpret_cast<uint64_t*>(scratch);
    if (holds) {
        store_columns<D, LP>(Zc, q, wave);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            uint64_t best = 0;
#pragma unroll
            for (int n = 0; n < I::NB; ++n)
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    best = max(best, entry_key<D>(q[n][c][t], eig_row<D>(16 * (wave + kEigWaves * n) + 4 * g + t)));
            keys[(4 * wave + g) * LP + 16 * c + i16] = best;
        }
    }
    __syncthreads();
    for (int e = tid; e < 8 * LP; e += kEigThreads) {    // eight lanes to a column
        const int c = e >> 3, u = e & 7;
        uint64_t best = 0;
#pragma unroll
        for (int w = 0; w < 4 * I::W; w += 8) best = max(best, keys[(w + u) * LP + c]);
#pragma unroll
        for (int m = 1; m < 8; m <<= 1) best = max(best, (uint64_t)__shfl_xor((unsigned long long)best, m));
        if (u == 0 && c < L && rankv[c] < r) {
            resid[c] = (best & 1) ? -1.f : 1.f;
            order[rankv[c]] = c;
            S[(size_t)b * r + rankv[c]] = __builtin_amdgcn_ldexpf(sqrtf(fmaxf(theta[c], 0.f)), sh_ge / 2);
        }
    }
    __syncthreads();
    // a row of V to a wave
    if (lane < r) {
        const int c = order[lane];
        const float sgn = resid[c];
#pragma unroll 4
        for (int p = wave; p < D; p += kEigWaves) V[((size_t)b * D + eig_row<D>(p)) * r + lane] = sgn * Zc[c * LD + p];
    }
    if (tid == 0 && info) info[b] = status;
}

template <int D, int L, bool MANY = false>
hipError_t launch_eig_t(const float* G, const float* partials, int nsplit, const int32_t* lengths, int B, int N,
                        int r, float* S, float* V, int32_t* info, const EigParams& prm, hipStream_t stream) {
    using C = EigCfg<D, L, MANY>;
    if constexpr (D == 64 && C::ritz) {
        if (B > 256) return launch_eig_t<D, L, true>(G, partials, nsplit, lengths, B, N, r, S, V, info, prm, stream);
    }
    if ((partials != nullptr) != C::GLDS) return hipErrorInvalidValue;
    const size_t lds = sizeof(float) * C::lds_floats;
    auto kern = eig_topr_kernel<D, L, MANY>;
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(B), dim3(kEigThreads), lds, stream, G, partials, nsplit, lengths, N, r, S, V,
                       info, prm);
    return hipGetLastError();
}

template <int D>
hipError_t launch_eig_d(const float* G, const float* partials, int nsplit, const int32_t* lengths, int B, int N,
                        int r, float* S, float* V, int32_t* info, const EigParams& prm, hipStream_t stream) {
    const int L = eig_block_columns(D, r);
#define SOLAR_EIG_CASE(LL)                                                                    \
    case LL:                                                                                  \
        if constexpr (LL <= D && (D < 256 || LL <= 40))                                       \
            return launch_eig_t<D, LL>(G, partials, nsplit, lengths, B, N, r, S, V, info, prm, stream); \
        else                                                                                  \
            return hipErrorInvalidValue;
    switch (L) {
        SOLAR_EIG_CASE(16)
        SOLAR_EIG_CASE(24)
        SOLAR_EIG_CASE(32)
        SOLAR_EIG_CASE(40)
        SOLAR_EIG_CASE(48)
        SOLAR_EIG_CASE(56)
        SOLAR_EIG_CASE(64)
        SOLAR_EIG_CASE(72)
        default: return hipErrorInvalidValue;
    }
#undef SOLAR_EIG_CASE
}

}  // namespace

EigParams eig_default_params() {
    EigParams p;
    p.tol_res = 5.0e-6f;
    p.tol_orth = kSweepDone;
    p.tol_orth_tied = kSweepDoneTied;
    p.max_iter = 40;
    p.sweeps = 12;
    p.mgs_steps = 2;
    p.direct = true;
    return p;
}

// Columns of the iterate block: r plus an oversampling of 8, rounded up to a multiple of 8.
int eig_block_columns(int d, int r) {
    int L = 8 * ((r + 8 + 7) / 8);
    if (L < 16) L = 16;
    if (L > d) L = d;
    return L;
}

hipError_t launch_eig(const float* G, const float* partials, int nsplit, const int32_t* lengths, int B, int N,
                      int d, int r, float* S, float* V, int32_t* info, const EigParams& prm, hipStream_t stream) {
    switch (d) {
        case 64: return launch_eig_d<64>(G, partials, nsplit, lengths, B, N, r, S, V, info, prm, stream);
        case 128: return launch_eig_d<128>(G, partials, nsplit, lengths, B, N, r, S, V, info, prm, stream);
        case 256: return launch_eig_d<256>(G, partials, nsplit, lengths, B, N, r, S, V, info, prm, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace solar
