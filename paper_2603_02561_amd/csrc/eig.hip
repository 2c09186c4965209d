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
// basis comes from one modified Gram-Schmidt pass.  After those, basis and small
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
// failed check doubles the number of Gram-Schmidt steps before the next Jacobi phase.
//
// The phase is bound by latency, not by throughput: Gram-Schmidt passes, the reduction of the dense solver and
// Jacobi sweeps are chains of dependent steps with a workgroup barrier after each (d = 128, 40 columns, thousands of cycles:
// staging and start 18, four products 33, two Gram-Schmidt passes 53, Ritz step 119, checks and output 28).  The
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

// Standard normal draw for start-block entry (b, j, i): counter-based, Box-Muller.
__device__ __forceinline__ float omega_entry(int b, int j, int i) {
    uint32_t c = mix32((uint32_t)b * 0x9e3779b9u + (uint32_t)j * 0x85ebca6bu + (uint32_t)i + 0x1234567u);
    uint32_t c2 = mix32(c ^ 0x68bc21ebu);
    float u1 = ((c >> 8) + 1u) * (1.0f / 16777217.0f);
    float u2 = (c2 >> 8) * (1.0f / 16777216.0f);
    return sqrtf(-2.0f * __logf(u1)) * __cosf(6.28318530718f * u2);
}

// Z = G Q with the float 16x16x4 MFMA, block rows of 16 dealt round-robin to the waves.  G is symmetric, and
// the order of the contraction is free, so lane (i, g) takes entries 16 j + 4 g .. + 3 of row i of G and of
// column i of Q with one 16-byte read each and feeds them to four products in turn.  The strides D + 4 of
// Gs and of the columns of Q and Z spread the 16 rows over all banks.  Gb has row stride GS: the copy of G
// in LDS or, when G does not fit there, G itself: then the whole rows are loaded ahead of the products.
// With a shift t the result is (G - t I) Q: the accumulators start from -t Q.
template <int D, int LP, int GS, bool SHIFTED = false>
__device__ __forceinline__ void gemm_gq(const float* Gb, const float* Qc, float* Zc, float shift = 0.f) {
    constexpr int LD = D + 4;
    constexpr int NRB = D / 16, NCB = LP / 16, NK = D / 16;
    constexpr bool AHEAD = D > 128;                     // G comes from memory
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i16 = lane & 15, g = lane >> 4;
    const float* qb = Qc + i16 * LD + 4 * g;
    constexpr int NB = (NRB + kEigWaves - 1) / kEigWaves;
    v4f ahead[AHEAD ? NB : 1][AHEAD ? NK : 1];
    if constexpr (AHEAD) {
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int j = 0; j < NK; ++j)
                ahead[n][j] = *reinterpret_cast<const v4f*>(Gb + (16 * (wave + n * kEigWaves) + i16) * GS + 16 * j + 4 * g);
    }
    // a wave takes whole block rows: the operand read from G serves all NCB column blocks, whose
    // accumulators are independent chains for the matrix unit
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        const int ib = wave + n * kEigWaves;
        if (NRB % kEigWaves != 0 && ib >= NRB) break;
        const float* ga = Gb + (16 * ib + i16) * GS + 4 * g;
        v4f acc[NCB];
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            if constexpr (SHIFTED)
                acc[cb] = -shift * *reinterpret_cast<const v4f*>(&Qc[(16 * cb + i16) * LD + 16 * ib + 4 * g]);
            else
                acc[cb] = v4f{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int j = 0; j < NK; ++j) {
            v4f a, q[NCB];
            if constexpr (AHEAD) a = ahead[n][j];
            else a = *reinterpret_cast<const v4f*>(ga + 16 * j);
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) q[cb] = *reinterpret_cast<const v4f*>(qb + 16 * cb * LD + 16 * j);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb) acc[cb] = mfma16x16x4(a[s], q[cb][s], acc[cb]);
        }
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
            *reinterpret_cast<v4f*>(&Zc[(16 * cb + i16) * LD + 16 * ib + 4 * g]) = acc[cb];
    }
}

// most power steps that a slow convergence rate may add before the first Jacobi phase
constexpr int kExtraStepsCap = 4;

// One pass of modified Gram-Schmidt over the L columns of Zc, normalized into Qc: a cheap
// orthonormal basis of span(Z) for the early power steps, where only the span matters.  The
// columns are taken in panels of kPanel: every team of TM lanes loads the panel and
// orthogonalizes it in registers (all teams do the same arithmetic in the same order, so they
// hold the same bits), team i writes panel column i, normalized, to Qc, and each team then
// projects the panel, column after column, out of the later columns it owns.  The order of
// the projections is that of column-by-column Gram-Schmidt; a panel costs one barrier where
// that costs kPanel.  Columns that collapse below dead2 (squared norm) are dropped (zero in Qc).
// The basis is orthonormal to about 2^-24 * cond(Z), which is all a power step needs.  pivot2[j]
// receives the squared norm column j had when it was normalized (the squared diagonal of the
// triangular factor, which tends to the eigenvalues of G in decreasing order).
constexpr int kPanel = 4;

template <int CH>
__device__ __forceinline__ float dot_ch(const v4f* a, const v4f* b) {
    float g = 0.f;
#pragma unroll
    for (int k = 0; k < CH; ++k) g += a[k].x * b[k].x + a[k].y * b[k].y + a[k].z * b[k].z + a[k].w * b[k].w;
    return g;
}

template <int D, int L>
__device__ __forceinline__ void mgs_orthonormalize(float* Zc, float* Qc, float* pivot2, float dead2) {
    static_assert(L % kPanel == 0, "the block is a whole number of panels");
    constexpr int LD = D + 4;
    constexpr int TM = min_c(16, D / 4);         // lanes per column
    constexpr int CH = D / (4 * TM);
    constexpr int NTEAM = kEigThreads / TM;
    static_assert(NTEAM >= kPanel, "one team per panel column");
    const int tid = threadIdx.x;
    const int team = tid / TM, u = tid % TM;
#pragma unroll 1
    for (int p0 = 0; p0 < L; p0 += kPanel) {
        v4f a[kPanel][CH];
        float inv[kPanel], nrm[kPanel];
#pragma unroll
        for (int i = 0; i < kPanel; ++i) {
            const float* zi = Zc + (p0 + i) * LD + 4 * u;
#pragma unroll
            for (int k = 0; k < CH; ++k) a[i][k] = *reinterpret_cast<const v4f*>(zi + 4 * TM * k);
        }
#pragma unroll
        for (int i = 0; i < kPanel; ++i) {
            float g[kPanel];
#pragma unroll
            for (int k = i; k < kPanel; ++k) g[k] = dot_ch<CH>(a[i], a[k]);
#pragma unroll
            for (int k = i; k < kPanel; ++k) g[k] = team_sum<TM>(g[k]);
            nrm[i] = g[i];
            inv[i] = g[i] > dead2 ? __builtin_amdgcn_rcpf(g[i]) : 0.f;   // 1 ulp: a projection coefficient
#pragma unroll
            for (int k = i + 1; k < kPanel; ++k) {
                const float c = g[k] * inv[i];
#pragma unroll
                for (int q = 0; q < CH; ++q) a[k][q] -= c * a[i][q];
            }
        }
        // team i owns panel column i: normalized into Qc (nobody reads Qc during the pass)
        if (team < kPanel) {
#pragma unroll
            for (int i = 0; i < kPanel; ++i) {
                if (team == i) {
                    const float sc = nrm[i] > dead2 ? __builtin_amdgcn_rsqf(nrm[i]) : 0.f;
                    if (u == 0) pivot2[p0 + i] = nrm[i];   // squared diagonal of the triangular factor
                    float* qi = Qc + (p0 + i) * LD + 4 * u;
#pragma unroll
                    for (int k = 0; k < CH; ++k) *reinterpret_cast<v4f*>(qi + 4 * TM * k) = a[i][k] * sc;
                }
            }
        }
        for (int c = p0 + kPanel + team; c < L; c += NTEAM) {
            float* zc = Zc + c * LD + 4 * u;
            v4f b[CH];
#pragma unroll
            for (int k = 0; k < CH; ++k) b[k] = *reinterpret_cast<const v4f*>(zc + 4 * TM * k);
            // the panel is orthogonal already, so its four projections can all be taken from the
            // column as it stands (they differ from the one-after-another values by the panel's
            // loss of orthogonality times rounding): four independent reductions instead of a
            // chain of four
            float g[kPanel];
#pragma unroll
            for (int i = 0; i < kPanel; ++i) g[i] = dot_ch<CH>(a[i], b);
#pragma unroll
            for (int i = 0; i < kPanel; ++i) g[i] = team_sum<TM>(g[i]) * inv[i];
#pragma unroll
            for (int i = 0; i < kPanel; ++i)
#pragma unroll
                for (int k = 0; k < CH; ++k) b[k] -= g[i] * a[i][k];
#pragma unroll
            for (int k = 0; k < CH; ++k) *reinterpret_cast<v4f*>(zc + 4 * TM * k) = b[k];
        }
        __syncthreads();
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
    const TriLds<D, RB> w(sm, nullptr);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
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
                                                             reinterpret_cast<int*>(w.wb), r);
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
    if (v < r) {
        tri_back<D, TB>(w.U, w.ih, w.dd, u, y);
        const double l = w.lam[v];
        const bool live = any && l > dead;
        // sign fixed by the largest-magnitude entry
        float best = -1.f, val = 0.f;
        int bi = 0;
#pragma unroll
        for (int q = 0; q < D / TB; ++q) {
            const float f = (float)y[q];
            if (fabsf(f) > best) { best = fabsf(f); bi = TB * q + u; val = f; }
        }
#pragma unroll
        for (int m = 1; m < TB; m <<= 1) {
            const float ob = __shfl_xor(best, m), ov = __shfl_xor(val, m);
            const int oi = __shfl_xor(bi, m);
            if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; val = ov; }
        }
        const float sgn = val < 0.f ? -1.f : 1.f;
#pragma unroll
        for (int q = 0; q < D / TB; ++q) V[(size_t)(TB * q + u) * r + v] = live ? sgn * (float)y[q] : 0.f;
        if (u == 0) S[v] = live ? (float)(l * bound * rsq64(l * bound)) : 0.f;
    }
    return true;
}

template <int D, int L, bool MANY>
__global__ __launch_bounds__(kEigThreads, (EigCfg<D, L, MANY>::groups * kEigWaves / 4)) void eig_topr_kernel(
    const float* __restrict__ G, const float* __restrict__ partials, int nsplit,
    const int32_t* __restrict__ lengths, int N, int r,
    float* __restrict__ S, float* __restrict__ V, int32_t* __restrict__ info, EigParams prm) {
    using C = EigCfg<D, L, MANY>;
    constexpr int LP = C::LP, LD = C::LD, TC = C::TC;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    float* Zc = smem;
    float* Qc = Zc + LP * LD;
    float* theta = Qc + LP * LD;   // [LP]
    float* resid = theta + LP;     // [LP] residuals, also column norms
    int* rankv = reinterpret_cast<int*>(resid + LP);              // [LP]
    float* Gs = resid + 2 * LP + 8;                               // [D][GS] when C::GLDS
    __shared__ int sh_bits;
    __shared__ int sh_bits2;
    __shared__ float sh_rate[2];
    __shared__ double sh_scal[1];
    __shared__ int sh_twist[64];
    const int tid = threadIdx.x;
    const int b = blockIdx.x;
    const float* Gb = G + (size_t)b * D * D;
    double* tri = reinterpret_cast<double*>(smem + C::base_floats);

    {
        const int raw = lengths ? lengths[b] : N;
        if (raw < r || raw > N) {  // uniform over the workgroup
            for (int e = tid; e < D * r; e += kEigThreads) V[(size_t)b * D * r + e] = 0.f;
            for (int e = tid; e < r; e += kEigThreads) S[(size_t)b * r + e] = 0.f;
            if (tid == 0 && info) info[b] = -1;
            return;
        }
    }
    if (tid == 0) { sh_bits = 0; sh_bits2 = 0; }
    // G to LDS where it fits; true if this thread met an entry that is not finite.  One that is not finite shows on
    // the diagonal too (|G_ij|^2 <= G_ii G_jj), which is what is looked at where G stays in memory.
    auto stage = [&]() __attribute__((always_inline)) {
    v4f probe = v4f{0.f, 0.f, 0.f, 0.f};                // NaN where an entry was not finite
    auto look = [&](v4f v) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 4; ++t) probe[t] = fmaf(v[t], 0.f, probe[t]);
    };
    if constexpr (C::GLDS) {
        if (partials) {
            // G from the split-N partial blocks of the Gram kernel: per chunk and fragment pair
            // (s1 <= s2 of CPL = D/16 column fragments) a 16 x 16 block in MFMA layout, lane
            // i2 + 16*(i1/4), component i1%4, holding G[CPL*i1 + s1][CPL*i2 + s2]; pairs with
            // s1 < s2 also supply the mirror image.  Chunks are summed in a fixed order.
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
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int i = 0; i < ITEMS; ++i) acc[i] += part[q][i];
            }
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {
                const int e = tid + i * kEigThreads;
                if (e < NP * 64) {
                    const int pair = e >> 6, ln = e & 63;
                    int s1 = 0, rest = pair;
                    while (rest >= CPL - s1) { rest -= CPL - s1; ++s1; }
                    const int s2 = s1 + rest;
                    look(acc[i]);
                    const int c = CPL * (ln & 15) + s2;
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const int a = CPL * (4 * (ln >> 4) + t) + s1;
                        Gs[a * C::GS + c] = acc[i][t];
                        if (s1 < s2) Gs[c * C::GS + a] = acc[i][t];
                    }
                }
            }
        } else {
            for (int e = tid; e < D * D / 4; e += kEigThreads) {
                const int i = e / (D / 4), c4 = e % (D / 4);
                const v4f v = *reinterpret_cast<const v4f*>(Gb + (size_t)i * D + 4 * c4);
                look(v);
                *reinterpret_cast<v4f*>(Gs + i * C::GS + 4 * c4) = v;
            }
        }
    } else {
        for (int e = tid; e < D; e += kEigThreads) probe[0] = fmaf(Gb[(size_t)e * D + e], 0.f, probe[0]);
    }
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
    const bool bad = stage();
    // wide blocks; a test that caps the power steps wants to see the iteration
    bool by_ritz = true;
    if constexpr (C::direct) {
        if (prm.direct) {
            if (__syncthreads_or(bad)) { not_finite(); return; }
            if (eig_direct<D, L - 8, C::RB, C::GS>(Gs, reinterpret_cast<double*>(smem), sh_scal, sh_twist, r,
                                            S + (size_t)b * r, V + (size_t)b * D * r)) {
                if (tid == 0 && info) info[b] = 0;
                return;
            }
            __syncthreads();
            stage();
        }
        by_ritz = false;
    }
    const float* Gop = C::GLDS ? Gs : Gb;
    // start block Omega (columns >= L stay zero so that the padded GEMM columns are zero)
    for (int e = tid; e < LP * D; e += kEigThreads) {
        const int j = e / D, i = e % D;
        Qc[j * LD + i] = (j < L) ? omega_entry(b, j, i) : 0.f;
        Zc[j * LD + i] = 0.f;
    }
    if (__syncthreads_or(bad)) { not_finite(); return; }   // uniform

    const int col = tid / TC, cu = tid % TC;
    // The iteration alternates cheap and full steps.  After a power step Z = G Q the block is
    // re-orthonormalized either by one Gram-Schmidt pass (`mgs_steps` times in a row: only the
    // span matters then) or by the Jacobi phase, which also rotates the basis to Ritz vectors;
    // the step after a Jacobi phase checks the residuals of those Ritz pairs.
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
        if (cheb_j < cheb_k) {
            const float shift = 0.5f * cheb_b * (1.f + __cosf((2 * cheb_j + 1) * 1.57079632679f / cheb_k));
            ++cheb_j;
            gemm_gq<D, LP, C::GS, true>(Gop, Qc, Zc, shift);
        } else {
            gemm_gq<D, LP, C::GS>(Gop, Qc, Zc);
        }
        __syncthreads();
        // column norms of Z (for the dead-column threshold), Rayleigh quotients and residuals
        if (col < L) {
            const float* q = Qc + col * LD;
            const float* z = Zc + col * LD;
            float th = 0.f, nn = 0.f;
            for (int i = cu; i < D; i += TC) { th += q[i] * z[i]; nn += z[i] * z[i]; }
            th = team_sum<TC>(th);
            nn = team_sum<TC>(nn);
            float rs = 0.f;
            for (int i = cu; i < D; i += TC) { const float e = z[i] - th * q[i]; rs += e * e; }
            rs = team_sum<TC>(rs);
            if (cu == 0) {
                theta[col] = th;
                resid[col] = sqrtf(rs);
                atomicMax(&sh_bits2, __float_as_int(nn));
            }
        }
        __syncthreads();
        const float dead2 = kDeadRel * kDeadRel * __int_as_float(sh_bits2);
        if (have_ritz) {
            if (tid < L) {
                const float th = theta[tid];
                int rk = 0;
                for (int k = 0; k < L; ++k) {
                    const float tk = theta[k];
                    rk += (tk > th || (tk == th && k < tid)) ? 1 : 0;
                }
                rankv[tid] = rk;
                if (rk < r) atomicMax(&sh_bits, __float_as_int(resid[tid]));
            }
            __syncthreads();
            const float maxres = __int_as_float(sh_bits);
            float thmax = 0.f;
            for (int k = 0; k < L; ++k) thmax = fmaxf(thmax, theta[k]);
            bool done = orth_ok && (maxres <= prm.tol_res * thmax);
            // stagnation at the rounding floor counts as converged
            if (orth_ok && it >= 3 && maxres > 0.5f * prev_res && maxres <= 1.0e-4f * thmax) done = true;
            prev_res = maxres;
            if (done) break;
            if (it >= prm.max_iter) { status = it; break; }
        }
        __syncthreads();
        if (tid == 0) { sh_bits = 0; sh_bits2 = 0; }
        if (cheap_left > 0) {
            --cheap_left;
            have_ritz = false;
            mgs_orthonormalize<D, L>(Zc, Qc, resid, dead2);
            if (cycle == 0 && cheap_left == 0 && it > 0) {   // the last of the initial cheap steps
                // Convergence rate seen by this pass: the smallest diagonal entry of the triangular
                // factor over the r-th largest estimates lambda_(L+1) / lambda_r.  A slowly decaying
                // spectrum (ratio above 0.3) would fail the check after the usual two steps and pay
                // a whole Jacobi phase for it, so cheap steps are added up front instead (each costs
                // a sixth to a tenth of that phase), and these k steps apply G - t_j I with the t_j
                // at the roots of the Chebyshev polynomial of degree k on [0, lambda_L]: together
                // they are the polynomial of degree k that is smallest on the unwanted part of the
                // spectrum relative to its value at lambda_r (at a ratio of 0.6, 1/44 after three
                // steps where three plain power steps give 1/4.6); the Gram-Schmidt pass between two
                // steps only changes the basis of the block, not its span.  Four filtered steps
                // leave the residuals of the first check ten times below the tolerance where five
                // plain ones left some users just above it, who then paid a second Jacobi phase.
                // (Ending the cheap steps after one when the
                // ratio is ~ 0, as for inputs of rank r, was tried: one user in eight then failed
                // the check by a small margin and took seven steps.)
                if (tid < L) {
                    const float v = resid[tid];
                    int rk = 0;
#pragma unroll 8
                    for (int k = 0; k < L; ++k) {
                        const float vk = resid[k];
                        rk += (vk > v || (vk == v && k < tid)) ? 1 : 0;
                    }
                    if (rk == r - 1) sh_rate[0] = v;
                    if (rk == L - 1) sh_rate[1] = v;
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
        // orthogonalize the columns of Z (this also rotates them to Ritz vectors)
        if constexpr (C::ritz) {
            if (by_ritz) {
                const TriLds<L, L> w(tri, reinterpret_cast<double*>(Qc));
                if (ritz_rotate<D, L>(Zc, Qc, w, sh_scal, sh_twist, resid, r)) {
                    orth_ok = true;
                    continue;
                }
                by_ritz = false;                         // close eigenvalues: sweeps, from here on
            }
        }
        orth_ok = false;
        for (int sw = 0; sw < prm.sweeps; ++sw) {
            const float mine = jacobi_sweep<D, L>(Zc, dead2);
            const bool any = __syncthreads_or(mine > prm.tol_orth);
            if (!any) { orth_ok = true; break; }
        }
        // normalize; drop columns that are numerically zero
        if (col < L) {
            const float* z = Zc + col * LD;
            float nn = 0.f;
            for (int i = cu; i < D; i += TC) nn += z[i] * z[i];
            nn = team_sum<TC>(nn);
            if (cu == 0) resid[col] = sqrtf(nn);
        }
        __syncthreads();
        if (col < L) {
            float nmax = 0.f;
            for (int k = 0; k < L; ++k) nmax = fmaxf(nmax, resid[k]);
            const float nj = resid[col];
            const float inv = (nj > kDeadRel * nmax && nj > 0.f) ? 1.f / nj : 0.f;
            const float* z = Zc + col * LD;
            float* q = Qc + col * LD;
            for (int i = cu; i < D; i += TC) q[i] = z[i] * inv;
        }
        __syncthreads();
    }

    // outputs: columns ranked by Ritz value, sign fixed by the largest-magnitude entry
    if (col < L && rankv[col] < r) {
        const int k = rankv[col];
        const float* q = Qc + col * LD;
        float best = -1.f;
        int bi = 0;
        for (int i = cu; i < D; i += TC) {
            const float a = fabsf(q[i]);
            if (a > best) { best = a; bi = i; }
        }
        for (int m = 1; m < TC; m <<= 1) {
            const float ob = __shfl_xor(best, m);
            const int oi = __shfl_xor(bi, m);
            if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
        }
        const float sgn = (q[bi] < 0.f) ? -1.f : 1.f;
        for (int i = cu; i < D; i += TC) V[((size_t)b * D + i) * r + k] = sgn * q[i];
        if (cu == 0) S[(size_t)b * r + k] = sqrtf(fmaxf(theta[col], 0.f));
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
    if (partials && !C::GLDS) return hipErrorInvalidValue;
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
