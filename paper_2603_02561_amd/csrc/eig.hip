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
// eigenvalues take one-sided (Hestenes) Jacobi sweeps over the columns of Z.  Both are insensitive
// to the huge dynamic range of the block (G Omega is dominated by the leading
// eigenvectors) and to rank deficiency (columns that vanish are dropped).  The power
// step after a Jacobi phase yields the residuals |G q_i - theta_i q_i| of the Ritz
// pairs; the iteration ends when every wanted pair is below tol_res * theta_max, and a
// failed check doubles the number of Gram-Schmidt steps before the next Jacobi phase.
//
// The phase is bound by latency, not by throughput: a Jacobi sweep is L-1 rounds of
// L/2 independent column rotations with a workgroup barrier after each round.  The
// kernel runs eight waves (two per SIMD), gives every column pair a team of up to 16
// lanes whose partial dot products are combined with DPP lane permutations, and keeps
// every trip count a compile-time constant.
#include "common.h"
#include "kernels.h"
#include "tridiag.h"
#include "xty_partials.h"

namespace solar {

namespace {

constexpr int kEigThreads = 512;
constexpr int kEigWaves = kEigThreads / 64;
// A column of the iterate whose norm falls below this fraction of the largest column norm
// is rounding noise of the float Gram matrix (about sqrt(d) * 2^-24 relative) and is dropped.
constexpr float kDeadRel = 1.0e-5f;
// Rotations are skipped below kSkipCos.  The Jacobi phase converges quadratically: a sweep whose
// largest |cos| was c leaves about c^2 behind (L * c^2 at worst), so the phase ends after the
// first sweep that met no |cos| above kSweepDone = 5e-4, with a few 1e-6 left; the residual
// check of the following power step is what accepts the result.  (1e-3 leaves V^T V up to 1.3e-5
// off the identity at 72 columns and 3e-3 up to 4e-5; 3e-2 makes the check fail and the iteration
// longer.  In a batch some user nearly always needs the sweep that a looser limit would save
// the others, so the launch is no shorter with 1e-3.)
constexpr float kSkipCos = 1.0e-7f;
constexpr float kSweepDone = 5.0e-4f;

__host__ __device__ constexpr int pow2floor_c(int x) {
    int p = 1;
    while (2 * p <= x) p *= 2;
    return p;
}
__host__ __device__ constexpr int min_c(int a, int b) { return a < b ? a : b; }

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

template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}

// Sum over a team of T consecutive lanes (T a power of two, team aligned to T); every
// lane of the team receives the same bits.  Up to 16 lanes the exchange is a DPP operand
// (quad permutes, then mirror within 8 and within 16 lanes).
template <int T>
__device__ __forceinline__ float team_sum(float v) {
    if constexpr (T >= 2) v += dpp_mov<0xB1>(v);    // quad_perm [1,0,3,2]
    if constexpr (T >= 4) v += dpp_mov<0x4E>(v);    // quad_perm [2,3,0,1]
    if constexpr (T >= 8) v += dpp_mov<0x141>(v);   // row_half_mirror
    if constexpr (T >= 16) v += dpp_mov<0x140>(v);  // row_mirror
    if constexpr (T >= 32) v += __shfl_xor(v, 16);
    if constexpr (T >= 64) v += __shfl_xor(v, 32);
    return v;
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

// Work arrays of one dense solve at `base` (doubles): reflectors, wa, wb, vectors of length N.
template <int N, int RB>
struct TriLds {
    using T = TriCfg<N, RB>;
    double *U, *wa, *wb, *dd, *ee, *ih, *es, *lam;
    double2* t;
    static constexpr size_t kDoublesNoWa = T::USZ + T::WB + T::VEC;
    static constexpr size_t kDoubles = kDoublesNoWa + T::WA;
    // wa == nullptr: behind the other arrays
    __device__ __forceinline__ TriLds(double* base, double* wa_) {
        U = base;
        wb = U + T::USZ;
        dd = wb + T::WB;
        ee = dd + N;
        ih = ee + N;
        es = ih + N;
        t = reinterpret_cast<double2*>(es + N);
        lam = reinterpret_cast<double*>(t + N + 8);
        wa = wa_ ? wa_ : dd + T::VEC;
    }
};

// MANY: for batches of more users than compute units
template <int D, int L, bool MANY = false>
struct EigCfg {
    static constexpr int LP = 16 * ((L + 15) / 16);
    static constexpr int LD = D + 4;
    // lanes per column outside the Jacobi rounds
    static constexpr int TC = min_c(min_c(64, D), pow2floor_c(kEigThreads / L));
    // G is staged in LDS when it fits beside the two iterate blocks
    static constexpr bool GLDS = D <= 128;
    static constexpr int GS = GLDS ? D + 4 : D;
    static constexpr size_t base_floats = (size_t)2 * LP * LD + 3 * LP + 8 + (GLDS ? (size_t)D * GS : 0);
    // Wide blocks are solved directly: the reduction of the whole matrix is then cheaper than the
    // power steps, Gram-Schmidt passes and Ritz steps of the iteration, and takes the same time for every
    // spectrum (16 users, d = 128, r = 64: 214 us per launch, where iterating took 360 for
    // inputs of rank r, 452 for singular values ~ k^-1/2 and 732 with the last ones in the noise; d = 64, r = 40:
    // 78 us against 122, 227 and 619; at d = 64, L = 24 and d = 128, L = 48 the two are about even on easy spectra).
    static constexpr bool direct = (D == 64 && L >= 32) || (D == 128 && L >= 56);
    // Narrower ones take the Ritz step of the iteration through the same solver instead of Jacobi sweeps
    // (16 users, inputs of rank r: d = 128, r = 32 from 142 to 113 us, r = 16 from 82 to 67; d = 256,
    // r = 32 from 253 to 178, of which 55 are the wider reads of the products G Q), except the narrowest,
    // where it is no faster (d = 64, r = 8: 38 us).  It takes the whole register file for one workgroup: at d = 64 the
    // sweeps, of which three fit a compute unit, are faster for more users than compute units (r = 16, 256 users 52
    // us against 58, 1024 users 196 against 128).
    static constexpr bool ritz = !direct && (D > 64 || L > 16) && !MANY;
    static constexpr size_t ritz_floats = ritz ? 2 * TriLds<ritz ? L : 16, ritz ? L : 16>::kDoublesNoWa : 0;
    static constexpr int RB = D == 128 || L <= 40 ? 32 : 64;   // eigenvectors per pass of the direct solution
    static constexpr size_t direct_floats = direct ? 2 * TriLds<direct ? D : 16, RB>::kDoubles : 0;
    static constexpr size_t lds_floats =
        base_floats + ritz_floats > direct_floats ? base_floats + ritz_floats : direct_floats;
    // Workgroups that registers and LDS let share a compute unit, which is what counts with more users than compute
    // units: the waves of one fill the gaps in the chains of the others.  1024 users at d = 64: r = 8 137 us with one, 84 with
    // six; r = 24, direct, 279 and 197 with two (where iterating takes 168 for inputs of rank r, 215 to 290 for
    // singular values ~ k^-1/2 and k^-1).  r > 32 takes the eigenvectors in one pass and 86 KB for it: alone
    // on its compute unit it is as fast for many users (r = 40: 309) as iterating is at best.
    static constexpr int groups = D == 64 && !ritz && L <= 40 ? 2 : 1;
    static_assert(groups * (sizeof(float) * lds_floats + 1024) <= 160 * 1024, "LDS");
};

// One cyclic sweep of one-sided Jacobi over the L columns of Zc; returns this thread's largest
// |cos| met in the sweep.
//
// A rotation needs two columns and a round of disjoint rotations touches every column, so a
// sweep that keeps the columns in LDS between rounds moves the whole block through LDS and meets
// a workgroup barrier once per round: 39 times per sweep at 40 columns, about 640 of a round's
// 1280 cycles.  Here the columns are dealt to the waves in half-groups of G = 64 / T columns (T
// lanes per column pair) and a wave keeps two half-groups A, B in registers for G rounds:
// team i of the wave holds A[i] and, in round j, B[(i + j) mod G], which the teams pass on with
// lane permutations; after G rounds every column of A has met every column of B.  The half-groups
// meet each other in a round-robin tournament of H - 1 such super-rounds, with LDS and the
// workgroup barrier only between them, and the pairs inside a half-group are taken first, G - 1
// rounds through LDS.  The number of rotations per sweep is that of any cyclic ordering; the
// barriers drop from L - 1 to (H - 1) + (G - 1).
// most power steps that a slow convergence rate may add before the first Jacobi phase
constexpr int kExtraStepsCap = 4;
// the widest team (at most 16 lanes, a float4 per lane at least) whose waves fit the workgroup
__host__ __device__ constexpr int jacobi_team_lanes(int d, int l) {
    for (int t = 16; t > 8; t /= 2) {
        const int g = 64 / t;
        if (4 * t <= d && (l + 2 * g - 1) / (2 * g) <= kEigWaves) return t;
    }
    return 8;
}

template <int D, int L>
struct JacobiCfg {
    static constexpr int T = jacobi_team_lanes(D, L);   // lanes per column pair
    static constexpr int G = 64 / T;                    // column pairs per wave = columns per half-group
    static constexpr int NW = (L + 2 * G - 1) / (2 * G);  // waves that hold columns
    static constexpr int H = 2 * NW;                    // half-groups
    static constexpr int LPAD = H * G;                  // columns including the (zero) padding
    static constexpr int CH = D / (4 * T);              // float4 per lane and column
    static_assert(NW <= kEigWaves, "one wave per pair of half-groups");
    static_assert(LPAD <= EigCfg<D, L>::LP, "the padding columns exist in LDS");
    static_assert(LPAD / 2 * T <= kEigThreads, "one team per pair in the rounds through LDS");
    static_assert(D % (4 * T) == 0 && CH >= 1, "whole float4 per lane");
};

// The rotation that makes the columns a, c of a pair orthogonal, from their squared norms al, be
// and inner product ga; the norms follow in closed form (al' = al - t ga, be' = be + t ga with
// t the tangent).  With d = be - al and g = ga, both divided by |a||c| so that squares cannot
// overflow, the rotation has cos^2 = x = 1/2 + |d| / (2 sqrt(d^2 + 4 g^2)) and
// sin = sign(d) g / (sqrt(d^2 + 4 g^2) cos): two dependent reciprocal square roots, where the
// route over zeta = d / 2g and the tangent takes four dependent transcendental steps.  Columns
// that have collapsed to rounding noise are left alone (dropped later), and so are pairs whose
// cosine is below kSkipCos.  With BRANCHLESS the rotation is always applied and a pair that is
// left alone gets the identity: no lane branches in the chain of dependent instructions, which
// pays while a lane holds up to eight elements per column.
template <int T, int CH, bool BRANCHLESS>
__device__ __forceinline__ void rotate_columns(v4f (&a)[CH], v4f (&c)[CH], float& al, float& be, float ga,
                                               float dead2, float& offmax) {
    const float ra = __builtin_amdgcn_rsqf(al), rb = __builtin_amdgcn_rsqf(be);
    const float gn = ga * ra * rb;   // cosine of the angle between the columns
    const float dn = (be - al) * ra * rb;
    const float cosv = fabsf(gn);
    const bool live = al > dead2 && be > dead2;
    const bool rot = live && cosv > kSkipCos;
    const float ih = __builtin_amdgcn_rsqf(dn * dn + 4.f * gn * gn);
    const float x = 0.5f + 0.5f * fabsf(dn) * ih;
    const float r = __builtin_amdgcn_rsqf(x);
    float cs = x * r;
    float sn = (dn >= 0.f ? gn : -gn) * ih * r;
    float tg = sn * r * ga;
    if constexpr (BRANCHLESS) {
        offmax = live ? fmaxf(offmax, cosv) : offmax;
        cs = rot ? cs : 1.f;
        sn = rot ? sn : 0.f;
        tg = rot ? tg : 0.f;
#pragma unroll
        for (int k = 0; k < CH; ++k) {
            const v4f x4 = a[k], y4 = c[k];
            a[k] = cs * x4 - sn * y4;
            c[k] = sn * x4 + cs * y4;
        }
        al -= tg;
        be += tg;
    } else {
        if (live) offmax = fmaxf(offmax, cosv);
        if (rot) {
#pragma unroll
            for (int k = 0; k < CH; ++k) {
                const v4f x4 = a[k], y4 = c[k];
                a[k] = cs * x4 - sn * y4;
                c[k] = sn * x4 + cs * y4;
            }
            al -= tg;
            be += tg;
        }
    }
}

template <int CH>
__device__ __forceinline__ float dot_ch(const v4f (&a)[CH], const v4f (&c)[CH]) {
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < CH; ++k) s += a[k].x * c[k].x + a[k].y * c[k].y + a[k].z * c[k].z + a[k].w * c[k].w;
    return s;
}

// pair number k of round rho of a round-robin tournament of n players (n even): player n - 1
// stays, the others go round
__device__ __forceinline__ void tournament_pair(int n, int rho, int k, int& p, int& q) {
    p = rho + k;
    q = rho - k;
    if (p >= n - 1) p -= n - 1;
    if (q < 0) q += n - 1;
    if (k == 0) p = n - 1;
}

template <int D, int L>
__device__ __forceinline__ float jacobi_sweep(float* Zc, float dead2) {
    using J = JacobiCfg<D, L>;
    constexpr int T = J::T, G = J::G, CH = J::CH, LD = EigCfg<D, L>::LD;
    constexpr bool NB = T == 16;   // measured: teams of 16 lanes gain from it, teams of 8 lose
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int u = tid % T;
    float offmax = 0.f;
    v4f a[CH], c[CH];
    auto load = [&](v4f (&dst)[CH], int col) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < CH; ++k) dst[k] = *reinterpret_cast<const v4f*>(Zc + col * LD + 4 * u + 4 * T * k);
    };
    auto store = [&](const v4f (&src)[CH], int col) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < CH; ++k) *reinterpret_cast<v4f*>(Zc + col * LD + 4 * u + 4 * T * k) = src[k];
    };
    // the pairs inside every half-group: G - 1 rounds through LDS, one team per pair
    if constexpr (G > 1) {
        const int team = tid / T;
        const int hg = team / (G / 2), k = team % (G / 2);
#pragma unroll 1
        for (int rho = 0; rho < G - 1; ++rho) {
            if (team < J::LPAD / 2) {
                int p, q;
                tournament_pair(G, rho, k, p, q);
                load(a, hg * G + p);
                load(c, hg * G + q);
                float al = team_sum<T>(dot_ch<CH>(a, a)), be = team_sum<T>(dot_ch<CH>(c, c));
                rotate_columns<T, CH, NB>(a, c, al, be, team_sum<T>(dot_ch<CH>(a, c)), dead2, offmax);
                store(a, hg * G + p);
                store(c, hg * G + q);
            }
            __syncthreads();
        }
    }
    // the pairs between half-groups: wave w holds the half-groups of pair w of the super-round
    const int i = lane / T;
#pragma unroll 1
    for (int s = 0; s < J::H - 1; ++s) {
        if (wave < J::NW) {
            int ha, hb;
            tournament_pair(J::H, s, wave, ha, hb);
            load(a, ha * G + i);
            load(c, hb * G + i);
            // squared norms once per super-round; they follow the rotations in closed form, and
            // that of a B column travels with the column
            float al = team_sum<T>(dot_ch<CH>(a, a)), be = team_sum<T>(dot_ch<CH>(c, c));
#pragma unroll
            for (int j = 0; j < G; ++j) {
                rotate_columns<T, CH, NB>(a, c, al, be, team_sum<T>(dot_ch<CH>(a, c)), dead2, offmax);
                if (j + 1 < G) {
                    // team i takes over the B column of team i + 1
                    be = __shfl(be, (lane + T) & 63);
#pragma unroll
                    for (int k = 0; k < CH; ++k) {
                        c[k].x = __shfl(c[k].x, (lane + T) & 63);
                        c[k].y = __shfl(c[k].y, (lane + T) & 63);
                        c[k].z = __shfl(c[k].z, (lane + T) & 63);
                        c[k].w = __shfl(c[k].w, (lane + T) & 63);
                    }
                }
            }
            store(a, ha * G + i);
            store(c, hb * G + (i + G - 1) % G);
        }
        __syncthreads();
    }
    return offmax;
}

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

// Two wanted eigenvalues closer than this (relative to the norm) leave their vectors, which are computed
// independently of each other, orthogonal only to about 1e-15 / kTriGap: the caller takes another route.
constexpr double kTriGap = 1.0e-9;
// A matrix of zeros comes out of the reduction with a norm of about 1e-89; one of floats, or of their
// squares, is above this.
constexpr double kTriZero = 1.0e-80;

// Gm[i][j] = z_i . z_j in double precision for the L columns of Zc (D values each, column stride LD)
template <int D, int L, int LD, int LG>
__device__ __forceinline__ void gram_columns64(const float* Zc, double* Gm) {
    constexpr int NT = (L + 15) / 16;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    for (int p = wave; p < NT * (NT + 1) / 2; p += kEigWaves) {
        int I = 0, rest = p;
        while (rest >= NT - I) { rest -= NT - I; ++I; }
        const int J = I + rest;
        const float* za = Zc + (16 * I + i16) * LD + g;
        const float* zb = Zc + (16 * J + i16) * LD + g;
        v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
        for (int k0 = 0; k0 < D; k0 += 4) acc = mfma16x16x4f64((double)za[k0], (double)zb[k0], acc);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int i = 16 * I + g + 4 * t, j = 16 * J + i16;
            if (i < L && j < L) {
                Gm[i * LG + j] = acc[t];
                Gm[j * LG + i] = acc[t];
            }
        }
    }
    __syncthreads();
}

// The Rayleigh-Ritz step on the N columns of Zc (LDS, column stride D + 4): with C = Z^T Z = W diag(l) W^T,
// formed and solved in double precision, the columns of Z W diag(l)^-1/2 are orthonormal and
// diagonalize the projected problem, which is what one-sided Jacobi sweeps over Z converge to.  They go
// to Qc (zero where sqrt(l) is below kDeadRel of the largest), in descending order of l; sig[k] receives
// sqrt(l_k).  Qc may share its memory with wa.  False (and Qc untouched unless it is wa): two of the
// `wanted` leading eigenvalues are too close for this route.
template <int D, int N>
__device__ __forceinline__ bool ritz_rotate(const float* Zc, float* Qc, const TriLds<N, N>& w, double* scal, int* twist,
                                            float* sig, int wanted) {
    using T = TriCfg<N, N>;
    constexpr int LD = D + 4, NT = (N + 15) / 16;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    double* Cm = w.wa;
    gram_columns64<D, N, LD, N>(Zc, Cm);
    TriRows<N> a;
    if (wave < kTriWaves) {
#pragma unroll
        for (int m = 0; m < T::RS; ++m)
#pragma unroll
            for (int c = 0; c < T::NC; ++c) {
                const int i = 16 * (m / 4) + 4 * wave + m % 4, j = (lane ^ (4 * wave)) + 64 * c;
                a[m][c] = i < N && j < N ? Cm[i * N + j] : 0.0;
            }
    }
    tri_reduce<N>(a, w.wb, w.U, w.dd, w.ee, w.ih);
    const double bound = tri_values<N, (N <= 32 ? 8 : 4)>(w.dd, w.ee, w.es, w.t, w.lam, scal,
                                                          reinterpret_cast<int*>(w.wb), N);
    const double l0 = w.lam[0], dead = (double)kDeadRel * kDeadRel * l0;
    const bool close = tid + 1 < wanted && w.lam[tid + 1] > dead && w.lam[tid] - w.lam[tid + 1] < kTriGap;
    if (__syncthreads_or(close) || !(bound > kTriZero) || !(l0 > 0.0)) return false;
    tri_vectors<N, N>(w.t, w.es, w.lam, w.wa, w.wb, twist, 0, N);
    constexpr int TB = 8;
    const int v = tid / TB, u = tid % TB;
    double y[N / TB];
    if (v < N) tri_load<N, N, TB>(w.wa, v, u, y);
    tri_cross<N>(w.U, w.dd);
    if (v < N) {
        tri_back<N, TB>(w.U, w.ih, w.dd, u, y);
        const double l = w.lam[v], rs = l > dead ? rsq64(l * bound) : 0.0;
        if (u == 0) sig[v] = (float)(l > 0.0 ? l * bound * rsq64(l * bound) : 0.0);
#pragma unroll
        for (int q = 0; q < N / TB; ++q) w.wb[v * N + TB * q + u] = l > dead ? y[q] * rs : 0.0;
    }
    __syncthreads();
    for (int J = wave; J < D / 16; J += kEigWaves) {
#pragma unroll
        for (int I = 0; I < NT; ++I) {
            const bool in = 16 * I + i16 < N;
            const double* wr = w.wb + (in ? 16 * I + i16 : 0) * N + g;
            const float* zr = Zc + g * LD + 16 * J + i16;
            v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int k0 = 0; k0 < N; k0 += 4) acc = mfma16x16x4f64(in ? wr[k0] : 0.0, (double)zr[k0 * LD], acc);
#pragma unroll
            for (int t = 0; t < 4; ++t) Qc[(16 * I + g + 4 * t) * LD + 16 * J + i16] = (float)acc[t];
        }
    }
    __syncthreads();
    return true;
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

// ---- small problems of Algorithm 1 -----------------------------------------------------------------------
// Cholesky factorization of the L x L matrix in A (LDS, row stride LR doubles, both triangles), in double precision
// by the whole workgroup: a thread keeps its entries in registers, so a step is the store of the pivot row, one
// barrier and a multiply-add.  The row of pivot k stays in A as it was when its turn came, A[k][j] = R[k][k] R[k][j];
// inv[k] receives 1 / R[k][k]^2 and rs[k] 1 / R[k][k].  A pivot k that is not above limit * d0[k]
// ends it (false, in every thread); with DROP, one that is not above `limit` drops its column (inv = rs = 0).
template <int L, int LR, bool DROP>
__device__ __forceinline__ bool cholesky64(double* A, double* inv, double* rs, const double* d0, double limit) {
    const int tid = threadIdx.x;
    constexpr int RP = kEigThreads / L, Q = (L + RP - 1) / RP;   // rows per pass of the threads, entries per thread
    const int j = tid % L, i0 = tid / L;
    double a[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) a[q] = i0 + q * RP < L ? A[(i0 + q * RP) * LR + j] : 0.0;
    __syncthreads();
    for (int k = 0; k < L; ++k) {
        double* row = A + k * LR;
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (i0 + q * RP == k) row[j] = a[q];
        __syncthreads();
        const double piv = row[k];
        if constexpr (!DROP) {
            if (!(piv > limit * d0[k]) || !(piv > 0.0)) return false;   // uniform
        }
        const bool live = !DROP || piv > limit;
        const double r1 = live ? rsq64(piv) : 0.0, f = live ? rcp64(piv) : 0.0;
        if (tid == 0) { inv[k] = f; rs[k] = r1; }
        const double m = row[j] * f;
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (i0 + q * RP < L) a[q] = fma(-m, row[i0 + q * RP], a[q]);
    }
    __syncthreads();
    return true;
}

// Z <- Z R^-1 for the factor that cholesky64 left in A, columns of Z at Zc + c * LD; one thread per row.
template <int D, int L, int LD, int LR>
__device__ __forceinline__ void solve_rows64(float* Zc, const double* A, const double* inv, const double* rs) {
    static_assert(LR % 2 == 0 && L % 2 == 0, "pairs of a row are read together");
    const int a = threadIdx.x;
    if (a < D) {
        double x[L];
#pragma unroll
        for (int c = 0; c < L; ++c) x[c] = (double)Zc[c * LD + a];
#pragma unroll
        for (int k = 0; k < L; ++k) {
            const double f = x[k] * inv[k];
            const double2* row = reinterpret_cast<const double2*>(A + k * LR);
#pragma unroll
            for (int c2 = (k + 1) / 2; c2 < L / 2; ++c2) {
                const double2 v = row[c2];
                if (2 * c2 > k) x[2 * c2] = fma(-f, v.x, x[2 * c2]);
                x[2 * c2 + 1] = fma(-f, v.y, x[2 * c2 + 1]);
            }
            Zc[k * LD + a] = (float)(x[k] * rs[k]);
        }
    }
    __syncthreads();
}

// LDS of the last step, in floats: the columns, their images (also the first work array of the dense solve), and
// the other work arrays; the Cholesky factor shares the memory of the latter.
template <int D, int L>
struct SmallCfg {
    using C = EigCfg<D, L>;
    static constexpr int LR = L + 2;
    static constexpr size_t zc = (size_t)C::LP * C::LD;
    static constexpr size_t qc = zc > 2 * (size_t)L * L ? zc : 2 * (size_t)L * L;
    static constexpr size_t tri = 2 * TriLds<L, L>::kDoublesNoWa;
    static_assert(tri >= 2 * ((size_t)L * LR + 3 * L), "the factor fits the work arrays");
    static_assert(zc % 4 == 0 && qc % 4 == 0, "16-byte alignment of the work arrays");
    static constexpr size_t floats = zc + qc + tri + 2 * C::LP;
};

// Last step of Algorithm 1 when it is run with passes over H: from W = H^T Y (d x r) and
// Gy = Y^T Y (r x r) of the final Y = H Omega, the QR factor R of Y is the Cholesky factor of
// Gy (Y = Q R  =>  Gy = R^T R), Q^T H = R^-T W^T, and the singular values s and right singular
// vectors of Q^T H are those of (Q^T H)^T = W R^-1, from the eigenpairs of its Gram matrix in double precision
// (ritz_rotate; one-sided Jacobi sweeps where two of its eigenvalues are too close for that route, or one is
// too small).  One workgroup per user, all of it in LDS.  The time is that of its dependent chains (64 users, d = 128,
// r = 32: 64 us, where float Cholesky with four barriers a column and the sweeps took 87).
// info: 0 ok, > 0 Jacobi sweeps exhausted, -1 bad length, -2 Gy is not numerically
// positive definite (Y has fewer than r independent columns).
template <int D, int L>
__global__ __launch_bounds__(kEigThreads) void rsvd_small_kernel(
    const float* __restrict__ partials, int nsplit, const int32_t* __restrict__ lengths, int N,
    float* __restrict__ S, float* __restrict__ V, int32_t* __restrict__ info, int max_sweeps) {
    using C = EigCfg<D, L>;
    using SC = SmallCfg<D, L>;
    constexpr int LD = C::LD, TC = C::TC, LR = SC::LR;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    float* Zc = smem;                  // [LP][LD] columns of W, then of W R^-1
    float* Qc = Zc + SC::zc;           // [LP][LD] singular vectors
    double* tri = reinterpret_cast<double*>(Qc + SC::qc);
    float* nrm = reinterpret_cast<float*>(tri) + SC::tri;         // [LP] column norms
    int* rankv = reinterpret_cast<int*>(nrm + C::LP);             // [LP]
    double* Rm = tri;                  // [L][LR] Gy, then its Cholesky factor
    double* inv = Rm + L * LR;         // [L]
    double* rs = inv + L;              // [L]
    double* d0 = rs + L;               // [L]
    __shared__ int sh_bits;
    __shared__ double sh_scal[1];
    __shared__ int sh_twist[64];
    const int tid = threadIdx.x, b = blockIdx.x;
    const int r = L;
    auto fail = [&](int code) {
        for (int e = tid; e < D * r; e += kEigThreads) V[(size_t)b * D * r + e] = 0.f;
        for (int e = tid; e < r; e += kEigThreads) S[(size_t)b * r + e] = 0.f;
        if (tid == 0 && info) info[b] = code;
    };
    {
        const int raw = lengths ? lengths[b] : N;
        if (raw < r || raw > N) { fail(-1); return; }   // uniform over the workgroup
    }
    if (tid == 0) sh_bits = 0;
    constexpr int NB = xty_blocks<D / 16, L / 16>();
    add_xty_partials<D, L, true, LD, LR, double>(partials + (size_t)b * nsplit * (NB * 256), nsplit, NB, kEigThreads, Zc, Rm);
    __syncthreads();
    if (tid < L) d0[tid] = Rm[tid * LR + tid];
    __syncthreads();
    // A pivot below 1e-5 of its diagonal entry counts as breakdown: the results would carry a relative error of
    // about 2^-24 / 1e-5, a percent (Gy is a float sum).
    if (!cholesky64<L, LR, false>(Rm, inv, rs, d0, 1.0e-5)) { fail(-2); return; }
    solve_rows64<D, L, LD, LR>(Zc, Rm, inv, rs);
    int status = 0;
    // singular values below this share of the largest go the other way: their squares would be short of digits
    constexpr float kSmallRel = 1.0e-4f;
    const float* cols = Qc;
    if (!ritz_rotate<D, L>(Zc, Qc, TriLds<L, L>(tri, reinterpret_cast<double*>(Qc)), sh_scal, sh_twist, nrm, L) ||
        !(nrm[L - 1] > kSmallRel * nrm[0])) {
        __syncthreads();
        cols = Zc;
        const int col = tid / TC, cu = tid % TC;
        auto column_norms = [&]() {
            if (col < L) {
                const float* z = Zc + col * LD;
                float nn = 0.f;
                for (int i = cu; i < D; i += TC) nn += z[i] * z[i];
                nn = team_sum<TC>(nn);
                if (cu == 0) { nrm[col] = nn; atomicMax(&sh_bits, __float_as_int(nn)); }
            }
            __syncthreads();
        };
        // padding columns of the sweeps are zero
        for (int e = tid; e < (C::LP - L) * LD; e += kEigThreads) Zc[L * LD + e] = 0.f;
        column_norms();
        const float dead2 = kDeadRel * kDeadRel * __int_as_float(sh_bits);
        status = max_sweeps;
        for (int sw = 0; sw < max_sweeps; ++sw) {
            const float mine = jacobi_sweep<D, L>(Zc, dead2);
            const bool any = __syncthreads_or(mine > kSweepDone);
            if (!any) { status = 0; break; }
        }
        column_norms();
        if (col < L && cu == 0) nrm[col] = __builtin_amdgcn_sqrtf(nrm[col]);
        __syncthreads();
    }
    if (tid < L) {
        const float th = nrm[tid];
        int rk = 0;
        for (int k = 0; k < L; ++k) {
            const float tk = nrm[k];
            rk += (tk > th || (tk == th && k < tid)) ? 1 : 0;
        }
        rankv[tid] = rk;
    }
    __syncthreads();
    // outputs: columns ranked by norm, normalized, sign fixed by the largest-magnitude entry
    const int col = tid / TC, cu = tid % TC;
    if (col < L) {
        const int k = rankv[col];
        const float* q = cols + col * LD;
        float best = -1.f, nn = 0.f;
        int bi = 0;
        for (int i = cu; i < D; i += TC) {
            const float a = fabsf(q[i]);
            nn += a * a;
            if (a > best) { best = a; bi = i; }
        }
        nn = team_sum<TC>(nn);
        const float scale = nn > 0.f ? __builtin_amdgcn_rsqf(nn) : 0.f;
        for (int m = 1; m < TC; m <<= 1) {
            const float ob = __shfl_xor(best, m);
            const int oi = __shfl_xor(bi, m);
            if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
        }
        const float sgn = (q[bi] < 0.f) ? -scale : scale;
        for (int i = cu; i < D; i += TC) V[((size_t)b * D + i) * r + k] = sgn * q[i];
        if (cu == 0) S[(size_t)b * r + k] = nrm[col];
    }
    if (tid == 0 && info) info[b] = status;
}

// Re-orthonormalisation of the power-iteration block between two passes over H when Algorithm 1
// is run as printed: W (d x r, row-major) is replaced by an orthonormal basis of its range.
// The printed algorithm has no such step; it changes nothing in exact arithmetic (every later
// quantity depends on the block only through its range), and in float it is what keeps the
// r columns from collapsing onto the leading singular vector: without it cond(H Omega) grows by
// (s_1/s_r)^2 per power step.  W R^-1 with the Cholesky factor of W^T W, all in double precision: orthonormal to
// about 1e-16 cond(W)^2, so one pass is enough where Gram-Schmidt in float took two (64 users, d = 128, r = 32:
// 17 us instead of 22); columns that vanish are dropped as zeros.
template <int D, int L>
__global__ __launch_bounds__(kEigThreads) void orthonormalize_block_kernel(
    const float* __restrict__ partials, int nsplit, int blocks, float* __restrict__ W) {
    using C = EigCfg<D, L>;
    constexpr int LD = C::LD, LR = L + 2;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    float* Zc = smem;                                                  // [LP][LD]
    double* Rm = reinterpret_cast<double*>(Zc + C::LP * LD);           // [L][LR]
    double* inv = Rm + L * LR;                                         // [L]
    double* rs = inv + L;                                              // [L]
    const int tid = threadIdx.x, b = blockIdx.x;
    add_xty_partials<D, L, false, LD, 1, double>(partials + (size_t)b * nsplit * (blocks * 256), nsplit, blocks,
                                                 kEigThreads, Zc, nullptr);
    __syncthreads();
    gram_columns64<D, L, LD, LR>(Zc, Rm);
    double top = 0.0;
    for (int k = 0; k < L; ++k) top = fmax(top, Rm[k * LR + k]);
    cholesky64<L, LR, true>(Rm, inv, rs, nullptr, (double)kDeadRel * kDeadRel * top);
    solve_rows64<D, L, LD, LR>(Zc, Rm, inv, rs);
    float* Wb = W + (size_t)b * D * L;
    for (int e = tid; e < D * L; e += kEigThreads) Wb[e] = Zc[(e % L) * LD + e / L];
}

template <int D, int L>
hipError_t launch_orthonormalize_t(const float* partials, int nsplit, bool gram, float* W, int B, hipStream_t stream) {
    using C = EigCfg<D, L>;
    const size_t lds = sizeof(float) * (size_t)C::LP * C::LD + sizeof(double) * ((size_t)L * (L + 2) + 2 * L);
    auto kern = orthonormalize_block_kernel<D, L>;
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(B), dim3(kEigThreads), lds, stream, partials, nsplit,
                       gram ? xty_blocks<D / 16, L / 16>() : (D / 16) * (L / 16), W);
    return hipGetLastError();
}

template <int D, int L>
hipError_t launch_rsvd_small_t(const float* partials, int nsplit, const int32_t* lengths, int B, int N,
                               float* S, float* V, int32_t* info, hipStream_t stream) {
    const size_t lds = sizeof(float) * SmallCfg<D, L>::floats;
    auto kern = rsvd_small_kernel<D, L>;
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(B), dim3(kEigThreads), lds, stream, partials, nsplit, lengths, N, S, V,
                       info, 30);
    return hipGetLastError();
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

hipError_t launch_orthonormalize_block(const float* partials, int nsplit, bool gram, float* W, int B, int d, int r,
                                       hipStream_t stream) {
#define SOLAR_ORTH_CASE(DD, LL) \
    if (d == DD && r == LL) return launch_orthonormalize_t<DD, LL>(partials, nsplit, gram, W, B, stream);
    SOLAR_ORTH_CASE(64, 16) SOLAR_ORTH_CASE(64, 32) SOLAR_ORTH_CASE(64, 48) SOLAR_ORTH_CASE(64, 64)
    SOLAR_ORTH_CASE(128, 16) SOLAR_ORTH_CASE(128, 32) SOLAR_ORTH_CASE(128, 48) SOLAR_ORTH_CASE(128, 64)
#undef SOLAR_ORTH_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_rsvd_small(const float* partials, int nsplit, const int32_t* lengths, int B, int N, int d,
                             int r, float* S, float* V, int32_t* info, hipStream_t stream) {
#define SOLAR_RSVD_CASE(DD, LL) \
    if (d == DD && r == LL) return launch_rsvd_small_t<DD, LL>(partials, nsplit, lengths, B, N, S, V, info, stream);
    SOLAR_RSVD_CASE(64, 16) SOLAR_RSVD_CASE(64, 32) SOLAR_RSVD_CASE(64, 48) SOLAR_RSVD_CASE(64, 64)
    SOLAR_RSVD_CASE(128, 16) SOLAR_RSVD_CASE(128, 32) SOLAR_RSVD_CASE(128, 48) SOLAR_RSVD_CASE(128, 64)
#undef SOLAR_RSVD_CASE
    return hipErrorInvalidValue;
}

}  // namespace solar
