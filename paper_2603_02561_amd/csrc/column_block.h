// Device code on d x L blocks of columns in LDS, one workgroup of 512 threads per user: what the eigensolver (eig.hip) and
// the small problems of Algorithm 1 (rsvd_small.hip) share.  One-sided Jacobi sweeps over the columns, and the
// Rayleigh-Ritz step through the dense solver of tridiag.h.  Every loop over columns or rows has a
// compile-time trip count.
#pragma once

#include "common.h"
#include "tridiag.h"

namespace solar {

namespace {

constexpr int kEigThreads = 512;
constexpr int kEigWaves = kEigThreads / 64;
// A column of the iterate whose norm falls below this fraction of the largest column norm
// is rounding noise of the float Gram matrix (about sqrt(d) * 2^-24 relative) and is dropped.
constexpr float kDeadRel = 1.0e-5f;
// The same between power steps, relative to the largest column of the first panel, which mixes all eigenvectors and is up to four
// times the largest eigenvalue, while what is left of a column when its turn comes in the panels can be a fraction of its own: with
// 1e-5 here too, values just above that limit were lost (d = 128, r = 40: s_k = k^-3/2, the last at 3.95e-3 s_1, for 467 of
// 512 users, levels of six down to 3.9e-3 for 29; now for none).  At 1e-6 columns of rounding noise make first checks fail, 1.3 to 1.8 times
// as long; at 3e-6 the slowest spectrum found takes 1.09 times as long (0.8^k, d = 128, r = 40).
constexpr float kBasisDead = 3.0e-6f;
// Rotations are skipped below kSkipCos.  The Jacobi phase converges quadratically: a sweep whose
// largest |cos| was c leaves about c^2 behind (L * c^2 at worst), so the phase ends after the
// first sweep that met no |cos| above kSweepDone = 5e-4, with a few 1e-6 left; the residual
// check of the following power step is what accepts the result.  (1e-3 leaves V^T V up to 1.3e-5
// off the identity at 72 columns and 3e-3 up to 4e-5; 3e-2 makes the check fail and the iteration
// longer.  In a batch some user nearly always needs the sweep that a looser limit would save
// the others, so the launch is no shorter with 1e-3.)
constexpr float kSkipCos = 1.0e-7f;
constexpr float kSweepDone = 5.0e-4f;
// The same where coinciding eigenvalues led to the sweeps: a rotation between two of those is by up to 45 degrees and carries what the
// sweep met over to columns that it had dealt with, so what is left is of the order of c and not of c^2.  With 5e-4 V^T V was more than
// 2e-5 off for one user in eight with six-fold eigenvalues, 3e-4 at most; now 1e-6.  It costs 3 to 9 % where pairs
// coincide and up to 16 % with larger groups, where it also saves checks that failed for it (d = 128: r = 64 502 -> 445 us, r = 16 132 -> 107).
constexpr float kSweepDoneTied = 2.0e-5f;

__host__ __device__ constexpr int pow2floor_c(int x) {
    int p = 1;
    while (2 * p <= x) p *= 2;
    return p;
}
__host__ __device__ constexpr int min_c(int a, int b) { return a < b ? a : b; }

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

// The iterate in registers: wave w holds the rows of the blocks w, w + 8 of 16 (d = 64: waves 4 .. 7 hold none),
// lane (i, g) = (l % 16, l / 16) of block n the rows 4 g + t of column 16 c + i in component t of [n][c].  That is how the
// matrix unit leaves a product, and it is an operand as it stands wherever rows are contracted (the order of a
// contraction is free).
template <int D, int LP>
struct Iterate {
    static constexpr int NB = D > 128 ? D / 128 : 1, NC = LP / 16;
    static constexpr int W = min_c(kEigWaves, D / 16);   // waves that hold rows
    static constexpr int LDI = D + 8;                    // bf16 elements per column of an image
    typedef v4f Regs[NB][NC];
};

// LDS of one pass over the panels of a block (basis_panels in eig.hip), in floats at `base`
template <int D, int LP>
struct BasisLds {
    using I = Iterate<D, LP>;
    static constexpr int kT = 20;                        // row stride of the 16 x 16 blocks that change hands
    static constexpr size_t gram = (size_t)I::W * 512, part = (size_t)I::W * (I::NC - 1) * 256, sum = (I::NC - 1) * 256;
    static constexpr size_t floats = gram + 512 + part + sum + 16 * kT + (size_t)I::W * I::NB * 16 * kT;
    double* gm;        // [W][16][16] the waves' shares of the panel's Gram matrix
    double* gs;        // [16][16] their sum
    float *cp, *cs;    // [W][NC-1][256] shares of Qp^T Z, [NC-1][256] their sums
    float* tm;         // [16][kT] per column the multipliers of the elimination and the reciprocal of the norm
    float* tr;         // [W][NB][16][kT] the wave's rows of the panel, rows first
    __device__ __forceinline__ explicit BasisLds(float* base) {
        gm = reinterpret_cast<double*>(base);
        gs = gm + I::W * 256;
        cp = base + gram + 512;
        cs = cp + part;
        tm = cs + sum;
        tr = tm + 16 * kT;
    }
};

// MANY: for batches of more users than compute units
template <int D, int L, bool MANY = false>
struct EigCfg {
    static constexpr int LP = 16 * ((L + 15) / 16);
    static constexpr int LD = D + 4;
    // lanes per column outside the Jacobi rounds
    static constexpr int TC = min_c(min_c(64, D), pow2floor_c(kEigThreads / L));
    // G is staged in LDS when it fits, on its way to registers or to the direct solution
    static constexpr bool GLDS = D <= 128;
    static constexpr int GS = D + 4;
    // two blocks of columns, or the images of one
    static constexpr size_t x_floats = (size_t)2 * LP * LD;
    static_assert(2 * x_floats >= (size_t)3 * LP * (D + 8), "three images of 16-bit values");
    static constexpr size_t base_floats = x_floats + 4 * LP;
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
    // sweeps, of which two fit a compute unit, are faster for more users than compute units (r = 16, 256 users 52
    // us against 58, 1024 users 196 against 128).
    static constexpr bool ritz = !direct && (D > 64 || L > 16) && !MANY;
    static constexpr size_t ritz_floats = ritz ? 2 * TriLds<ritz ? L : 16, ritz ? L : 16>::kDoublesNoWa : 0;
    static constexpr int RB = D == 128 || L <= 40 ? 32 : 64;   // eigenvectors per pass of the direct solution
    static constexpr size_t direct_floats = direct ? 2 * TriLds<direct ? D : 16, RB>::kDoubles : 0;
    static constexpr size_t scratch_floats = ritz_floats > BasisLds<D, LP>::floats ? ritz_floats : BasisLds<D, LP>::floats;
    static constexpr size_t stage_floats = GLDS ? (size_t)D * GS : 0;
    static constexpr size_t own_floats = base_floats + scratch_floats > stage_floats ? base_floats + scratch_floats : stage_floats;
    static constexpr size_t lds_floats = own_floats > direct_floats ? own_floats : direct_floats;
    // Workgroups that registers and LDS let share a compute unit, which is what counts with more users than compute
    // units: the waves of one fill the gaps in the chains of the others.  1024 users at d = 64: r = 8 78 us with
    // two, 97 with three, whose 80 registers spill 46 (r = 16 121 and 151); r = 20, direct, 172 with two.  r > 32 takes the
    // eigenvectors in one pass and 104 KB for it: alone on its compute unit 274 (r = 40).
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
    const int tid = fresh_tid(), lane = tid & 63, wave = tid >> 6;
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
    const int tid = fresh_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
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
    // stride of the columns of W: a multiple of 16 would put 16 lanes on four banks
    constexpr int LW = N + 2;
    static_assert(LW * N <= T::WB, "W in a work array");
    constexpr int LD = D + 4, NT = (N + 15) / 16;
    const int tid = fresh_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
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
                                                          w.wb, N);
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
        for (int q = 0; q < N / TB; ++q) w.wb[v * LW + TB * q + u] = l > dead ? y[q] * rs : 0.0;
    }
    __syncthreads();
    for (int J = wave; J < D / 16; J += kEigWaves) {
        double zr[N / 4];
#pragma unroll
        for (int k = 0; k < N / 4; ++k) zr[k] = (double)Zc[(4 * k + g) * LD + 16 * J + i16];
#pragma unroll
        for (int I = 0; I < NT; ++I) {
            const bool in = 16 * I + 15 < N || 16 * I + i16 < N;
            const double* wr = w.wb + (in ? 16 * I + i16 : 0) * LW + g;
            v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int k = 0; k < N / 4; ++k) acc = mfma16x16x4f64(in ? wr[4 * k] : 0.0, zr[k], acc);
#pragma unroll
            for (int t = 0; t < 4; ++t) Qc[(16 * I + g + 4 * t) * LD + 16 * J + i16] = (float)acc[t];
        }
    }
    __syncthreads();
    return true;
}

}  // namespace

}  // namespace solar
