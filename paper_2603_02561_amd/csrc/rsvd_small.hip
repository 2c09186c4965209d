// The small problems of Algorithm 1 run with passes over H (rsvd.hip): the basis of the block between two power
// steps, and the factorization of the last projection.  One workgroup per user, in LDS, double precision where
// squares of singular values meet.  Bound by chains of dependent steps like eig.hip, but built without its
// scheduling flag, which drove these kernels to the whole register file and, in part, into scratch: 256 registers and 24
// spilled instead of 104 for the basis at d = 128, r = 32.
#include "column_block.h"
#include "common.h"
#include "kernels.h"
#include "xty_partials.h"

namespace solar {

namespace {

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
// r = 32: 60 us, where float Cholesky with four barriers a column and the sweeps took 87).
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
            const bool any = __syncthreads_or(mine > kSweepDoneTied);
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
// 18 us instead of 22); columns that vanish are dropped as zeros.
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

}  // namespace

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
