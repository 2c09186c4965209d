// The two contractions over the sequence axis that Algorithm 1 ("Randomized SVD with Power
// Iteration") needs beside Y = H Omega, when it is run as printed, with passes over H:
//   W  = H^T Y   (d x r): the power iteration Omega <- H^T (H Omega), and, after the last
//                          pass, the factor of Q^T H = R^-T (H^T Y)^T for Y = Q R;
//   Gy = Y^T Y   (r x r): the Gram matrix whose Cholesky factor is the R of that QR.
// H is the row-major X (bf16 or float), Y is float [N][r].  As in the Gram kernel the
// sequence axis is the contraction axis of the MFMA and both operands of a product come from
// the same rows: a wave streams 16 rows per step with 16 lanes per row, lane j holding CPL =
// d/16 consecutive columns of X and CY = r/16 consecutive columns of Y; fragment pair (s, c)
// yields the 16x16 block {W[CPL*i+s][CY*j+c]}, pair (c1 <= c2) of Y fragments the block
// {Gy[CY*i+c1][CY*j+c2]}.  Y is a float quantity of unbounded dynamic range (no
// normalisation between power steps in the printed algorithm).  Float inputs take the float
// 16x16x4 MFMA (xty_partial_kernel, with Y in memory); bf16 inputs take power_pass_kernel, which forms
// the rows of Y where they are consumed.
// Split-N with a fixed-order reduction (waves in LDS; the chunks are added by the kernel that uses the
// sums, add_xty_partials in xty_partials.h): results are bitwise reproducible.  A wave keeps a ring of row
// blocks, all but one of them as loads in flight (the scheme of the Gram kernel).
#include "common.h"
#include "kernels.h"
#include "xty_partials.h"

namespace solar {

namespace {

constexpr int kWaves = 4;

// Partial blocks of more than kParallelReduceBlocks fragment pairs do not fit the LDS four times
// over; their waves are added one after another into one region instead.
constexpr int kParallelReduceBlocks = 36;

template <int CPL, int CY>
__global__ __launch_bounds__(kWaves * 64) void xty_partial_kernel(
    const float* __restrict__ X, const float* __restrict__ Y, const int32_t* __restrict__ lengths, int N,
    int nsplit, float* __restrict__ partials) {
    constexpr int D = 16 * CPL, R = 16 * CY;
    constexpr int NB = xty_blocks<CPL, CY>();
    constexpr int STEP = 16;
    const int b = blockIdx.y, split = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane & 15, h = lane >> 4;
    const int len = user_len(lengths, b, N);
    const int chunk = ceil_div(ceil_div(len, nsplit), STEP) * STEP;
    const int r0 = split * chunk;
    const int r1 = min(len, r0 + chunk);
    const float* Yb = Y + (size_t)b * N * R + CY * j;
    const float* Xb = X + (size_t)b * N * D + CPL * j;

    v4f acc[NB];
#pragma unroll
    for (int p = 0; p < NB; ++p) acc[p] = v4f{0.f, 0.f, 0.f, 0.f};

    // A block is 16 rows: lane (j, h) holds rows 4t + h, t = 0..3, as loaded.  Loads carry no predicate and sit behind no branch: the row index is
    // clamped to the chunk's last row and the rows of Y past it count as zero when a ragged
    // block is multiplied (a zero row of Y contributes to neither W nor Gy).  With a branch
    // around a prefetch the compiler waits for all outstanding loads before every block.
    struct Rows { float x[4][CPL]; float y[4][CY]; };
    const int row_max = max(r1 - 1, 0);
    auto load = [&](Rows& dst, int base) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const size_t row = (size_t)min(base + 4 * t + h, row_max);
            const float* px = Xb + row * D;
#pragma unroll
            for (int q = 0; q < CPL / 4; ++q) {
                const v4f v = *reinterpret_cast<const v4f*>(px + 4 * q);
                dst.x[t][4 * q + 0] = v.x; dst.x[t][4 * q + 1] = v.y;
                dst.x[t][4 * q + 2] = v.z; dst.x[t][4 * q + 3] = v.w;
            }
            const float* py = Yb + row * R;
            if constexpr (CY == 4) {
                const v4f v = *reinterpret_cast<const v4f*>(py);
                dst.y[t][0] = v.x; dst.y[t][1] = v.y; dst.y[t][2] = v.z; dst.y[t][3] = v.w;
            } else if constexpr (CY == 2) {
                const float2 v = *reinterpret_cast<const float2*>(py);
                dst.y[t][0] = v.x; dst.y[t][1] = v.y;
            } else {
#pragma unroll
                for (int c = 0; c < CY; ++c) dst.y[t][c] = py[c];
            }
        }
    };
    auto compute = [&](const Rows& src) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
#pragma unroll
            for (int s = 0; s < CPL; ++s)
#pragma unroll
                for (int c = 0; c < CY; ++c)
                    acc[s * CY + c] = mfma16x16x4(src.x[t][s], src.y[t][c], acc[s * CY + c]);
            int p = CPL * CY;
#pragma unroll
            for (int c1 = 0; c1 < CY; ++c1)
#pragma unroll
                for (int c2 = c1; c2 < CY; ++c2) {
                    acc[p] = mfma16x16x4(src.y[t][c1], src.y[t][c2], acc[p]);
                    ++p;
                }
        }
    };
    auto compute_tail = [&](Rows& src, int base) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (base + 4 * t + h >= r1) {
#pragma unroll
                for (int c = 0; c < CY; ++c) src.y[t][c] = 0.f;
            }
        compute(src);
    };
    // ring of kRing row blocks per wave: kRing - 1 blocks of loads stay in flight while one block
    // is multiplied; the steady-state loop takes kRing whole blocks per trip and has no branch in
    // its body, at most kRing - 1 whole blocks and one ragged block are left for the tail
    constexpr int kRing = 3;
    Rows ring[kRing];
    constexpr int stride = kWaves * STEP;
    const int base0 = r0 + wave * STEP;
    const int nblk = base0 < r1 ? ceil_div(r1 - base0, stride) : 0;
    const int nwhole = r1 - base0 >= STEP ? (r1 - base0 - STEP) / stride + 1 : 0;
#pragma unroll
    for (int k = 0; k < kRing - 1; ++k) load(ring[k], base0 + k * stride);
    int i = 0;
    for (; i + kRing <= nwhole; i += kRing) {
#pragma unroll
        for (int k = 0; k < kRing; ++k) {
            load(ring[(k + kRing - 1) % kRing], base0 + (i + k + kRing - 1) * stride);
            __builtin_amdgcn_sched_barrier(0);   // the prefetch is issued before the block is used
            compute(ring[k]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int k = 0; k < kRing; ++k) {
        if (i + k < nblk) {
            if (i + k + kRing - 1 < nblk) load(ring[(k + kRing - 1) % kRing], base0 + (i + k + kRing - 1) * stride);
            compute_tail(ring[k], base0 + (i + k) * stride);
        }
    }

    // Fixed-order sum over the waves of the workgroup (wave 0 + 1 + 2 + 3), then one coalesced store.
    extern __shared__ __attribute__((aligned(16))) v4f red[];
    v4f* out = reinterpret_cast<v4f*>(partials) + ((size_t)b * nsplit + split) * (NB * 64);
    if constexpr (NB <= kParallelReduceBlocks) {
        // every wave parks its blocks in its own region: one barrier
#pragma unroll
        for (int p = 0; p < NB; ++p) red[(wave * NB + p) * 64 + lane] = acc[p];
        __syncthreads();
        for (int e = threadIdx.x; e < NB * 64; e += kWaves * 64) {
            v4f v = red[e];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) v += red[w * NB * 64 + e];
            out[e] = v;
        }
    } else {
        for (int w = 0; w < kWaves; ++w) {
            if (wave == w) {
#pragma unroll
                for (int p = 0; p < NB; ++p) {
                    if (w == 0) red[p * 64 + lane] = acc[p];
                    else red[p * 64 + lane] += acc[p];
                }
            }
            __syncthreads();
        }
        for (int e = threadIdx.x; e < NB * 64; e += kWaves * 64) out[e] = red[e];
    }
}

// a, b as the sum of three bf16 values each (truncation: 8 + 8 + 8 bits of the significand, exact), packed in part[0..2][u]
__device__ __forceinline__ void split_bf16x3(float a, float b, uint32_t (&part)[3][4], int u) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const uint32_t x = __float_as_uint(a), y = __float_as_uint(b);
        part[q][u] = __builtin_amdgcn_perm(y, x, 0x07060302u);
        a -= __uint_as_float(x & 0xffff0000u);
        b -= __uint_as_float(y & 0xffff0000u);
    }
}

// One power step of Algorithm 1 on bf16 inputs in one pass over H: W = H^T (H Omega) and, with GRAM, Gy = Y^T Y,
// where the rows of Y = H Omega go from the accumulators of one product straight into the next and are never
// stored.  Bound by HBM: X is read once.  At B = 64, N = 10000, d = 128, r = 32 (164 MB) a pass takes 35 us, with
// Y^T Y 45 us; with Y written by a projection and read back by a contraction on the float instruction, which
// bound it, the two took 45 + 62 us and a third launch added the chunks.
//   * A wave loads 32 rows as the Gram kernel does (16 lanes per row, CPL columns per lane) and transposes them in
//     registers into the operand of W = X^T Y; it also parks them in its own LDS tile and reads them back row by
//     row as the operand of Y = X Omega (Omega in three bf16 terms).
//   * A lane's accumulators of Y are rows 4h..4h+3 and 16+4h..+3 of the block for rank CY*(l%16) + c.  The loader
//     gives lane group h those same rows, so they are the contraction slots of the next product as they stand.
//   * X is exact in bf16, and Omega and Y split into three bf16 terms without loss, so X^T Y takes three bf16
//     products per 32 rows where the float instruction takes eight of twice the length.
//     Y^T Y stays on the float instruction; only the last pass needs it.
template <int CPL, int CY>
struct PassCfg {
    static constexpr int D = 16 * CPL, KK = D / 32;
    static constexpr int waves = CPL * CY <= 16 ? 8 : 4;      // two waves per SIMD where the registers allow it
    static constexpr int ring = CPL * CY >= 16 && waves == 8 ? 2 : 3;
    static constexpr int LDX = D + 8;                         // bf16 elements per row of a tile
    static constexpr size_t omega_bytes = (size_t)KK * CY * 3 * 64 * sizeof(v4u);
    static constexpr size_t tile_bytes = (size_t)32 * LDX * 2;
    static constexpr size_t loop_bytes = omega_bytes + waves * tile_bytes;
    static constexpr int nb(bool gram) { return gram ? xty_blocks<CPL, CY>() : CPL * CY; }
    // regions that the waves' sums are parked in: as many as fit LDS
    static constexpr int regions(bool gram) {
        int g = waves;
        while (g > 1 && (size_t)g * nb(gram) * 1024 > 156 * 1024) g /= 2;
        return g;
    }
    static constexpr size_t lds(bool gram) {
        const size_t red = (size_t)regions(gram) * nb(gram) * 1024;
        return red > loop_bytes ? red : loop_bytes;
    }
};

template <int CPL, int CY, bool GRAM>
__global__ __launch_bounds__((PassCfg<CPL, CY>::waves * 64)) void power_pass_kernel(
    const uint16_t* __restrict__ Xv, const float* __restrict__ Omega, const int32_t* __restrict__ lengths, int N,
    int nsplit, float* __restrict__ partials) {
    using C = PassCfg<CPL, CY>;
    constexpr int D = C::D, R = 16 * CY, KK = C::KK, LDX = C::LDX, STEP = 32, W = CPL / 2;
    constexpr int NW = CPL * CY, NB = C::nb(GRAM), nthr = C::waves * 64;
    extern __shared__ __attribute__((aligned(16))) v4u lds[];
    const int b = blockIdx.y, split = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane & 15, h = lane >> 4;
    v4u* om = lds;                                             // [KK][CY][three terms][64]
    uint16_t* tile = reinterpret_cast<uint16_t*>(lds + KK * CY * 3 * 64) + wave * (32 * LDX);
    const int len = user_len(lengths, b, N);
    const int chunk = ceil_div(ceil_div(len, nsplit), STEP) * STEP;
    const int r0 = split * chunk;
    const int r1 = min(len, r0 + chunk);

    const uint32_t* X = reinterpret_cast<const uint32_t*>(Xv) + (size_t)b * N * (D / 2) + W * j;
    const int row_max = max(r1 - 1, 0);
    // rows of lane group h: 4h .. 4h+3 and 16+4h .. 16+4h+3 of the block
    auto row_of = [&](int t) __attribute__((always_inline)) { return 4 * h + (t & 3) + 16 * (t >> 2); };
    auto load = [&](uint32_t (&dst)[8][W], int base) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const uint32_t* p = X + (size_t)min(base + row_of(t), row_max) * (D / 2);
            if constexpr (W == 2) {
                const uint2 v = *reinterpret_cast<const uint2*>(p);
                dst[t][0] = v.x; dst[t][1] = v.y;
            } else {
                static_assert(W == 4, "d = 128");
                const v4u v = *reinterpret_cast<const v4u*>(p);
                dst[t][0] = v.x; dst[t][1] = v.y; dst[t][2] = v.z; dst[t][3] = v.w;
            }
        }
    };
    constexpr int kRing = C::ring;
    uint32_t ring[kRing][8][W];
    constexpr int stride = C::waves * STEP;
    const int base0 = r0 + wave * STEP;
    const int nblk = base0 < r1 ? ceil_div(r1 - base0, stride) : 0;
    const int nwhole = r1 - base0 >= STEP ? (r1 - base0 - STEP) / stride + 1 : 0;
#pragma unroll
    for (int k = 0; k < kRing - 1; ++k) load(ring[k], base0 + k * stride);

    // operands of Omega: slot (g, u) of chunk kk is column 32 kk + 8 g + u, lane j supplies rank CY j + c
    for (int e = threadIdx.x; e < KK * CY * 64; e += nthr) {
        const int ln = e & 63, c = (e >> 6) % CY, kk = (e >> 6) / CY;
        const float* src = Omega + ((size_t)b * D + 32 * kk + 8 * (ln >> 4)) * R + CY * (ln & 15) + c;
        uint32_t part[3][4];
#pragma unroll
        for (int u2 = 0; u2 < 4; ++u2) split_bf16x3(src[(size_t)(2 * u2) * R], src[(size_t)(2 * u2 + 1) * R], part, u2);
#pragma unroll
        for (int q = 0; q < 3; ++q)
            om[((kk * CY + c) * 3 + q) * 64 + ln] = v4u{part[q][0], part[q][1], part[q][2], part[q][3]};
    }
    v4f acc[NB];
#pragma unroll
    for (int p = 0; p < NB; ++p) acc[p] = v4f{0.f, 0.f, 0.f, 0.f};
    __syncthreads();

    auto compute = [&](const uint32_t (&src)[8][W]) __attribute__((always_inline)) {
        wave_order();
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            uint16_t* d = tile + row_of(t) * LDX + CPL * j;
            if constexpr (W == 2) *reinterpret_cast<uint2*>(d) = uint2{src[t][0], src[t][1]};
            else *reinterpret_cast<v4u*>(d) = v4u{src[t][0], src[t][1], src[t][2], src[t][3]};
        }
        wave_order();
        // Y of the block: y[rt][c][t] is row 16 rt + 4 h + t, rank CY j + c
        v4f y[2][CY];
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int c = 0; c < CY; ++c) y[rt][c] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            v4u xa[2];
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
                xa[rt] = *reinterpret_cast<const v4u*>(tile + (16 * rt + j) * LDX + 32 * kk + 8 * h);
#pragma unroll
            for (int c = 0; c < CY; ++c) {
#pragma unroll
                for (int q = 2; q >= 0; --q) {
                    const v4u w = om[((kk * CY + c) * 3 + q) * 64 + lane];
#pragma unroll
                    for (int rt = 0; rt < 2; ++rt) y[rt][c] = mfma16x16x32bf16(xa[rt], w, y[rt][c]);
                }
            }
        }
        // fragment s: column CPL j + s of the lane's eight rows
        v4u frag[CPL];
#pragma unroll
        for (int s = 0; s < CPL; ++s) {
            uint32_t o[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                o[u] = __builtin_amdgcn_perm(src[2 * u + 1][s / 2], src[2 * u][s / 2],
                                             (s & 1) ? 0x07060302u : 0x05040100u);
            frag[s] = v4u{o[0], o[1], o[2], o[3]};
        }
#pragma unroll
        for (int c = 0; c < CY; ++c) {
            uint32_t part[3][4];
#pragma unroll
            for (int u = 0; u < 4; ++u) split_bf16x3(y[u >> 1][c][2 * (u & 1)], y[u >> 1][c][2 * (u & 1) + 1], part, u);
#pragma unroll
            for (int q = 2; q >= 0; --q) {
                const v4u yb = v4u{part[q][0], part[q][1], part[q][2], part[q][3]};
#pragma unroll
                for (int s = 0; s < CPL; ++s) acc[s * CY + c] = mfma16x16x32bf16(frag[s], yb, acc[s * CY + c]);
            }
        }
        if constexpr (GRAM) {
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    int p = NW;
#pragma unroll
                    for (int c1 = 0; c1 < CY; ++c1)
#pragma unroll
                        for (int c2 = c1; c2 < CY; ++c2) {
                            acc[p] = mfma16x16x4(y[rt][c1][t], y[rt][c2][t], acc[p]);
                            ++p;
                        }
                }
        }
    };
    // a block of the tail: rows at or past the end of the chunk count as zero
    auto compute_tail = [&](uint32_t (&src)[8][W], int base) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 8; ++t)
            if (base + row_of(t) >= r1) {
#pragma unroll
                for (int w = 0; w < W; ++w) src[t][w] = 0u;
            }
        compute(src);
    };
    int i = 0;
    for (; i + kRing <= nwhole; i += kRing) {
#pragma unroll
        for (int k = 0; k < kRing; ++k) {
            load(ring[(k + kRing - 1) % kRing], base0 + (i + k + kRing - 1) * stride);
            __builtin_amdgcn_sched_barrier(0);   // the prefetch is issued before the block is used
            compute(ring[k]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int k = 0; k < kRing; ++k) {
        if (i + k < nblk) {
            if (i + k + kRing - 1 < nblk) load(ring[(k + kRing - 1) % kRing], base0 + (i + k + kRing - 1) * stride);
            compute_tail(ring[k], base0 + (i + k) * stride);
        }
    }

    // Sum over the waves in a fixed order: `regions` of them at a time into regions of LDS, then the regions.
    constexpr int G = C::regions(GRAM);
    v4f* red = reinterpret_cast<v4f*>(lds);
    __syncthreads();                                          // the tiles and Omega are done with
#pragma unroll
    for (int q = 0; q < C::waves / G; ++q) {
        if (wave / G == q) {
            v4f* mine = red + (wave % G) * (NB * 64) + lane;
#pragma unroll
            for (int p = 0; p < NB; ++p) {
                if (q == 0) mine[p * 64] = acc[p];
                else mine[p * 64] += acc[p];
            }
        }
        __syncthreads();
    }
    v4f* out = reinterpret_cast<v4f*>(partials) + ((size_t)b * nsplit + split) * (NB * 64);
    for (int e = threadIdx.x; e < NB * 64; e += nthr) {
        v4f v = red[e];
#pragma unroll
        for (int w = 1; w < G; ++w) v += red[w * NB * 64 + e];
        out[e] = v;
    }
}

template <int CPL, int CY>
hipError_t launch_xty_t(const float* X, const float* Y, const int32_t* lengths, int B, int N, float* partials,
                        hipStream_t stream) {
    constexpr int NB = xty_blocks<CPL, CY>();
    constexpr size_t lds = sizeof(v4f) * 64 * NB * (NB <= kParallelReduceBlocks ? kWaves : 1);
    const int nsplit = gram_nsplit(B, N);
    auto kern = xty_partial_kernel<CPL, CY>;
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(nsplit, B), dim3(kWaves * 64), lds, stream, X, Y, lengths, N, nsplit, partials);
    return hipGetLastError();
}

template <int CPL, int CY, bool GRAM>
hipError_t launch_pass_g(const uint16_t* X, const float* Omega, const int32_t* lengths, int B, int N, float* partials,
                         hipStream_t stream) {
    using C = PassCfg<CPL, CY>;
    constexpr size_t lds = C::lds(GRAM);
    static_assert(lds <= 160 * 1024, "fits LDS");
    const int nsplit = gram_nsplit(B, N);
    auto kern = power_pass_kernel<CPL, CY, GRAM>;
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(nsplit, B), dim3(C::waves * 64), lds, stream, X, Omega, lengths, N, nsplit, partials);
    return hipGetLastError();
}

template <int CPL, int CY>
hipError_t launch_pass_t(const uint16_t* X, const float* Omega, const int32_t* lengths, int B, int N, bool gram,
                         float* partials, hipStream_t stream) {
    return gram ? launch_pass_g<CPL, CY, true>(X, Omega, lengths, B, N, partials, stream)
                : launch_pass_g<CPL, CY, false>(X, Omega, lengths, B, N, partials, stream);
}

}  // namespace

bool rsvd_supported(int d, int r) { return (d == 64 || d == 128) && r >= 16 && r <= 64 && r % 16 == 0 && r <= d; }

size_t xty_partial_floats(int B, int N, int d, int r) {
    const int cpl = d / 16, cy = r / 16;
    return (size_t)B * gram_nsplit(B, N) * (cpl * cy + cy * (cy + 1) / 2) * 256;
}

#define SOLAR_FOR_SHAPE(CALL)                   \
    if (d == 64 && r == 16) return CALL(4, 1);  \
    if (d == 64 && r == 32) return CALL(4, 2);  \
    if (d == 64 && r == 48) return CALL(4, 3);  \
    if (d == 64 && r == 64) return CALL(4, 4);  \
    if (d == 128 && r == 16) return CALL(8, 1); \
    if (d == 128 && r == 32) return CALL(8, 2); \
    if (d == 128 && r == 48) return CALL(8, 3); \
    if (d == 128 && r == 64) return CALL(8, 4); \
    return hipErrorInvalidValue;

hipError_t launch_xty(const float* X, const float* Y, const int32_t* lengths, int B, int N, int d, int r,
                      float* partials, hipStream_t stream) {
#define SOLAR_XTY(CPL, CY) launch_xty_t<CPL, CY>(X, Y, lengths, B, N, partials, stream)
    SOLAR_FOR_SHAPE(SOLAR_XTY)
#undef SOLAR_XTY
}

hipError_t launch_power_pass(const uint16_t* X, const float* Omega, const int32_t* lengths, int B, int N, int d, int r,
                             bool gram, float* partials, hipStream_t stream) {
#define SOLAR_PASS(CPL, CY) launch_pass_t<CPL, CY>(X, Omega, lengths, B, N, gram, partials, stream)
    SOLAR_FOR_SHAPE(SOLAR_PASS)
#undef SOLAR_PASS
}
#undef SOLAR_FOR_SHAPE

}  // namespace solar
