// Row-times-matrix products around the attention operators:
//   * linear attention Attn_lin = Query (Key^T Value) (Preliminaries) with Key = Value = X:
//     O_b = scale * Q_b G_b, G_b = X_b^T X_b from the Gram kernel;
//   * the learnable projections W_Q, W_K, W_V of the Preliminaries, folded around an operator
//     that works on H itself: Q' = C (W_Q W_K^T) before it and O' = O W_V after it.
// Both are Out[rows x d] = scale * In[rows x d] * W[d x d] with a float matrix W, per user or shared.
//
// Bound by memory.  W is split once per workgroup into three bf16 matrices that add up to it exactly (24
// bits; fewer for values below 2^-110, whose terms are below the smallest bf16) and kept in LDS; the products run on the
// 32x32x16 bf16 instruction with float accumulation.  A bf16
// row takes three of them, each product exact; a float row is split the same way and takes the six whose
// size is above 2^-24 of the leading one, which is the rounding of a float product.  That is a third (or
// two thirds) of the time of the float instruction for the same precision: 64000 rows of d = 128 take
// 12.6 us from bf16 to bf16 (2.6 TB/s) and 22 from float to float, of d = 256 35 and 62; with the
// float instruction, 16 rows per wave and a copy of W per 64 rows 31.5, 38.5, 155 and 189.
#include "common.h"
#include "kernels.h"

namespace solar {

namespace {

constexpr int kRowWaves = 8;

__device__ __forceinline__ v16f mfma32x32x16bf16(v8bf a, v8bf b, v16f c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ v16f mfma32x32x2(float a, float b, v16f c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// x = s[0] + s[1] + s[2] to 24 bits
__device__ __forceinline__ void split3(const float (&x)[8], v8bf (&s)[3]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const __bf16 h = (__bf16)x[i];
        const float r = x[i] - (float)h;
        const __bf16 m = (__bf16)r;
        s[0][i] = h;
        s[1][i] = m;
        s[2][i] = (__bf16)(r - (float)m);
    }
}

template <int D>
struct RowCfg {
    static constexpr int NC = D < 128 ? D : (D == 128 ? 128 : 64);   // output columns per workgroup (LDS)
    static constexpr int LDW = D + 8;                                // bf16 stride of a column: conflict-free
    static constexpr size_t lds_bytes = (size_t)3 * NC * LDW * 2;
};

// One wave takes blocks of 32 rows: lane (i, h) holds entries 16 s + 8 h .. + 7 of row i for every step s of
// the contraction, the next block's rows are loaded while this one is multiplied.
// IN_PLACE: Out is In, and the columns of a row are spread over workgroups otherwise (d = 256): a workgroup then keeps
// its rows in registers and takes the column chunks one after another.
template <int D, bool IN_BF16, bool OUT_BF16, bool IN_PLACE>
__global__ __launch_bounds__(kRowWaves * 64) void rowgemm_kernel(
    const void* In, const float* __restrict__ W, size_t w_stride, int rows, float scale, void* Out) {
    using C = RowCfg<D>;
    constexpr int NC = C::NC, LDW = C::LDW, NS = D / 16, NT = NC / 32;
    constexpr int VS = IN_BF16 ? 1 : 2;                  // 16-byte loads per step
    constexpr bool AHEAD = NS * VS < 16;                 // two blocks of rows fit the registers
    extern __shared__ __attribute__((aligned(16))) __bf16 img[];     // [3][NC][LDW]
    const int b = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i32 = lane & 31, h = lane >> 5;
    const int nblk = ceil_div(rows, 32), stride = gridDim.x * kRowWaves;
    const char* in = reinterpret_cast<const char*>(In) + (size_t)b * rows * D * (IN_BF16 ? 2 : 4);
    v4u raw[AHEAD ? 2 : 1][NS][VS];
    auto load = [&](int blk, v4u (&r)[NS][VS]) __attribute__((always_inline)) {
        int row = 32 * blk + i32;
        row = row < rows ? row : rows - 1;
        const char* p = in + ((size_t)row * D + 8 * h) * (IN_BF16 ? 2 : 4);
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int v = 0; v < VS; ++v)
                r[s][v] = *reinterpret_cast<const v4u*>(p + s * (IN_BF16 ? 32 : 64) + 16 * v);
    };
    int blk = blockIdx.x * kRowWaves + wave;
    if (blk < nblk) load(blk, raw[0]);
    const float* Wb = W + (size_t)b * w_stride;
    // the images of the NC columns from c0 on
    auto stage = [&](int c0) __attribute__((always_inline)) {
        for (int e = tid; e < NC * (D / 8); e += kRowWaves * 64) {
            const int c = e % NC, k8 = e / NC;
            float x[8];
            v8bf s[3];
#pragma unroll
            for (int k = 0; k < 8; ++k) x[k] = Wb[(size_t)(8 * k8 + k) * D + c0 + c];
            split3(x, s);
#pragma unroll
            for (int p = 0; p < 3; ++p) *reinterpret_cast<v8bf*>(img + (p * NC + c) * LDW + 8 * k8) = s[p];
        }
    };
    if constexpr (!IN_PLACE) {
        stage(blockIdx.z * NC);
        __syncthreads();
    }
    const __bf16* wb = img + i32 * LDW + 8 * h;
    auto multiply = [&](int at, const v4u (&r)[NS][VS], int c0) __attribute__((always_inline)) {
        v16f acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
        // the operands from LDS one step ahead of the products, and no further: left alone, the compiler
        // reads all steps' at once and spills
        v8bf w[2][NT][3];
        auto read = [&](int s, v8bf (&d)[NT][3]) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    d[t][p] = *reinterpret_cast<const v8bf*>(wb + (p * NC + 32 * t) * LDW + 16 * s);
        };
        read(0, w[0]);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (s + 1 < NS) read(s + 1, w[(s + 1) & 1]);
            v8bf a[3];
            if constexpr (IN_BF16) {
                a[0] = __builtin_bit_cast(v8bf, r[s][0]);
            } else {
                float x[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) x[k] = __uint_as_float(r[s][k / 4][k % 4]);
                if constexpr (IN_PLACE) {                // or the terms of all steps are formed once and kept
#pragma unroll
                    for (int k = 0; k < 8; ++k) asm volatile("" : "+v"(x[k]));
                }
                split3(x, a);
            }
            auto product = [&](int i, int j) __attribute__((always_inline)) {
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] = mfma32x32x16bf16(a[i], w[s & 1][t][j], acc[t]);
            };
            // the small products first
            product(0, 2);
            if constexpr (!IN_BF16) {
                product(1, 1);
                product(2, 0);
                product(1, 0);
            }
            product(0, 1);
            product(0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        // component e is row 8 (e / 4) + 4 h + e % 4 of the block, column i32 of the tile
        auto store = [&]() __attribute__((always_inline)) {
            const int row0 = 32 * at + 4 * h;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int row = row0 + 8 * (e / 4) + e % 4;
                if (row < rows) {
                    const size_t o = ((size_t)b * rows + row) * D + c0 + i32;
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        const float v = scale * acc[t][e];
                        if constexpr (OUT_BF16) reinterpret_cast<__bf16*>(Out)[o + 32 * t] = (__bf16)v;
                        else reinterpret_cast<float*>(Out)[o + 32 * t] = v;
                    }
                }
            }
        };
        store();
        // An infinity, or a value that rounds to one as a bf16 (above 3.39e38), has terms inf, inf - inf and NaN, and
        // the terms of a product that overflows can cancel to NaN: a block with a sum that is not finite is taken
        // again on the float instruction.  The look at the sums costs 0.1 us a launch, 1 to 2 % of 64000 rows.
        constexpr int kChains = 8;   // a zero each, NaN if any sum is not finite
        float probe[kChains];
#pragma unroll
        for (int i = 0; i < kChains; ++i) probe[i] = 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int e = 0; e < 16; ++e) probe[e % kChains] = fmaf(acc[t][e], 0.f, probe[e % kChains]);
#pragma unroll
        for (int i = kChains / 2; i; i /= 2)
#pragma unroll
            for (int k = 0; k < i; ++k) probe[k] += probe[k + i];
        if (__builtin_expect(__any(probe[0] != 0.f), 0)) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                uint32_t at_w = (16 * s + 8 * h) * D + i32;
                asm volatile("" : "+v"(at_w));   // or these loads are taken ahead of the loop over the blocks
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    float a;
                    if constexpr (IN_BF16) a = (k & 1) ? bf16_hi(r[s][0][k / 2]) : bf16_lo(r[s][0][k / 2]);
                    else a = __uint_as_float(r[s][k / 4][k % 4]);
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        acc[t] = mfma32x32x2(a, (Wb + c0)[at_w + k * D + 32 * t], acc[t]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            store();
        }
    };
    if constexpr (IN_PLACE) {
        for (int first = blockIdx.x * kRowWaves; first < nblk; first += stride, blk += stride) {   // uniform
            if (first > (int)blockIdx.x * kRowWaves && blk < nblk) load(blk, raw[0]);
#pragma unroll 1
            for (int c0 = 0; c0 < D; c0 += NC) {
                __syncthreads();                         // the image of the last chunk is done with
                stage(c0);
                __syncthreads();
                if (blk < nblk) multiply(blk, raw[0], c0);
            }
        }
    } else if constexpr (AHEAD) {
        for (; blk < nblk; blk += 2 * stride) {
            if (blk + stride < nblk) load(blk + stride, raw[1]);
            multiply(blk, raw[0], blockIdx.z * NC);
            if (blk + stride >= nblk) break;
            if (blk + 2 * stride < nblk) load(blk + 2 * stride, raw[0]);
            multiply(blk + stride, raw[1], blockIdx.z * NC);
        }
    } else {
        while (blk < nblk) {
            multiply(blk, raw[0], blockIdx.z * NC);
            blk += stride;
            if (blk < nblk) load(blk, raw[0]);
        }
    }
}

template <int D>
hipError_t launch_d(const void* In, const float* W, size_t w_stride, int B, int rows, float scale, bool in_bf16,
                    bool out_bf16, void* Out, hipStream_t stream) {
    using C = RowCfg<D>;
    // one workgroup per compute unit (the images of W take more than half of its LDS), none without a block
    // of rows for every wave
    constexpr int NZ = D / C::NC;
    const bool in_place = NZ > 1 && In == Out && in_bf16 == out_bf16;
    const int nz = in_place ? 1 : NZ;
    const int want = ceil_div(ceil_div(rows, 32), kRowWaves), room = ceil_div(256, B * nz);
    const dim3 grid(want < room ? want : room, B, nz), block(kRowWaves * 64);
#define SOLAR_ROWGEMM(IB, OB)                                                                        \
    do {                                                                                             \
        auto kern = rowgemm_kernel<D, IB, OB, false>;                                                \
        if constexpr (NZ > 1 && IB == OB) {                                                          \
            if (in_place) kern = rowgemm_kernel<D, IB, OB, true>;                                    \
        }                                                                                            \
        hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), C::lds_bytes);         \
        if (e != hipSuccess) return e;                                                               \
        hipLaunchKernelGGL(kern, grid, block, C::lds_bytes, stream, In, W, w_stride, rows, scale, Out); \
    } while (0)
    if (in_bf16 && out_bf16) SOLAR_ROWGEMM(true, true);
    else if (in_bf16) SOLAR_ROWGEMM(true, false);
    else if (out_bf16) SOLAR_ROWGEMM(false, true);
    else SOLAR_ROWGEMM(false, false);
#undef SOLAR_ROWGEMM
    return hipGetLastError();
}

}  // namespace

// Out[b] = scale * In[b] * W[b * w_stride ...]; w_stride = 0 shares one matrix among the users.
hipError_t launch_rowgemm(const void* In, const float* W, size_t w_stride, int B, int rows, int d, float scale,
                          bool in_bf16, bool out_bf16, void* Out, hipStream_t stream) {
    switch (d) {
        case 64: return launch_d<64>(In, W, w_stride, B, rows, scale, in_bf16, out_bf16, Out, stream);
        case 128: return launch_d<128>(In, W, w_stride, B, rows, scale, in_bf16, out_bf16, Out, stream);
        case 256: return launch_d<256>(In, W, w_stride, B, rows, scale, in_bf16, out_bf16, Out, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace solar
