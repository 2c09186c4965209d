// SVD-Attention, Attn_SVD = MatMul(MatMul(Query, Key_r^T), Value_r) (Section
// "SVD-Attention"), on gfx950.
//
// attention_seq_kernel -- softmax over the N sequence positions, evaluated in
// factor space:   O = softmax_n(scale * Qt P^T) P V^T,   Qt = Q V,  P = X V.
// The M x N score matrix is never stored: the kernel walks over tiles of P with an
// online softmax (running row maximum and row sum), keeps Z = sum_n w_n P_n in the
// matrix-unit accumulators and only at the end maps Z / l back to d columns with
// V^T.  Key and value are the same tile of P, so one LDS tile feeds both products.
// The transposed forms S^T = P Qt^T and Z^T = P^T W^T are used so that a
// query is a lane (column l%16 of every accumulator): the softmax statistics of a
// query are then combined over 4 lane groups only, and the accumulator of one
// product is directly the B operand of the next with no data movement (the
// contraction index may be enumerated in any order as long as A and B agree).
//
// Both products over the sequence keep float accuracy on the bf16 instruction: P, Qt and the weights W are each
// the sum of three bf16 terms (rounded to nearest: what is left is below 2^-26), and a product is
// taken as the six products of terms that are not below 2^-25 of it, with float accumulators.  Per 16 queries,
// 64 rows and 16 ranks that is 384 cycles of the matrix unit where the float 16x16x4 instruction takes 1024; the
// tile of P is split once, when it is stored to LDS, the weights by the wave that formed them (about a
// hundred vector instructions per 64 rows).  B = 32, N = 4096, M = 512,
// d = 128, r = 16: 64.8 -> 61.2 us, 58.2 with the loads two steps ahead; B = 64, N = 1500, M = 1200, r = 64: 422 -> 289 -> 274; errors against double precision fall
// from 7.7e-7 to 5.8e-7 (geometric mean over twelve shapes).
// Values of P or Qt below 2^-110 keep fewer bits (there is no bf16 below 2^-133).
// The products with V in the prologue and the epilogue stay on the float instruction.
//
// attention_tokens_kernel -- the literal r-token form, with or without softmax:
//   O = softmax_k(scale * Q T^T) T   or   O = scale * (Q T^T) T,   T = diag(S) V^T.
#include <cstdlib>

#include "common.h"
#include "kernels.h"

namespace solar {

namespace {

constexpr float kLog2e = 1.4426950408889634f;
// the six products of terms that count, smallest first
__device__ constexpr int kTermA[6] = {0, 2, 1, 0, 1, 0}, kTermB[6] = {2, 0, 1, 1, 0, 0};

// Ranks of a row in a tile image.  Lane group g holds ranks 16*ib + 4*g + t of Qt in component t of block ib, and
// these are its contraction slots: an instruction takes 32 ranks (blocks 2c and 2c+1, eight slots per lane), so
// the image of such a chunk lists the quads of four ranks as 0 4 1 5 2 6 3 7 and a lane's eight are one 16-byte
// read.  An odd last block fills an instruction with two terms of its 16 ranks; it is stored as it is.
template <int RB>
__device__ __forceinline__ constexpr int quad_at(int q) {   // where quad q (ranks 4q .. 4q+3) is, in quads
    return q < 8 * (RB / 2) ? (q & ~7) + 2 * (q & 3) + ((q >> 2) & 1) : q;
}

// a, b as three bf16 terms each, packed in t[0..2].  A value above 3.39e38 rounds to infinity as a bf16 and leaves
// inf - inf and NaN for the other terms; with CLAMP its leading term is the largest bf16, and every finite
// value is the sum of its terms.
template <bool CLAMP = false>
__device__ __forceinline__ void split3_pair(float a, float b, uint32_t (&t)[3]) {
    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
    constexpr float kTop = 3.38953139e38f;   // the largest bf16
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const v2bf v = CLAMP && q == 0 ? v2bf{(__bf16)fminf(fmaxf(a, -kTop), kTop), (__bf16)fminf(fmaxf(b, -kTop), kTop)}
                                       : v2bf{(__bf16)a, (__bf16)b};
        t[q] = __builtin_bit_cast(uint32_t, v);
        a -= bf16_lo(t[q]);
        b -= bf16_hi(t[q]);
    }
}

// four rows of one rank out of a row-major image: within 16 lanes, lane i passes the address of row i/4, quad i%4
// and receives element i of the 16 for rows 0..3
__device__ __forceinline__ uint2 read_transposed(const uint16_t* p) {
    typedef short v4s __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) v4s* lds_v4s_ptr;
    const v4s v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_ptr)(p));
    return __builtin_bit_cast(uint2, v);
}

// V, and two buffers of NS tiles of three images of NT rows
constexpr size_t seq_lds(int D, int RB, int NS, int NT) {
    return sizeof(float) * (size_t)D * (16 * RB + 4) + sizeof(uint16_t) * (size_t)2 * NS * 3 * NT * (16 * RB + 8);
}

// The waves of a workgroup are NS groups of QG.  The waves of a group have queries of their own (QB blocks of 16 each);
// group sp takes every NS-th tile of NT rows of the sequence for the same queries, and the groups'
// partial results (reference, row sum, Z) are merged in a fixed order at the end.  NS > 1 gives a small
// batch, whose workgroups do not fill the GPU's wave slots, NS independent chains of products and
// exponentials per SIMD; QG = 1 gives a single request four times the workgroups.
template <int D, int RB, bool BF16, int QB, int NS, int QG, int NT>
__global__ __launch_bounds__(64 * QG * NS) void attention_seq_kernel(
    const void* __restrict__ Qv, const float* __restrict__ V, const float* __restrict__ P,
    const int32_t* __restrict__ lengths, int B, int N, int r, int M, float scale, float* __restrict__ O) {
    constexpr int RP = 16 * RB;
    constexpr int LDV = RP + 4;
    constexpr int LDP = RP + 8;             // bf16 elements per row of an image; reads are free of bank conflicts
    constexpr int kImg = NT * LDP;         // one term of a tile
    constexpr int FC = RB / 2;              // chunks of 32 ranks, then possibly one of 16
    constexpr bool HALF = RB % 2 != 0;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    float* Vs = smem;                                               // [D][LDV]
    uint16_t* Ps = reinterpret_cast<uint16_t*>(Vs + D * LDV);       // [2][NS][3 terms][NT][LDP]
    constexpr int NTHR = 64 * QG * NS;
    // Workgroups are dealt to the 8 XCDs round-robin by linear id.  All M-tiles of a user
    // get ids that agree modulo 8, so they share one XCD and its L2 holds that user's P once.
    const int mtiles = ceil_div(M, QG * QB * 16);
    // Fewer than eight users take consecutive ids, so that no XCD idles, and every XCD reads its own copy.
    const int slot = B < 8 ? (int)blockIdx.x : (int)(blockIdx.x >> 3);
    const int b = B < 8 ? slot / mtiles : (slot / mtiles) * 8 + (int)(blockIdx.x & 7);
    if (b >= B) return;   // uniform over the workgroup
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = (tid >> 6) % QG;       // queries of the wave
    const int sp = (tid >> 6) / QG;         // its share of the sequence (0 when NS == 1)
    const int i16 = lane & 15, g = lane >> 4;
    const int len = user_len(lengths, b, N);
    const int m_wave = (slot % mtiles) * (QG * QB * 16) + wave * (QB * 16);
    const float* Pb = P + (size_t)b * N * r;

    for (int e = tid; e < D * RP; e += NTHR) {
        const int k = e / RP, c = e % RP;
        Vs[k * LDV + c] = (c < r) ? V[((size_t)b * D + k) * r + c] : 0.f;
    }
    __syncthreads();

    // ---- prologue: Qt^T = V^T Q^T, scaled by scale*log2(e) -------------------------
    v4f qt[QB][RB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
        for (int ib = 0; ib < RB; ++ib) qt[qb][ib] = v4f{0.f, 0.f, 0.f, 0.f};
        const int m = m_wave + 16 * qb + i16;
        const bool valid = m < M;
        const size_t row = ((size_t)b * M + (valid ? m : 0)) * D;
        for (int kk = 0; kk < D / 16; ++kk) {
            v4f q4;
            if constexpr (BF16) {
                uint2 w = reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(Qv) + row)[4 * kk + g];
                q4 = v4f{bf16_lo(w.x), bf16_hi(w.x), bf16_lo(w.y), bf16_hi(w.y)};
            } else {
                q4 = reinterpret_cast<const v4f*>(reinterpret_cast<const float*>(Qv) + row)[4 * kk + g];
            }
            if (!valid) q4 = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float* vrow = Vs + (16 * kk + 4 * g + t) * LDV;
#pragma unroll
                for (int ib = 0; ib < RB; ++ib)
                    qt[qb][ib] = mfma16x16x4(vrow[16 * ib + i16], q4[t], qt[qb][ib]);
            }
        }
#pragma unroll
        for (int ib = 0; ib < RB; ++ib) qt[qb][ib] *= scale * kLog2e;
    }

    // B operands of the score product: three terms of every chunk of 32 ranks; of an odd last block the pairs of terms
    // that the pairs of P (0, 1), (0, 1) and (0, 2) are multiplied with
    v4u qf[QB][FC > 0 ? FC : 1][3], qh[QB][3];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        uint32_t w[RB][2][3];
#pragma unroll
        for (int ib = 0; ib < RB; ++ib)
#pragma unroll
            for (int e = 0; e < 2; ++e) split3_pair<true>(qt[qb][ib][2 * e], qt[qb][ib][2 * e + 1], w[ib][e]);
#pragma unroll
        for (int c = 0; c < FC; ++c)
#pragma unroll
            for (int q = 0; q < 3; ++q)
                qf[qb][c][q] = v4u{w[2 * c][0][q], w[2 * c][1][q], w[2 * c + 1][0][q], w[2 * c + 1][1][q]};
        if constexpr (HALF) {
            constexpr int first[3] = {0, 1, 2}, second[3] = {1, 0, 0};
#pragma unroll
            for (int k = 0; k < 3; ++k)
                qh[qb][k] = v4u{w[RB - 1][0][first[k]], w[RB - 1][1][first[k]], w[RB - 1][0][second[k]], w[RB - 1][1][second[k]]};
        }
    }

    // ---- main loop over tiles of P -------------------------------------------------
    v4f z[QB][RB];
    float mrun[QB], lrun[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        mrun[qb] = -INFINITY;
        lrun[qb] = 0.f;
#pragma unroll
        for (int ib = 0; ib < RB; ++ib) z[qb][ib] = v4f{0.f, 0.f, 0.f, 0.f};
    }

    const int ntiles = ceil_div(ceil_div(len, NT), NS);   // steps of NS tiles
    constexpr int kRows = NS * NT;                        // rows loaded per step
    // A thread moves kItems quads of ranks per step; row and quad follow from compile-time divisors.  The loads of a
    // step are issued two steps ahead and stay in registers while a tile is multiplied: rows are clamped to the last
    // valid one instead of being predicated, and count as zero when they are split and stored.
    constexpr int kQuads = 4 * RB, kItems = kRows * kQuads / NTHR;
    static_assert(kItems * NTHR == kRows * kQuads, "whole items per thread");
    v4f st[kItems];
    auto fetch = [&](int tile) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kItems; ++i) {
            const int e = tid + i * NTHR, nn = e / kQuads, c0 = 4 * (e % kQuads);
            const float* row = Pb + (size_t)min(tile * kRows + nn, len - 1) * r;
            if ((r & 3) == 0) {   // uniform: rows of 16-byte multiples
                st[i] = *reinterpret_cast<const v4f*>(row + min(c0, r - 4));
            } else {
#pragma unroll
                for (int t = 0; t < 4; ++t) st[i][t] = row[min(c0 + t, r - 1)];
            }
        }
    };
    auto commit = [&](int tile, uint16_t* dst) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kItems; ++i) {
            const int e = tid + i * NTHR, nn = e / kQuads, c4 = e % kQuads;
            const bool on = tile * kRows + nn < len;
            v4f v;
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] = on && 4 * c4 + t < r ? st[i][t] : 0.f;
            uint32_t lo[3], hi[3];
            split3_pair(v[0], v[1], lo);
            split3_pair(v[2], v[3], hi);
            uint16_t* at = dst + (nn / NT) * (3 * kImg) + (nn % NT) * LDP + 4 * quad_at<RB>(c4);
#pragma unroll
            for (int q = 0; q < 3; ++q) *reinterpret_cast<uint2*>(at + q * kImg) = uint2{lo[q], hi[q]};
        }
    };
    if (ntiles > 0) {
        fetch(0);
        commit(0, Ps);
        fetch(1);
    }
    __syncthreads();

    for (int tile = 0; tile < ntiles; ++tile) {
        const uint16_t* pt = Ps + ((tile & 1) * NS + sp) * (3 * kImg);
        const int n0 = (tile * NS + sp) * NT;
        if (n0 < len) {   // uniform over the wave: only the last step can leave a group without rows

        // scores S^T[n][m] for the blocks of 16 rows
        v4f s[QB][NT / 16];
#pragma unroll
        for (int nb = 0; nb < NT / 16; ++nb) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) s[qb][nb] = v4f{0.f, 0.f, 0.f, 0.f};
            const uint16_t* prow = pt + (16 * nb + i16) * LDP;
#pragma unroll
            for (int c = 0; c < FC; ++c) {
                v4u a[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) a[q] = *reinterpret_cast<const v4u*>(prow + q * kImg + 32 * c + 8 * g);
#pragma unroll
                for (int k = 0; k < 6; ++k)
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb)
                        s[qb][nb] = mfma16x16x32bf16(a[kTermA[k]], qf[qb][c][kTermB[k]], s[qb][nb]);
            }
            if constexpr (HALF) {
                uint2 a[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) a[q] = *reinterpret_cast<const uint2*>(prow + q * kImg + 32 * FC + 4 * g);
                const v4u a01 = v4u{a[0].x, a[0].y, a[1].x, a[1].y}, a02 = v4u{a[0].x, a[0].y, a[2].x, a[2].y};
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
                    s[qb][nb] = mfma16x16x32bf16(a02, qh[qb][2], s[qb][nb]);
                    s[qb][nb] = mfma16x16x32bf16(a01, qh[qb][1], s[qb][nb]);
                    s[qb][nb] = mfma16x16x32bf16(a01, qh[qb][0], s[qb][nb]);
                }
            }
        }
        // mask rows past the valid length (component t of block nb is row 16*nb + 4*g + t)
        if (n0 + NT > len) {
#pragma unroll
            for (int nb = 0; nb < NT / 16; ++nb)
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (n0 + 16 * nb + 4 * g + t >= len) {
#pragma unroll
                        for (int qb = 0; qb < QB; ++qb) s[qb][nb][t] = -INFINITY;
                    }
        }
        // online softmax per query (= per lane column), weights overwrite the scores
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            float mt = -INFINITY;
#pragma unroll
            for (int nb = 0; nb < NT / 16; ++nb)
#pragma unroll
                for (int t = 0; t < 4; ++t) mt = fmaxf(mt, s[qb][nb][t]);
            mt = wave_xor_max(mt, 16);
            mt = wave_xor_max(mt, 32);
            const float mnew = fmaxf(mrun[qb], mt);   // finite: row 0 of tile 0 is valid
            const float alpha = __builtin_amdgcn_exp2f(mrun[qb] - mnew);
            mrun[qb] = mnew;
            float lsum = 0.f;
#pragma unroll
            for (int nb = 0; nb < NT / 16; ++nb)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float w = __builtin_amdgcn_exp2f(s[qb][nb][t] - mnew);
                    s[qb][nb][t] = w;
                    lsum += w;
                }
            lrun[qb] = lrun[qb] * alpha + lsum;
#pragma unroll
            for (int ib = 0; ib < RB; ++ib) z[qb][ib] *= alpha;
        }
        // Z^T += P^T W^T, 32 rows at a time: slots 0..3 of lane group g are rows 4*g .. +3 of block 2c, slots 4..7
        // those of block 2c + 1
#pragma unroll
        for (int c = 0; c < NT / 32; ++c) {
            v4u w[QB][3];
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                uint32_t t[4][3];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    split3_pair(s[qb][2 * c + e / 2][2 * (e % 2)], s[qb][2 * c + e / 2][2 * (e % 2) + 1], t[e]);
#pragma unroll
                for (int q = 0; q < 3; ++q) w[qb][q] = v4u{t[0][q], t[1][q], t[2][q], t[3][q]};
            }
            const uint16_t* zrow = pt + (32 * c + 4 * g + (i16 >> 2)) * LDP;
#pragma unroll
            for (int ib = 0; ib < RB; ++ib) {
                v4u a[3];
                const int col = 4 * quad_at<RB>(4 * ib + (i16 & 3));
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const uint2 lo = read_transposed(zrow + q * kImg + col);
                    const uint2 hi = read_transposed(zrow + q * kImg + 16 * LDP + col);
                    a[q] = v4u{lo.x, lo.y, hi.x, hi.y};
                }
#pragma unroll
                for (int k = 0; k < 6; ++k)
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb)
                        z[qb][ib] = mfma16x16x32bf16(a[kTermA[k]], w[qb][kTermB[k]], z[qb][ib]);
            }
        }
        }
        commit(tile + 1, Ps + ((tile + 1) & 1) * (NS * 3 * kImg));
        fetch(tile + 2);
        __syncthreads();
    }

    // A value of P above 3.39e38 makes its scores NaN, and so can a product that overflows (its terms have different signs)
    // where the float product is an infinity and its weight zero.  A wave whose sums are not finite
    // walks its share again on the float instruction, P read from memory and Qt put together again.  The loop above is
    // the same instruction for instruction (72 shapes: 1.000 of the time on average, 0.86 to 1.04 by register count).
    bool finite = true;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        finite &= finite32(lrun[qb]);
#pragma unroll
        for (int ib = 0; ib < RB; ++ib)
#pragma unroll
            for (int t = 0; t < 4; ++t) finite &= finite32(z[qb][ib][t]);
    }
    if (__builtin_expect(__any(!finite), 0)) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            mrun[qb] = -INFINITY;
            lrun[qb] = 0.f;
#pragma unroll
            for (int ib = 0; ib < RB; ++ib) z[qb][ib] = v4f{0.f, 0.f, 0.f, 0.f};
        }
        auto query = [&](int qb, int ib, int t) __attribute__((always_inline)) {
            float v = 0.f;
#pragma unroll
            for (int q = 2; q >= 0; --q) {
                uint32_t word = HALF && ib == RB - 1 ? qh[qb][q][t / 2] : qf[qb][ib / 2][q][2 * (ib % 2) + t / 2];
                asm volatile("" : "+v"(word));   // or all of Qt is put together ahead of the loop, and kept
                v += t % 2 ? bf16_hi(word) : bf16_lo(word);
            }
            return v;
        };
        auto p_at = [&](int n, int c) __attribute__((always_inline)) {
            return n < len && c < r ? Pb[(size_t)n * r + c] : 0.f;
        };
#pragma unroll 1
        for (int step = 0; step < ntiles * (NT / 16); ++step) {
            const int n0 = ((step / (NT / 16)) * NS + sp) * NT + 16 * (step % (NT / 16));
            if (n0 >= len) break;   // uniform; later steps are further on
            v4f s[QB];
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) s[qb] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ib = 0; ib < RB; ++ib)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float a = p_at(n0 + i16, 16 * ib + 4 * g + t);
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb) s[qb] = mfma16x16x4(a, query(qb, ib, t), s[qb]);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                float mt = -INFINITY;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    if (n0 + 4 * g + t >= len) s[qb][t] = -INFINITY;
                    mt = fmaxf(mt, s[qb][t]);
                }
                mt = wave_xor_max(mt, 16);
                mt = wave_xor_max(mt, 32);
                const float mnew = fmaxf(mrun[qb], mt);
                const float alpha = __builtin_amdgcn_exp2f(mrun[qb] - mnew);
                mrun[qb] = mnew;
                lrun[qb] *= alpha;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    s[qb][t] = __builtin_amdgcn_exp2f(s[qb][t] - mnew);
                    lrun[qb] += s[qb][t];
                }
#pragma unroll
                for (int ib = 0; ib < RB; ++ib) z[qb][ib] *= alpha;
            }
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int ib = 0; ib < RB; ++ib) {
                    const float a = p_at(n0 + 4 * g + t, 16 * ib + i16);
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb) z[qb][ib] = mfma16x16x4(a, s[qb][t], z[qb][ib]);
                    __builtin_amdgcn_sched_barrier(0);
                }
        }
    }

    // ---- merge of the sequence shares (group 0 takes the others in order) -----------------
    if constexpr (NS > 1) {
        constexpr int kState = QB * (4 * RB + 2);   // floats per lane
        float* st = reinterpret_cast<float*>(Ps);    // [NS-1][QG waves][kState][64 lanes]
        if (sp > 0) {
            float* mine = st + ((sp - 1) * QG + wave) * (kState * 64) + lane;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                mine[(qb * (4 * RB + 2) + 0) * 64] = mrun[qb];
                mine[(qb * (4 * RB + 2) + 1) * 64] = lrun[qb];
#pragma unroll
                for (int ib = 0; ib < RB; ++ib)
#pragma unroll
                    for (int t = 0; t < 4; ++t) mine[(qb * (4 * RB + 2) + 2 + 4 * ib + t) * 64] = z[qb][ib][t];
            }
        }
        __syncthreads();
        if (sp > 0) return;
        for (int o = 0; o < NS - 1; ++o) {
            const float* other = st + (o * QG + wave) * (kState * 64) + lane;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const float mo = other[(qb * (4 * RB + 2) + 0) * 64];
                const float lo = other[(qb * (4 * RB + 2) + 1) * 64];
                const float mnew = fmaxf(mrun[qb], mo);
                // a share without rows has reference -inf and contributes nothing
                const float a0 = mrun[qb] > -INFINITY ? __builtin_amdgcn_exp2f(mrun[qb] - mnew) : 0.f;
                const float a1 = mo > -INFINITY ? __builtin_amdgcn_exp2f(mo - mnew) : 0.f;
                mrun[qb] = mnew;
                lrun[qb] = lrun[qb] * a0 + lo * a1;
#pragma unroll
                for (int ib = 0; ib < RB; ++ib)
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        z[qb][ib][t] = z[qb][ib][t] * a0 + other[(qb * (4 * RB + 2) + 2 + 4 * ib + t) * 64] * a1;
            }
        }
    }

    // ---- epilogue: O^T = V (Z / l)^T ------------------------------------------------
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        float l = lrun[qb];
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        const float inv = l > 0.f ? 1.f / l : 0.f;
#pragma unroll
        for (int ib = 0; ib < RB; ++ib) z[qb][ib] *= inv;
        const int m = m_wave + 16 * qb + i16;
        for (int cb = 0; cb < D / 16; ++cb) {
            v4f o = v4f{0.f, 0.f, 0.f, 0.f};
            const float* vrow = Vs + (16 * cb + i16) * LDV;
#pragma unroll
            for (int ib = 0; ib < RB; ++ib)
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    o = mfma16x16x4(vrow[16 * ib + 4 * g + t], z[qb][ib][t], o);
            if (m < M) *reinterpret_cast<v4f*>(O + ((size_t)b * M + m) * D + 16 * cb + 4 * g) = o;
        }
    }
}

// Literal r-token form.  One wave per candidate at a time; lane k holds token k.
template <bool BF16>
__global__ __launch_bounds__(256) void attention_tokens_kernel(
    const void* __restrict__ Qv, const float* __restrict__ S, const float* __restrict__ V, int d,
    int r, int M, float scale, int softmax, float* __restrict__ O) {
    extern __shared__ __attribute__((aligned(16))) float smem[];
    const int LDT = d + 1;
    float* T = smem;               // [r][LDT]  T[k][j] = S[k] V[j][k]
    const int b = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int e = tid; e < d * r; e += 256) {
        const int j = e / r, k = e % r;
        T[k * LDT + j] = S[(size_t)b * r + k] * V[((size_t)b * d + j) * r + k];
    }
    __syncthreads();
    const int rows_per_block = 64;
    for (int mi = wave; mi < rows_per_block; mi += 4) {
        const int m = blockIdx.x * rows_per_block + mi;
        if (m >= M) break;   // uniform over the wave
        // lane holds q[lane], q[lane+64], ... ; values are handed round with shuffles
        float qreg[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int j = lane + 64 * c;
            qreg[c] = 0.f;
            if (j < d) {
                const size_t idx = ((size_t)b * M + m) * d + j;
                qreg[c] = BF16 ? __uint_as_float((uint32_t)reinterpret_cast<const uint16_t*>(Qv)[idx] << 16)
                               : reinterpret_cast<const float*>(Qv)[idx];
            }
        }
        float sc = 0.f;
        const float* tk = T + (lane < r ? lane : 0) * LDT;
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (64 * c < d)
                for (int jj = 0; jj < 64; ++jj) sc += __shfl(qreg[c], jj) * tk[64 * c + jj];
        sc *= scale;
        float w;
        if (softmax) {
            float mx = lane < r ? sc : -INFINITY;
            for (int msk = 1; msk < 64; msk <<= 1) mx = fmaxf(mx, __shfl_xor(mx, msk));
            float ex = lane < r ? __builtin_amdgcn_exp2f((sc - mx) * kLog2e) : 0.f;
            float sum = ex;
            for (int msk = 1; msk < 64; msk <<= 1) sum += __shfl_xor(sum, msk);
            w = ex / sum;
        } else {
            w = lane < r ? sc : 0.f;
        }
        for (int j = lane; j < d; j += 64) {
            float acc = 0.f;
            for (int k = 0; k < r; ++k) acc += __shfl(w, k) * T[k * LDT + j];
            O[((size_t)b * M + m) * d + j] = acc;
        }
    }
}

}  // namespace

template <int D, int RB, int QB, int NS, int QG = 4, int NT = 64>
static hipError_t launch_seq_q(const void* Q, const float* V, const float* P,
                               const int32_t* lengths, int B, int N, int r, int M, float scale,
                               bool bf16, float* O, hipStream_t stream) {
    constexpr size_t lds = seq_lds(D, RB, NS, NT);
    dim3 grid(ceil_div(M, QG * QB * 16) * (B < 8 ? B : 8 * ceil_div(B, 8))), block(64 * QG * NS);
    auto kern = bf16 ? attention_seq_kernel<D, RB, true, QB, NS, QG, NT> : attention_seq_kernel<D, RB, false, QB, NS, QG, NT>;
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, grid, block, lds, stream, Q, V, P, lengths, B, N, r, M, scale, O);
    return hipGetLastError();
}

// A wave takes two 16-query blocks (each row of P read from LDS serves both) unless that leaves
// fewer workgroups than compute units; then one block per wave fills the GPU.  If the workgroups
// of four waves still leave the SIMDs with fewer than four waves each, the sequence is shared
// out among two or four groups of waves per workgroup (as far as the tile buffers fit LDS).
template <int D, int RB, int QB>
static hipError_t launch_seq_n(const void* Q, const float* V, const float* P,
                               const int32_t* lengths, int B, int N, int r, int M, float scale,
                               bool bf16, float* O, hipStream_t stream) {
    const long long wgs = (long long)B * ceil_div(M, 64 * QB);
    int ns = wgs >= 1024 ? 1 : (wgs >= 512 ? 2 : 4);
    // two query blocks per wave leave room for two groups only (four would hold 16 waves to 128
    // registers each, which that variant does not fit; nor does it fit 256 at d = 256, r > 48)
    constexpr int kMaxNs = QB == 1 ? 4 : ((D == 256 && RB == 4) ? 1 : 2);
    if (ns > kMaxNs) ns = kMaxNs;
    while (ns > 1 && seq_lds(D, RB, ns, 64) > 160 * 1024) ns /= 2;
    while (ns > 1 && N <= (ns / 2) * 64) ns /= 2;   // no more groups than tiles
    if constexpr (kMaxNs >= 4 && seq_lds(D, RB, 4, 64) <= 160 * 1024) {
        if (ns == 4) return launch_seq_q<D, RB, QB, 4>(Q, V, P, lengths, B, N, r, M, scale, bf16, O, stream);
    }
    if constexpr (kMaxNs >= 2 && seq_lds(D, RB, 2, 64) <= 160 * 1024) {
        if (ns == 2) return launch_seq_q<D, RB, QB, 2>(Q, V, P, lengths, B, N, r, M, scale, bf16, O, stream);
    }
    return launch_seq_q<D, RB, QB, 1>(Q, V, P, lengths, B, N, r, M, scale, bf16, O, stream);
}

// Up to 64 workgroups of 64 queries leave three compute units of four idle: sixteen queries to a workgroup then, and
// its eight waves (four where the images of eight do not fit LDS) share out the sequence in tiles of 32 rows.
// One user, N = 10000, M = 1000, d = 128, r = 21: 189 -> 85 us (with the loads two steps ahead); two users, N = 20000,
// M = 200, d = 64, r = 30: 419 -> 158; one user, N = 1024, M = 64, d = 64, r = 8: 16 -> 10.
template <int D, int RB>
static hipError_t launch_seq_t(const void* Q, const float* V, const float* P,
                               const int32_t* lengths, int B, int N, int r, int M, float scale,
                               bool bf16, float* O, hipStream_t stream) {
    constexpr int kShares = seq_lds(D, RB, 8, 32) <= 160 * 1024 ? 8 : 4;
    if ((long long)B * ceil_div(M, 64) <= 64 && N > 32 * kShares)
        return launch_seq_q<D, RB, 1, kShares, 1, 32>(Q, V, P, lengths, B, N, r, M, scale, bf16, O, stream);
    if ((long long)B * ceil_div(M, 128) < 256)
        return launch_seq_n<D, RB, 1>(Q, V, P, lengths, B, N, r, M, scale, bf16, O, stream);
    return launch_seq_n<D, RB, 2>(Q, V, P, lengths, B, N, r, M, scale, bf16, O, stream);
}

template <int D>
static hipError_t launch_seq_d(const void* Q, const float* V, const float* P,
                               const int32_t* lengths, int B, int N, int r, int M, float scale,
                               bool bf16, float* O, hipStream_t stream) {
    switch ((r + 15) / 16) {
        case 1: return launch_seq_t<D, 1>(Q, V, P, lengths, B, N, r, M, scale, bf16, O, stream);
        case 2: return launch_seq_t<D, 2>(Q, V, P, lengths, B, N, r, M, scale, bf16, O, stream);
        case 3: return launch_seq_t<D, 3>(Q, V, P, lengths, B, N, r, M, scale, bf16, O, stream);
        case 4: return launch_seq_t<D, 4>(Q, V, P, lengths, B, N, r, M, scale, bf16, O, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_attention_seq(const void* Q, const float* V, const float* P,
                                const int32_t* lengths, int B, int N, int d, int r, int M,
                                float scale, bool bf16, float* O, hipStream_t stream) {
    switch (d) {
        case 64: return launch_seq_d<64>(Q, V, P, lengths, B, N, r, M, scale, bf16, O, stream);
        case 128: return launch_seq_d<128>(Q, V, P, lengths, B, N, r, M, scale, bf16, O, stream);
        case 256: return launch_seq_d<256>(Q, V, P, lengths, B, N, r, M, scale, bf16, O, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_attention_tokens(const void* Q, const float* S, const float* V, int B, int d,
                                   int r, int M, float scale, bool softmax, bool bf16, float* O,
                                   hipStream_t stream) {
    const size_t lds = sizeof(float) * ((size_t)r * (d + 1));
    dim3 grid(ceil_div(M, 64), B), block(256);
    if (bf16) {
        auto kern = attention_tokens_kernel<true>;
        hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, grid, block, lds, stream, Q, S, V, d, r, M, scale, softmax ? 1 : 0, O);
    } else {
        auto kern = attention_tokens_kernel<false>;
        hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, grid, block, lds, stream, Q, S, V, d, r, M, scale, softmax ? 1 : 0, O);
    }
    return hipGetLastError();
}

}  // namespace solar
