// Partial blocks of the contractions W = H^T Y (d x r) and Gy = Y^T Y (r x r) over a chunk of the sequence, as
// rsvd.hip writes them and the small kernels of Algorithm 1 read them: per chunk, 16 x 16 blocks in MFMA layout
// (register q of lane l is element (4*(l/16)+q, l%16)); with CPL = d/16 and CY = r/16, block s*CY + c holds
// {W[CPL*i+s][CY*j+c]}, and behind those, where the pass formed Gy, the blocks (c1 <= c2) hold {Gy[CY*i+c1][CY*j+c2]}.
#pragma once

#include "common.h"

namespace solar {

template <int CPL, int CY>
__host__ __device__ constexpr int xty_blocks() { return CPL * CY + CY * (CY + 1) / 2; }

// Adds the chunks of one user in their order: W goes to Zc, column c at Zc + c * LD; with GRAM, Gy to Gm, row u at
// Gm + u * LG.  `blocks` is what a chunk holds (with or without those of Gy).  Called by all `threads` threads; the
// loads of four chunks are in flight together.
template <int D, int R, bool GRAM, int LD, int LG, typename TG>
__device__ __forceinline__ void add_xty_partials(const float* partials, int nsplit, int blocks, int threads, float* Zc,
                                                 TG* Gm) {
    constexpr int CPL = D / 16, CY = R / 16, NW = CPL * CY, NB = GRAM ? xty_blocks<CPL, CY>() : NW;
    const v4f* src = reinterpret_cast<const v4f*>(partials);
    for (int e = threadIdx.x; e < NB * 64; e += threads) {
        v4f sum = v4f{0.f, 0.f, 0.f, 0.f};
        int s = 0;
        for (; s + 4 <= nsplit; s += 4) {
            v4f part[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) part[q] = src[(size_t)(s + q) * (blocks * 64) + e];
#pragma unroll
            for (int q = 0; q < 4; ++q) sum += part[q];
        }
        for (; s < nsplit; ++s) sum += src[(size_t)s * (blocks * 64) + e];
        const int blk = e >> 6, j = e & 15, i0 = 4 * ((e >> 4) & 3);
        if (blk < NW) {
            const int col = CY * j + blk % CY, row = blk / CY;
#pragma unroll
            for (int q = 0; q < 4; ++q) Zc[col * LD + CPL * (i0 + q) + row] = sum[q];
        } else if constexpr (GRAM) {
            int c1 = 0, rest = blk - NW;
            while (rest >= CY - c1) { rest -= CY - c1; ++c1; }
            const int v = CY * j + c1 + rest;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int u = CY * (i0 + q) + c1;
                Gm[u * LG + v] = (TG)sum[q];
                if (rest) Gm[v * LG + u] = (TG)sum[q];
            }
        }
    }
}

}  // namespace solar
