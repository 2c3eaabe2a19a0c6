// One 16 x 16 tile of a product over k < K on FP64 MFMA by one wavefront, for
// the density matrices and the renormalized operators.
//
// Lane (g, i), g = lane / 16, takes row i of the first operand and column i of
// the second; step j of a block of 16 takes k = k0 + 4 g + j, so that an operand
// whose k are neighbours in memory comes in 16-byte loads.  The tiles are few
// and small (a density block of order 361: 78 tiles of 32 x 32, 23 blocks of k),
// so the loads' latency bounds them: DEPTH blocks are on their way while one is
// multiplied.  Density matrices of Heisenberg m = 2048: 32.5 -> 24.2 us (8-byte
// loads through flat addresses, one block at a time, before), the two stages of
// an m = 1024 block's operators 12.4 -> 10.1 us each.
#pragma once

#include "internal.h"

namespace dmrg {

typedef double v4d_p __attribute__((ext_vector_type(4)));
typedef double pair_p __attribute__((ext_vector_type(2), aligned(8)));

// x[j] = p[(k + j) * stride], j < 4 (CONTIG: stride 1)
template <bool CONTIG>
__device__ __forceinline__ void load_k4(double (&x)[4], gptr p, int64_t stride, int k) {
    if (CONTIG) {
        const pair_p lo = *(gptr_of<pair_p>)(p + k), hi = *(gptr_of<pair_p>)(p + k + 2);
        x[0] = lo.x;
        x[1] = lo.y;
        x[2] = hi.x;
        x[3] = hi.y;
    } else {
        gptr q = p + k * stride;
#pragma unroll
        for (int j = 0; j < 4; ++j, q += stride) x[j] = *q;
    }
}

// Accumulator value v of lane (g, i) of the result is D[4 v + g][i].  a and b: the
// lane's row and column (both inside the operands), at k = 0.
template <bool ACONTIG, bool BCONTIG>
__device__ __forceinline__ v4d_p tile_product(gptr a, int64_t sa, gptr b, int64_t sb, int K) {
    constexpr int DEPTH = 4;
    const int g4 = 4 * ((threadIdx.x & 63) >> 4);
    const int nb = K >> 4;  // whole blocks
    v4d_p acc = {0.0, 0.0, 0.0, 0.0};
    double ta[4], tb[4];  // the rest, k clamped to the operands
    const int rest = K & 15;
    if (rest) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t k = min(16 * nb + g4 + j, K - 1);
            ta[j] = a[ACONTIG ? k : k * sa];
            tb[j] = b[BCONTIG ? k : k * sb];
        }
    }
    if (nb) {
        double xa[DEPTH][4], xb[DEPTH][4];
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            const int k = 16 * min(u, nb - 1) + g4;
            load_k4<ACONTIG>(xa[u], a, sa, k);
            load_k4<BCONTIG>(xb[u], b, sb, k);
        }
        for (int n = 0; n < nb; n += DEPTH) {
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
                if (n + u < nb) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[u][j], xb[u][j], acc, 0, 0, 0);
                }
                const int k = 16 * min(n + u + DEPTH, nb - 1) + g4;
                load_k4<ACONTIG>(xa[u], a, sa, k);
                load_k4<BCONTIG>(xb[u], b, sb, k);
            }
        }
    }
    if (rest) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool in = g4 + j < rest;
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? ta[j] : 0.0, in ? tb[j] : 0.0, acc, 0, 0, 0);
        }
    }
    return acc;
}

}  // namespace dmrg
