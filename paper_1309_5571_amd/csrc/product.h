// One 32 x 32 tile of a product over k < K on FP64 MFMA by one workgroup of four
// wavefronts, a 16 x 16 quarter each, for the density matrices and the
// renormalized operators.
//
// Both operands go through LDS, 32 k at a time: two wavefronts use each row, and
// what bounds the kernels is the first-level cache's lines per load.  (Each
// wavefront loading its own operands in the layout of the matrix instruction, 16
// rows by 32 bytes, took 32.5 us for the density matrices of Heisenberg m = 2048,
// with those loads issued four blocks ahead 36.)  Here a load takes whole lines,
// 16 bytes a lane along whichever index is contiguous, and two panels are on
// their way while one is multiplied: 17.1 us.  The products are summed in the
// order of k.
#pragma once

#include "internal.h"

namespace dmrg {

typedef double v4d_p __attribute__((ext_vector_type(4)));
typedef double pair_p __attribute__((ext_vector_type(2), aligned(8)));

constexpr int PANEL = 32;                // rows (or columns) of a tile, and k of a panel
constexpr int PANEL_LD[2] = {40, 36};    // LDS strides, [k][row] and [row][k]: no bank more than twice a read
constexpr int PANEL_SIZE = PANEL * 40;
constexpr int PANELS_LDS = 4 * PANEL_SIZE;  // doubles: two operands, two buffers

// Element (row r, k) of an operand at p[r * s + k] (CONTIG) or p[k * s + r], rows
// rows from p on; a row past them is the last one, k past K is zero.
struct Operand {
    gptr p;
    int64_t s;
    int rows;
};

// This thread's part of the panel from k0 on: the four entries along the
// contiguous index are o = 2 (t % 16), o + 1 of the lines t / 16 and t / 16 + 16.
template <bool CONTIG>
__device__ __forceinline__ void panel_load(double (&x)[4], const Operand &m, int K, int k0) {
    const int o = 2 * (threadIdx.x & 15), line = threadIdx.x >> 4;
    if (k0 + PANEL <= K && (CONTIG || m.rows >= PANEL)) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int l = line + 16 * h;
            const pair_p v = *(gptr_of<pair_p>)(CONTIG ? m.p + min(l, m.rows - 1) * m.s + (k0 + o)
                                                       : m.p + (k0 + l) * m.s + o);
            x[2 * h] = v.x;
            x[2 * h + 1] = v.y;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int l = line + 16 * (e >> 1), c = o + (e & 1);
            const int r = min(CONTIG ? l : c, m.rows - 1), k = k0 + (CONTIG ? c : l), kc = min(k, K - 1);
            const double v = m.p[CONTIG ? r * m.s + kc : kc * m.s + r];
            x[e] = k < K ? v : 0.0;
        }
    }
}

template <bool CONTIG>
__device__ __forceinline__ void panel_store(const double (&x)[4], double *lds) {
    double *d = lds + (threadIdx.x >> 4) * PANEL_LD[CONTIG] + 2 * (threadIdx.x & 15);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        d[16 * h * PANEL_LD[CONTIG]] = x[2 * h];
        d[16 * h * PANEL_LD[CONTIG] + 1] = x[2 * h + 1];
    }
}

// Accumulator value v of lane (g, i), g = lane / 16, of the result is D[4 v +
// g][i] of the quarter (wave / 2, wave % 2).  All 256 threads call it;
// lds: PANELS_LDS doubles.
template <bool ACONTIG, bool BCONTIG>
__device__ __forceinline__ v4d_p tile_product(const Operand a, const Operand b, int K, double *lds) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = lane & 15, g = lane >> 4;
    const int ra = 16 * (wave >> 1) + i, rb = 16 * (wave & 1) + i;
    constexpr int LA = PANEL_LD[ACONTIG], LB = PANEL_LD[BCONTIG];
    const int fa = ACONTIG ? ra * LA + g : g * LA + ra, fb = BCONTIG ? rb * LB + g : g * LB + rb;
    double *la = lds, *lb = lds + 2 * PANEL_SIZE;
    v4d_p acc = {0.0, 0.0, 0.0, 0.0};
    if (K < 1) return acc;
    double xa[2][4], xb[2][4];
    auto fetch = [&](int h, int k0) {
        if (k0 >= K) return;
        panel_load<ACONTIG>(xa[h], a, K, k0);
        panel_load<BCONTIG>(xb[h], b, K, k0);
    };
    auto store = [&](int h) {
        panel_store<ACONTIG>(xa[h], la + h * PANEL_SIZE);
        panel_store<BCONTIG>(xb[h], lb + h * PANEL_SIZE);
    };
    fetch(0, 0);
    fetch(1, PANEL);
    store(0);
    __syncthreads();
    for (int k0 = 0; k0 < K; k0 += 2 * PANEL) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int kp = k0 + h * PANEL;
            if (kp >= K) break;
            fetch(h, kp + 2 * PANEL);
#pragma unroll
            for (int s = 0; s < PANEL / 4; ++s)
                if (kp + 4 * s < K)
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(la[h * PANEL_SIZE + fa + 4 * s * (ACONTIG ? 1 : LA)],
                                                               lb[h * PANEL_SIZE + fb + 4 * s * (BCONTIG ? 1 : LB)],
                                                               acc, 0, 0, 0);
            if (kp + PANEL < K) {
                store(h ^ 1);  // the next panel; this one's buffer is read up to the barrier
                __syncthreads();
            }
        }
    }
    return acc;
}

}  // namespace dmrg
