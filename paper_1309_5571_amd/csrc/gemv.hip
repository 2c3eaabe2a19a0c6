// The tall-skinny products of dmrg_gemv_t, dmrg_gemv_t_noalloc and
// dmrg_gemv_n: s = V^T x and y = beta y + V s, V of n rows and k <= 64 columns.
//
// Both read V once and do two operations per element, so HBM bounds them from
// some 1e5 rows on, and what counts is the bytes in flight.  A thread takes two
// neighbouring rows and all columns (20 at most of V^T x): one 16-byte load per column (8-byte
// alignment is enough for it), issued back to back because the number of
// columns is a template argument (in steps of GROUP).  The columns that round k
// up to a whole group are read from the last column, whose lines are on their
// way already, and their results are not used: no branch between the loads.
//
// n = 4e6, k = 20 (640 MB): V^T x 111 + 5 us, V s 109 us (6.1 TB/s, what a
// plain read reaches); with 8-byte loads behind a branch j < k each, one in
// flight per wavefront, they took 183 + 14 and 156 us.  n = 1e6, k = 64: 95
// and 88 us from 288 and 136; n = 1e5, k = 20: 9.7 and 6.5 us from 16.3 and 7.8,
// the calls' own time.
#include <algorithm>
#include <utility>

#include "gemv.h"
#include "internal.h"

namespace dmrg {

namespace {

constexpr int GROUP = 4;
constexpr int MAX_GROUPS = GEMV_PART_COLS / GROUP;
constexpr int FINAL_THREADS = 256;
constexpr int ROWS = 2 * GEMV_THREADS;  // rows of a block at a time
// Groups of columns of one block of V^T x.  With the sums of 64 columns a
// thread has registers for four loads in flight and a CU for 12 wavefronts:
// 521 us at n = 4e6, k = 64 against 349 with four blocks of 16 columns, which
// read x four times.
constexpr int PART_GROUPS = 5;
constexpr int FILL = 1024;              // blocks that fill the chip
constexpr int MAX_BLOCKS = 1 << 20;     // grid cap of y = beta y + V s

// Rows e and e + 1 of one column; columns start at any multiple of 8 bytes.
typedef double pair_t __attribute__((ext_vector_type(2), aligned(8)));

__device__ __forceinline__ pair_t rows2(const double *p) { return *(const pair_t *)p; }

// The address in column j + 1 from that in column j, the last column's again
// after column k - 1; SURE columns are there (1 <= SURE <= k).  (All column
// addresses held at once spill the scalar registers from 20 columns on.)
template <int SURE>
__device__ __forceinline__ const double *next_column(const double *p, int j, int k, int64_t ldv) {
    return p + (j + 1 < SURE || j + 1 < k ? ldv : 0);
}

// First stage of s = V^T x: block (b, y) takes the columns from y * KB on and
// leaves its sum for column j at part[j * gridDim.x + b].
template <int G>
__global__ __launch_bounds__(GEMV_THREADS) void k_gemv_t_part(int64_t n, int k, const double *__restrict__ V,
                                                              int64_t ldv, const double *__restrict__ x,
                                                              double *__restrict__ part) {
    constexpr int KB = G * GROUP;
    const int j0 = blockIdx.y * KB;
    V += (int64_t)j0 * ldv;
    k = min(k - j0, KB);
    __shared__ double lds[GEMV_THREADS / 64 * KB];
    double acc[KB];
#pragma unroll
    for (int j = 0; j < KB; ++j) acc[j] = 0.0;
    const int64_t first = (int64_t)blockIdx.x * GEMV_THREADS + threadIdx.x;
    for (int64_t e = 2 * first; e + 1 < n; e += (int64_t)gridDim.x * ROWS) {
        const pair_t xv = rows2(x + e);
        const double *p = V + e;
#pragma unroll
        for (int j = 0; j < KB; p = next_column<1>(p, j++, k, ldv)) {
            const pair_t v = rows2(p);
            acc[j] += v.x * xv.x;
            acc[j] += v.y * xv.y;
        }
    }
    if ((n & 1) && first == 0) {  // the last row of an odd number
        const double xv = x[n - 1];
        const double *p = V + n - 1;
#pragma unroll
        for (int j = 0; j < KB; p = next_column<1>(p, j++, k, ldv)) acc[j] += *p * xv;
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < KB; ++j) {
        const double sum = wave_reduce(acc[j]);
        if (lane == 0) lds[w * KB + j] = sum;
    }
    __syncthreads();
    const int j = threadIdx.x;
    if (j < k) {
        double sum = 0.0;
#pragma unroll
        for (int q = 0; q < GEMV_THREADS / 64; ++q) sum += lds[q * KB + j];
        part[(size_t)(j0 + j) * gridDim.x + blockIdx.x] = sum;
    }
}

// Second stage: one block a column.  (One block for all columns took 14 us at
// 1024 partials of 20 columns, a chain of dependent loads.)
__global__ __launch_bounds__(FINAL_THREADS) void k_gemv_t_final(int nblk, const double *__restrict__ part,
                                                                double *__restrict__ s) {
    __shared__ double lds[FINAL_THREADS / 64];
    const double *p = part + (size_t)blockIdx.x * nblk;
    double v[GEMV_PART_BLOCKS / FINAL_THREADS];
#pragma unroll
    for (int q = 0; q < GEMV_PART_BLOCKS / FINAL_THREADS; ++q) {
        const int b = q * FINAL_THREADS + threadIdx.x;
        v[q] = b < nblk ? p[b] : 0.0;
    }
    double sum = 0.0;
#pragma unroll
    for (int q = 0; q < GEMV_PART_BLOCKS / FINAL_THREADS; ++q) sum += v[q];
    sum = wave_reduce(sum);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        double total = 0.0;
#pragma unroll
        for (int w = 0; w < FINAL_THREADS / 64; ++w) total += lds[w];
        s[blockIdx.x] = total;
    }
}

// y = beta y + V s.  The blocks take the rows from the last to the first: the
// product V^T x that comes before it in an orthogonalization has read them from
// the first to the last, and what it read last is still in the 256 MB cache.
template <int G>
__global__ __launch_bounds__(GEMV_THREADS) void k_gemv_n(int64_t n, int k, const double *__restrict__ V, int64_t ldv,
                                                         const double *__restrict__ s, double beta,
                                                         double *__restrict__ y) {
    constexpr int KB = G * GROUP, SURE = KB - GROUP + 1;  // SURE <= k <= KB
    const int64_t chunks = (n + ROWS - 1) / ROWS;
    for (int64_t c = chunks - 1 - blockIdx.x; c >= 0; c -= gridDim.x) {
        const int64_t e = c * ROWS + 2 * threadIdx.x;
        const double *p = V + e;
        if (e + 1 < n) {
            pair_t v[KB];
#pragma unroll
            for (int j = 0; j < KB; p = next_column<SURE>(p, j++, k, ldv)) v[j] = rows2(p);
            pair_t acc = {0.0, 0.0};
            if (beta != 0.0) acc = beta * rows2(y + e);
#pragma unroll
            for (int j = 0; j < KB; ++j)
                if (j < SURE || j < k) {
                    acc.x += v[j].x * s[j];
                    acc.y += v[j].y * s[j];
                }
            *(pair_t *)(y + e) = acc;
        } else if (e < n) {  // the last row of an odd number
            double acc = (beta == 0.0) ? 0.0 : beta * y[e];
            for (int j = 0; j < k; ++j) acc += p[(int64_t)j * ldv] * s[j];
            y[e] = acc;
        }
    }
}

using PartFn = void (*)(int64_t, int, const double *, int64_t, const double *, double *);
using GemvNFn = void (*)(int64_t, int, const double *, int64_t, const double *, double, double *);

template <size_t... I>
PartFn part_kernel(int g, std::index_sequence<I...>) {
    static const PartFn table[] = {k_gemv_t_part<(int)I + 1>...};
    return table[g - 1];
}

template <size_t... I>
GemvNFn n_kernel(int g, std::index_sequence<I...>) {
    static const GemvNFn table[] = {k_gemv_n<(int)I + 1>...};
    return table[g - 1];
}

}  // namespace

int gemv_t_blocks(int64_t n) { return (int)std::min<int64_t>((n + ROWS - 1) / ROWS, GEMV_PART_BLOCKS); }

dmrg_status gemv_t_launch(int64_t n, int32_t k, const double *V, int64_t ldv, const double *x, double *s,
                          double *part, hipStream_t st) {
    const int nblk = gemv_t_blocks(n);
    // At most PART_GROUPS groups a block, as even as they go, and fewer while
    // the blocks do not fill the chip (n = 1e5: 196 blocks of rows; k = 32 in
    // one part and in four: 14.4 and 9.5 us).
    const int groups = (k + GROUP - 1) / GROUP;
    int parts = (groups + PART_GROUPS - 1) / PART_GROUPS;
    while (2 * parts <= groups && nblk * 2 * parts <= FILL) parts *= 2;
    const int per = (groups + parts - 1) / parts;
    parts = (groups + per - 1) / per;
    const PartFn fn = part_kernel(per, std::make_index_sequence<PART_GROUPS>{});
    hipLaunchKernelGGL(fn, dim3(nblk, parts), dim3(GEMV_THREADS), 0, st, n, (int)k, V, ldv, x, part);
    hipLaunchKernelGGL(k_gemv_t_final, dim3(k), dim3(FINAL_THREADS), 0, st, nblk, (const double *)part, s);
    DMRG_HIP(hipGetLastError());
    return DMRG_OK;
}

dmrg_status gemv_n_launch(int64_t n, int32_t k, const double *V, int64_t ldv, const double *s, double beta, double *y,
                          hipStream_t st) {
    const int nblk = (int)std::min<int64_t>((n + ROWS - 1) / ROWS, MAX_BLOCKS);
    const GemvNFn fn = n_kernel((k + GROUP - 1) / GROUP, std::make_index_sequence<MAX_GROUPS>{});
    hipLaunchKernelGGL(fn, dim3(nblk), dim3(GEMV_THREADS), 0, st, n, (int)k, V, ldv, s, beta, y);
    DMRG_HIP(hipGetLastError());
    return DMRG_OK;
}

}  // namespace dmrg
