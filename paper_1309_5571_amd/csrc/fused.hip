// Output tiles of plans whose tiles all fit 16 x 16 (gfx950): FP64, and the
// FP32 phase of a mixed solve.
//
// Small sectors (Hubbard m = 2048: 421 tiles, block orders 1 to 36) leave a
// tile a chain of latencies and hardly any arithmetic: descriptor, operands,
// products, reduction, store.  So the operand loads of a two-sided segment --
// A, X and B -- are in flight at once, and its intermediate T = A X never leaves
// the registers: formed transposed, X^T A^T, it is in the operand layout of
// the second product.  The descriptors of a tile lie at a fixed stride (see
// pack_tiles in plan.cpp), so their load does not wait for the tile's record, and
// the diagonal terms are one round of loads on the wavefronts with fewer
// segments.  Hubbard m = 2048 projection, calls back to back: 12.8 us with
// the task kernel (loads of one 16-long block of a product at a time, T
// through LDS), 8.1 us here.  A tile takes 6 us of which 0.6 is descriptors, 1.3
// operands, 2 to 4 the products (two tiles per compute unit).  Six wavefronts a
// tile (168 registers) leave half of the tiles for a second round: 10.4 us.
// Starting a wavefront's second segment before the first one's products: 2 %
// slower.
#include <type_traits>

#include "internal.h"
#include "terms.h"

namespace dmrg {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int FW = 4;  // wavefronts of a tile
constexpr int LONG = 9;  // MFMA steps of a piece of a contraction (registers)

template <int PREC>
struct Ft;
template <>
struct Ft<DMRG_F64> {
    typedef double val;  // operands, stored operator blocks and intermediates
    typedef v4d acc;
    // accumulator value e of lane group g is row 4 e + g
    __device__ static int row(int g, int e) { return 4 * e + g; }
    __device__ static acc mma(val a, val b, acc c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
};
template <>
struct Ft<DMRG_F32> {
    typedef float val;
    typedef v4f acc;
    __device__ static int row(int g, int e) { return 4 * g + e; }
    __device__ static acc mma(val a, val b, acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
};

template <class T>
__device__ __forceinline__ T load_at(gptr_of<T> base, uint32_t bytes) {
    return *(gptr_of<T>)((gptr_of<char>)base + bytes);
}

// Two-sided segment: for every 16-wide column sub-tile c of the intermediate,
// T_c = A X_c (NS steps of the contraction at a time), then acc += T_c B_c^T;
// in the adjoint pass T_c = A^T X_c and acc += T_c B_c, the same blocks read
// along their other index.
// With one piece (K <= 4 NS) A is loaded once and the loads of the next
// sub-tile's X and B are issued before a sub-tile's products.
template <int PREC, bool ADJ, int NS, bool ONE>
__device__ __forceinline__ void two_sided(typename Ft<PREC>::acc &acc, const Seg &s, const Task &tk, gptr in, int i,
                                          int g) {
    typedef typename Ft<PREC>::val V;
    typedef typename Ft<PREC>::acc A4;
    const gptr_of<V> A = (gptr_of<V>)(uintptr_t)s.p, R = (gptr_of<V>)(uintptr_t)s.r;
    const gptr X = in + s.q;
    // byte offsets; contraction indices and columns are clamped to the last one
    const uint32_t row = tk.row0 + min(i, tk.m - 1), col = tk.col0 + min(i, tk.n - 1);
    const uint32_t arow = ADJ ? row : row * s.ldp, ak = (ADJ ? s.ldp : 1) * (uint32_t)sizeof(V);
    const uint32_t amax = arow * sizeof(V) + (s.K - 1) * ak, xmax = (uint32_t)(s.K - 1) * s.ldq * 8u;
    V a[NS], r[2][4];
    double x[2][NS];
    auto load_a = [&](int k0) {
        const uint32_t o = arow * sizeof(V) + (k0 + g) * ak;
#pragma unroll
        for (int j = 0; j < NS; ++j) a[j] = load_at<V>(A, min(o + j * (4 * ak), amax));
    };
    auto load_x = [&](double (&to)[NS], int c, int k0) {
        const uint32_t xc = min(16 * c + i, s.K2 - 1) * 8u, o = (uint32_t)(k0 + g) * s.ldq * 8u;
#pragma unroll
        for (int j = 0; j < NS; ++j) to[j] = load_at<double>(X, min(o + j * (4u * s.ldq * 8u), xmax) + xc);
    };
    auto load_r = [&](V (&to)[4], int c) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t k = min(16 * c + Ft<PREC>::row(g, e), s.K2 - 1);
            to[e] = load_at<V>(R, (ADJ ? k * s.ldr + col : col * s.ldr + k) * sizeof(V));
        }
    };
    auto first = [&](A4 &t, const double (&xs)[NS], int rem) {
#pragma unroll
        for (int j = 0; j < NS; ++j)
            if (4 * j < rem) {
                const bool in_k = 4 * j + g < rem;
                t = Ft<PREC>::mma(in_k ? (V)xs[j] : (V)0, in_k ? a[j] : (V)0, t);
            }
    };
    auto second = [&](const A4 &t, const V (&rs)[4], int c) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (16 * c + Ft<PREC>::row(0, e) < s.K2) {
                const bool in_k = 16 * c + Ft<PREC>::row(g, e) < s.K2;
                acc = Ft<PREC>::mma(in_k ? t[e] : (V)0, in_k ? rs[e] : (V)0, acc);
            }
    };
    const int nc = (s.K2 + 15) >> 4;
    if (ONE) {
        load_a(0);
        load_x(x[0], 0, 0);
        load_r(r[0], 0);
        for (int c = 0; c < nc; c += 2) {
            if (c + 1 < nc) {
                load_x(x[1], c + 1, 0);
                load_r(r[1], c + 1);
            }
            A4 t = {0, 0, 0, 0};
            first(t, x[0], s.K);
            second(t, r[0], c);
            if (c + 1 >= nc) break;
            if (c + 2 < nc) {
                load_x(x[0], c + 2, 0);
                load_r(r[0], c + 2);
            }
            t = A4{0, 0, 0, 0};
            first(t, x[1], s.K);
            second(t, r[1], c + 1);
        }
    } else {
        for (int c = 0; c < nc; ++c) {
            A4 t = {0, 0, 0, 0};
            load_r(r[0], c);
            for (int k0 = 0; k0 < s.K; k0 += 4 * NS) {
                load_a(k0);
                load_x(x[0], c, k0);
                first(t, x[0], s.K - k0);
            }
            second(t, r[0], c);
        }
    }
}

// One-sided segment (or the second product of a two-stage one): op(P) op(Q),
// contraction in pieces of 4 LONG, an operand from the call's input in FP64 with its
// row (column) scale.  load() requests the first piece.
template <int PREC>
struct OneSided {
    typedef typename Ft<PREC>::val V;
    static constexpr int NS = LONG;
    double x[NS];  // the operand from the call's input, else P
    V y[NS];       // the other one
    double scale;
    bool xp;       // x is P
    __device__ __forceinline__ void load(const Seg &s, const Task &tk, gptr in, const void *tmp, int i, int g, int k0) {
        const bool pin = s.pkind == OPD_IN, qin = s.qkind == OPD_IN;
        xp = pin || !qin;
        const uint64_t xs = xp ? s.p : s.q, ys = xp ? s.q : s.p;
        const int xkind = xp ? s.pkind : s.qkind, ykind = xp ? s.qkind : s.pkind;
        // row (column) of the operand, its byte offset and the bytes from one contraction index to the next
        const uint32_t pr = tk.row0 + min(i, tk.m - 1), qc = tk.col0 + min(i, tk.n - 1);
        const uint32_t pb = s.ptrans ? pr : pr * s.ldp, pk = s.ptrans ? s.ldp : 1;
        const uint32_t qb = s.qtrans ? qc * s.ldq : qc, qk = s.qtrans ? 1 : s.ldq;
        const uint32_t xb = xp ? pb : qb, xk = xp ? pk : qk, yb = xp ? qb : pb, yk = xp ? qk : pk;
        const gptr_of<V> Y = (ykind == OPD_ABS ? (gptr_of<V>)(uintptr_t)ys : (gptr_of<V>)tmp + ys);
        if (pin || qin || PREC == DMRG_F64) {
            const gptr X = xkind == OPD_IN ? in + xs : xkind == OPD_ABS ? as_global(xs) : (gptr)tmp + xs;
#pragma unroll
            for (int j = 0; j < NS; ++j) x[j] = load_at<double>(X, (xb + min(k0 + 4 * j + g, s.K - 1) * xk) * 8u);
        } else {
            const gptr_of<V> X = (xkind == OPD_ABS ? (gptr_of<V>)(uintptr_t)xs : (gptr_of<V>)tmp + xs);
#pragma unroll
            for (int j = 0; j < NS; ++j)
                x[j] = load_at<V>(X, (xb + min(k0 + 4 * j + g, s.K - 1) * xk) * (uint32_t)sizeof(V));
        }
#pragma unroll
        for (int j = 0; j < NS; ++j)
            y[j] = load_at<V>(Y, (yb + min(k0 + 4 * j + g, s.K - 1) * yk) * (uint32_t)sizeof(V));
        scale = 1.0;
        if (k0 == 0 && pin && s.pscale) scale = as_global(s.pscale)[pr];
        if (k0 == 0 && qin && s.qscale) scale = as_global(s.qscale)[qc];
    }
    __device__ __forceinline__ void piece(typename Ft<PREC>::acc &acc, int rem, int g) {
#pragma unroll
        for (int j = 0; j < NS; ++j)
            if (4 * j < rem) {
                const bool in_k = 4 * j + g < rem;
                const V a = in_k ? (V)(x[j] * scale) : (V)0, b = in_k ? y[j] : (V)0;
                acc = xp ? Ft<PREC>::mma(a, b, acc) : Ft<PREC>::mma(b, a, acc);
            }
    }
    __device__ __forceinline__ void finish(typename Ft<PREC>::acc &acc, const Seg &s, const Task &tk, gptr in,
                                           const void *tmp, int i, int g) {
        piece(acc, s.K, g);
        for (int k0 = 4 * NS; k0 < s.K; k0 += 4 * NS) {
            const double keep = scale;
            load(s, tk, in, tmp, i, g, k0);
            scale = keep;
            typename Ft<PREC>::acc next = {0, 0, 0, 0};  // (a sum of its own: a shorter chain of roundings)
            piece(next, s.K - k0, g);
            acc += next;
        }
    }
};

// The first n diagonal terms (at most DIAG_AHEAD) of two output elements, the
// descriptors in a register, word by word over the lanes (10 words each): all
// slices are requested before the first is used.
constexpr int DIAG_AHEAD = 6;
static_assert(sizeof(DiagTerm) == 40, "read word by word");
__device__ __forceinline__ void diag_ahead(double (&v)[2], uint32_t dw, int n, const double *__restrict__ coef,
                                           const double (&x)[2], const int64_t (&rr)[2], const int64_t (&cc)[2]) {
    auto word = [&](int k) { return (uint32_t)__builtin_amdgcn_readlane(dw, k); };
    auto pair = [&](int k) { return (uint64_t)word(k + 1) << 32 | word(k); };
    double l[DIAG_AHEAD][2], r[DIAG_AHEAD][2], c[DIAG_AHEAD];
#pragma unroll
    for (int d = 0; d < DIAG_AHEAD; ++d) {
        l[d][0] = l[d][1] = r[d][0] = r[d][1] = 1.0;
        c[d] = 0.0;
        if (d < n) {
            const gptr vl = as_global(pair(10 * d)), vr = as_global(pair(10 * d + 2));
            c[d] = coef[word(10 * d + 4)];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                if (vl) l[d][q] = vl[rr[q] * (int)word(10 * d + 6)];
                if (vr) r[d][q] = vr[cc[q] * (int)word(10 * d + 7)];
            }
        }
    }
#pragma unroll
    for (int d = 0; d < DIAG_AHEAD; ++d)
        if (d < n) {
            const double w = c[d] * __longlong_as_double((long long)pair(10 * d + 8));
#pragma unroll
            for (int q = 0; q < 2; ++q) v[q] += w * x[q] * l[d][q] * r[d][q];
        }
}

struct GradArgs {  // the coefficient gradient's other vector and its partials
    const double *xg;
    double *partials;
};

// The tile's product sums: segment w, w + FW, ... of the list on wavefront w, the
// wavefronts' sums added in order.  stride, dstride: distance of consecutive tiles'
// descriptors, 0 if not packed.  ADJ: a tile of the adjoint; with GRAD also the
// coefficient gradient's share <grad.xg, segment product> of every segment and diagonal
// term (out, and with it coef, may be null then).  Hubbard m = 2048, calls back to
// back, us for the adjoint / the gradient / both in one pass: 8.9 / 14.4 / 15.0 against
// 25.2 / 29.2 / 32.1 on 32 x 32 tiles (two launches; contractions below 16 value by
// value) and 19.8 / 23.1 / 43.1 on the task kernel.
template <int PREC, bool ADJ, bool GRAD>
__global__ __launch_bounds__(64 * FW) __attribute__((amdgpu_waves_per_eu(2))) void k_fused(
    const Task *__restrict__ tasks, const Seg *__restrict__ segs, const DiagTerm *__restrict__ diags, int stride,
    int dstride, const double *__restrict__ in, const double *__restrict__ coef, const int32_t *__restrict__ mask,
    const void *__restrict__ tmp, double *__restrict__ out, const double *__restrict__ dfold,
    std::conditional_t<GRAD, GradArgs, RayArgs> extra) {
    RayArgs ray{};
    GradArgs grad{};
    if constexpr (GRAD)
        grad = extra;
    else
        ray = extra;
    typedef typename Ft<PREC>::acc A4;
    __shared__ double red[FW][16][17];
    __shared__ double wtile[256];  // first the diagonal terms' sums, then the output values
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int i = lane & 15, g = lane >> 4;
    // the packed descriptors of this wavefront's first two segments and of the diagonal terms
    Seg s{}, next{};
    uint32_t dw = 0;
    if (stride) {
        s = segs[(int)blockIdx.x * stride + min(wave, stride - 1)];
        next = segs[(int)blockIdx.x * stride + min(wave + FW, stride - 1)];
    }
    if (dstride) dw = ((gptr_of<uint32_t>)(diags + (int64_t)blockIdx.x * dstride))[min(lane, 10 * dstride - 1)];
    const Task tk = tasks[blockIdx.x];
    if (mask && !mask[tk.member]) return;
    const int cnt = tk.m * tk.n;
    const int nseg = tk.seg_end - tk.seg_begin, ndiag = tk.diag_end - tk.diag_begin;
    // epilogue inputs of this thread's element, requested before the products
    auto offset = [&](int el) { return (int64_t)(tk.row0 + el / tk.n) * tk.ldc + tk.col0 + el % tk.n; };
    double pre_x = 0.0, pre_d = 0.0;
    if (dfold) {
        const int64_t o = offset(min((int)threadIdx.x, cnt - 1));
        pre_x = in[tk.x_off + o];
        pre_d = dfold[tk.c_off + o];
    }
    // xg at this lane's elements of a product
    double gx[4];
    bool inside[4];
    if (GRAD) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = Ft<PREC>::row(g, v);
            inside[v] = r < tk.m && i < tk.n;
            gx[v] = grad.xg[tk.c_off + (int64_t)(tk.row0 + min(r, tk.m - 1)) * tk.ldc + tk.col0 + min(i, tk.n - 1)];
        }
    }
    double tot[4] = {0.0, 0.0, 0.0, 0.0};
    if (!stride && nseg > 0) {  // (a tile may have no segment, and a plan no descriptor at all)
        s = segs[tk.seg_begin + min(wave, nseg - 1)];
        next = segs[tk.seg_begin + min(wave + FW, nseg - 1)];
    }
    for (int si = wave; si < nseg; si += FW) {
        const double c = GRAD && !out ? 0.0 : (s.coef >= 0 ? coef[s.coef] : 1.0) * s.w;
        double part = 0.0;
        auto add = [&](int v, double x) {
            tot[v] += c * x;
            // (outside the tile the product holds duplicated rows and columns, not zeros)
            if (GRAD && inside[v]) part += gx[v] * x;
        };
        A4 acc = {0, 0, 0, 0};
        if (s.fused == 2) {  // copy segment
            const gptr X = (gptr)in + s.q, vl = as_global(s.pscale), vr = as_global(s.qscale);
            const int64_t col = tk.col0 + min(i, tk.n - 1);
            const double sc = vr ? vr[col] : 1.0;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t row = tk.row0 + min(Ft<PREC>::row(g, v), tk.m - 1);
                add(v, X[row * s.ldq + col] * (vl ? vl[row] : 1.0) * sc);
            }
        } else if (s.fused) {
            if (s.K <= 16)
                two_sided<PREC, ADJ, 4, true>(acc, s, tk, (gptr)in, i, g);
            else if (s.K <= 4 * LONG)
                two_sided<PREC, ADJ, LONG, true>(acc, s, tk, (gptr)in, i, g);
            else
                two_sided<PREC, ADJ, LONG, false>(acc, s, tk, (gptr)in, i, g);
#pragma unroll
            for (int v = 0; v < 4; ++v) add(v, (double)acc[v]);
        } else {
            OneSided<PREC> one;
            one.load(s, tk, (gptr)in, tmp, i, g, 0);
            one.finish(acc, s, tk, (gptr)in, tmp, i, g);
#pragma unroll
            for (int v = 0; v < 4; ++v) add(v, (double)acc[v]);
        }
        if (GRAD) {
            part = group_sum<64>(part) * s.w;
            if (lane == 0) grad.partials[tk.part0 + si] = part;
        }
        s = next;
        next = segs[tk.seg_begin + min(si + 2 * FW, nseg - 1)];
    }
    if (GRAD) {
        // diagonal terms: <xg, d v_l v_r in> over the tile, one wavefront per term
        for (int d = tk.diag_begin + wave; d < tk.diag_end; d += FW) {
            double part = 0.0;
            for (int e = lane; e < cnt; e += 64) {
                const int64_t rr = tk.row0 + e / tk.n, cc = tk.col0 + e % tk.n, o = rr * tk.ldc + cc;
                part += diag_sum(diags, d, d + 1, nullptr, in[tk.x_off + o], rr, cc) * grad.xg[tk.c_off + o];
            }
            part = group_sum<64>(part);
            if (lane == 0) grad.partials[tk.part0 + nseg + (d - tk.diag_begin)] = part;
        }
        if (!out) return;
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave][Ft<PREC>::row(g, v)][i] = tot[v];
    if (!dfold && ndiag && wave >= FW - 2) {  // two elements a lane on the last two wavefronts (fewer segments)
        const int e0 = 128 * (wave - (FW - 2)) + lane;
        double x[2], v[2] = {0.0, 0.0};
        int64_t r2[2], c2[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int el = min(e0 + 64 * q, cnt - 1);
            r2[q] = tk.row0 + el / tk.n;
            c2[q] = tk.col0 + el % tk.n;
            x[q] = in[tk.x_off + r2[q] * tk.ldc + c2[q]];
        }
        const int ahead = dstride ? min(ndiag, DIAG_AHEAD) : 0;
        diag_ahead(v, dw, ahead, coef, x, r2, c2);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (ndiag > ahead) v[q] += diag_sum(diags, tk.diag_begin + ahead, tk.diag_end, coef, x[q], r2[q], c2[q]);
            wtile[e0 + 64 * q] = v[q];
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < cnt) {
        const int e = rare((int)threadIdx.x), r = e / tk.n, cl = e % tk.n;
        double val = 0.0;
#pragma unroll
        for (int v = 0; v < FW; ++v) val += red[v][r][cl];
        if (dfold)
            val += pre_d * pre_x;
        else if (ndiag)
            val += wtile[e];
        out[tk.c_off + offset(e)] = val;
        if (ray.V) wtile[e] = val;
    }
    if (ray.V) {
        // the tile's share of [V(:, :i-1), x]^T y, columns w, w + FW, ... on wavefront w
        __syncthreads();
        double wv[4];
        int64_t off[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int q = min(lane + 64 * k, cnt - 1);
            off[k] = tk.c_off + (int64_t)(tk.row0 + q / tk.n) * tk.ldc + tk.col0 + q % tk.n;
            wv[k] = lane + 64 * k < cnt ? wtile[q] : 0.0;
        }
        for (int j = wave; j < ray.i; j += FW) {
            const gptr Vj = (gptr)((j == ray.i - 1) ? in : ray.V + (int64_t)j * ray.n);
            double dot = 0.0;
#pragma unroll
            for (int k = 0; k < 4; ++k) dot += Vj[off[k]] * wv[k];
            dot = group_sum<64>(dot);
            if (lane == 0) ray.part[j * ray.ld + tk.rslot] = dot;
        }
    }
}

dmrg_status launch_fused(const PassSet &ps, int prec, bool adjoint, const double *coef, const double *in,
                         const void *tmp, double *out, hipStream_t s, const int32_t *mask, const double *dfold,
                         const RayArgs *ray, const double *xg, double *partials) {
    const Lists &l = ps.stageB;
    if (l.ntask) {
        auto go = [&](auto kernel, auto extra) {
            hipLaunchKernelGGL(kernel, dim3(l.ntask), dim3(64 * FW), 0, s, l.tasks, (const Seg *)ps.segs,
                               (const DiagTerm *)ps.diags, l.stride, l.dstride, in, coef, mask, tmp, out, dfold, extra);
        };
        const RayArgs ra = ray ? *ray : RayArgs{};
        if (prec == DMRG_F32)
            go(k_fused<DMRG_F32, false, false>, ra);
        else if (partials)
            go(k_fused<DMRG_F64, true, true>, GradArgs{xg, partials});
        else if (adjoint)
            go(k_fused<DMRG_F64, true, false>, ra);
        else
            go(k_fused<DMRG_F64, false, false>, ra);
    }
    DMRG_HIP(hipGetLastError());
    return DMRG_OK;
}

}  // namespace dmrg
