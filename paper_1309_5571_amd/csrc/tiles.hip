// FP64 projection passes over 32 x 32 and 64 x 64 output tiles (gfx950).
//
// Every output sub-matrix of a pass is the sum of its segments c P Q (see
// Seg).  A tile's contraction is the concatenation of its segments'
// contractions, cut into items of 16 (four MFMA steps of v_mfma_f64_16x16x4).
//
//   k_tiles32  one workgroup per 32 x 32 tile, the items dealt to its
//              wavefronts in equal contiguous runs (Split, made with the
//              plan): a single superblock has fewer tiles than the chip has
//              compute units, so a tile's contraction is what can be spread.
//              Operands go from memory to the MFMA registers, two items ahead.
//   k_tiles64  one workgroup of four wavefronts per 64 x 64 tile, a quarter
//              each, the operands shared through LDS: half the operand
//              traffic per product, for plans with tiles enough to fill the
//              chip.
//
// What bounds them.  At m = 1024 (Heisenberg, 172 output tiles of 720
// contraction indices, 328 intermediates) a pass is a chain of cold misses:
// descriptors 1 us, operands 1.5 us, then 2 us (stage A) and 5 us (B) of
// matrix instructions per compute unit.  Projection 37.9 us with the
// 32-long items of the task kernel (no load ahead of its use; generic-pointer
// loads, which can only be waited for all together), 25.3 us with k_tiles32; at
// m = 2048 147 us -> 95 us.  For 64 members of m = 256 .. 2048 the matrix
// instructions take 291 us: 1596 us with the task kernel, 950 us
// with k_tiles32, 535 us (35 TFLOP/s) with k_tiles64.  Vector instructions do
// not overlap the FP64 matrix instructions of their SIMD, so both keep what
// is not a load or a product out of the item loop.
#include "internal.h"
#include "terms.h"

namespace dmrg {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int KI = 16;  // contraction length of one item: four MFMA steps of 4

// What an item's consumer needs besides its operands (uniform in the wavefront).
struct Item {
    int si, k0;  // segment, first contraction index of the window
    int skip;    // window entries before the item (a segment's last 16 indices, part of them done before)
    int flags;
};
enum : int {
    IT_PU = 1, IT_QU = 2,  // the operands' contraction is contiguous
    IT_SLOW = 4,           // nothing was fetched: see slow_item
    IT_LAST = 8            // last item of its segment, or of the run
};

__device__ __forceinline__ gptr operand(gptr in, gptr tmp, uint64_t a, int32_t kind) {
    return kind == OPD_ABS ? as_global(a) : (kind == OPD_IN ? in : tmp) + a;
}

// ------------------------------------------------------------------ 32 x 32 tiles, the contraction split

// Lane l = (g = l / 16, i = l % 16) works on rows (columns) 2 i + t of the
// tile in sub-tile t, and at MFMA step j of an item on entry kofs(g, j) of its
// window of 16 contraction indices.  Both are so that 16-byte loads carry two
// useful values whichever way an operand lies in memory: two steps (j, j + 1)
// of one row where the contraction is contiguous, both sub-tiles of one step
// where the rows are.  An item is eight such loads, always (so that the number
// in flight is known); the window of a segment's last item is its last 16
// indices, with those before the item zeroed.
__device__ __forceinline__ int kofs(int g, int j) { return 8 * (j >> 1) + 2 * g + (j & 1); }
__device__ __forceinline__ int sub(int t, int i) { return 2 * i + t; }

typedef double v2d __attribute__((ext_vector_type(2)));
typedef double v2d_mem __attribute__((ext_vector_type(2), aligned(8)));
typedef const __attribute__((address_space(1))) v2d_mem *gptr2;

// One operand of an item, as loaded: value h = 4 t + j (contiguous contraction)
// or 2 j + t is step j of sub-tile t, values 2 q and 2 q + 1 in x[q].
struct Half {
    v2d x[4];
    template <bool UNIT>
    __device__ __forceinline__ double get(int t, int j) const {
        return UNIT ? x[2 * t + (j >> 1)][j & 1] : x[j][t];
    }
    // the window's first `skip` entries count as zero
    __device__ __forceinline__ void cut(bool unit, int g, int skip) {
#pragma unroll
        for (int h = 0; h < 8; ++h)
            x[h >> 1][h & 1] = (unit ? kofs(g, h & 3) : kofs(g, h >> 1)) >= skip ? x[h >> 1][h & 1] : 0.0;
    }
    // not contiguous, odd tile: the last row's pair was read one to the left
    __device__ __forceinline__ void unswap(bool swap) {
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j][0] = swap ? x[j][1] : x[j][0];
    }
};
struct Frag {
    Half p, q;
};

typedef const __attribute__((address_space(1))) char *gbytes;

// One operand of a segment as a wavefront reads it.  Everything but the two
// offsets is uniform, and all in bytes: an item costs a handful of scalar
// additions besides its loads (with addresses computed from indices, the
// instructions between the products cost as much as the products).
struct Side {
    gbytes b;         // the tile's first row at the window's first contraction index
    int64_t d1, d2;   // loads at b, b + d1 (offset o0) and b + d2, b + d2 + d1 (offset o1)
    int64_t ks;       // from one contraction index to the next
    uint32_t o0, o1;  // this lane's offsets
};

// Odd tiles: lane i's pair would end one past the tile's last row.
__device__ __forceinline__ bool pair_swaps(int n, int i) { return min(2 * i, n - 1) + 1 >= n; }

__device__ __forceinline__ Side side_of(gptr a, bool unit, int64_t ld, int row0, int n, int i, int g) {
    Side s;
    const int r0 = min(2 * i, n - 1), r1 = min(2 * i + 1, n - 1);
    s.b = (gbytes)(a + (unit ? row0 * ld : row0));
    s.ks = unit ? 8 : ld * 8;
    s.d1 = unit ? 64 : ld * 8;  // load q's contraction index: 8 (q & 1), or kofs(0, q)
    s.d2 = unit ? 0 : ld * 64;
    s.o0 = (uint32_t)((unit ? r0 * ld + 2 * g : 2 * g * ld + r0 - (pair_swaps(n, i) ? 1 : 0)) * 8);
    s.o1 = unit ? (uint32_t)((r1 * ld + 2 * g) * 8) : s.o0;
    return s;
}

__device__ __forceinline__ v2d load_pair(gbytes base, uint32_t o) { return *(gptr2)(base + o); }

__device__ __forceinline__ void load_half(Half &h, const Side &s) {
    const gbytes b2 = s.b + s.d2;
    h.x[0] = load_pair(s.b, s.o0);
    h.x[1] = load_pair(s.b + s.d1, s.o0);
    h.x[2] = load_pair(b2, s.o1);
    h.x[3] = load_pair(b2 + s.d1, s.o1);
}

// The item's 16 MFMA steps.
template <bool PU, bool QU>
__device__ __forceinline__ void products(v4d (&acc)[2][2], const Frag &f) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(f.p.get<PU>(a, j), f.q.get<QU>(b, j), acc[a][b], 0, 0, 0);
}

// A run's segment descriptors, staged by its wavefront: 2 x SEG_HALF of them,
// the half behind the walk refilled as it moves on.  A descriptor read from
// memory where a segment begins costs the run several cold misses in a row
// (0.8 us each).
constexpr int SEG_HALF = 8;
constexpr int SEG_WORDS = sizeof(Seg) / 8;
static_assert(sizeof(Seg) % 8 == 0, "descriptors are staged in 8-byte words");
struct SegWindow {
    uint64_t w[2 * SEG_HALF * SEG_WORDS];
};

__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ uint32_t uni(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint64_t uni(uint64_t v) {
    return (uint64_t)uni((uint32_t)(v >> 32)) << 32 | uni((uint32_t)v);
}

// Segments whose items are not fetched ahead: contractions shorter than a
// window, single rows or columns where pairs are needed, rows too long for 32-bit
// offsets, and copies.
__device__ __forceinline__ bool slow_seg(int fused, int K, int ptrans, int qtrans, int ldp, int ldq, int m, int n) {
    return fused == 2 || K < KI || (ptrans && m == 1) || (!qtrans && n == 1) || ldp >= (1 << 23) || ldq >= (1 << 23);
}

// Column of sub-tile b of NB, lane i.
template <int NB>
__device__ __forceinline__ int col_of(int b, int i) { return NB * i + b; }

// Such an item, value by value; a copy leaves X in the accumulator.
template <int NB>
__device__ __forceinline__ void slow_item(v4d (&acc)[2][NB], const Seg &s, gptr in, gptr tmp, int row0, int col0, int m,
                                          int n, int i, int g, int k0, int skip) {
    i = rare(i);
    g = rare(g);
    if (s.fused == 2) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const gptr x = in + s.q + (row0 + min(sub(a, 4 * e + g), m - 1)) * (int64_t)s.ldq + col0;
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[a][b][e] = x[min(col_of<NB>(b, i), n - 1)];
            }
        return;
    }
    const gptr P = operand(in, tmp, s.p, s.pkind), Q = operand(in, tmp, s.q, s.qkind);
    const int64_t pr = s.ptrans ? 1 : s.ldp, pk = s.ptrans ? s.ldp : 1, qc = s.qtrans ? s.ldq : 1,
                  qk = s.qtrans ? 1 : s.ldq;
#pragma unroll 1
    for (int j = 0; j < 4; ++j) {
        const int e = kofs(g, j);
        const bool on = e >= skip && k0 + e >= 0 && k0 + e < s.K;
        const int64_t k = min(max(k0 + e, 0), s.K - 1);
        double p[2], q[NB];
#pragma unroll
        for (int a = 0; a < 2; ++a) p[a] = P[(row0 + min(sub(a, i), m - 1)) * pr + k * pk];
#pragma unroll
        for (int b = 0; b < NB; ++b) q[b] = Q[(col0 + min(col_of<NB>(b, i), n - 1)) * qc + k * qk];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < NB; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(on ? p[a] : 0.0, on ? q[b] : 0.0, acc[a][b], 0, 0, 0);
    }
}

// Row and column scales (diagonal factors) of a finished segment product.
template <int NB>
__device__ __forceinline__ void scale_rows(v4d (&acc)[2][NB], gptr ps, gptr qs, int row0, int col0, int m, int n, int i,
                                           int g) {
    if (ps) {
        g = rare(g);
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double v = ps[row0 + min(sub(a, 4 * e + g), m - 1)];
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[a][b][e] *= v;
            }
    }
    if (qs) {
        i = rare(i);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const double v = qs[col0 + min(col_of<NB>(b, i), n - 1)];
            acc[0][b] *= v;
            acc[1][b] *= v;
        }
    }
}

// The fields of a staged descriptor that an operand walk needs, made uniform.
struct SegHead {
    int K, ldp, ldq;
    bool ptrans, qtrans, slow;
    gptr p, q;
};
__device__ __forceinline__ SegHead head_of(const Seg &s, gptr in, gptr tmp, int m, int n) {
    SegHead h;
    const int fused = uni(s.fused);
    h.ldp = uni(s.ldp);
    h.ldq = uni(s.ldq);
    h.ptrans = uni(s.ptrans);
    h.qtrans = uni(s.qtrans);
    h.slow = slow_seg(fused, uni(s.K), h.ptrans, h.qtrans, h.ldp, h.ldq, m, n);
    h.K = fused == 2 ? KI : uni(s.K);
    h.p = operand(in, tmp, uni(s.p), uni(s.pkind));
    h.q = operand(in, tmp, uni(s.q), uni(s.qkind));
    return h;
}
__device__ __forceinline__ double uni(double v) {
    return __longlong_as_double((long long)uni((uint64_t)__double_as_longlong(v)));
}

// One run's walk over its items: fetch() issues the loads of the next item.
struct Walk {
    const Seg *segs;
    SegWindow *win;
    gptr in, tmp, coef;
    int row0, col0, m, n;
    int i, g, lane;
    int first, end;  // segments of the run's tile from the run's first on
    double cw;       // lane s: the coefficient of window slot s
    // current segment
    int si, kleft, k0, left, skip, flags;
    Side P, Q;

    __device__ __forceinline__ int slot(int s) const { return (s - first) & (2 * SEG_HALF - 1); }
    __device__ __forceinline__ const Seg &staged(int s) const {
        return *reinterpret_cast<const Seg *>(win->w + slot(s) * SEG_WORDS);
    }
    // coefficient * constant of a segment
    __device__ __forceinline__ double scale_of(int s) const {
        const double w = uni(staged(s).w);
        return coef ? readlane_f64(cw, slot(s)) * w : w;
    }
    __device__ __forceinline__ void stage(int s0) {
        const uint64_t *src = reinterpret_cast<const uint64_t *>(segs);
        uint64_t v[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int x = min(rare(lane) + 64 * q, SEG_HALF * SEG_WORDS - 1);
            const int s = min(s0 + x / SEG_WORDS, end - 1);
            v[q] = src[(int64_t)s * SEG_WORDS + x % SEG_WORDS];
        }
        const int to = slot(s0) * SEG_WORDS;
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (lane + 64 * q < SEG_HALF * SEG_WORDS) win->w[to + lane + 64 * q] = v[q];
        wave_lds_order();
        if (coef) {
            const double c = coef[staged(s0 + (rare(lane) & (SEG_HALF - 1))).coef];
            cw = (lane & SEG_HALF) == (slot(s0) & SEG_HALF) ? c : cw;
        }
    }
    __device__ __forceinline__ void open(int s_, int kb) {
        si = s_;
        if (((si - first) & (SEG_HALF - 1)) == 0) stage(si);
        const SegHead h = head_of(staged(si), in, tmp, m, n);
        flags = (h.ptrans ? 0 : IT_PU) | (h.qtrans ? IT_QU : 0) | (h.slow ? IT_SLOW : 0);
        k0 = kb * KI;
        kleft = h.K - k0;
        // a slow segment's loads go to a descriptor: valid memory, never used
        const gptr none = (gptr)segs;
        const bool sl = h.slow;
        P = side_of(sl ? none : h.p, !h.ptrans, sl ? 0 : h.ldp, sl ? 0 : row0, sl ? 2 : m, sl ? 0 : i, sl ? 0 : g);
        Q = side_of(sl ? none : h.q, h.qtrans, sl ? 0 : h.ldq, sl ? 0 : col0, sl ? 2 : n, sl ? 0 : i, sl ? 0 : g);
        if (sl) P.ks = Q.ks = 0;
        P.b += k0 * P.ks;
        Q.b += k0 * Q.ks;
        window();
    }
    // the current item's window: its 16 indices, or the segment's last 16
    __device__ __forceinline__ void window() {
        skip = 0;
        if (kleft < KI) {
            skip = KI - kleft;
            P.b -= skip * P.ks;
            Q.b -= skip * Q.ks;
        }
    }
    __device__ __forceinline__ void fetch(Frag &f, Item &it) {
        load_half(f.p, P);
        load_half(f.q, Q);
        it.si = si;
        it.k0 = k0 - skip;
        it.skip = skip;
        it.flags = flags | (kleft <= KI || left <= 1 ? IT_LAST : 0);
        if (left > 1) {  // past the run's end the last item is fetched again, and never used
            --left;
            kleft -= KI;
            if (kleft <= 0) {
                open(si + 1, 0);
            } else {
                k0 += KI;
                P.b += KI * P.ks;
                Q.b += KI * Q.ks;
                window();
            }
        }
    }
};

// Wavefronts (runs) of a 32 x 32 tile: an output tile's contraction is several
// times that of an intermediate, of which there are more.
template <int MODE>
constexpr int waves_of() { return MODE == 0 ? TWA : TWB; }

constexpr int RED_LD = 34;  // even: a lane's two columns are one 16-byte access
template <int MODE>
constexpr size_t tiles32_lds() {
    return (size_t)(waves_of<MODE>() * 32 * RED_LD + (MODE ? 1024 : 0)) * sizeof(double) +
           waves_of<MODE>() * sizeof(SegWindow);
}

// MODE 0: intermediates (stage A).  MODE 1: output tiles with the diagonal
// epilogue and, inside Davidson, their Rayleigh rows.  MODE 2: output tiles
// of the adjoint (out may be null) and the coefficient-gradient partials
// <x, segment product> of the tile.
template <int MODE>
__global__ __launch_bounds__(64 * waves_of<MODE>()) __attribute__((amdgpu_waves_per_eu(2))) void k_tiles32(
    const Task *__restrict__ tasks, const Split *__restrict__ splits, const Seg *__restrict__ segs,
    const DiagTerm *__restrict__ diags, const double *__restrict__ in, const double *__restrict__ tmp,
    double *__restrict__ out, const double *__restrict__ coef, const int32_t *__restrict__ mask,
    const double *__restrict__ dfold, RayArgs ray, const double *__restrict__ xg, double *__restrict__ partials) {
    constexpr int TW = waves_of<MODE>();
    extern __shared__ __align__(16) double smem[];
    double(*red)[32][RED_LD] = reinterpret_cast<double(*)[32][RED_LD]>(smem);  // the runs' sums
    SegWindow *win = reinterpret_cast<SegWindow *>(smem + TW * 32 * RED_LD);
    double *wtile = reinterpret_cast<double *>(win + TW);  // the tile's output values (Rayleigh rows), MODE 2: its x
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int i16 = lane & 15, g = lane >> 4;
    const Task tk = tasks[blockIdx.x];
    if (mask && !mask[tk.member]) return;
    Split sp;
    if (MODE == 0) {
        const int b = tk.nitem * wave / TW;
        sp = Split{tk.seg_begin, b, tk.nitem * (wave + 1) / TW - b, 0};
    } else {
        sp = splits[(int64_t)blockIdx.x * TW + wave];
    }
    const int cnt = tk.m * tk.n;
    constexpr int NQ = 1024 / (64 * TW);  // tile elements per thread
    DiagTerm dt0{};
    if (MODE != 0 && tk.diag_end > tk.diag_begin) dt0 = diags[tk.diag_begin];
    if (MODE == 2) {  // x on the tile, zero outside
        for (int e = threadIdx.x; e < 1024; e += 64 * TW) {
            const int r = e >> 5, c = e & 31;
            wtile[e] = r < tk.m && c < tk.n ? xg[tk.c_off + (int64_t)(tk.row0 + r) * tk.ldc + tk.col0 + c] : 0.0;
        }
        __syncthreads();
    }
    // the run's sum over its segments lies in LDS (its registers go to operands in flight)
    auto run_sum = [&](int a, int e) -> v2d & {
        return *reinterpret_cast<v2d *>(&red[wave][sub(a, 4 * e + g)][2 * i16]);
    };
    v4d acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        acc[a][0] = acc[a][1] = v4d{0, 0, 0, 0};
#pragma unroll
        for (int e = 0; e < 4; ++e) run_sum(a, e) = v2d{0.0, 0.0};
    }
    Walk wk;
    wk.segs = segs;
    wk.win = win + wave;
    wk.in = (gptr)in;
    wk.tmp = (gptr)tmp;
    wk.coef = MODE == 0 ? nullptr : (gptr)coef;
    wk.row0 = tk.row0;
    wk.col0 = tk.col0;
    wk.m = tk.m;
    wk.n = tk.n;
    wk.i = i16;
    wk.g = g;
    wk.lane = lane;
    wk.first = sp.seg;
    wk.end = tk.seg_end;
    wk.left = sp.n;
    int slot = sp.part;  // MODE 2: the run's next partial
    auto use = [&](Frag &f, const Item &it) {
        if (it.flags & IT_SLOW) {
            slow_item<2>(acc, wk.staged(it.si), (gptr)in, (gptr)tmp, tk.row0, tk.col0, tk.m, tk.n, i16, g, it.k0, it.skip);
        } else {
            if (!(it.flags & IT_PU) && (tk.m & 1)) f.p.unswap(pair_swaps(tk.m, i16));
            if (!(it.flags & IT_QU) && (tk.n & 1)) f.q.unswap(pair_swaps(tk.n, i16));
            if (it.skip) {
                f.p.cut(it.flags & IT_PU, g, it.skip);
                f.q.cut(it.flags & IT_QU, g, it.skip);
            }
            switch (it.flags & (IT_PU | IT_QU)) {
            case IT_PU | IT_QU: products<true, true>(acc, f); break;
            case IT_PU: products<true, false>(acc, f); break;
            case IT_QU: products<false, true>(acc, f); break;
            default: products<false, false>(acc, f); break;
            }
        }
        if (it.flags & IT_LAST) {
            const Seg &s = wk.staged(it.si);
            const gptr ps = as_global(uni(s.pscale)), qs = as_global(uni(s.qscale));
            const double c = wk.scale_of(it.si);
            scale_rows<2>(acc, ps, qs, tk.row0, tk.col0, tk.m, tk.n, i16, g);
            double part = 0.0;
#pragma unroll
            for (int a = 0; a < 2; ++a) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const v2d v = {acc[a][0][e], acc[a][1][e]};
                    run_sum(a, e) += c * v;
                    // (outside the tile the accumulator holds duplicated rows and columns, not zeros)
                    if (MODE == 2) {
                        const v2d x = *reinterpret_cast<v2d *>(&wtile[sub(a, 4 * e + g) * 32 + 2 * i16]);
                        if (sub(a, 4 * e + g) < tk.m && 2 * i16 < tk.n) part += x[0] * v[0];
                        if (sub(a, 4 * e + g) < tk.m && 2 * i16 + 1 < tk.n) part += x[1] * v[1];
                    }
                }
                acc[a][0] = acc[a][1] = v4d{0, 0, 0, 0};
            }
            if (MODE == 2) {
                part = group_sum<64>(part) * uni(s.w);
                if (lane == 0) partials[slot] = part;
                ++slot;
            }
        }
    };
    Frag f0, f1, f2;
    Item i0, i1, i2;
    if (sp.n > 0) {
        wk.open(sp.seg, sp.kb);
        wk.fetch(f0, i0);
        wk.fetch(f1, i1);
    }
    // epilogue inputs: the folded diagonal, or the first diagonal term's slices, and the matching
    // input entries are requested here and first used after the products
    const bool dg = MODE != 0 && (MODE == 1 || out);
    const bool fold = MODE == 1 && dfold, first_diag = dg && !fold && tk.diag_end > tk.diag_begin;
    double pre_x[NQ], pre_l[NQ], pre_r[NQ];
    if (fold || first_diag) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int e = min((int)threadIdx.x + q * 64 * TW, cnt - 1);
            const int64_t rr = tk.row0 + e / tk.n, cc = tk.col0 + e % tk.n, o = rr * tk.ldc + cc;
            pre_x[q] = in[tk.x_off + o];
            pre_l[q] = fold ? dfold[tk.c_off + o] : *(dt0.vl ? as_global(dt0.vl) + rr * dt0.sl : (gptr)in);
            pre_r[q] = fold ? 0.0 : *(dt0.vr ? as_global(dt0.vr) + cc * dt0.sr : (gptr)in);
        }
    }
    if (sp.n > 0) {
        for (int q = 0;; q += 3) {
            wk.fetch(f2, i2);
            __builtin_amdgcn_sched_barrier(0);
            use(f0, i0);
            if (q + 1 >= sp.n) break;
            wk.fetch(f0, i0);
            __builtin_amdgcn_sched_barrier(0);
            use(f1, i1);
            if (q + 2 >= sp.n) break;
            wk.fetch(f1, i1);
            __builtin_amdgcn_sched_barrier(0);
            use(f2, i2);
            if (q + 3 >= sp.n) break;
        }
    }
    if (MODE == 2) {
        // diagonal terms: <x, d v_l v_r in> over the tile, one wavefront per term
        for (int d = tk.diag_begin + wave; d < tk.diag_end; d += TW) {
            double part = 0.0;
            for (int e = lane; e < cnt; e += 64) {
                const int64_t rr = tk.row0 + e / tk.n, cc = tk.col0 + e % tk.n;
                part += diag_sum(diags, d, d + 1, nullptr, in[tk.x_off + rr * tk.ldc + cc], rr, cc) *
                        xg[tk.c_off + rr * tk.ldc + cc];
            }
            part = group_sum<64>(part);
            if (lane == 0) partials[tk.part0 + (d - tk.diag_begin)] = part;
        }
        if (!out) return;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int e = threadIdx.x + q * 64 * TW;
        if (e >= cnt) break;
        const int r = e / tk.n, c = e % tk.n;
        // the runs' sums in pairs: a chain of eight has half as much rounding again
        double part[TW];
#pragma unroll
        for (int v = 0; v < TW; ++v) part[v] = red[v][r][c];
#pragma unroll
        for (int w = TW / 2; w > 0; w /= 2)
#pragma unroll
            for (int v = 0; v < w; ++v) part[v] += part[v + w];
        double val = part[0];
        const int64_t rr = tk.row0 + r, cc = tk.col0 + c;
        const int64_t o = tk.c_off + rr * tk.ldc + cc;
        if (fold) {  // sum_d c_d vl vr, folded once for fixed coefficients
            val += pre_l[q] * pre_x[q];
        } else if (first_diag) {
            double d = (coef ? coef[dt0.coef] : 1.0) * dt0.w * pre_x[q];
            if (dt0.vl) d *= pre_l[q];
            if (dt0.vr) d *= pre_r[q];
            val += d + diag_sum(diags, tk.diag_begin + 1, tk.diag_end, coef, pre_x[q], rr, cc);
        }
        out[o] = val;
        if (MODE == 1 && ray.V) wtile[e] = val;
    }
    if (MODE == 1 && ray.V) {
        // the tile's share of [V(:, :i-1), x]^T y: wavefront w takes columns w,
        // w + TW, ...; its lanes run over the tile's elements (coalesced along
        // tile rows) and combine in a fixed order
        __syncthreads();
        constexpr int JW = KM / TW;
        const int ii = ray.i;
        double dot[JW];
#pragma unroll
        for (int jj = 0; jj < JW; ++jj) dot[jj] = 0.0;
        for (int e0 = 0; e0 < cnt; e0 += 4 * 64) {
            int64_t off[4];
            double wv[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int e = min(e0 + lane + 64 * k, cnt - 1);
                off[k] = tk.c_off + (int64_t)(tk.row0 + e / tk.n) * tk.ldc + tk.col0 + e % tk.n;
                wv[k] = e0 + lane + 64 * k < cnt ? wtile[e] : 0.0;
            }
#pragma unroll
            for (int jj = 0; jj < JW; ++jj) {
                if (wave + TW * jj < ii) {
                    const int j = wave + TW * jj;
                    const double *Vj = (j == ii - 1) ? in : ray.V + (int64_t)j * ray.n;
#pragma unroll
                    for (int k = 0; k < 4; ++k) dot[jj] += Vj[off[k]] * wv[k];
                }
            }
        }
#pragma unroll
        for (int jj = 0; jj < JW; ++jj) {
            const int j = wave + TW * jj;
            if (j < ii) {
                const double v = group_sum<64>(dot[jj]);
                if (lane == 0) ray.part[j * ray.ld + tk.rslot] = v;
            }
        }
    }
}

// ------------------------------------------------------------------ 64 x 64 tiles, operands through LDS

// One operand of an item in LDS: window entry k of row r at [k][r].  With this
// stride the column-wise writes of a contiguous contraction (8 rows x 4 pairs
// of entries per half wavefront) fall on different banks; even, so that two
// rows are one 16-byte read.
constexpr int LS = 68;
struct Panel {
    double v[KI * LS];
};
struct Stage64 {
    Panel p, q;
};

// One operand of a segment as a thread fetches it for the workgroup: two pairs
// of values per item.  Contiguous contraction: row tid / 4, window entries
// 2 (tid % 4) (+ 1) and the same + 8.  Else: window entry tid / 16, rows
// 2 (tid % 16) (+ 1) and the same + 32.
struct Fetch64 {
    gbytes b;         // the tile's first row at the window's first contraction index (uniform)
    int64_t ks;       // from one contraction index to the next
    uint32_t o0, o1;  // byte offsets of the two pairs
    int to;           // element of the panel that the first pair goes to
};

__device__ __forceinline__ Fetch64 fetch64_of(gptr a, bool unit, int64_t ld, int row0, int n, int tid) {
    Fetch64 s;
    s.b = (gbytes)(a + (unit ? row0 * ld : row0));
    s.ks = unit ? 8 : ld * 8;
    if (unit) {
        s.o0 = (uint32_t)((min(tid >> 2, n - 1) * ld + 2 * (tid & 3)) * 8);
        s.o1 = s.o0 + 64;
        s.to = 2 * (tid & 3) * LS + (tid >> 2);
    } else {
        const int i = tid & 15;
        const int64_t k = (tid >> 4) * ld;
        s.o0 = (uint32_t)((k + min(2 * i, n - 1) - (pair_swaps(n, i) ? 1 : 0)) * 8);
        s.o1 = (uint32_t)((k + min(2 * i + 32, n - 1) - (pair_swaps(n, i + 16) ? 1 : 0)) * 8);
        s.to = (tid >> 4) * LS + 2 * i;
    }
    return s;
}

// A fetched item into LDS.  edge: an odd tile whose last pair was read one to
// the left, or a window whose first `skip` entries count as zero (both rare, and
// kept out of the common path: vector instructions do not overlap the FP64
// matrix instructions of the same SIMD).
__device__ __forceinline__ void put64(Panel &panel, v2d x0, v2d x1, bool unit, bool edge, int to, int n, int tid,
                                      int skip) {
    if (unit) {
        if (edge) {
            const int k = 2 * (rare(tid) & 3);
            x0 = v2d{k >= skip ? x0[0] : 0.0, k + 1 >= skip ? x0[1] : 0.0};
            x1 = v2d{k + 8 >= skip ? x1[0] : 0.0, k + 9 >= skip ? x1[1] : 0.0};
        }
        double *d = panel.v + to;
        d[0] = x0[0];
        d[LS] = x0[1];
        d[8 * LS] = x1[0];
        d[9 * LS] = x1[1];
    } else {
        if (edge) {
            const int k = rare(tid) >> 4, i = rare(tid) & 15;
            if (n & 1) {
                x0[0] = pair_swaps(n, i) ? x0[1] : x0[0];
                x1[0] = pair_swaps(n, i + 16) ? x1[1] : x1[0];
            }
            x0 = k >= skip ? x0 : v2d{0.0, 0.0};
            x1 = k >= skip ? x1 : v2d{0.0, 0.0};
        }
        v2d *d = reinterpret_cast<v2d *>(panel.v + to);
        d[0] = x0;
        d[16] = x1;
    }
}

// Operands of one item from LDS (p and q at this lane's first rows), and one
// of its four MFMA steps on a quarter of the tile.
struct Lane64 {
    v2d x[4], y[4];
    __device__ __forceinline__ void read(const double *p, const double *q) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            x[j] = *reinterpret_cast<const v2d *>(p + kofs(0, j) * LS);
            y[j] = *reinterpret_cast<const v2d *>(q + kofs(0, j) * LS);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    __device__ __forceinline__ void step(v4d (&acc)[2][2], int j) const {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[j][a], y[j][b], acc[a][b], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
};

// MODE 0: intermediates, MODE 1: output tiles, as k_tiles32.  Three workgroups
// per compute unit (168 registers) against two: 600 us against 658 us for the
// 64-member projection, before its tiles were ordered for the XCDs (an item's
// products wait for LDS and the barrier).
template <int MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_tiles64(
    const Task *__restrict__ tasks, const Seg *__restrict__ segs, const DiagTerm *__restrict__ diags,
    const double *__restrict__ in, const double *__restrict__ tmp, double *__restrict__ out,
    const double *__restrict__ coef, const int32_t *__restrict__ mask, const double *__restrict__ dfold, RayArgs ray) {
    __shared__ __align__(16) Stage64 st[2];
    __shared__ SegWindow win;
    __shared__ double dots[4][KM];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int i16 = lane & 15, g = lane >> 4;
    const Task tk = tasks[blockIdx.x];
    if (mask && !mask[tk.member]) return;
    // this wavefront's quarter
    const int r0 = 32 * (wave >> 1), c0 = 32 * (wave & 1);
    const bool mine = r0 < tk.m && c0 < tk.n;
    const int qm = min(tk.m - r0, 32), qn = min(tk.n - c0, 32);

    // descriptors: staged by the whole workgroup, see SegWindow
    auto staged = [&](int s) -> const Seg & {
        return *reinterpret_cast<const Seg *>(win.w + ((s - tk.seg_begin) & (2 * SEG_HALF - 1)) * SEG_WORDS);
    };
    v4d acc[2][2];
    double tot[2][2][4];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) tot[a][b][e] = 0.0;
    const double *lp = st[0].p.v + 2 * g * LS + r0 + 2 * i16, *lq = st[0].q.v + 2 * g * LS + c0 + 2 * i16;
    constexpr int FLIP = sizeof(Stage64) / sizeof(double);
    for (int si = tk.seg_begin; si < tk.seg_end; ++si) {
        if (((si - tk.seg_begin) & (SEG_HALF - 1)) == 0) {
            const int x = min(tid, SEG_HALF * SEG_WORDS - 1);
            const int s = min(si + x / SEG_WORDS, tk.seg_end - 1);
            const uint64_t v = reinterpret_cast<const uint64_t *>(segs)[(int64_t)s * SEG_WORDS + x % SEG_WORDS];
            if (tid < SEG_HALF * SEG_WORDS)
                win.w[((si - tk.seg_begin) & (2 * SEG_HALF - 1)) * SEG_WORDS + tid] = v;
            __syncthreads();
        }
        const Seg &s = staged(si);
        const SegHead h = head_of(s, (gptr)in, (gptr)tmp, tk.m, tk.n);
        double c = uni(s.w);
        if (MODE != 0) c *= coef[uni(s.coef)];
        const bool pu = !h.ptrans, qu = h.qtrans;
        const int n_items = (h.K + KI - 1) / KI, cut = n_items * KI - h.K;
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) acc[a][b] = v4d{0, 0, 0, 0};
        if (h.slow) {
            for (int q = 0; mine && q < n_items; ++q) {
                const int skip = q == n_items - 1 ? cut : 0;
                slow_item<2>(acc, s, (gptr)in, (gptr)tmp, tk.row0 + r0, tk.col0 + c0, qm, qn, i16, g, q * KI - skip, skip);
            }
        } else {
            Fetch64 P = fetch64_of(h.p, pu, h.ldp, tk.row0, tk.m, tid);
            Fetch64 Q = fetch64_of(h.q, qu, h.ldq, tk.col0, tk.n, tid);
            const bool podd = !pu && (tk.m & 1), qodd = !qu && (tk.n & 1);
            v2d p0, p1, q0, q1;
            auto fetch = [&](int item) {
                if (item == n_items - 1) {  // the window is the segment's last 16 indices
                    P.b -= cut * P.ks;
                    Q.b -= cut * Q.ks;
                }
                p0 = load_pair(P.b, P.o0);
                p1 = load_pair(P.b, P.o1);
                q0 = load_pair(Q.b, Q.o0);
                q1 = load_pair(Q.b, Q.o1);
                P.b += KI * P.ks;
                Q.b += KI * Q.ks;
            };
            auto put = [&](int item) {
                const int skip = item == n_items - 1 ? cut : 0;
                Stage64 &to = st[item & 1];
                put64(to.p, p0, p1, pu, podd || skip, P.to, tk.m, tid, skip);
                put64(to.q, q0, q1, qu, qodd || skip, Q.to, tk.n, tid, skip);
            };
            fetch(0);
            put(0);
            if (n_items > 1) fetch(1);
            __syncthreads();
            for (int q = 0; q < n_items; ++q) {
                // the next item into the other buffer and the one after it on its
                // way, both behind products that are already running
                Lane64 l;
                if (mine) {
                    l.read(lp + (q & 1) * FLIP, lq + (q & 1) * FLIP);
                    l.step(acc, 0);
                }
                if (q + 1 < n_items) put(q + 1);
                if (mine) l.step(acc, 1);
                if (q + 2 < n_items) fetch(q + 2);
                if (mine) {
                    l.step(acc, 2);
                    l.step(acc, 3);
                }
                __syncthreads();
            }
        }
        if (mine) {
            scale_rows<2>(acc, as_global(uni(s.pscale)), as_global(uni(s.qscale)), tk.row0 + r0, tk.col0 + c0, qm, qn,
                          i16, g);
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int e = 0; e < 4; ++e) tot[a][b][e] += c * acc[a][b][e];
        }
    }
    if (mine) {
        // element (a, e, b): row sub(a, 4 e + g), column 2 i16 + b of the quarter, clamped to it for the loads
        int64_t rr[2][4], cc[2];
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            cc[a] = tk.col0 + c0 + min(2 * i16 + a, qn - 1);
#pragma unroll
            for (int e = 0; e < 4; ++e) rr[a][e] = tk.row0 + r0 + min(sub(a, 4 * e + g), qm - 1);
        }
        const bool fold = MODE == 1 && dfold;
        if (fold || (MODE == 1 && tk.diag_end > tk.diag_begin)) {
            double x[2][4][2], d[2][4][2];
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        const int64_t o = rr[a][e] * tk.ldc + cc[b];
                        x[a][e][b] = in[tk.x_off + o];
                        d[a][e][b] = fold ? dfold[tk.c_off + o] : 0.0;
                    }
            if (fold) {
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int b = 0; b < 2; ++b) tot[a][b][e] += d[a][e][b] * x[a][e][b];
            } else {
                for (int t = tk.diag_begin; t < tk.diag_end; ++t) {
                    const DiagTerm dt = diags[t];
                    double l[2][4], r[2];
#pragma unroll
                    for (int a = 0; a < 2; ++a) {
                        r[a] = dt.vr ? as_global(dt.vr)[cc[a] * dt.sr] : 1.0;
#pragma unroll
                        for (int e = 0; e < 4; ++e) l[a][e] = dt.vl ? as_global(dt.vl)[rr[a][e] * dt.sl] : 1.0;
                    }
                    const double cd = (coef ? coef[dt.coef] : 1.0) * dt.w;
#pragma unroll
                    for (int a = 0; a < 2; ++a)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
#pragma unroll
                            for (int b = 0; b < 2; ++b) d[a][e][b] += cd * x[a][e][b] * l[a][e] * r[b];
                }
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int b = 0; b < 2; ++b) tot[a][b][e] += d[a][e][b];
            }
        }
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    if (sub(a, 4 * e + g) < qm && 2 * i16 + b < qn)
                        out[tk.c_off + rr[a][e] * tk.ldc + cc[b]] = tot[a][b][e];
                    else
                        tot[a][b][e] = 0.0;
                }
    }
    if (MODE == 1 && ray.V) {
        // the tile's share of [V(:, :i-1), x]^T y: every wavefront its quarter's
        // (its elements are in registers), summed over the quarters in order
        for (int j = 0; j < ray.i; ++j) {
            const gptr Vj = (gptr)((j == ray.i - 1) ? in : ray.V + (int64_t)j * ray.n) + tk.c_off;
            double d = 0.0;
            if (mine) {
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const gptr row = Vj + (int64_t)(tk.row0 + r0 + min(sub(a, 4 * e + g), qm - 1)) * tk.ldc + tk.col0 + c0;
#pragma unroll
                        for (int b = 0; b < 2; ++b) d += row[min(2 * i16 + b, qn - 1)] * tot[a][b][e];
                    }
            }
            d = group_sum<64>(d);
            if (lane == 0) dots[wave][j] = d;
        }
        __syncthreads();
        if (tid < ray.i) ray.part[tid * ray.ld + tk.rslot] = (dots[0][tid] + dots[1][tid]) + (dots[2][tid] + dots[3][tid]);
    }
}

// ------------------------------------------------------------------ launchers

template <int MODE>
static void launch32(const PassSet &ps, const Lists &l, const double *in, const double *tmp, double *out,
                     const double *coef, hipStream_t s, const int32_t *mask, const double *dfold, const RayArgs &ray,
                     const double *xg, double *partials) {
    if (l.ntask)
        hipLaunchKernelGGL(k_tiles32<MODE>, dim3(l.ntask), dim3(64 * waves_of<MODE>()), tiles32_lds<MODE>(), s, l.tasks, l.splits,
                           (const Seg *)ps.segs, (const DiagTerm *)ps.diags, in, tmp, out, coef, mask, dfold, ray, xg,
                           partials);
}

template <int MODE>
static void launch64(const PassSet &ps, const Lists &l, const double *in, const double *tmp, double *out,
                     const double *coef, hipStream_t s, const int32_t *mask, const double *dfold, const RayArgs &ray) {
    if (l.ntask)
        hipLaunchKernelGGL(k_tiles64<MODE>, dim3(l.ntask), dim3(256), 0, s, l.tasks, (const Seg *)ps.segs,
                           (const DiagTerm *)ps.diags, in, tmp, out, coef, mask, dfold, ray);
}

dmrg_status launch_tiles(const PassSet &ps, const double *coef, const double *in, double *tmp, double *out,
                         hipStream_t s, const int32_t *mask, const double *dfold, const RayArgs *ray,
                         const double *xg, double *partials) {
    const RayArgs ra = ray ? *ray : RayArgs{};
    if (ps.wide == 64) {
        launch64<0>(ps, ps.stageA, in, tmp, tmp, coef, s, mask, nullptr, RayArgs{});
        launch64<1>(ps, ps.stageB, in, tmp, out, coef, s, mask, dfold, ra);
    } else {
        launch32<0>(ps, ps.stageA, in, tmp, tmp, coef, s, mask, nullptr, RayArgs{}, nullptr, nullptr);
        if (partials)
            launch32<2>(ps, ps.stageB, in, tmp, out, coef, s, mask, nullptr, RayArgs{}, xg, partials);
        else
            launch32<1>(ps, ps.stageB, in, tmp, out, coef, s, mask, dfold, ra, nullptr, nullptr);
    }
    DMRG_HIP(hipGetLastError());
    return DMRG_OK;
}

}  // namespace dmrg
