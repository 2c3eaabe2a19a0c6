// Eigen-decomposition of symmetric blocks (Alg. 1, step 6: the eigenvalues of
// each block's density matrix decide which states the block keeps).
// One workgroup per block, two methods by order d:
//
// d <= 8: cyclic two-sided Jacobi in LDS with the round-robin ("circle")
// ordering: each round pairs every index with one other, the d/2 plane
// rotations J of a round are independent, so all of them are found together
// and then applied at once, A <- J^T A J and V <- V J.  With the indices
// grouped by pair, A splits into 2x2 sub-blocks A_kl (rows of pair k, columns
// of pair l) that transform on their own, J_k^T A_kl J_l, so each thread takes
// whole sub-blocks.  A sweep is d - 1 rounds (every pair once); the method
// stops after a sweep with no rotation.
//
// 8 < d <= 2048: Householder reduction to tridiagonal form T = Q^T A Q (the last
// 180 rows in registers, those before them in global memory, where the block
// stays cache-resident), then T's eigenpairs.  Orders up to 512: Cuppen's divide and
// conquer on T (leaves of 4 to 16 rows by implicit QL, one wavefront each; merges
// by deflation, the secular equation on a group of lanes per root and Gu and
// Eisenstat's recomputed weights), then the reflectors of Q applied to its
// eigenvectors, 16 columns a workgroup.  Larger orders: Q formed, and the
// implicit QL iteration with
// Wilkinson's shift on T (the tql2 procedure of Bowdler, Martin, Reinsch and
// Wilkinson), whose plane rotations are applied to the columns of Q: the QL
// recurrence is sequential and runs on one lane, writing each sweep's
// rotations to LDS, which the whole workgroup then applies to the rows of Q
// (Q is stored column-major, so a rotation of columns i, i+1 is a coalesced
// read of two columns).
#include <hip/hip_runtime.h>

#include "internal.h"
#include "lanes.h"

namespace dmrg {

constexpr int EIG_TPB = 256;        // selection kernel
constexpr int EIG_LDS_DIM = 8;  // largest order of the Jacobi method (larger ones are faster on the tridiagonal path)
constexpr int EIG_MAX_DIM = 2048;
constexpr int EIG_MAX_SWEEPS = 40;
constexpr int TRI_TPB = 1024;  // tridiagonal path
constexpr int TRI_WAVES = TRI_TPB / 64;
constexpr int QL_MAXIT = 60;  // QL iterations per eigenvalue before the block is reported unconverged

// LDS writes of a wavefront's lanes are visible to its other lanes after it
__device__ __forceinline__ void wave_sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Pair k of round r of the circle ordering on n' = m + 1 (even) indices:
// k = 0 pairs r with the fixed index m, k > 0 pairs r + k with r - k (mod m).
__device__ __forceinline__ void circle_pair(int r, int k, int m, int &p, int &q) {
    if (k == 0) {
        p = r;
        q = m;
    } else {
        p = (r + k) % m;
        q = (r - k + m) % m;
    }
}

// One block of order d <= EIG_LDS_DIM, by one wavefront; lds: its JAC_LDS doubles.
constexpr int JAC_LDS = 3 * EIG_LDS_DIM * EIG_LDS_DIM + 5 * EIG_LDS_DIM;
__device__ __forceinline__ void eigh_jacobi(int d, const double *in, double *wb, double *out, int32_t *info,
                                            double *lds) {
    constexpr int NP = EIG_LDS_DIM / 2;  // pairs per round
    constexpr int NE = EIG_LDS_DIM * EIG_LDS_DIM;
    constexpr int NT = 64;
    static_assert(NT >= NE, "an element a lane");
    double *V = lds, *part = V + NE, *A = part + NE, *diag = A + NE + EIG_LDS_DIM;
    double *rc = diag + EIG_LDS_DIM, *rs = rc + NP;
    int *rp = (int *)(rs + NP), *rq = rp + NP, *rf = rq + NP;
    const int tid = threadIdx.x & 63;
    const int lda = d + 1;
    if (tid < NE) part[tid] = tid < d * d ? in[tid] * in[tid] : 0.0;
    wave_sync_lds();
    if (tid == 0) {
        double s = 0.0;
        for (int i = 0; i < NE; ++i) s += part[i];
        part[0] = sqrt(s);
    }
    wave_sync_lds();
    // rotations below this size are skipped: the off-diagonal part left is
    // at the rounding level of the matrix norm
    const double thr = part[0] * 0x1p-53 / d;
    for (int e = tid; e < d * d; e += NT) {
        const int r = e / d, c = e % d;
        A[r * lda + c] = in[e];
        V[r * d + c] = (r == c) ? 1.0 : 0.0;
    }
    wave_sync_lds();
    const int m = d + (d & 1) - 1;  // rounds per sweep; index m is a dummy when d is odd
    const int np = (m + 1) / 2;
    int sweep = 0;
    bool done = false;
    for (; sweep < EIG_MAX_SWEEPS && !done; ++sweep) {
        int rotated = 0;
        for (int r = 0; r < m; ++r) {
            int any = 0;
            for (int k = tid; k < np; k += NT) {
                int p, q;
                circle_pair(r, k, m, p, q);
                double c = 1.0, s = 0.0;
                bool rot = false;
                if (p < d && q < d) {
                    const double apq = A[p * lda + q];
                    if (fabs(apq) > thr) {
                        const double app = A[p * lda + p], aqq = A[q * lda + q];
                        const double tau = (aqq - app) / (2.0 * apq);
                        // the smaller root of t^2 + 2 tau t - 1 = 0 (rotation angle <= pi/4)
                        const double t = fabs(tau) > 1e150 ? 0.5 / tau
                                                            : (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
                        c = 1.0 / sqrt(1.0 + t * t);
                        s = t * c;
                        rot = true;
                    }
                }
                rc[k] = c;
                rs[k] = s;
                rp[k] = p;
                rq[k] = q;
                rf[k] = rot;
                any |= rot;
            }
            any = __builtin_amdgcn_ballot_w64(any) != 0;
            wave_sync_lds();
            if (!any) continue;
            rotated = 1;
            // A_kl <- J_k^T A_kl J_l for every pair of pairs; the rotated
            // element of a pair (k == l) is zero in exact arithmetic and is set
            // so (its rounding residue would otherwise be rotated again)
            for (int it = tid; it < np * np; it += NT) {
                const int k = it / np, l = it - k * np;
                if (!rf[k] && !rf[l]) continue;
                const int pk = rp[k], qk = rq[k], pl = rp[l], ql = rq[l];
                const bool vpk = pk < d, vqk = qk < d, vpl = pl < d, vql = ql < d;
                const int ipp = (vpk && vpl) ? pk * lda + pl : 0, ipq = (vpk && vql) ? pk * lda + ql : 0;
                const int iqp = (vqk && vpl) ? qk * lda + pl : 0, iqq = (vqk && vql) ? qk * lda + ql : 0;
                double xpp = A[ipp], xpq = A[ipq], xqp = A[iqp], xqq = A[iqq];
                xpp = (vpk && vpl) ? xpp : 0.0;
                xpq = (vpk && vql) ? xpq : 0.0;
                xqp = (vqk && vpl) ? xqp : 0.0;
                xqq = (vqk && vql) ? xqq : 0.0;
                const double ck = rc[k], sk = rs[k], cl = rc[l], sl = rs[l];
                const double tpp = ck * xpp - sk * xqp, tpq = ck * xpq - sk * xqq;  // rows (pair k)
                const double tqp = sk * xpp + ck * xqp, tqq = sk * xpq + ck * xqq;
                double ypp = cl * tpp - sl * tpq, ypq = sl * tpp + cl * tpq;  // columns (pair l)
                double yqp = cl * tqp - sl * tqq, yqq = sl * tqp + cl * tqq;
                if (k == l) ypq = yqp = 0.0;
                if (vpk && vpl) A[ipp] = ypp;
                if (vpk && vql) A[ipq] = ypq;
                if (vqk && vpl) A[iqp] = yqp;
                if (vqk && vql) A[iqq] = yqq;
            }
            // V <- V J: columns p, q of every rotated pair
            for (int it = tid; it < d * np; it += NT) {
                const int i = it / np, l = it - i * np;
                if (!rf[l]) continue;
                const int pl = rp[l], ql = rq[l];
                const double cl = rc[l], sl = rs[l];
                const double vp = V[i * d + pl], vq = V[i * d + ql];
                V[i * d + pl] = cl * vp - sl * vq;
                V[i * d + ql] = sl * vp + cl * vq;
            }
            wave_sync_lds();
        }
        done = !rotated;
    }
    // eigenvalues in descending order (ties by index), eigenvectors with the
    // first entry of largest magnitude positive
    for (int i = tid; i < d; i += NT) diag[i] = A[i * lda + i];
    wave_sync_lds();
    for (int i = tid; i < d; i += NT) {
        const double wi = diag[i];
        int rank = 0;
        for (int j = 0; j < d; ++j) {
            const double wj = diag[j];
            rank += (wj > wi) || (wj == wi && j < i);
        }
        int kmax = 0;
        double vmax = -1.0;
        for (int r = 0; r < d; ++r) {
            const double av = fabs(V[r * d + i]);
            if (av > vmax) {
                vmax = av;
                kmax = r;
            }
        }
        const double sg = V[kmax * d + i] < 0.0 ? -1.0 : 1.0;
        wb[rank] = wi;
        for (int r = 0; r < d; ++r) out[r * d + rank] = sg * V[r * d + i];
    }
    if (tid == 0 && info) *info = done ? sweep : -2;
}

// Sum over the workgroup of one value per thread, and the value `lead` of
// thread 0, both returned to every thread (the same total in every thread).
// Two barriers: after it, every thread may overwrite what the block read before.
__device__ __forceinline__ double block_sum_lead(double x, double lead, double *red, double *lead_out) {
    x = group_sum<64>(x);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) red[wv] = x;
    if (threadIdx.x == 0) red[TRI_WAVES] = lead;
    __syncthreads();
    double t = 0.0;
    for (int i = 0; i < TRI_WAVES; ++i) t += red[i];
    *lead_out = red[TRI_WAVES];
    __syncthreads();
    return t;
}

// Sum over the workgroup with one barrier, and the value `lead` of the thread
// where `own` holds, to every thread: the caller alternates two buffers of
// TRI_WAVES + 1, so that a buffer is rewritten only after another barrier
__device__ __forceinline__ double block_sum1(double x, bool own, double lead, double *buf, double *lead_out) {
    x = group_sum<64>(x);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) buf[wv] = x;
    if (own) buf[TRI_WAVES] = lead;
    __syncthreads();
    double t = 0.0;
    for (int i = 0; i < TRI_WAVES; ++i) t += buf[i];
    *lead_out = buf[TRI_WAVES];
    return t;
}

// sqrt(x^2 + y^2) without overflow or harmful underflow
__device__ __forceinline__ double hyp(double x, double y) {
    const double ax = fabs(x), ay = fabs(y);
    const double mx = fmax(ax, ay), mn = fmin(ax, ay);
    if (mx == 0.0) return 0.0;
    if (mx > 0x1p-500 && mx < 0x1p+500) return sqrt(x * x + y * y);
    const double q = mn / mx;
    return mx * sqrt(1.0 + q * q);
}

constexpr int TRI_UB = 16;  // rows of a column read per batch of loads (Householder step)
constexpr int QL_B = 8;     // rotations applied per batch of loads (QL; the next batch is fetched ahead)
constexpr int Q_REG = 8;    // column entries per lane kept in registers (Q formation, L <= 512)
constexpr int QB = 16;      // factors per block of the Q formation (their vectors: QB x 512 doubles of LDS)
constexpr int HH_WAVES = TRI_WAVES - 1;       // wavefronts with rows of the block (Householder reduction in registers)
constexpr int HH_REG_DIM = HH_WAVES * 4 * 3;  // largest order reduced there: 12 rows of three columns a thread
constexpr int HH_VEC = 64 * 3;                // LDS vectors of that reduction
static_assert(HH_REG_DIM <= HH_VEC, "vectors as long as the order");
static_assert(5 * HH_VEC <= EIG_MAX_DIM && TRI_WAVES * HH_VEC <= 2 * EIG_MAX_DIM, "its LDS in the pool of the larger orders");
// Blocks of the Jacobi method per workgroup of k_eigh_hh, a wavefront each, in the
// partial products' place: one while there are no more blocks than compute units
// (a wavefront is faster alone: order 8, 40 us against 55 with four on a compute unit), then so many
// that their workgroups, which hold a compute unit each, fit the chip at once.  Odd,
// so that the first blocks of the groups fall on all XCDs and their quarters (workgroup
// b's place follows b mod 32).  With one block a workgroup always, calls on 300 / 1000 /
// 3000 blocks of order 8 took 193 / 274 / 718 us, here 131 / 138 / 222; with a kernel of
// their own 119 / 131 / 205, but its launch adds 40 us where larger blocks are among them.
constexpr int JAC_MAX = 13, CUS = 256;
static_assert(JAC_MAX <= TRI_WAVES && JAC_MAX * JAC_LDS <= TRI_WAVES * HH_VEC, "room for the blocks");
static int jacobi_per(int nblk) { return nblk <= CUS ? 1 : std::min((nblk + CUS - 1) / CUS | 1, JAC_MAX); }

// ------------------------------------------------------------------ divide and conquer
// The symmetric tridiagonal eigenproblem of orders up to DC_MAX by Cuppen's
// divide and conquer (eigenvectors by Gu and Eisenstat's recomputed weights):
// T is torn at the boundaries of a bisection tree, T = blockdiag(T_i) + sum
// |e_b| v_b v_b^T (v_b = e_{b-1} + sign(e_b) e_b, the torn diagonals reduced by
// |e_b|); the leaves (at most DC_LEAF) are solved by implicit QL, one wavefront
// each; then the tree is merged bottom-up.  A merge of two solved halves is the
// rank-one eigenproblem D + rho z z^T (z: the last row of the left half's
// eigenvectors and the first row of the right half's): deflation of
// negligible weights and of nearly equal poles (a plane rotation), the roots
// of the secular equation 1 + rho sum z_i^2 / (d_i - lambda) = 0 from the
// nearer pole (a group of lanes per root: a two-pole rational model,
// bracketed), the weights recomputed from the roots, and the rows of the
// merged block of eigenvectors multiplied by the merge's eigenvector matrix
// (FP64 MFMA, in place).  The merges of a level of the tree run side by side.
constexpr int DC_MAX = 512;
constexpr int DC_LEAF = 16;
constexpr int DC_ITMAX = 100;  // root-finder steps per root (they end at the resolution, typically after 3-8)

// Product over aligned groups of G lanes (G a power of two, 1 <= G <= 64), the
// same bits on every lane of a group (as group_sum); all lanes active
template <int G>
__device__ __forceinline__ double group_prod(double v) {
    if (G >= 2) v *= dpp_f64<DPP_XOR1>(v);
    if (G >= 4) v *= dpp_f64<DPP_XOR2>(v);
    if (G >= 8) v *= dpp_f64<DPP_HALF_MIRROR>(v);
    if (G >= 16) v *= dpp_f64<DPP_MIRROR>(v);
    if (G == 32) v *= __shfl_xor(v, 16, 64);
    if (G == 64) v = (readlane_f64(v, 0) * readlane_f64(v, 16)) * (readlane_f64(v, 32) * readlane_f64(v, 48));
    return v;
}
__device__ __forceinline__ double group_prod(double v, int G) {
    switch (G) {
    case 1: return v;
    case 2: return group_prod<2>(v);
    case 4: return group_prod<4>(v);
    case 8: return group_prod<8>(v);
    case 16: return group_prod<16>(v);
    case 32: return group_prod<32>(v);
    default: return group_prod<64>(v);
    }
}

// 1/x: the hardware reciprocal refined by one Newton step
__device__ __forceinline__ double rcpd(double x) {
    const double r = __builtin_amdgcn_rcp(x);
    return fma(fma(-x, r, 1.0), r, r);
}
constexpr int DC_NLEAF = 32;    // most leaves: orders <= DC_MAX need at most 2^5 of at most DC_LEAF
static_assert((DC_MAX + DC_NLEAF - 1) / DC_NLEAF <= DC_LEAF, "leaf count");
// the pool (5 EIG_MAX_DIM doubles) holds the leaves, then the scratch of a merge
static_assert(DC_NLEAF * DC_LEAF * (DC_LEAF + 1) + TRI_WAVES * (2 * DC_LEAF + 2) <= 5 * EIG_MAX_DIM, "leaf scratch");
static_assert(13 * DC_MAX <= 5 * EIG_MAX_DIM, "merge scratch");
// a level's merges run on TRI_TPB >> t threads each: one wavefront at least, an
// order of at most half as many threads, two panels of 16 roots a wavefront
static_assert(DC_NLEAF / 2 <= TRI_WAVES && 2 * DC_MAX <= TRI_TPB && DC_MAX / 16 <= 2 * TRI_WAVES, "merge teams");
typedef double v4d_eig __attribute__((ext_vector_type(4)));
static_assert(QB * 64 * Q_REG <= 4 * EIG_MAX_DIM, "Q formation: factor vectors in the pool past the factors' t");

// Implicit QL (as the large-order path) on a leaf of order m <= DC_LEAF, one
// wavefront: d (LDS, length m) becomes its eigenvalues, e (length m,
// e[m-1] = 0) is destroyed, Zl (row-major m x m, LDS, row stride DC_LEAF) its
// eigenvectors.  Lane 0 runs each iteration's chase and leaves its rotations
// in rot (cosines, then sines, by index); then lane r applies them, in the
// chase's order, to row r of Zl.  wctl: four ints of LDS.  Every lane returns
// the iteration count, or -1 if an eigenvalue needed more than QL_MAXIT.
__device__ __forceinline__ int ql_leaf(int m, double *d, double *e, double *Zl, double *rot, int *wctl) {
    const int lane = threadIdx.x & 63;
    for (int i = lane; i < m * DC_LEAF; i += 64) Zl[i] = i / DC_LEAF == i % DC_LEAF ? 1.0 : 0.0;
    double *rc = rot, *rs = rot + DC_LEAF;
    int l = 0, it_l = 0, its = 0;
    double tol = 0.0;
    if (lane == 0) {
        double anorm = 0.0;
        for (int i = 0; i < m; ++i) anorm = fmax(anorm, fabs(d[i]) + fabs(e[i]) + (i ? fabs(e[i - 1]) : 0.0));
        tol = anorm * 0x1p-53;
    }
    for (;;) {
        if (lane == 0) {
            // the next iteration: status 0 and the rotation range [lo, hi], 1 when
            // every eigenvalue has converged, -1 when one did not
            int status = 1, lo = 0, hi = -1;
            while (l < m) {
                int mm = l;
                while (mm < m - 1 && fabs(e[mm]) > tol) ++mm;
                if (mm == l) {
                    ++l;
                    it_l = 0;
                    continue;
                }
                if (it_l >= QL_MAXIT) {
                    status = -1;
                    break;
                }
                ++it_l;
                ++its;
                double g = (d[l + 1] - d[l]) / (2.0 * e[l]);
                double r = hyp(g, 1.0);
                g = d[mm] - d[l] + e[l] / (g + copysign(r, g));
                double s = 1.0, c = 1.0, p = 0.0;
                bool early = false;
                int i = mm - 1;
                for (; i >= l; --i) {
                    const double f = s * e[i], bb = c * e[i];
                    r = hyp(f, g);
                    e[i + 1] = r;
                    if (r == 0.0) {
                        d[i + 1] -= p;
                        e[mm] = 0.0;
                        early = true;
                        break;
                    }
                    s = f / r;
                    c = g / r;
                    g = d[i + 1] - p;
                    r = (d[i] - g) * s + 2.0 * c * bb;
                    p = s * r;
                    d[i + 1] = g + p;
                    g = c * r - bb;
                    rc[i] = c;
                    rs[i] = s;
                }
                if (!early) {
                    d[l] -= p;
                    e[l] = g;
                    e[mm] = 0.0;
                }
                status = 0;
                lo = i + 1;  // (l when the chase ran through)
                hi = mm - 1;
                break;
            }
            wctl[0] = status;
            wctl[1] = lo;
            wctl[2] = hi;
            wctl[3] = its;
        }
        wave_sync_lds();
        const int status = wctl[0], lo = wctl[1], hi = wctl[2];
        if (status != 0) {
            const int n_its = wctl[3];
            wave_sync_lds();  // (wctl is rewritten by the next leaf of this wavefront)
            return status < 0 ? -1 : n_its;
        }
        if (lane < m) {
            double *zr = Zl + lane * DC_LEAF;
            for (int i = hi; i >= lo; --i) {
                const double c = rc[i], s = rs[i], h = zr[i + 1];
                zr[i + 1] = s * zr[i] + c * h;
                zr[i] = c * zr[i] - s * h;
            }
        }
        wave_sync_lds();  // the next chase rewrites rc, rs
    }
}

// Scratch of one merge (LDS, carved from the pool): doubles of length DC_MAX
struct DcScratch {
    double *zz, *ds, *rc, *rs, *delta, *zeta, *tau, *zhat, *invn, *lamn;
    int *perm, *defl, *rj, *ri, *nd, *tmp;
};

// The wavefronts that do one merge: 2^t merges of a level run side by side,
// each on size = TRI_TPB >> t threads.  Every barrier is the workgroup's, so
// all teams pass the same number of them.  A merge's time is a chain of
// latencies (barriers, the root finder's iterations, the chains of
// rotations) that more threads do not shorten; order 180, 15 merges one after the
// other: 1.22 ms for the solve, four levels side by side: 0.63 ms, with smaller
// leaves and the deflation scanned by a wavefront: 0.48 ms.
struct DcTeam {
    int size, waves, tid, wv;  // wv: the wavefront's index in the team
};

__device__ __forceinline__ double team_sum(double x, const DcTeam &tm, double *red) {
    x = group_sum<64>(x);
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) red[wv] = x;
    __syncthreads();
    double t = 0.0;
    for (int i = 0; i < tm.waves; ++i) t += red[wv - tm.wv + i];
    return t;
}

// Rank of v[i] among v[0..cnt) (ties by index), on G lanes that share i.
__device__ __forceinline__ int dc_rank(const double *v, int cnt, int i, int g, int G) {
    const double x = v[i];
    int rk = 0;
    for (int j = g; j < cnt; j += G) {
        const double y = v[j];
        rk += (y < x) || (y == x && j < i);
    }
    return (int)group_sum((double)rk, G);
}

// Rows [lo, hi) of the eigenvectors times the merge's eigenvector matrix
// W(i, j) = zhat_i / (delta_i - lambda_j) / norm_j on FP64 MFMA, in place in the
// columns of the k poles that are left.  A wavefront takes NP panels of 16 roots
// and RT tiles of 16 rows at a time; its lanes form the entries of W (pole 4 s +
// lane / 16, root lane % 16) where the product takes them, each once per group
// of rows.  The team holds the products of a group of rows in registers until
// all of it has read them.  (One wavefront per two rows, a reciprocal for every
// entry of W and pair of rows, was bound by them: order 512, 23.1 ms for the
// whole solve against 16.9.)
template <int NP, int RT>
__device__ __forceinline__ void dc_rows(int n, int lo, int hi, int k, int mmax, double *Zt, const DcScratch &S,
                                        const DcTeam &tm) {
    const int lane = threadIdx.x & 63, r16 = lane & 15, g = lane >> 4;
    const size_t N = (size_t)n;
    const double *dl = S.delta, *zh = S.zhat;
    const int *col = S.tmp;
    const int steps = (k + 3) >> 2;
    double dj[NP], tj[NP];  // origin pole and offset of this lane's roots
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int j = min(16 * (tm.wv + p * tm.waves) + r16, max(k - 1, 0));
        dj[p] = k > 0 ? S.zeta[j] : 0.0;
        tj[p] = k > 0 ? S.tau[j] : 0.0;
    }
    for (int c0 = 0; c0 < mmax; c0 += 16 * RT) {
        const int row0 = lo + c0, nt = min(RT, (hi - row0 + 15) >> 4);  // uniform
        const bool work = 16 * tm.wv < k && nt > 0;
        v4d_eig acc[NP][RT];
        if (work) {
            int off[RT];
#pragma unroll
            for (int q = 0; q < RT; ++q) {
                off[q] = min(row0 + 16 * q + r16, hi - 1);
#pragma unroll
                for (int p = 0; p < NP; ++p) acc[p][q] = v4d_eig{0.0, 0.0, 0.0, 0.0};
            }
            auto load = [&](double (&x)[RT], int s) {
                const double *c = Zt + (size_t)col[min(4 * s + g, k - 1)] * N;
#pragma unroll
                for (int q = 0; q < RT; ++q)
                    if (q < nt) x[q] = c[off[q]];
            };
            auto step = [&](const double (&x)[RT], int s) {
                const int i = min(4 * s + g, k - 1);
                const double di = dl[i], zi = 4 * s + g < k ? zh[i] : 0.0;
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    const double wij = zi * rcpd((di - dj[p]) - tj[p]);
#pragma unroll
                    for (int q = 0; q < RT; ++q)
                        if (q < nt) acc[p][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(wij, x[q], acc[p][q], 0, 0, 0);
                }
            };
            double x0[RT], x1[RT];
            load(x0, 0);
            for (int s = 0; s < steps; s += 2) {
                load(x1, s + 1);
                step(x0, s);
                load(x0, s + 2);
                if (s + 1 < steps) step(x1, s + 1);
            }
        }
        __syncthreads();
        if (work) {
            // value v of lane (g, r16) is root 4 v + g of the panel, row r16 of the tile
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int j = 16 * (tm.wv + p * tm.waves) + 4 * v + g;
                    if (j >= k) continue;
                    const double inv = S.invn[j];
                    double *c = Zt + (size_t)col[j] * N;
#pragma unroll
                    for (int q = 0; q < RT; ++q) {
                        const int r = row0 + 16 * q + r16;
                        if (r < hi) c[r] = acc[p][q][v] * inv;
                    }
                }
        }
    }
}

// Merge of the solved halves [lo, mid) and [mid, hi) coupled by rho, by one
// team of the workgroup (mmax: the largest order of the level's merges).  Zt:
// column-major n x n eigenvectors of T (rows and columns of the block only).
// The columns keep their places: the eigenvalues of a merge are not sorted.
__device__ __forceinline__ void dc_merge(int n, int lo, int mid, int hi, int mmax, double rho, double *sd, double *Zt,
                                         const DcScratch &S, const DcTeam &tm, double *red, int *ctl) {
    const int tid = tm.tid;
    const size_t N = (size_t)n;
    const int m = hi - lo;
    // z: row mid - 1 of the left half's eigenvectors, row mid of the right half's
    double part = 0.0;
    for (int c = tid; c < m; c += tm.size) {
        const int col = lo + c;
        double v = col < mid ? Zt[col * N + (mid - 1)] : Zt[col * N + mid];
        if (col >= mid && rho < 0.0) v = -v;
        S.zz[c] = v;
        S.perm[c] = c;  // (poles that are not numbers have no rank)
        part += v * v;
    }
    const double nz2 = team_sum(part, tm, red);
    const double rh = fabs(rho) * nz2;  // rho of the normalized z
    const bool on = rh > 0.0;           // else no coupling: the halves are already solved
    const double inz = 1.0 / sqrt(nz2);
    // ascending order of the poles (ties by index)
    {
        int G = 64;
        while (G > 1 && G * m > tm.size) G >>= 1;
        if (64 * tm.wv < G * m) {
            const int c = min(tid / G, m - 1), g = tid & (G - 1);
            const int rk = dc_rank(sd + lo, m, c, g, G);
            if (tid / G < m && g == 0) {
                S.perm[rk] = c;
                S.ds[rk] = sd[lo + c];
                S.zeta[rk] = S.zz[c] * inz;  // (zeta used as the sorted z during deflation)
            }
        }
    }
    __syncthreads();
    // deflation: a negligible weight leaves its pole; two poles closer than the
    // resolution are rotated so that one weight vanishes, in pole order.  One
    // wavefront: the weights and the neighbours are tested side by side, and only
    // the chains of rotations that start at a close pair are followed one by one
    // (a rotation changes the pole and weight that the next test takes; past the
    // end of a chain the tests hold again).  The rotation test |(d_t - d_p) c s|
    // <= tol is taken as |d_t - d_p| |z_t z_p| <= tol (z_p^2 + z_t^2) (no root: the
    // weights left are above tol / rh >= 8u, so the squares do not underflow).
    if (tm.wv == 0) {
        const int lane = tid & 63;
        const uint64_t below = (1ull << lane) - 1;
        double *zs = S.zeta, *ds = S.ds;
        int *cand = S.nd;
        const double tol = 8.0 * 0x1p-53 * fmax(fmax(fabs(ds[0]), fabs(ds[m - 1])), rh);
        auto close = [&](double zp, double dp, double zt, double dt) {
            return fabs(dt - dp) * fabs(zt * zp) <= tol * (zp * zp + zt * zt);
        };
        int kc = 0, nrot = 0, k = 0;
        for (int t0 = 0; on && t0 < m; t0 += 64) {
            const int t = t0 + lane;
            const bool keep = t < m && !(rh * fabs(zs[min(t, m - 1)]) <= tol);
            const uint64_t mask = __builtin_amdgcn_ballot_w64(keep);
            if (t < m) S.defl[t] = !keep;
            if (keep) cand[kc + __builtin_popcountll(mask & below)] = t;
            kc += __builtin_popcountll(mask);
        }
        wave_sync_lds();
        for (int i0 = 1, skip = 0; i0 < kc; i0 += 64) {
            const int ii = min(i0 + lane, kc - 1), pp = cand[ii - 1], tt = cand[ii];
            uint64_t mask = __builtin_amdgcn_ballot_w64(i0 + lane < kc && close(zs[pp], ds[pp], zs[tt], ds[tt]));
            while (mask) {
                int i = i0 + __builtin_ctzll(mask);
                mask &= mask - 1;
                if (i < skip) continue;  // in the last chain
                int prev = cand[i - 1];
                double zp = zs[prev], dp = ds[prev];
                for (; i < kc; ++i) {
                    const int t = cand[i];
                    const double zt = zs[t], dt = ds[t];
                    if (!close(zp, dp, zt, dt)) break;
                    const double h = hyp(zp, zt);
                    const double c = zt / h, sn = -zp / h;
                    const double dpn = dp * c * c + dt * sn * sn;
                    const double dtn = dp * sn * sn + dt * c * c;
                    if (lane == 0) {
                        zs[t] = h;
                        zs[prev] = 0.0;
                        ds[prev] = dpn;
                        ds[t] = dtn;
                        S.rj[nrot] = prev;
                        S.ri[nrot] = t;
                        S.rc[nrot] = c;
                        S.rs[nrot] = sn;
                        S.defl[prev] = 1;
                    }
                    ++nrot;
                    prev = t;
                    zp = h;
                    dp = dtn;
                }
                skip = i + 1;
            }
            wave_sync_lds();
        }
        for (int i0 = 0; i0 < kc; i0 += 64) {
            const int t = cand[min(i0 + lane, kc - 1)];
            const bool keep = i0 + lane < kc && !S.defl[t];
            const uint64_t mask = __builtin_amdgcn_ballot_w64(keep);
            if (keep) S.tmp[k + __builtin_popcountll(mask & below)] = t;
            k += __builtin_popcountll(mask);
        }
        if (lane == 0) {
            ctl[0] = k;
            ctl[1] = nrot;
        }
    }
    __syncthreads();
    const int k = ctl[0], nrot = ctl[1];
    // the non-deflated poles in ascending order (a rotation may move one by a rounding);
    // the poles by slot are in ds, those left are gathered in delta first
    for (int j = tid; j < k; j += tm.size) {
        S.nd[j] = S.tmp[j];
        S.delta[j] = S.ds[S.tmp[j]];
    }
    __syncthreads();
    int G = 64;
    while (G > 1 && G * k > tm.size) G >>= 1;
    if (64 * tm.wv < G * k) {
        const int j = min(tid / G, k - 1), g = tid & (G - 1);
        const int rk = dc_rank(S.delta, k, j, g, G);
        if (tid / G < k && g == 0) S.nd[rk] = S.tmp[j];
    }
    __syncthreads();
    for (int j = tid; j < k; j += tm.size) {
        const int t = S.nd[j];
        S.delta[j] = S.ds[t];
        S.zz[j] = S.zeta[t];           // zz: the weights of the non-deflated poles
        S.tmp[j] = lo + S.perm[t];     // tmp: their columns
    }
    __syncthreads();
    // roots of the secular equation: root j lies between delta[j] and delta[j+1]
    // (the last one below delta[k-1] + rh sum z^2), in coordinates centred on
    // the nearer pole.  Each step fits the sums over the poles below and above
    // the gap with one pole each (value and slope at the iterate) and moves to
    // the root of that model; a step that leaves the bracket bisects instead.
    // G lanes per root (aligned groups inside a wavefront) split the sums over
    // the poles and combine them with group sums, so every lane of a group
    // holds the same values and takes the same steps; a wavefront iterates
    // until all of its roots have stopped, finished roots keeping their value.
    const double *dl = S.delta, *zw = S.zz;
    if (64 * tm.wv < G * k) {  // wavefronts past the last root's group have nothing to do
        const int g = tid & (G - 1), jr = tid / G, j = min(jr, k - 1);
        double part = 0.0;
        for (int i = g; i < k; i += G) part += zw[i] * zw[i];
        const double zsum = group_sum(part, G);
        const bool last = j + 1 == k;
        const double lo_d = dl[j], hi_d = last ? dl[j] + rh * zsum : dl[j + 1];
        const double half = 0.5 * (hi_d - lo_d);
        // the sums over the poles below and above the gap at x from origin org
        double psi, dpsi, phi, dphi;
        auto sums = [&](double org, double x) {
            psi = dpsi = phi = dphi = 0.0;
#pragma unroll 4
            for (int i = g; i < k; i += G) {
                const double r = rcpd((dl[i] - org) - x);
                const double t = zw[i] * zw[i] * r;
                const bool below = i <= j;
                psi += below ? t : 0.0;
                dpsi += below ? t * r : 0.0;
                phi += below ? 0.0 : t;
                dphi += below ? 0.0 : t * r;
            }
            psi = group_sum(psi, G);
            dpsi = group_sum(dpsi, G);
            phi = group_sum(phi, G);
            dphi = group_sum(dphi, G);
        };
        // from x to the root of the model that the sums at x give.  (Its quotients
        // by rcpd make single roots take twice the steps, and their wavefronts wait.)
        auto model = [&](double dj, double dj1, double x, double bnd) {
            const double u = dj - x, qq = dpsi * u * u, pp = psi - dpsi * u;
            if (last) {
                const double C = 1.0 + rh * (pp + phi);
                return C != 0.0 ? dj + rh * qq / C : bnd;
            }
            const double v = dj1 - x, ss = dphi * v * v, rr = phi - dphi * v;
            const double C = 1.0 + rh * (pp + rr), A1 = rh * qq, A2 = rh * ss;
            // C (u - eta)(v - eta) + A1 (v - eta) + A2 (u - eta) = 0, root inside the gap
            const double qb = -(C * (u + v) + A1 + A2), qc = C * u * v + A1 * v + A2 * u;
            const double disc = qb * qb - 4.0 * C * qc;
            const double sq = sqrt(fmax(disc, 0.0));
            const double q1 = -0.5 * (qb + copysign(sq, qb));
            const double e1 = q1 / C, e2 = qc / q1;
            const double x1 = x + e1, x2 = x + e2;
            return dj < x1 && x1 < dj1 ? x1 : x2;
        };
        sums(lo_d, half);
        const double f = 1.0 + rh * (psi + phi);
        int o;
        double a, bnd, x;
        if (last || f >= 0.0) {
            o = j;
            a = f >= 0.0 ? 0.0 : half;
            bnd = f >= 0.0 ? half : hi_d - lo_d;
            x = half;
        } else {
            o = j + 1;
            a = -half;
            bnd = 0.0;
            x = -half;
        }
        const double dorg = dl[o];
        const double dj = dl[j] - dorg, dj1 = last ? 0.0 : dl[j + 1] - dorg;
        {
            const double xn = model(dj, dj1, x, bnd);
            x = (a < xn && xn < bnd) ? xn : 0.5 * (a + bnd);
        }
        bool done = false;
        for (int it = 0; it < DC_ITMAX; ++it) {
            if (__builtin_amdgcn_ballot_w64(!done) == 0) break;  // every root of the wavefront has stopped
            sums(dorg, x);
            if (done) continue;
            const double fx = 1.0 + rh * (psi + phi);
            if (fx > 0.0)
                bnd = x;
            else
                a = x;
            const double err = 8.0 * 0x1p-53 * (1.0 + rh * (fabs(psi) + fabs(phi)) + fabs(x) * rh * (dpsi + dphi));
            if (fabs(fx) <= err || bnd - a <= 2.0 * 0x1p-53 * fmax(fabs(a), fabs(bnd))) {
                done = true;
                continue;
            }
            const double xn = model(dj, dj1, x, bnd);
            x = (a < xn && xn < bnd) ? xn : 0.5 * (a + bnd);
        }
        if (jr < k && g == 0) {
            S.zeta[j] = dorg;  // (the sorted z is not needed any more)
            S.tau[j] = x;
        }
    }
    __syncthreads();
    // weights recomputed from the roots (their signs kept), then the norms of
    // the eigenvectors zhat_i / (delta_i - lambda_j); G lanes per weight (per
    // norm) split the product (the sum) over the poles, as for the roots
    if (64 * tm.wv < G * k) {
        const int g = tid & (G - 1), ir = tid / G, i = min(ir, k - 1);
        const double di = dl[i];
        double prod = 1.0;
#pragma unroll 4
        for (int j = g; j < k; j += G)
            if (j != i) prod *= ((S.zeta[j] - di) + S.tau[j]) * rcpd(dl[j] - di);
        prod = group_prod(prod, G) * (((S.zeta[i] - di) + S.tau[i]) / rh);
        if (ir < k && g == 0) S.zhat[i] = copysign(sqrt(fmax(prod, 0.0)), zw[i]);
    }
    __syncthreads();
    if (64 * tm.wv < G * k) {
        const int g = tid & (G - 1), jr = tid / G, j = min(jr, k - 1);
        const double dj = S.zeta[j], tj = S.tau[j];
        double q = 0.0;
#pragma unroll 4
        for (int i = g; i < k; i += G) {
            const double x = S.zhat[i] * rcpd((dl[i] - dj) - tj);
            q += x * x;
        }
        q = group_sum(q, G);
        if (jr < k && g == 0) {
            S.invn[j] = 1.0 / sqrt(q);
            S.lamn[j] = dj + tj;
        }
    }
    // the deflation rotations on the columns of the block (in pole order), each
    // thread on its own rows.  A column is the later one of at most one rotation,
    // and if it is the earlier one of another, then of the next: its value is
    // carried, and every load takes a column that no rotation has changed.
    constexpr int ROT = 4;  // rotations per batch of loads
    for (int r = lo + tid; r < hi; r += tm.size) {
        double carry = 0.0;
        int have = -1;  // slot of the carried column
        for (int q0 = 0; q0 < nrot; q0 += ROT) {
            double xj[ROT], xi[ROT];
#pragma unroll
            for (int u = 0; u < ROT; ++u) {
                const int q = min(q0 + u, nrot - 1);
                xj[u] = Zt[(size_t)(lo + S.perm[S.rj[q]]) * N + r];
                xi[u] = Zt[(size_t)(lo + S.perm[S.ri[q]]) * N + r];
            }
#pragma unroll
            for (int u = 0; u < ROT; ++u) {
                const int q = q0 + u;
                if (q >= nrot) break;
                const int sj = S.rj[q], si = S.ri[q];
                const double c = S.rc[q], sn = S.rs[q];
                const double yj = sj == have ? carry : xj[u], yi = xi[u];
                Zt[(size_t)(lo + S.perm[sj]) * N + r] = c * yj + sn * yi;
                carry = c * yi - sn * yj;
                have = si;
                if (q + 1 == nrot || S.rj[q + 1] != si) Zt[(size_t)(lo + S.perm[si]) * N + r] = carry;
            }
        }
    }
    __syncthreads();
    if (n <= 256)
        dc_rows<1, 6>(n, lo, hi, k, mmax, Zt, S, tm);
    else
        dc_rows<2, 4>(n, lo, hi, k, mmax, Zt, S, tm);
    if (on) {
        for (int t = tid; t < m; t += tm.size)
            if (S.defl[t]) sd[lo + S.perm[t]] = S.ds[t];
        for (int j = tid; j < k; j += tm.size) sd[S.tmp[j]] = S.lamn[j];
    }
    __syncthreads();
}

// The whole tridiagonal solve: sd becomes the eigenvalues of T (unordered) and
// Zt (n x n global, column-major: u) its eigenvectors.  ctl[2]: set to 1 if a
// leaf did not converge; ctl[3]: leaf QL iterations + merges.
__device__ __forceinline__ void dc_solve(int n, double *sd, double *se, double *pool, int *ipool, double *Zt,
                                         double *red, int *ctl) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const size_t N = (size_t)n;
    // the smallest leaves (4 at most) that DC_NLEAF of them allow: their QL chases
    // are serial on one lane, a level more of merges costs less (order 64, leaves
    // of 8: 168 us, of 4: 135; order 128, of 16: 446, of 8: 332; order
    // 180, of 16: 603, of 8: 483 with the merges as they were then)
    const int lmax = n <= 4 * DC_NLEAF ? 4 : (n <= 8 * DC_NLEAF ? 8 : DC_LEAF);
    int T = 0;
    while (((n + (1 << T) - 1) >> T) > lmax) ++T;
    const int nleaf = 1 << T;
    auto bnd = [&](int t, int i) { return (n * i) >> t; };
    for (int c = wv; c < n; c += TRI_WAVES)
        for (int r = lane; r < n; r += 64) Zt[c * N + r] = 0.0;
    // tear at the leaf boundaries (leaves hold at least 2 rows: no index is shared)
    if (tid >= 1 && tid < nleaf) {
        const int b0 = bnd(T, tid);
        const double r = fabs(se[b0 - 1]);
        sd[b0 - 1] -= r;
        sd[b0] -= r;
    }
    if (tid == 0) ctl[3] = 0;
    __syncthreads();
    // leaves: one wavefront each (its lane 0), eigenvectors in LDS, then into Zt
    double *leafZ = pool;                              // [nleaf][DC_LEAF][DC_LEAF]
    double *leafE = pool + DC_NLEAF * DC_LEAF * DC_LEAF;  // [nleaf][DC_LEAF]
    double *leafR = leafE + DC_NLEAF * DC_LEAF + wv * 2 * DC_LEAF;  // this wavefront's rotations
    int *leafC = (int *)(leafE + DC_NLEAF * DC_LEAF + TRI_WAVES * 2 * DC_LEAF) + 4 * wv;
    for (int lf = wv; lf < nleaf; lf += TRI_WAVES) {
        const int lo = bnd(T, lf), m = bnd(T, lf + 1) - lo;
        double *el = leafE + lf * DC_LEAF;
        for (int i = lane; i < m; i += 64) el[i] = i + 1 < m ? se[lo + i] : 0.0;
        wave_sync_lds();
        const int it = ql_leaf(m, sd + lo, el, leafZ + lf * DC_LEAF * DC_LEAF, leafR, leafC);
        if (lane == 0) {
            if (it < 0) ctl[2] = 1;
            else atomicAdd(&ctl[3], it);
        }
    }
    __syncthreads();
    for (int lf = wv; lf < nleaf; lf += TRI_WAVES) {
        const int lo = bnd(T, lf), m = bnd(T, lf + 1) - lo;
        const double *Zl = leafZ + lf * DC_LEAF * DC_LEAF;
        for (int e = lane; e < m * m; e += 64) {
            const int r = e / m, c = e % m;
            Zt[(size_t)(lo + c) * N + lo + r] = Zl[r * DC_LEAF + c];
        }
    }
    __syncthreads();
    // merges, deepest level first
    DcScratch S;
    for (int t = T - 1; t >= 0; --t) {
        DcTeam tm;
        tm.size = TRI_TPB >> t;
        tm.waves = TRI_WAVES >> t;
        tm.tid = tid & (tm.size - 1);
        tm.wv = wv & (tm.waves - 1);
        const int i = tid / tm.size;
        const int lo = bnd(t, i), mid = bnd(t + 1, 2 * i + 1), hi = bnd(t, i + 1);
        S.zz = pool + lo;
        S.ds = S.zz + DC_MAX;
        S.rc = S.ds + DC_MAX;
        S.rs = S.rc + DC_MAX;
        S.delta = S.rs + DC_MAX;
        S.zeta = S.delta + DC_MAX;
        S.tau = S.zeta + DC_MAX;
        S.zhat = S.tau + DC_MAX;
        S.invn = S.zhat + DC_MAX;
        S.lamn = S.invn + DC_MAX;
        S.perm = (int *)(pool + 10 * DC_MAX) + lo;
        S.defl = S.perm + DC_MAX;
        S.rj = S.defl + DC_MAX;
        S.ri = S.rj + DC_MAX;
        S.nd = S.ri + DC_MAX;
        S.tmp = S.nd + DC_MAX;
        int *tctl = ipool + 2 * i;
        dc_merge(n, lo, mid, hi, (n + (1 << t) - 1) >> t, se[mid - 1], sd, Zt, S, tm, red, tctl);
    }
    if (tid == 0) ctl[3] += nleaf - 1;  // merges
    __syncthreads();
}

// Householder reduction with the block in registers, R = 4 NQ rows by NQ
// columns a thread: the wavefront wv keeps the rows R wv .. of the columns lane
// + 64 q, so that only vectors pass through LDS (zero past the order, so that
// rows and columns past it add nothing).  The last wavefront keeps no rows but
// the vectors, and forms each step's scalars between two barriers.  Step k: row
// k (left in srow by the previous step's pass, with step k - 1's update (v', w')
// still to apply) gives the diagonal and the reflector v (into LDS, and stored
// in row k beyond k + 1 for the back-transformation); then rows and columns k +
// 1.. take step k - 1's update and are multiplied by v in one pass, which also
// leaves row k + 1 in srow; the wavefronts' partial products meet in LDS (spart)
// as p = t A v, and w = p - K v goes next to v, the next step's pending update.
// Each entry is updated by its own thread (A(i, j) and A(j, i) may differ by
// roundings).  D: the stride of the rows of Z, the block, and of A, which may be
// the same; P0: the update (v', w') pending before step 0, zero past the order.
// What bounds it: the LDS reads that every lane makes of a row's entries (one
// serves NQ columns; with one column a thread they took most of a step) and the
// chain of the scalars, which one wavefront does in the shortest time: with all
// 16 forming them, or joining reductions for them, 4 wavefronts a SIMD issue the
// same instructions.  Order 180: 612 -> 299 us (1.7 us a step), 32: 54 -> 25.
template <int NQ>
__device__ __forceinline__ double hh_pick(const double (&x)[NQ], int q) {  // x[q], q uniform
    const double x1 = x[NQ > 1 ? 1 : 0], x2 = x[NQ > 2 ? 2 : 0];
    double y = x[0];
    if (NQ > 1) y = q >= 1 ? x1 : y;
    if (NQ > 2) y = q >= 2 ? x2 : y;
    return y;
}

template <int NQ>
__device__ __forceinline__ void hh_reduce(int d, size_t D, const double *Z, double *A, double *wb, double2 *P0,
                                          double2 *P1, double *srow, double *spart) {
    constexpr int R = 4 * NQ, LD = 64 * NQ;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);  // (so that the rows, and their tests, are scalar)
    for (int j = tid; j < HH_VEC; j += TRI_TPB) {
        P1[j] = make_double2(0.0, 0.0);
        srow[j] = j < d ? Z[j] : 0.0;  // row 0
    }
    __syncthreads();
    double2 *cur = P0, *nxt = P1;
    if (wv < HH_WAVES) {
        const int j0 = wv * R;
        double a[R][NQ];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int c = lane + 64 * q;
                a[r][q] = (j0 + r < d && c < d) ? Z[(size_t)(j0 + r) * D + c] : 0.0;
            }
        for (int k = 0; k + 2 < d; ++k) {
            __syncthreads();  // v of step k and w of step k - 1 are in LDS
            // rows and columns k + 1..: step k - 1's update, and the product with v;
            // row k + 1 into srow
            if (j0 + R > k + 1 && j0 < d) {  // (uniform: rows that are not finished)
                double2 pc[NQ];
                double acc[NQ];
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    pc[q] = cur[lane + 64 * q];
                    acc[q] = 0.0;
                }
                const double2 *pr = cur + j0, *pn = nxt + j0;
                // each row's LDS reads are issued one row ahead, so that their
                // latency overlaps the previous row's work; v is zero up to row k
                double2 nr = pr[0];
                double nv = pn[0].x;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const double2 pj = nr;
                    const double vr = nv;
                    if (r + 1 < R) {
                        nr = pr[r + 1];
                        nv = pn[r + 1].x;
                    }
#pragma unroll
                    for (int q = 0; q < NQ; ++q) {
                        const double x = fma(-pj.x, pc[q].y, fma(-pj.y, pc[q].x, a[r][q]));
                        a[r][q] = x;
                        acc[q] = fma(x, vr, acc[q]);
                    }
                    if (j0 + r == k + 1) {  // (uniform)
#pragma unroll
                        for (int q = 0; q < NQ; ++q) srow[lane + 64 * q] = a[r][q];
                    }
                }
#pragma unroll
                for (int q = 0; q < NQ; ++q) spart[wv * LD + 64 * q + lane] = acc[q];
            }
            __syncthreads();
            double2 *tmp = cur;
            cur = nxt;
            nxt = tmp;
        }
        __syncthreads();
        // the entry (d - 1, d - 1) after the last step's update
        const double2 pd = cur[d - 1];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int q = 0; q < NQ; ++q)
                if (j0 + r == d - 1 && lane + 64 * q == d - 1) wb[d - 1] = fma(-pd.x, pd.y, fma(-pd.y, pd.x, a[r][q]));
    } else {
        const int G = (d + R - 1) / R;  // wavefronts that have rows
        double v[NQ], w[NQ], t = 0.0;   // the last step's reflector, the update pending before it
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            v[q] = cur[lane + 64 * q].x;
            w[q] = cur[lane + 64 * q].y;
        }
        // p = t A v, K = t p.v / 2, w = p - K v: step k's update, pending in buf
        auto update = [&](int k, double2 *buf) {
            double p[NQ], pv = 0.0;
#pragma unroll
            for (int q = 0; q < NQ; ++q) p[q] = 0.0;
#pragma unroll 4
            for (int g = (k + 1) / R; g < G; ++g)  // (the rows past k)
#pragma unroll
                for (int q = 0; q < NQ; ++q) p[q] += spart[g * LD + 64 * q + lane];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                p[q] = lane + 64 * q > k ? t * p[q] : 0.0;
                pv += p[q] * v[q];
            }
            const double K = 0.5 * t * group_sum<64>(pv);
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                w[q] = p[q] - K * v[q];
                buf[lane + 64 * q].y = w[q];
            }
        };
        for (int k = 0; k + 2 < d; ++k) {
            if (k > 0) update(k - 1, cur);
            // row k after step k - 1's update: the diagonal and x
            const double vk = readlane_f64(hh_pick<NQ>(v, k >> 6), k & 63);
            const double wk = readlane_f64(hh_pick<NQ>(w, k >> 6), k & 63);
            double x[NQ], part = 0.0;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int j = lane + 64 * q;
                x[q] = fma(-v[q], wk, fma(-w[q], vk, srow[j]));
                part += j > k + 1 ? x[q] * x[q] : 0.0;  // (zero past the order)
            }
            const double sigma = group_sum<64>(part);
            const double alpha = readlane_f64(hh_pick<NQ>(x, (k + 1) >> 6), (k + 1) & 63);
            double beta = alpha, scale = 0.0;
            t = 0.0;  // sigma = 0: the row is already reduced
            if (sigma != 0.0) {
                beta = -copysign(sqrt(alpha * alpha + sigma), alpha);
                t = (beta - alpha) / beta;
                scale = 1.0 / (alpha - beta);
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int j = lane + 64 * q;
                v[q] = j <= k ? 0.0 : (j == k + 1 ? 1.0 : (sigma != 0.0 ? x[q] * scale : 0.0));
                nxt[j].x = v[q];
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int j = lane + 64 * q;
                if (j > k + 1 && j < d) A[k * D + j] = v[q];
                if (j == k) wb[k] = x[q];
                if (j == k + 1) A[j * D + k] = beta;
                if (j == k + 2) A[j * D + k] = t;
            }
            __syncthreads();
            double2 *tmp = cur;
            cur = nxt;
            nxt = tmp;
        }
        update(d - 3, cur);
        // the diagonal entry and the coupling of row d - 2 after the last step's update
        const int k = d - 2;
        const double vk = readlane_f64(hh_pick<NQ>(v, k >> 6), k & 63);
        const double wk = readlane_f64(hh_pick<NQ>(w, k >> 6), k & 63);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int j = lane + 64 * q;
            const double x = fma(-v[q], wk, fma(-w[q], vk, srow[j]));
            if (j == k) wb[k] = x;
            if (j == k + 1) A[j * D + k] = x;
        }
        __syncthreads();
    }
}

// Householder reduction of the blocks of orders EIG_LDS_DIM + 1 .. HH_REG_DIM to
// tridiagonal form T = Q^T A Q (Q = H_0 ... H_{d-3}, H_k = I - t_k v_k v_k^T on
// indices k + 1.., v_k(k + 1) = 1), one workgroup per block, the block held in
// registers.  Output for k_eigh_tri: the diagonal of T in w (block b's slice),
// T(k + 1, k) at u(k + 1, k), t_k at u(k + 2, k), and v_k(j) at u(k, j) for
// j >= k + 2 (u row-major, block b at off[b]); a is only read.
__global__ __launch_bounds__(TRI_TPB) void k_eigh_hh(int nblk, const int64_t *__restrict__ off,
                                                     const int32_t *__restrict__ dim, const int64_t *__restrict__ woff,
                                                     const double *__restrict__ a, double *__restrict__ w,
                                                     double *__restrict__ u, int32_t *__restrict__ info, int per) {
    __shared__ double2 P0[HH_VEC], P1[HH_VEC];  // (v, w) of two steps
    __shared__ double srow[HH_VEC];
    __shared__ double spart[TRI_WAVES * HH_VEC];
    const int b = blockIdx.x;
    if (b >= nblk) return;
    const int d = dim[b];
    if (d < 1 || d > EIG_MAX_DIM) {
        if (threadIdx.x == 0 && info) info[b] = -1;  // unsupported order
        return;
    }
    if (d > HH_REG_DIM) return;  // reduced by k_eigh_tri
    if (d <= EIG_LDS_DIM) {
        // the first such block of a group of per: all of the group's, a wavefront each
        const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g0 = b / per * per;
        const int dl = lane < per && g0 + lane < nblk ? dim[g0 + lane] : 0;
        const uint64_t mask = __builtin_amdgcn_ballot_w64(dl >= 1 && dl <= EIG_LDS_DIM);
        if (g0 + __builtin_ctzll(mask) != b || !(mask >> wave & 1)) return;
        const int bj = g0 + wave;
        eigh_jacobi(dim[bj], a + off[bj], w + woff[bj], u + off[bj], info ? info + bj : nullptr, spart + wave * JAC_LDS);
        return;
    }
    const double *Z = a + off[b];
    double *A = u + off[b], *wb = w + woff[b];
    for (int j = threadIdx.x; j < HH_VEC; j += TRI_TPB) P0[j] = make_double2(0.0, 0.0);  // no update is pending
    if (d <= HH_WAVES * 4)
        hh_reduce<1>(d, d, Z, A, wb, P0, P1, srow, spart);
    else if (d <= HH_WAVES * 8)
        hh_reduce<2>(d, d, Z, A, wb, P0, P1, srow, spart);
    else
        hh_reduce<3>(d, d, Z, A, wb, P0, P1, srow, spart);
}

// Tridiagonal path of the orders EIG_LDS_DIM + 1 .. EIG_MAX_DIM, one workgroup
// per block: T handed over by k_eigh_hh (orders up to HH_REG_DIM) or reduced
// here, in global memory as far as the block exceeds the registers (11 us a step
// at order 256), the last HH_REG_DIM rows there (1.7): order 256, 3.12 -> 2.28 ms.  Orders up to DC_MAX: divide and conquer on T, which
// leaves the eigenvectors of T in a, the reflectors in u and the order of the
// eigenvalues on its diagonal, for k_eigh_back and k_eigh_out.  Larger orders: Q formed,
// implicit QL on T applied to it, and the ordered output written here.
__global__ __launch_bounds__(TRI_TPB) void k_eigh_tri(int nblk, const int64_t *__restrict__ off,
                                                      const int32_t *__restrict__ dim, const int64_t *__restrict__ woff,
                                                      double *__restrict__ a, double *__restrict__ w,
                                                      double *__restrict__ u, int32_t *__restrict__ info) {
    __shared__ double sd[EIG_MAX_DIM];  // diagonal of T, then the eigenvalues
    __shared__ double se[EIG_MAX_DIM];  // se[i] couples i and i + 1
    __shared__ double pool[5 * EIG_MAX_DIM];
    double *sq = pool;                     // Householder factors; QL: cosines (second buffer)
    double *sx = pool + EIG_MAX_DIM;       // Householder vector; QL: cosines (first buffer)
    double *sy = pool + 2 * EIG_MAX_DIM;   // p, then w = p - K v; QL: sines (first buffer)
    double *sz = pool + 3 * EIG_MAX_DIM;   // QL: sines (second buffer)
    double *spart = pool + 4 * EIG_MAX_DIM;  // row-group partial sums of p
    // (the divide-and-conquer path, which forms no Q, uses the whole pool once the factors are stored)
    __shared__ int srank[EIG_MAX_DIM];
    __shared__ double red[TRI_WAVES + 1];
    __shared__ double red2[TRI_WAVES + 1];  // second buffer of the reductions of the Householder steps
    __shared__ int ctl[4];
    const int b = blockIdx.x;
    if (b >= nblk) return;
    const int d = dim[b];
    if (d <= EIG_LDS_DIM || d > EIG_MAX_DIM) return;  // done (or rejected) by k_eigh_hh
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const size_t D = (size_t)d;
    double *A = u + off[b];  // working matrix (row-major, both triangles), then Householder vectors
    double *Z = a + off[b];  // Q, then the eigenvectors; column-major: Z[c * d + r] = Q(r, c)
    if (d <= HH_REG_DIM) {
        // reduced by k_eigh_hh: the diagonal in w, the off-diagonal and the
        // factors t below the diagonal of u, the reflectors in its rows
        const double *wb = w + woff[b];
        for (int j = tid; j < d; j += TRI_TPB) {
            sd[j] = wb[j];
            se[j] = j + 1 < d ? A[(j + 1) * D + j] : 0.0;
        }
        __syncthreads();
    } else {
        for (int r = wv; r < d; r += TRI_WAVES)
            for (int c = lane; c < d; c += 64) A[r * D + c] = Z[r * D + c];
        __syncthreads();

        // ---- Householder reduction: step k zeroes A(k, k+2..) and A(k+2.., k) with
        // H = I - t v v^T acting on indices k+1.., v(0) = 1 (stored in row k beyond it).
        // A stays symmetric up to roundings (the two products of an update may be
        // fused differently for A(i, j) and A(j, i)), so column i of the trailing
        // block is read as its row i: each thread owns columns (coalesced across
        // the threads of a row).  Step k
        // needs p = t A22 v, w = p - K v and A22 -= v w^T + w v^T; the update of
        // step k and the product of step k + 1 are one pass over the block: row
        // k + 1 is updated first (it yields the next reflector), then every other
        // element is updated, stored and multiplied by the next v at once.
        // sv: v of the current step, sn: v of the next one, sy: p, then w.
        double *sv = sx, *sn = sz;
        double t = 0.0;  // the current step's factor
        {
            // step 0's reflector from row 0 and its product p = t A22 v
            const int L = d - 1;
            double part = 0.0;
            for (int j = tid; j < L; j += TRI_TPB) {
                const double x = A[1 + j];
                sv[j] = x;
                if (j) part += x * x;
            }
            double alpha;
            const double sigma = block_sum_lead(part, tid == 0 ? A[1] : 0.0, red, &alpha);
            if (sigma == 0.0) {
                if (tid == 0) {
                    sd[0] = A[0];
                    se[0] = alpha;
                    sq[0] = 0.0;
                }
                for (int j = tid; j < L; j += TRI_TPB) sv[j] = j ? 0.0 : 1.0;  // with t = 0: no reflection
            } else {
                const double beta = -copysign(sqrt(alpha * alpha + sigma), alpha);
                t = (beta - alpha) / beta;
                const double scale = 1.0 / (alpha - beta);
                for (int j = tid; j < L; j += TRI_TPB) sv[j] = j ? sv[j] * scale : 1.0;
                if (tid == 0) {
                    sd[0] = A[0];
                    se[0] = beta;
                    sq[0] = t;
                }
            }
            __syncthreads();
            const int G = max(1, min(TRI_TPB / L, 32)), R = (L + G - 1) / G;
            for (int q = tid; q < G * L; q += TRI_TPB) {
                const int i = q % L, g = q / L;
                const int j0 = g * R, j1 = min(L, j0 + R);
                const double *col = A + D + 1 + i;
                double acc = 0.0;
                for (int jb = j0; jb < j1; jb += TRI_UB) {
                    double av[TRI_UB];
    #pragma unroll
                    for (int u = 0; u < TRI_UB; ++u) av[u] = col[min(jb + u, j1 - 1) * D];
    #pragma unroll
                    for (int u = 0; u < TRI_UB; ++u)
                        if (jb + u < j1) acc += av[u] * sv[jb + u];
                }
                spart[q] = acc;
            }
            __syncthreads();
        }
        const int first = d - HH_REG_DIM;  // the block from here on is reduced in registers
        for (int k = 0; k < first; ++k) {
            const int L = d - k - 1, G = max(1, min(TRI_TPB / L, 32));
            // p and w of step k (the groups' partial products meet in LDS)
            double pv = 0.0;
            for (int i = tid; i < L; i += TRI_TPB) {
                double acc = 0.0;
                for (int g = 0; g < G; ++g) acc += spart[g * L + i];
                const double pi = t * acc;
                sy[i] = pi;
                pv += pi * sv[i];
            }
            double unused;
            const double K = 0.5 * t * block_sum1(pv, false, 0.0, red, &unused);
            for (int j = tid; j < L; j += TRI_TPB) sy[j] -= K * sv[j];  // w
            __syncthreads();
            for (int j = 1 + tid; j < L; j += TRI_TPB) A[k * D + k + 1 + j] = sv[j];
            if (k + 1 == first) break;  // its update is left pending
            // row k + 1 after step k's update (the same expression as for the
            // rest of the block): its diagonal, and the vector x of step k + 1 into sn
            double part = 0.0, diag = 0.0, lead = 0.0;
            for (int i = tid; i < L; i += TRI_TPB) {
                const double val = A[(k + 1) * D + k + 1 + i] - __dadd_rn(__dmul_rn(sv[0], sy[i]), __dmul_rn(sy[0], sv[i]));
                if (i == 0) diag = val;
                if (i == 1) lead = val;
                if (i >= 1) sn[i - 1] = val;
                if (i >= 2) part += val * val;
            }
            double alpha;  // x(0), handed over by the thread that formed it (sn[0] is rescaled below)
            const double sigma = block_sum1(part, tid == 1, lead, red2, &alpha);
            double tn = 0.0;
            if (sigma == 0.0) {  // the column is already reduced
                if (tid == 0) {
                    sd[k + 1] = diag;
                    se[k + 1] = alpha;
                    sq[k + 1] = 0.0;
                }
                for (int j = tid; j < L - 1; j += TRI_TPB) sn[j] = j ? 0.0 : 1.0;  // with t = 0: no reflection
            } else {
                const double beta = -copysign(sqrt(alpha * alpha + sigma), alpha);
                tn = (beta - alpha) / beta;
                const double scale = 1.0 / (alpha - beta);
                for (int j = tid; j < L - 1; j += TRI_TPB) sn[j] = j ? sn[j] * scale : 1.0;
                if (tid == 0) {
                    sd[k + 1] = diag;
                    se[k + 1] = beta;
                    sq[k + 1] = tn;
                }
            }
            __syncthreads();
            // the rest of A22 (indices k + 2..): updated, stored, and summed into the
            // next step's p; thread (i, g) on the rows of group g
            // of column i, loads in batches
            const int L1 = L - 1, G1 = max(1, min(TRI_TPB / L1, 32)), R1 = (L1 + G1 - 1) / G1;
            for (int q = tid; q < G1 * L1; q += TRI_TPB) {
                const int i = q % L1, g = q / L1;
                const int j0 = g * R1, j1 = min(L1, j0 + R1);
                double *col = A + (k + 2) * D + k + 2 + i;
                const double vi = sv[i + 1], wi = sy[i + 1];
                double acc = 0.0;
                for (int jb = j0; jb < j1; jb += TRI_UB) {
                    double av[TRI_UB];
    #pragma unroll
                    for (int u = 0; u < TRI_UB; ++u) av[u] = col[min(jb + u, j1 - 1) * D];
    #pragma unroll
                    for (int u = 0; u < TRI_UB; ++u) {
                        const int j = jb + u;
                        if (j < j1) {
                            const double val = av[u] - __dadd_rn(__dmul_rn(sv[j + 1], wi), __dmul_rn(sy[j + 1], vi));
                            col[j * D] = val;
                            acc += val * sn[j];
                        }
                    }
                }
                spart[q] = acc;
            }
            __syncthreads();
            double *tmp = sv;  // the next step's v becomes the current one
            sv = sn;
            sn = tmp;
            t = tn;
        }
        // the last HH_REG_DIM rows and columns, with step first - 1's update
        // pending, in registers (their vectors in the pool past the factors' t)
        double2 *P0 = (double2 *)sx, *P1 = P0 + HH_VEC;
        const double v0 = tid < HH_REG_DIM ? sv[tid] : 0.0, w0 = tid < HH_REG_DIM ? sy[tid] : 0.0;
        __syncthreads();
        if (tid < HH_VEC) P0[tid] = make_double2(v0, w0);
        double *B = A + first * D + first;
        hh_reduce<3>(HH_REG_DIM, D, B, B, sd + first, P0, P1, (double *)(P1 + HH_VEC), sy);
        __syncthreads();
        for (int j = first + tid; j < d; j += TRI_TPB) {
            se[j] = j + 1 < d ? A[(j + 1) * D + j] : 0.0;
            if (j + 2 < d) sq[j] = A[(j + 2) * D + j];
        }
        __syncthreads();
    }
    if (d <= DC_MAX) {
        // the reflectors (rows of u beyond k + 1) and their factors t (at
        // (k + 2, k)) stay in u for k_eigh_back; divide and conquer on T, its
        // eigenvectors into a, which the input no longer needs, its eigenvalues
        // in descending order (ties by index) into w, and the index of the
        // eigenvector that column c of the result takes into u(c, c)
        if (d > HH_REG_DIM)
            for (int k = tid; k + 2 < d; k += TRI_TPB) A[(k + 2) * D + k] = sq[k];
        if (tid == 0) ctl[2] = 0;
        __syncthreads();  // the factors in the pool are read up to here
        dc_solve(d, sd, se, pool, (int *)srank, Z, red, ctl);
        double *wb = w + woff[b];
        for (int c = tid; c < d; c += TRI_TPB) {  // (values that are not numbers have no rank)
            wb[c] = sd[c];
            A[c * D + c] = c;
        }
        __syncthreads();
        int G = 64;
        while (G > 1 && G * d > TRI_TPB) G >>= 1;
        if (64 * wv < G * d) {
            const int i = min(tid / G, d - 1), g = tid & (G - 1);
            const double wi = sd[i];
            int above = 0;
            for (int j = g; j < d; j += G) {
                const double wj = sd[j];
                above += (wj > wi) || (wj == wi && j < i);
            }
            const int rk = (int)group_sum((double)above, G);
            if (tid / G < d && g == 0) {
                wb[rk] = wi;
                A[rk * D + rk] = i;
            }
        }
        if (tid == 0 && info) info[b] = ctl[2] ? -2 : 1 + ctl[3];
        return;
    }
    // ---- Q = H_0 H_1 ... H_{d-3}, accumulated from the last factor; H_k Q only
    // changes the trailing block from index k + 1: y_c = v^T Q(:, c), then
    // Q(:, c) -= t y_c v.
    for (int c = wv; c < d; c += TRI_WAVES)
        for (int r = lane; r < d; r += 64) Z[c * D + r] = r == c ? 1.0 : 0.0;
    __syncthreads();
    if (d - 1 <= 64 * Q_REG) {
        // QB factors at a time: their vectors staged in LDS (rows from the
        // block's first touched index r0 = klo + 1, zero above each factor's
        // own start), then every wave applies all of them, last first, to four
        // columns at a time held in registers: one load and one store of each
        // column per block instead of per factor.  A factor meets zeros in the
        // rows and columns it does not reach, which leaves them unchanged.
        double *sv = sx;  // [QB][L0] (the pool past the factors' t)
        for (int khi = d - 3; khi >= 0; khi -= QB) {
            const int klo = max(0, khi - QB + 1), r0 = klo + 1, L0 = d - r0;
            for (int i = tid; i < (khi - klo + 1) * L0; i += TRI_TPB) {
                const int kk = i / L0, j = i - kk * L0, k = klo + kk, r = r0 + j;
                sv[i] = r == k + 1 ? 1.0 : (r > k + 1 ? A[k * D + r] : 0.0);
            }
            __syncthreads();
            for (int c0 = 4 * wv; c0 < L0; c0 += 4 * TRI_WAVES) {
                double cv[4][Q_REG];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double *col = Z + (r0 + min(c0 + e, L0 - 1)) * D + r0;
#pragma unroll
                    for (int q = 0; q < Q_REG; ++q) {
                        if (64 * q >= L0) break;  // uniform: the row slots past L0 are not used
                        cv[e][q] = col[min(lane + 64 * q, L0 - 1)];
                    }
                }
                for (int k = khi; k >= klo; --k) {
                    const double t = sq[k];
                    if (t == 0.0) continue;
                    const double *v = sv + (k - klo) * L0;
                    double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int q = 0; q < Q_REG; ++q) {
                        if (64 * q >= L0) break;
                        const int r = lane + 64 * q;
                        const double vr = r < L0 ? v[r] : 0.0;
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[e] += vr * cv[e][q];
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const double ty = t * group_sum<64>(acc[e]);
#pragma unroll
                        for (int q = 0; q < Q_REG; ++q) {
                            if (64 * q >= L0) break;
                            const int r = lane + 64 * q;
                            if (r < L0) cv[e][q] -= ty * v[r];
                        }
                    }
                }
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (c0 + e < L0) {
                        double *col = Z + (r0 + c0 + e) * D + r0;
#pragma unroll
                        for (int q = 0; q < Q_REG; ++q) {
                            const int r = lane + 64 * q;
                            if (r < L0) col[r] = cv[e][q];
                        }
                    }
            }
            __syncthreads();  // the next block reads these columns and rewrites sv
        }
    } else {
        // one factor at a time, one wave per column (or four columns)
        for (int k = d - 3; k >= 0; --k) {
            const double t = sq[k];
            if (t == 0.0) continue;
            const int L = d - k - 1;
            for (int j = tid; j < L; j += TRI_TPB) sx[j] = j ? A[k * D + k + 1 + j] : 1.0;
            __syncthreads();
            if (L <= 64 * Q_REG) {
                // four columns per wave at a time: all their loads in flight together
                for (int c0 = 4 * wv; c0 < L; c0 += 4 * TRI_WAVES) {
                    double cv[4][Q_REG];
                    double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const double *col = Z + (k + 1 + min(c0 + e, L - 1)) * D + k + 1;
#pragma unroll
                        for (int q = 0; q < Q_REG; ++q) cv[e][q] = col[min(lane + 64 * q, L - 1)];
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int q = 0; q < Q_REG; ++q) {
                            const int r = lane + 64 * q;
                            if (r < L) acc[e] += sx[r] * cv[e][q];
                        }
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const double ty = t * group_sum<64>(acc[e]);
                        if (c0 + e < L) {
                            double *col = Z + (k + 1 + c0 + e) * D + k + 1;
#pragma unroll
                            for (int q = 0; q < Q_REG; ++q) {
                                const int r = lane + 64 * q;
                                if (r < L) col[r] = cv[e][q] - ty * sx[r];
                            }
                        }
                    }
                }
            } else {
                for (int c = wv; c < L; c += TRI_WAVES) {
                    double *col = Z + (k + 1 + c) * D + k + 1;
                    double acc = 0.0;
                    for (int r = lane; r < L; r += 64) acc += sx[r] * col[r];
                    const double ty = t * group_sum<64>(acc);
                    for (int r = lane; r < L; r += 64) col[r] -= ty * sx[r];
                }
            }
            __syncthreads();
        }
    }

    int its = 0, bad = 0;
    {
    // ---- implicit QL on T (sd, se).  Lane 0 of wave 0 runs the recurrence and
    // leaves each iteration's rotations (indices lo..hi) in one of two LDS
    // buffers; in the same interval the other waves apply the previous
    // iteration's rotations to the rows of Z.
    int l = 0, it_l = 0;
    double tol = 0.0;
    // one QL iteration into buffer `buf` (lane 0 of wave 0 only); ctl[2 buf] = lo,
    // ctl[2 buf + 1] = hi, lo = -1 when every eigenvalue has converged
    auto ql_next = [&](int buf) {
        int lo = -1, hi = -1;
        double *rc = buf ? sq : sx, *rs = buf ? sz : sy;
        while (l < d) {
            // m: the first index >= l whose coupling counts as zero (se[d - 1] = 0);
            // eight couplings tested per round of LDS loads
            int m = l;
            for (;;) {
                double ev[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) ev[u] = se[min(m + u, d - 1)];
                int found = -1;
#pragma unroll
                for (int u = 7; u >= 0; --u)
                    if (fabs(ev[u]) <= tol || m + u >= d - 1) found = min(m + u, d - 1);
                if (found >= 0) {
                    m = found;
                    break;
                }
                m += 8;
            }
            if (m == l) {  // sd[l] is an eigenvalue
                ++l;
                it_l = 0;
                continue;
            }
            if (++it_l > QL_MAXIT) {
                bad = 1;
                l = d;
                break;
            }
            ++its;
            // shift: the eigenvalue of the leading 2 x 2 of the segment nearer sd[l]
            const double dl = sd[l];
            double g = (sd[l + 1] - dl) / (2.0 * se[l]);
            double r = hyp(g, 1.0);
            g = sd[m] - dl + se[l] / (g + copysign(r, g));
            double s = 1.0, c = 1.0, p = 0.0;
            // every value read below is still the one from before this iteration
            // (iteration i writes index i + 1), so the next ones are fetched ahead
            double dip1 = sd[m], di = sd[m - 1], ei = se[m - 1];
            int i = m - 1;
            bool early = false;
            for (; i >= l; --i) {
                const int in = i > l ? i - 1 : i;
                const double dn = sd[in], en = se[in];
                const double f = s * ei, bb = c * ei;
                // T is scaled to a norm in [1, 2), so f and g cannot overflow; a
                // rotation norm below 2^-500 (135 orders of magnitude below the
                // deflation threshold) counts as zero: the chase splits there and
                // the iteration is repeated on the shorter segment
                const double r2 = f * f + g * g;
                if (__builtin_expect(r2 <= 0x1p-1000, 0)) {
                    se[i + 1] = 0.0;
                    sd[i + 1] = dip1 - p;
                    se[m] = 0.0;
                    early = true;
                    break;
                }
                const double ir = rsqrt(r2);
                r = r2 * ir;
                se[i + 1] = r;
                s = f * ir;
                c = g * ir;
                g = dip1 - p;
                r = (di - g) * s + 2.0 * c * bb;
                p = s * r;
                sd[i + 1] = g + p;
                g = c * r - bb;
                rc[i] = c;
                rs[i] = s;
                dip1 = di;
                di = dn;
                ei = en;
            }
            if (!early) {
                sd[l] -= p;
                se[l] = g;
                se[m] = 0.0;
            }
            lo = early ? i + 1 : l;
            hi = m - 1;
            break;
        }
        ctl[2 * buf] = lo;
        ctl[2 * buf + 1] = hi;
    };
    double scale = 1.0;  // power of two: T * scale has a norm in [1, 2) (exact)
    if (tid == 0) {
        double anorm = 0.0;
        for (int i = 0; i < d; ++i)
            anorm = fmax(anorm, fabs(sd[i]) + fabs(se[i]) + (i ? fabs(se[i - 1]) : 0.0));
        if (anorm > 0.0 && isfinite(anorm)) {
            scale = ldexp(1.0, -ilogb(anorm));
            for (int i = 0; i < d; ++i) {
                sd[i] *= scale;
                se[i] *= scale;
            }
            anorm *= scale;
        }
        tol = anorm * 0x1p-53;
        ql_next(0);
    }
    __syncthreads();
    for (int step = 0;; ++step) {
        const int cur = step & 1;
        const int lo = ctl[2 * cur], hi = ctl[2 * cur + 1];
        if (lo < 0) break;
        if (wv == 0) {
            if (lane == 0) ql_next(cur ^ 1);
        } else if (hi >= lo) {
            // rotation i acts on columns i, i + 1, from hi down to lo: the column
            // i + 1 entering rotation i is the one rotation i + 1 left (carried),
            // column i is still the old one (fetched ahead in batches)
            const double *rc = cur ? sq : sx, *rs = cur ? sz : sy;
            for (int r = tid - 64; r < d; r += TRI_TPB - 64) {
                double carry = Z[(hi + 1) * D + r];
                double zv[QL_B], zn[QL_B];
#pragma unroll
                for (int q = 0; q < QL_B; ++q) zv[q] = Z[max(hi - q, lo) * D + r];
                for (int i0 = hi; i0 >= lo; i0 -= QL_B) {
                    // the next batch's columns lie below every column this batch writes
#pragma unroll
                    for (int q = 0; q < QL_B; ++q) zn[q] = Z[max(i0 - QL_B - q, lo) * D + r];
#pragma unroll
                    for (int q = 0; q < QL_B; ++q) {
                        const int i = i0 - q;
                        if (i >= lo) {
                            const double c = rc[i], s = rs[i];
                            Z[(i + 1) * D + r] = s * zv[q] + c * carry;
                            carry = c * zv[q] - s * carry;
                        }
                    }
#pragma unroll
                    for (int q = 0; q < QL_B; ++q) zv[q] = zn[q];
                }
                Z[lo * D + r] = carry;
            }
        }
        __syncthreads();
    }

    if (tid == 0 && scale != 1.0) {
        const double inv = 1.0 / scale;  // a power of two: exact
        for (int i = 0; i < d; ++i) sd[i] *= inv;
    }
    }  // QL
    __syncthreads();
    // ---- descending order (ties by index), first entry of largest magnitude positive
    for (int i = tid; i < d; i += TRI_TPB) {
        const double wi = sd[i];
        int rank = 0;
        for (int j = 0; j < d; ++j) {
            const double wj = sd[j];
            rank += (wj > wi) || (wj == wi && j < i);
        }
        srank[i] = rank;
    }
    __syncthreads();
    double *wb = w + woff[b];
    for (int i = wv; i < d; i += TRI_WAVES) {
        const double *col = Z + i * D;
        double best = -1.0;
        int bi = 0;
        for (int r = lane; r < d; r += 64) {
            const double av = fabs(col[r]);
            if (av > best) {
                best = av;
                bi = r;
            }
        }
        for (int o = 32; o > 0; o >>= 1) {
            const double ob = __shfl_xor(best, o, 64);
            const int oi = __shfl_xor(bi, o, 64);
            if (ob > best || (ob == best && oi < bi)) {
                best = ob;
                bi = oi;
            }
        }
        const double sg = col[bi] < 0.0 ? -1.0 : 1.0;
        const int rk = srank[i];
        for (int r = lane; r < d; r += 64) A[r * D + rk] = sg * col[r];
        if (lane == 0) wb[rk] = sd[i];
    }
    if (tid == 0 && info) info[b] = bad ? -2 : 1 + its;
}

constexpr int BK_COLS = 16;                  // columns of a block per workgroup of k_eigh_back
constexpr int BK_PANELS = DC_MAX / BK_COLS;  // its grid's second dimension
constexpr int BK_TPB = 256;                  // four wavefronts
constexpr int BK_LD = DC_MAX + 4;            // row stride of the staged reflectors (spreads the LDS banks)
static_assert(QB == 16 && BK_TPB == 16 * QB && BK_COLS == 16, "sixteen reflectors by sixteen columns");

// Apply the reflectors to the columns [cp, cp + 16) of Z, NT tiles of 16 rows a
// wavefront (tile q = wave + 4 i), held in registers throughout in the layout in
// which the matrix instruction leaves a product and takes its second operand.
template <int NT>
__device__ __forceinline__ void back_apply(int d, int cp, const double *__restrict__ H, double *__restrict__ Z,
                                           double *sv, double *st, double (*red)[2][256]) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 15, g = lane >> 4;
    const size_t D = (size_t)d;
    double *col = Z + (size_t)min(cp + c, d - 1) * D;
    v4d_eig z[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = 16 * (wave + 4 * i) + 4 * v + g;
            const double x = col[min(r, d - 1)];
            z[i][v] = r < d ? x : 0.0;
        }
    // this thread's part of a block: reflector klo + kk, rows c + 16 j
    const int kk = tid >> 4;
    double pre[4 * NT], pt = 0.0;
    auto fetch = [&](int khi) {
        const int klo = max(0, khi - QB + 1), k = min(klo + kk, khi);
#pragma unroll
        for (int j = 0; j < 4 * NT; ++j)
            if (16 * j + 15 > klo && 16 * j < d) pre[j] = H[(size_t)k * D + min(c + 16 * j, d - 1)];
        pt = H[(size_t)(k + 2) * D + k];
    };
    if (d >= 3) fetch(d - 3);
    for (int khi = d - 3; khi >= 0; khi -= QB) {
        const int klo = max(0, khi - QB + 1), k = klo + kk;
        const int q0 = (klo + 1) >> 4;  // first tile that the block reaches
#pragma unroll
        for (int j = 0; j < 4 * NT; ++j) {
            const int r = c + 16 * j;
            if (j >= q0 && 16 * j < d)
                sv[kk * BK_LD + r] = k > khi || r > d - 1 || r < k + 1 ? 0.0 : (r == k + 1 ? 1.0 : pre[j]);
        }
        if (c == 0) st[kk] = k <= khi ? pt : 0.0;
        __syncthreads();
        if (khi - QB >= 0) fetch(khi - QB);
        // Y = V^T Z and G = V^T V over this wavefront's rows
        v4d_eig y4 = {0.0, 0.0, 0.0, 0.0}, g4 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const int q = wave + 4 * i;
            if (q >= q0 && 16 * q < d) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const double x = sv[c * BK_LD + 16 * q + 4 * v + g];
                    y4 = __builtin_amdgcn_mfma_f64_16x16x4f64(x, z[i][v], y4, 0, 0, 0);
                    g4 = __builtin_amdgcn_mfma_f64_16x16x4f64(x, x, g4, 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            red[wave][0][16 * (4 * v + g) + c] = y4[v];
            red[wave][1][16 * (4 * v + g) + c] = g4[v];
        }
        __syncthreads();
#pragma unroll
        for (int h = 0; h < 2; ++h) red[0][h][tid] = (red[0][h][tid] + red[1][h][tid]) + (red[2][h][tid] + red[3][h][tid]);
        __syncthreads();
        // H_klo ... H_khi Z = Z - V y, y_j = t_j (v_j.z - sum_{i > j} v_j.v_i y_i)
        const double *Y = red[0][0], *G = red[0][1];
        double y[QB];
#pragma unroll
        for (int j = 0; j < QB; ++j) y[j] = Y[16 * j + c];
#pragma unroll
        for (int j = QB - 1; j >= 0; --j) {
            y[j] *= st[j];
#pragma unroll
            for (int i = 0; i < j; ++i) y[i] -= G[16 * j + i] * y[j];
        }
        double yb[4];  // the second operand of step s: -y[4 s + g]
#pragma unroll
        for (int s = 0; s < 4; ++s)
            yb[s] = -(g == 0 ? y[4 * s] : (g == 1 ? y[4 * s + 1] : (g == 2 ? y[4 * s + 2] : y[4 * s + 3])));
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const int q = wave + 4 * i;
            if (q >= q0 && 16 * q < d) {
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    z[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(sv[(4 * s + g) * BK_LD + 16 * q + c], yb[s], z[i], 0, 0, 0);
            }
        }
        __syncthreads();  // the next block restages sv and red
    }
    if (cp + c < d) {
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = 16 * (wave + 4 * i) + 4 * v + g;
                if (r < d) col[r] = z[i][v];
            }
    }
}

// Eigenvectors of the divide-and-conquer blocks (orders EIG_LDS_DIM + 1 ..
// DC_MAX): E = H_0 H_1 ... H_{d-3} Z, the reflectors (rows of u beyond k + 1,
// t_k at u(k + 2, k)) applied to the eigenvectors Z of T (a, column-major), the
// last one first, in place.  Workgroup (b, p) owns columns [16 p, 16 p + 16) of
// block b.  Sixteen reflectors V at a time go through LDS (the next sixteen are
// on their way meanwhile) and are applied at once: V^T Z and V^T V on FP64
// MFMA, sixteen steps of substitution in every lane, Z - V y on FP64 MFMA.  The
// chain of these blocks bounds it: 44 us at order 180, 211 at 512 (two reflectors
// at a time with a reduction over the wavefront for each took 163 and 775).
__global__ __launch_bounds__(BK_TPB) void k_eigh_back(int nblk, const int64_t *__restrict__ off,
                                                      const int32_t *__restrict__ dim, double *__restrict__ a,
                                                      const double *__restrict__ u) {
    __shared__ double sv[QB * BK_LD];
    __shared__ double st[QB];
    __shared__ double red[BK_TPB / 64][2][256];
    const int b = blockIdx.x;
    if (b >= nblk) return;
    const int d = dim[b];
    if (d <= EIG_LDS_DIM || d > DC_MAX) return;
    const int cp = blockIdx.y * BK_COLS;
    if (cp >= d) return;
    const double *H = u + off[b];
    double *Z = a + off[b];
    if (d <= 64)
        back_apply<1>(d, cp, H, Z, sv, st, red);
    else if (d <= 192)
        back_apply<3>(d, cp, H, Z, sv, st, red);
    else
        back_apply<8>(d, cp, H, Z, sv, st, red);
}

constexpr int OUT_COLS = 32;  // columns of u per workgroup of k_eigh_out
constexpr int OUT_TPB = 256;
constexpr int OUT_FILL = 16384;

// Output of the divide-and-conquer blocks: the columns of E (a, column-major)
// into u (row-major), column c the one whose index k_eigh_tri left at u(c, c),
// with its first entry of largest magnitude positive.  Workgroup (b, p) owns
// columns [32 p, 32 p + 32) of u (and those a grid of panels further), 32 x 32 tiles through LDS, read down the
// columns of E and written along the rows of u: 13 us at order 180, a chain of
// three reads (48 us with one workgroup per block and a staging copy).  Most
// workgroups find no columns where blocks are small, and a thousand blocks fill the
// chip with one panel each: OUT_FILL of them at most.  (10000 blocks of order 1, which
// have none: 327 us a call with all 16 panels, 286.)
__global__ __launch_bounds__(OUT_TPB) void k_eigh_out(int nblk, const int64_t *__restrict__ off,
                                                      const int32_t *__restrict__ dim, const double *__restrict__ a,
                                                      double *__restrict__ u) {
    constexpr int NC = OUT_COLS / (OUT_TPB / 64);  // columns of a wavefront
    constexpr int NR = OUT_TPB / 32;               // rows of a tile at a time
    __shared__ double ssg[OUT_COLS];
    __shared__ int src[OUT_COLS];
    __shared__ double tile[2][32][33];
    const int b = blockIdx.x;
    if (b >= nblk) return;
    const int d = dim[b];
    if (d <= EIG_LDS_DIM || d > DC_MAX) return;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const size_t D = (size_t)d;
    const double *E = a + off[b];
    double *U = u + off[b];
    for (int c0 = blockIdx.y * OUT_COLS; c0 < d; c0 += gridDim.y * OUT_COLS) {
        if (tid < OUT_COLS) {
            const int c = min(c0 + tid, d - 1);
            src[tid] = min(max((int)U[c * D + c], 0), d - 1);
        }
        __syncthreads();
        double best[NC];
        int bi[NC];  // twice the row, and the sign
#pragma unroll
        for (int e = 0; e < NC; ++e) {
            best[e] = -1.0;
            bi[e] = 0;
        }
        for (int r = lane; r < d; r += 64) {
            double av[NC];
#pragma unroll
            for (int e = 0; e < NC; ++e) av[e] = E[src[NC * wv + e] * D + r];
#pragma unroll
            for (int e = 0; e < NC; ++e)
                if (fabs(av[e]) > best[e]) {
                    best[e] = fabs(av[e]);
                    bi[e] = 2 * r + (av[e] < 0.0);
                }
        }
#pragma unroll
        for (int e = 0; e < NC; ++e) {
            for (int o = 32; o > 0; o >>= 1) {
                const double ob = __shfl_xor(best[e], o, 64);
                const int oi = __shfl_xor(bi[e], o, 64);
                if (ob > best[e] || (ob == best[e] && oi < bi[e])) {
                    best[e] = ob;
                    bi[e] = oi;
                }
            }
            if (lane == 0) ssg[NC * wv + e] = (bi[e] & 1) ? -1.0 : 1.0;
        }
        __syncthreads();
        const int tr = tid & 31, tc = tid >> 5;
        double x[32 / NR];
        auto fetch = [&](int rr) {
#pragma unroll
            for (int q = 0; q < 32 / NR; ++q) x[q] = E[src[tc + NR * q] * D + min(rr + tr, d - 1)];
        };
        fetch(0);
        for (int rr = 0, h = 0; rr < d; rr += 32, h ^= 1) {
#pragma unroll
            for (int q = 0; q < 32 / NR; ++q) tile[h][tc + NR * q][tr] = ssg[tc + NR * q] * x[q];
            __syncthreads();  // (the other buffer is read up to here: two are enough)
            if (rr + 32 < d) fetch(rr + 32);
#pragma unroll
            for (int q = 0; q < 32 / NR; ++q) {
                const int r = rr + tc + NR * q, c = c0 + tr;
                if (r < d && c < d) U[r * D + c] = tile[h][tr][tc + NR * q];
            }
        }
        __syncthreads();  // src, ssg and tile are the next columns'
    }
}

// State selection (Alg. 1, step 7: a block keeps its states of largest
// density-matrix eigenvalue).  One workgroup per group of sector blocks whose
// eigenvalues lie contiguous in w.  The m-th largest value is found by a radix
// select on order-preserving 64-bit keys (eight passes of 8 bits, a 256-bin
// histogram each); values above it are kept, and of the values equal to it the
// first ones in storage order (block order, then index order), by a scan.  A
// block keeps a prefix of its values because each block's values are stored
// in descending order.
constexpr int TRUNC_MAX = 16384;

// order-preserving key: a > b  <=>  key(a) > key(b), a == b  <=>  key(a) ==
// key(b) (for non-NaN values; -0 is taken as +0)
__device__ __forceinline__ uint64_t order_key(double v) {
    const uint64_t b = (uint64_t)__double_as_longlong(v == 0.0 ? 0.0 : v);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

__global__ __launch_bounds__(EIG_TPB) void k_truncate(int ngroup, const int32_t *__restrict__ gblk,
                                                      const int32_t *__restrict__ dim,
                                                      const int64_t *__restrict__ woff, const double *__restrict__ w,
                                                      const int32_t *__restrict__ m_keep, int32_t *__restrict__ keep,
                                                      double *__restrict__ discarded) {
    __shared__ unsigned char kept[TRUNC_MAX];
    __shared__ double part[EIG_TPB];
    __shared__ int hist[256];
    __shared__ int cnt[EIG_TPB];
    __shared__ uint64_t sel_key;
    __shared__ int sel_rem;
    const int g = blockIdx.x, tid = threadIdx.x;
    if (g >= ngroup) return;
    const int b0 = gblk[g], b1 = gblk[g + 1];
    if (b1 <= b0) {
        if (tid == 0 && discarded) discarded[g] = 0.0;
        return;
    }
    const int64_t base = woff[b0];
    const int64_t N64 = woff[b1 - 1] + dim[b1 - 1] - base;
    if (N64 < 0 || N64 > TRUNC_MAX) {
        for (int b = b0 + tid; b < b1; b += EIG_TPB) keep[b] = -1;
        if (tid == 0 && discarded) discarded[g] = __builtin_nan("");
        return;
    }
    const int N = (int)N64;
    const int m = m_keep[g];
    const double *wg = w + base;
    // thread tid owns values [lo, hi)
    const int per = (N + EIG_TPB - 1) / EIG_TPB;
    const int lo = min(N, tid * per), hi = min(N, lo + per);
    if (m <= 0 || m >= N) {  // nothing or everything kept
        for (int e = lo; e < hi; ++e) kept[e] = m > 0;
    } else {
        // radix select of the m-th largest key, most significant digit first
        uint64_t prefix = 0;
        int rem = m;  // rank still to be found inside the current prefix
        for (int pass = 0; pass < 8; ++pass) {
            const int shift = 56 - 8 * pass;
            for (int i = tid; i < 256; i += EIG_TPB) hist[i] = 0;
            __syncthreads();
            const uint64_t hmask = pass == 0 ? 0 : (~0ull << (shift + 8));
            for (int e = lo; e < hi; ++e) {
                const uint64_t k = order_key(wg[e]);
                if ((k & hmask) == prefix) atomicAdd(&hist[(k >> shift) & 255], 1);
            }
            __syncthreads();
            if (tid == 0) {
                int acc = 0, digit = 255;
                for (; digit > 0; --digit) {
                    if (acc + hist[digit] >= rem) break;
                    acc += hist[digit];
                }
                sel_key = prefix | ((uint64_t)digit << shift);
                sel_rem = rem - acc;
            }
            __syncthreads();
            prefix = sel_key;
            rem = sel_rem;
            __syncthreads();  // sel_* are rewritten by the next pass
        }
        // values equal to the cut: the first rem of them in storage order
        int c = 0;
        for (int e = lo; e < hi; ++e) c += order_key(wg[e]) == prefix;
        cnt[tid] = c;
        __syncthreads();
        if (tid == 0) {
            int run = 0;
            for (int i = 0; i < EIG_TPB; ++i) {
                const int t = cnt[i];
                cnt[i] = run;
                run += t;
            }
        }
        __syncthreads();
        int before = cnt[tid];
        for (int e = lo; e < hi; ++e) {
            const uint64_t k = order_key(wg[e]);
            bool keepit = k > prefix;
            if (k == prefix) keepit = before++ < rem;
            kept[e] = keepit;
        }
    }
    __syncthreads();
    double dsum = 0.0;
    for (int b = b0 + tid; b < b1; b += EIG_TPB) {
        const int64_t s = woff[b] - base;
        int kc = 0;
        for (int j = 0; j < dim[b]; ++j) {
            if (kept[s + j])
                ++kc;
            else
                dsum += wg[s + j];
        }
        keep[b] = kc;
    }
    part[tid] = dsum;
    __syncthreads();
    if (tid == 0 && discarded) {
        double t = 0.0;
        for (int i = 0; i < EIG_TPB; ++i) t += part[i];
        discarded[g] = t;
    }
}

}  // namespace dmrg

// ================================================================== ABI

using namespace dmrg;

extern "C" {

dmrg_status dmrg_eigh_blocks(int32_t nblk, const int64_t *off, const int32_t *dim, const int64_t *woff,
                             double *a, double *w, double *u, int32_t *info, void *stream) {
    clear_error();
    if (nblk < 0) return set_error(DMRG_E_INVALID_ARG, "negative block count");
    if (nblk == 0) return DMRG_OK;
    if (!off || !dim || !woff || !a || !w || !u) return set_error(DMRG_E_INVALID_ARG, "null argument");
    if (a == u || a == w || u == w) return set_error(DMRG_E_INVALID_ARG, "a, w and u must not overlap");
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(k_eigh_hh, dim3(nblk), dim3(TRI_TPB), 0, s, nblk, off, dim, woff, (const double *)a, w, u, info,
                       jacobi_per(nblk));
    hipLaunchKernelGGL(k_eigh_tri, dim3(nblk), dim3(TRI_TPB), 0, s, nblk, off, dim, woff, a, w, u, info);
    hipLaunchKernelGGL(k_eigh_back, dim3(nblk, BK_PANELS), dim3(BK_TPB), 0, s, nblk, off, dim, a, (const double *)u);
    const int panels = std::min(DC_MAX / OUT_COLS, std::max(1, OUT_FILL / nblk));
    hipLaunchKernelGGL(k_eigh_out, dim3(nblk, panels), dim3(OUT_TPB), 0, s, nblk, off, dim, (const double *)a, u);
    DMRG_HIP(hipGetLastError());
    return DMRG_OK;
}

dmrg_status dmrg_truncate(int32_t ngroup, const int32_t *gblk, const int32_t *dim, const int64_t *woff,
                          const double *w, const int32_t *m_keep, int32_t *keep, double *discarded, void *stream) {
    clear_error();
    if (ngroup < 0) return set_error(DMRG_E_INVALID_ARG, "negative group count");
    if (ngroup == 0) return DMRG_OK;
    if (!gblk || !dim || !woff || !w || !m_keep || !keep) return set_error(DMRG_E_INVALID_ARG, "null argument");
    hipLaunchKernelGGL(k_truncate, dim3(ngroup), dim3(EIG_TPB), 0, (hipStream_t)stream, ngroup, gblk, dim, woff, w,
                       m_keep, keep, discarded);
    DMRG_HIP(hipGetLastError());
    return DMRG_OK;
}

}  // extern "C"
