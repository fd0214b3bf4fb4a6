// Chirally split block basis, restrictor / prolongator, Galerkin coarse
// operator and coarse gamma matrices.
//
// * Basis (eq:mg_basis with eq:chirality:B): for block y and chirality alpha
//   the fields P_alpha theta_{B_y} v_c, c < Nv, orthonormalised in order c.
//   The result is the unique QR factor with positive real diagonal; it is
//   computed as Cholesky QR done twice (Gram matrix, Cholesky factor R,
//   W R^{-1}), which reaches the same factor as Gram-Schmidt to rounding.
//   Storage: B[y][alpha][c][3 s' + col][l], s' the spin inside the chirality,
//   l the block-local site, so one basis vector is 6*Vb contiguous complex.
// * R and T (eq:res_mg, eq:pro_mg): per block, a (2 Nv) x (12 Vb) complex
//   matrix times the right-hand sides.
// * D_1 = R M T (fig:A): nine nc x nc blocks per coarse site, entry [y][dir]
//   holding the fine hops that leave block y through face dir (dir 0: the
//   clover term and the hops inside the block).  Built by prolonging coarse
//   unit vectors, applying the matching piece of M and restricting.
// * (gamma5 gamma_k)_1 per block time slice (eq:coarse:gamma with an open
//   time index): only the alpha = 0 rows x alpha = 1 columns block is stored;
//   the other block is minus its adjoint (gamma5 gamma_k is anti-Hermitian and
//   flips chirality).
#include "mglma_internal.h"

int mg_galerkin(mglma_ctx* c, double2* tmp);

// ---------------------------------------------------------------------------
// basis construction
// ---------------------------------------------------------------------------
// field offset of column k: s'col V + l
__device__ __forceinline__ size_t col_off(int k, int Vb, size_t V) {
    int s = 0;
#pragma unroll
    for (int m = 1; m < 6; ++m) s += k >= m * Vb;
    return (size_t)s * (V - Vb) + (uint32_t)k;
}

// One pass of a Cholesky QR over sets of Nv vectors of K columns each, on the
// FP64 matrix cores:
//   APPLY: w_d = sum_{c <= d} src_c X[c][d], written to B (and its FP32 and FP16
//          copies where given);
//   GRAM:  G[c][d] = <w_c, w_d> for c <= d (without APPLY: of the source).
// The source is B itself (in place: a wavefront has read all vectors of its 16
// columns before it writes them) or, TV, the test vectors: set (y, a), column k
// = (s'col, l) is component 6 a + s'col at site y Vb + l, so the first pass also
// does the block projection and chiral split.
// One workgroup per set, wavefronts over tiles of 16 columns, no barrier between
// tiles.  APPLY: the rows of D = X^T W are vectors, its columns are contiguous in
// memory for loads and stores; X lies in LDS in the order of the lanes, upper
// triangle only.  GRAM: the tile goes through the wavefront's part of LDS (rows
// in, fragments out, slots exchanged within a row against bank conflicts), and each
// tile's products are summed for themselves first: |<w, w> - 1| is 2.0e-16 on
// average (4.0e-16 with one running sum a wavefront, 1.35e-15 with one a set).
//
// Bound: memory (read, write) and, with both, as much the matrix cores.  The
// three passes of a basis (Gram; apply and Gram; apply) on 48 x 24^3, 24
// vectors: 1.0 + 1.9 + 1.8 ms (0.65 + 1.3 + 1.4 at the rate of a copy), against
// 1.2 for the projection and twice 1.1 + 1.5 on the vector units, one pass each.
template <int NTR, bool APPLY, bool GRAM, bool TV>
__global__ __launch_bounds__(256) void k_qr_pass(Geo g, int Nv, int K, const double2* __restrict__ tv, double2* B,
                                                 const double2* __restrict__ X, double2* __restrict__ G,
                                                 float2* __restrict__ B32, __half2* __restrict__ B16) {
    typedef Mfma<double> MF;
    typedef MF::v4 V4;
    constexpr int NS = 4 * NTR, NX = APPLY ? 2 * NTR * (NTR + 1) : 0, NP = NTR * (NTR + 1) / 2;
    extern __shared__ double2 shx[];                   // X fragments, then the wavefronts' tiles
    const int ya = blockIdx.x, w = threadIdx.x >> 6, nw = blockDim.x >> 6, lane = threadIdx.x & 63;
    const int lr = lane & 15, lq = lane >> 4, ns = (Nv + 3) / 4;
    double2* sh = shx + NX * 64 + (GRAM ? w * NTR * 256 : 0);
    double2* Wb = B + (size_t)ya * Nv * K;
    // source (c, k): S[c * cs + off(k)]
    const double2* S = TV ? tv + (size_t)(ya & 1) * 6 * g.V + (size_t)(ya >> 1) * g.Vb : Wb;
    const size_t cs = TV ? (size_t)12 * g.V : (size_t)K;
    auto off = [&](int k) { return TV ? col_off(k, g.Vb, g.V) : (size_t)(uint32_t)k; };
    if constexpr (APPLY) {
        const double2* Xs = X + (size_t)ya * Nv * Nv;
        for (int e = w; e < NX; e += nw) {
            int t = 0;
            while (2 * (t + 1) * (t + 2) <= e) ++t;
            const int d = 16 * t + lr, c = 4 * (e - 2 * t * (t + 1)) + lq;
            shx[e * 64 + lane] = c < Nv && d < Nv ? Xs[c * Nv + d] : make_double2(0.0, 0.0);
        }
        __syncthreads();
    }
    V4 gr[GRAM ? NP : 1], gi[GRAM ? NP : 1];
#pragma unroll
    for (int p = 0; p < (GRAM ? NP : 1); ++p) {
        gr[p] = V4{0, 0, 0, 0};
        gi[p] = V4{0, 0, 0, 0};
    }
    const int nt = (K + 15) / 16;
    for (int q = w; q < nt; q += nw) {
        const int k = 16 * q + lr;
        const bool kok = k < K;
        const size_t ko = kok ? off(k) : 0;
        if constexpr (APPLY) {
            double2 b[NS];
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                if (s < ns) {
                    const int c = 4 * s + lq;
                    b[s] = S[(size_t)(c < Nv ? c : Nv - 1) * cs + ko];
                    b[s].x = kok ? b[s].x : 0.0;
                    b[s].y = kok ? b[s].y : 0.0;
                }
            }
#pragma unroll
            for (int t = 0; t < NTR; ++t) {
                V4 dr = {0, 0, 0, 0}, di = {0, 0, 0, 0};
#pragma unroll
                for (int s = 0; s < 4 * (t + 1); ++s) {
                    if (s < ns) {
                        const double2 x = shx[(2 * t * (t + 1) + s) * 64 + lane];
                        dr = MF::mac(x.x, b[s].x, dr);
                        di = MF::mac(x.x, b[s].y, di);
                        dr = MF::mac(-x.y, b[s].y, dr);
                        di = MF::mac(x.y, b[s].x, di);
                    }
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = MF::row(lq, r), d = 16 * t + i;
                    const double2 v = make_double2(dr[r], di[r]);
                    if (GRAM) sh[t * 256 + i * 16 + (lr ^ i)] = v;
                    if (kok && d < Nv) {
                        const size_t o = (size_t)d * K + k, og = (size_t)ya * Nv * K + o;
                        Wb[o] = v;
                        if (B32) B32[og] = make_float2((float)v.x, (float)v.y);
                        if (B16) B16[og] = __floats2half2_rn((float)v.x, (float)v.y);
                    }
                }
            }
        } else {
#pragma unroll
            for (int t = 0; t < NTR; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = 4 * r + lq, c = 16 * t + i;
                    double2 v = make_double2(0.0, 0.0);
                    if (kok && c < Nv) v = S[(size_t)c * cs + ko];
                    sh[t * 256 + i * 16 + (lr ^ i)] = v;
                }
        }
        if constexpr (GRAM) {
            wave_lds_fence();
            // the tile's products in sums of their own
            int p = 0;
#pragma unroll
            for (int i = 0; i < NTR; ++i)
#pragma unroll
                for (int j = i; j < NTR; ++j, ++p) {
                    V4 tr = {0, 0, 0, 0}, ti = {0, 0, 0, 0};
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        const int u = lr * 16 + ((4 * s + lq) ^ lr);
                        const double2 fi = sh[i * 256 + u], fj = sh[j * 256 + u];
                        tr = MF::mac(fi.x, fj.x, tr);
                        ti = MF::mac(fi.x, fj.y, ti);
                        tr = MF::mac(fi.y, fj.y, tr);
                        ti = MF::mac(-fi.y, fj.x, ti);
                    }
                    gr[p] += tr;
                    gi[p] += ti;
                    if (NTR > 2) __builtin_amdgcn_sched_barrier(0);   // bounded register use
                }
            wave_lds_fence();
        }
    }
    if constexpr (GRAM) {
        double* red = (double*)(shx + NX * 64);        // [wavefronts][re, im][64 lanes][4]
        double2* Gs = G + (size_t)ya * Nv * Nv;
        int p = 0;
#pragma unroll
        for (int i = 0; i < NTR; ++i)
#pragma unroll
            for (int j = i; j < NTR; ++j, ++p) {
                __syncthreads();
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    red[w * 512 + lane * 4 + r] = gr[p][r];
                    red[w * 512 + 256 + lane * 4 + r] = gi[p][r];
                }
                __syncthreads();
                for (int e = threadIdx.x; e < 256; e += blockDim.x) {
                    const int c = 16 * i + MF::row(e >> 6, e & 3), d = 16 * j + ((e >> 2) & 15);
                    if (c > d || d >= Nv) continue;
                    double sr = 0.0, si = 0.0;
                    for (int ww = 0; ww < nw; ++ww) {
                        sr += red[ww * 512 + e];
                        si += red[ww * 512 + 256 + e];
                    }
                    Gs[c * Nv + d] = make_double2(sr, si);
                }
            }
    }
}

// G (upper) = R^+ R; Rinv = R^{-1} (upper).  R is formed in LDS.
__global__ void k_chol_inv(int Nv, const double2* __restrict__ G, double2* __restrict__ Rinv, double tol, int* bad) {
    const int ya = blockIdx.x;
    extern __shared__ double2 R[];
    for (int e = threadIdx.x; e < Nv * Nv; e += blockDim.x) R[e] = G[(size_t)ya * Nv * Nv + e];
    __syncthreads();
    double2* X = Rinv + (size_t)ya * Nv * Nv;
    __shared__ double diag;
    for (int j = 0; j < Nv; ++j) {
        if (threadIdx.x == 0) {
            double g0 = R[j * Nv + j].x;
            double s = g0;
            for (int i = 0; i < j; ++i) s -= R[i * Nv + j].x * R[i * Nv + j].x + R[i * Nv + j].y * R[i * Nv + j].y;
            if (!(s > tol * tol * g0) || !(g0 > 0.0)) {
                atomicOr(bad, 1);
                s = 1.0;
            }
            diag = sqrt(s);
            R[j * Nv + j] = make_double2(diag, 0.0);
        }
        __syncthreads();
        for (int k = j + 1 + threadIdx.x; k < Nv; k += blockDim.x) {
            cx<double> s = cmk(R[j * Nv + k].x, R[j * Nv + k].y);
            for (int i = 0; i < j; ++i) {
                cx<double> a = cmk(R[i * Nv + j].x, -R[i * Nv + j].y);
                cx<double> b = cmk(R[i * Nv + k].x, R[i * Nv + k].y);
                s = s - a * b;
            }
            R[j * Nv + k] = make_double2(s.re / diag, s.im / diag);
        }
        __syncthreads();
    }
    for (int d = threadIdx.x; d < Nv; d += blockDim.x) {
        for (int cc = 0; cc < Nv; ++cc) X[cc * Nv + d] = make_double2(0.0, 0.0);
        X[d * Nv + d] = make_double2(1.0 / R[d * Nv + d].x, 0.0);
        for (int cc = d - 1; cc >= 0; --cc) {
            cx<double> s = cmk(0.0, 0.0);
            for (int e = cc + 1; e <= d; ++e)
                cmac(s, cmk(R[cc * Nv + e].x, R[cc * Nv + e].y), cmk(X[e * Nv + d].x, X[e * Nv + d].y));
            double rd = R[cc * Nv + cc].x;
            X[cc * Nv + d] = make_double2(-s.re / rd, -s.im / rd);
        }
    }
}

// ---------------------------------------------------------------------------
// restrict / prolong
// ---------------------------------------------------------------------------
// The products below are GEMMs with one long side: per (block, chirality) the
// basis is a matrix of Nv rows and K = 6 Vb contiguous columns k = (s'col, l),
// the other operand has up to 16 right-hand sides in a tile.  Both run on the
// matrix cores (16x16x4) so that each basis and field entry is loaded once, in
// the lane that multiplies it; they are bound by memory.

template <typename S, typename R> __device__ __forceinline__ void ld1c(const S* p, R& re, R& im) {
    const cx<R> v = ldc<S, R>(p);
    re = v.re;
    im = v.im;
}

// coarse[r][y][p] = sum_k conj(B[y][p][k]) fine[r][6 alpha(p) + s'col][y*Vb + l]
// grid (V1, 2 chiralities, ceil(nrhs/16)).  Rows p in NTR tiles of 16; the K
// columns in chunks of 16 dealt round-robin to the wavefronts, whose partial
// tiles are added in LDS in wave order.  Lane (lr, lq) takes four columns of a
// chunk: VEC (FP32 fields with Vb % 4 == 0 and 16-byte alignment) the
// contiguous 4 lq + s, else lq + 4 s, where the four lq of a row read one
// contiguous piece (FP64: 64 bytes).  One chunk in flight: two or four (more
// loads, more lines of the 16 rows open) cost 5-20 %.  48 x 24^3, 4^4 blocks,
// 24 vectors, 12 right-hand sides, against chunks of lane-contiguous columns in
// every precision: FP16 basis 422 -> 382 us, FP32 522 -> 450, FP64 894 -> 855;
// 18 x 12^3, 3^4 blocks, 10 vectors, 5 right-hand sides in FP64, against the
// block staged in LDS and multiplied on the vector units: 117 -> 22 us.
template <typename R, typename BS, int NTR, bool VEC>
__global__ __launch_bounds__(512) void k_restrict(Geo g, int Nv, const BS* __restrict__ B,
                                                  const typename VT<R>::c2* __restrict__ fine,
                                                  typename VT<R>::c2* __restrict__ coarse, int nrhs) {
    typedef typename VT<R>::c2 C2;
    typedef typename Mfma<R>::v4 V4;
    extern __shared__ char shraw[];
    R* red = (R*)shraw;                       // [waves][re, im][64 lanes][4]
    const int y = blockIdx.x, a = blockIdx.y, n0 = blockIdx.z * 16;
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6, lane = threadIdx.x & 63;
    const int lr = lane & 15, lq = lane >> 4;
    const int Vb = g.Vb, K = 6 * Vb, nc = 2 * Nv;
    const size_t V = g.V;
    // rows past Nv and right-hand sides past nrhs repeat the last one: their results are not written
    const BS* Bp[NTR];
#pragma unroll
    for (int t = 0; t < NTR; ++t)
        Bp[t] = B + ((size_t)(y * 2 + a) * Nv + (t * 16 + lr < Nv ? t * 16 + lr : Nv - 1)) * K;
    const C2* F = fine + ((size_t)(n0 + lr < nrhs ? n0 + lr : nrhs - 1) * 12 + 6 * a) * V + (size_t)y * Vb;
    V4 cr[NTR], ci[NTR];
#pragma unroll
    for (int t = 0; t < NTR; ++t) {
        cr[t] = V4{0, 0, 0, 0};
        ci[t] = V4{0, 0, 0, 0};
    }
    const int nfull = K / 16, nchunk = (K + 15) / 16;
    for (int q = w; q < nchunk; q += nw) {
        R fr[4], fi[4], br[NTR][4], bi[NTR][4];
        if (q < nfull) {
            if constexpr (VEC) {
                const int k = q * 16 + 4 * lq;
                ld4c(F + col_off(k, Vb, V), fr, fi);
#pragma unroll
                for (int t = 0; t < NTR; ++t) ld4c(Bp[t] + k, br[t], bi[t]);
            } else {
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const int k = q * 16 + lq + 4 * s;
                    ld1c<C2, R>(F + col_off(k, Vb, V), fr[s], fi[s]);
#pragma unroll
                    for (int t = 0; t < NTR; ++t) ld1c<BS, R>(Bp[t] + k, br[t][s], bi[t][s]);
                }
            }
        } else {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int k = q * 16 + (VEC ? 4 * lq + s : lq + 4 * s);
                fr[s] = fi[s] = (R)0;
                if (k < K) ld1c<C2, R>(F + col_off(k, Vb, V), fr[s], fi[s]);
#pragma unroll
                for (int t = 0; t < NTR; ++t) {
                    br[t][s] = bi[t][s] = (R)0;
                    if (k < K) ld1c<BS, R>(Bp[t] + k, br[t][s], bi[t][s]);
                }
            }
        }
#pragma unroll
        for (int t = 0; t < NTR; ++t) {
            // conj(b) f; FP64: a step's products in sums of their own
            V4 tr = sizeof(R) == 8 ? V4{0, 0, 0, 0} : cr[t], ti = sizeof(R) == 8 ? V4{0, 0, 0, 0} : ci[t];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                tr = Mfma<R>::mac(br[t][s], fr[s], tr);
                tr = Mfma<R>::mac(bi[t][s], fi[s], tr);
                ti = Mfma<R>::mac(br[t][s], fi[s], ti);
                ti = Mfma<R>::mac(-bi[t][s], fr[s], ti);
            }
            cr[t] = sizeof(R) == 8 ? cr[t] + tr : tr;
            ci[t] = sizeof(R) == 8 ? ci[t] + ti : ti;
            if (sizeof(R) == 8) __builtin_amdgcn_sched_barrier(0);   // bounded register use
        }
    }
    // thread -> (row p, rhs n) of a tile, p fastest
    const int pl = threadIdx.x & 15, nl = (threadIdx.x >> 4) & 15;
    const int src = (sizeof(R) == 8 ? ((pl & 3) * 16 + nl) * 4 + (pl >> 2) : ((pl >> 2) * 16 + nl) * 4 + (pl & 3));
#pragma unroll
    for (int t = 0; t < NTR; ++t) {
        R* o = red + (size_t)w * 512 + lane * 4;
        if (t) __syncthreads();
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            o[j] = cr[t][j];
            o[256 + j] = ci[t][j];
        }
        __syncthreads();
        if (threadIdx.x < 256 && t * 16 + pl < Nv && n0 + nl < nrhs) {
            R sr = 0, si = 0;
            for (int ww = 0; ww < nw; ++ww) {
                sr += red[ww * 512 + src];
                si += red[ww * 512 + 256 + src];
            }
            coarse[((size_t)(n0 + nl) * g.V1 + y) * nc + a * Nv + t * 16 + pl] = C2{sr, si};
        }
    }
}

// fine[r][6a + s'col][y*Vb + l] = sum_c B[y][a][c][k] coarse[r][y][a*Nv + c]
// grid (V1, 2 chiralities, groups of right-hand sides x ns).  The coarse
// vectors stay in registers (NS steps of four basis vectors; zero past Nv);
// each wavefront walks tiles of 16 W columns, lane lr the W columns from
// W lr on, so that a row of 16 lanes reads and writes 16 W contiguous entries.
// W = 4 (FP32 fields) needs Vb % 4 == 0 and 16-byte alignment.  At the rate of
// a copy: sizes as above, against one thread a site on the vector units, FP16
// basis 461 -> 318 us (4.6 TB/s), FP32 531 -> 520, FP64 1031 -> 860; 3^4
// blocks, FP64: 38 -> 18 us; 8^4, 4^4 blocks, 8 vectors, one right-hand side:
// 15 -> 5 us (ns workgroups a block).  A kernel for every number of steps: with
// 3, 5, 6, 8 and 16 alone, on 48 x 24^3, FP16 basis, 4 right-hand sides, 16 vectors
// took 194 instead of 167 us, 36 took 557 instead of 335.
template <typename R, typename BS, int NS, int W>
__global__ __launch_bounds__(256) void k_prolong(Geo g, int Nv, const BS* __restrict__ B,
                                                 const typename VT<R>::c2* __restrict__ coarse,
                                                 typename VT<R>::c2* __restrict__ fine, int nrhs, int ns) {
    typedef typename VT<R>::c2 C2;
    typedef typename Mfma<R>::v4 V4;
    const int y = blockIdx.x, a = blockIdx.y, ng = blockIdx.z / ns, n0 = ng * 16;
    const int w = (threadIdx.x >> 6) + 4 * (blockIdx.z - ng * ns), lane = threadIdx.x & 63;
    const int lr = lane & 15, lq = lane >> 4;
    const int Vb = g.Vb, K = 6 * Vb, nc = 2 * Nv;
    const size_t V = g.V;
    R xr[NS], xi[NS];
    const C2* X = coarse + ((size_t)(n0 + lr < nrhs ? n0 + lr : nrhs - 1) * g.V1 + y) * nc + a * Nv;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int c = 4 * s + lq;
        const C2 v = X[c < Nv ? c : Nv - 1];
        xr[s] = c < Nv ? v.x : (R)0;
        xi[s] = c < Nv ? v.y : (R)0;
    }
    const BS* Bya = B + (size_t)(y * 2 + a) * Nv * K;
    C2* F = fine + ((size_t)n0 * 12 + 6 * a) * V + (size_t)y * Vb;
    const int nt = (K + 16 * W - 1) / (16 * W);
    for (int q = w; q < nt; q += 4 * ns) {
        const int k = (q * 16 + lr) * W;
        const bool kok = k < K;
        const BS* bp = Bya + (kok ? k : 0);
        V4 dr[W], di[W];
#pragma unroll
        for (int u = 0; u < W; ++u) {
            dr[u] = V4{0, 0, 0, 0};
            di[u] = V4{0, 0, 0, 0};
        }
        R br[NS][W], bi[NS][W];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int c = 4 * s + lq;
            const BS* p = bp + (size_t)(c < Nv ? c : Nv - 1) * K;
            if constexpr (W == 4) ld4c(p, br[s], bi[s]);
            else ld1c<BS, R>(p, br[s][0], bi[s][0]);
        }
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int u = 0; u < W; ++u) {
                dr[u] = Mfma<R>::mac(xr[s], br[s][u], dr[u]);
                dr[u] = Mfma<R>::mac(-xi[s], bi[s][u], dr[u]);
                di[u] = Mfma<R>::mac(xi[s], br[s][u], di[u]);
                di[u] = Mfma<R>::mac(xr[s], bi[s][u], di[u]);
            }
        if (kok) {
            C2* f = F + col_off(k, Vb, V);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int n = Mfma<R>::row(lq, j);
                if (n0 + n < nrhs) {
                    C2* o = f + (size_t)n * 12 * V;
                    if constexpr (W == 4) {
                        *(float4*)o = make_float4(dr[0][j], di[0][j], dr[1][j], di[1][j]);
                        *(float4*)(o + 2) = make_float4(dr[2][j], di[2][j], dr[3][j], di[3][j]);
                    } else {
                        o[0] = C2{dr[0][j], di[0][j]};
                    }
                }
            }
        }
    }
}

// The same sums for few vectors on a large lattice, one thread per fine site:
// there the matrix cores' time for 16 right-hand sides and a multiple of four
// vectors exceeds that of the bytes.  The coarse vectors of the workgroup's
// blocks lie in LDS, PS_RHS right-hand sides at a time; a coarse value serves
// three basis entries.  48 x 24^3, 4^4 blocks, 5 vectors, 1 / 12 right-hand sides,
// against the matrix cores: FP16 basis 76 -> 46 / 257 -> 211 us, FP32 102 -> 79 /
// 265 -> 227, FP64 188 -> 153 / 438 -> 443.
#define PS_RHS 16
template <typename R, typename BS>
__global__ __launch_bounds__(256) void k_prolong_site(Geo g, int Nv, const BS* __restrict__ B,
                                                      const typename VT<R>::c2* __restrict__ coarse,
                                                      typename VT<R>::c2* __restrict__ fine, int nrhs, int nbw) {
    typedef typename VT<R>::c2 C2;
    extern __shared__ char shraw[];
    C2* cs = (C2*)shraw;                      // [nbw][nc][PS_RHS]
    const int i0 = blockIdx.x * 256, i = i0 + threadIdx.x;
    const int Vb = g.Vb, nc = 2 * Nv, y0 = i0 / Vb, y = i / Vb, l = i - y * Vb;
    const size_t V = g.V;
    for (int r0 = 0; r0 < nrhs; r0 += PS_RHS) {
        const int nr = nrhs - r0 < PS_RHS ? nrhs - r0 : PS_RHS;
        __syncthreads();
        for (int e = threadIdx.x; e < nbw * nc * nr; e += 256) {
            const int r = e % nr, t = e / nr, j = t % nc, yy = y0 + t / nc;
            cs[t * PS_RHS + r] = yy < g.V1 ? coarse[((size_t)(r0 + r) * g.V1 + yy) * nc + j] : C2{0, 0};
        }
        __syncthreads();
        if (i >= g.V) continue;
        const C2* cy = cs + (size_t)(y - y0) * nc * PS_RHS;
        for (int s0 = 0; s0 < 12; s0 += 3) {
            const int a = s0 / 6;
            cx<R> acc[3][PS_RHS];
#pragma unroll
            for (int u = 0; u < 3; ++u)
#pragma unroll
                for (int q = 0; q < PS_RHS; ++q) acc[u][q] = cmk((R)0, (R)0);
            for (int c = 0; c < Nv; ++c) {
                const BS* bp = B + (((size_t)y * nc + a * Nv + c) * 6 + s0 - 6 * a) * Vb + l;
                cx<R> b[3];
#pragma unroll
                for (int u = 0; u < 3; ++u) b[u] = ldc<BS, R>(bp + (size_t)u * Vb);
#pragma unroll
                for (int q = 0; q < PS_RHS; ++q) {
                    if (q < nr) {
                        const cx<R> x = ldc<C2, R>(cy + (a * Nv + c) * PS_RHS + q);
#pragma unroll
                        for (int u = 0; u < 3; ++u) cmac(acc[u][q], b[u], x);
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < PS_RHS; ++q) {
                if (q < nr) {
#pragma unroll
                    for (int u = 0; u < 3; ++u) stc<C2, R>(fine + ((size_t)(r0 + q) * 12 + s0 + u) * V + i, acc[u][q]);
                }
            }
        }
    }
}

// FP32 fields: four columns a lane at once
static bool cols4(const Geo& g, const void* fine) { return g.Vb % 4 == 0 && (uintptr_t)fine % 16 == 0; }

template <typename R, typename BS, bool VEC>
static int restrict_launch(mglma_ctx* c, const BS* B, const void* fine, void* coarse, int nrhs) {
    typedef typename VT<R>::c2 C2;
    const Geo& g = c->geo;
    const dim3 grid(g.V1, 2, (nrhs + 15) / 16);
    // few blocks: eight wavefronts share a block's columns (16 blocks, one right-hand side: 18 -> 12 us; 192
    // blocks, R and T of 12 FP16 78 -> 66), in FP32 with at least two chunks of columns for each up to 511 blocks (288
    // blocks of 4^4, 16 vectors, 1 / 12 / 20 right-hand sides: FP16 basis 34 -> 29 / 37 -> 30 / 50 -> 48 us, FP32 36 ->
    // 31 / 39 -> 34 / 57 -> 57; FP64 on 384 blocks of 3^4, 10 vectors, 5: R and T 42 with four, 47 with eight).  From 512
    // blocks on four: 20 there 73 against 80.  Not by the number of right-hand sides, as the order of the sums depends on
    // it (192 blocks, 20 FP16 / FP64: 106 -> 96 / 234 -> 245).
    const int nw = g.V1 < (sizeof(R) == 4 && 6 * g.Vb >= 256 ? 512 : 256) ? 8 : 4;
    const size_t shb = (size_t)nw * 512 * sizeof(R);
    switch ((c->Nv + 15) / 16) {
#define CASE(N)                                                                                                   \
    case N:                                                                                                       \
        hipLaunchKernelGGL((k_restrict<R, BS, N, VEC>), grid, dim3(64 * nw), shb, c->stream, g, c->Nv, B,         \
                           (const C2*)fine, (C2*)coarse, nrhs);                                                   \
        break;
        CASE(1) CASE(2) CASE(3) CASE(4)
#undef CASE
        default: return MGLMA_ERR_SHAPE;
    }
    HIP_TRY(hipGetLastError());
    return MGLMA_OK;
}

int mg_restrict(mglma_ctx* c, int prec, const void* fine, void* coarse, int nrhs) {
    if (nrhs <= 0) return MGLMA_OK;
    const bool v = cols4(c->geo, fine);
    if (prec == MGLMA_F16) {
        // FP32 fields, FP16 basis (four columns at once), else the FP32 basis
        if (v) return restrict_launch<float, __half2, true>(c, c->B16, fine, coarse, nrhs);
        prec = MGLMA_F32;
    }
    if (prec == MGLMA_F64) return restrict_launch<double, double2, false>(c, c->B64, fine, coarse, nrhs);
    if (prec != MGLMA_F32) return MGLMA_ERR_ARG;
    MG_TRY(mg_need_b32(c));
    if (v) return restrict_launch<float, float2, true>(c, c->B32, fine, coarse, nrhs);
    return restrict_launch<float, float2, false>(c, c->B32, fine, coarse, nrhs);
}

template <typename R, typename BS, int W>
static int prolong_launch(mglma_ctx* c, const BS* B, const void* coarse, void* fine, int nrhs) {
    typedef typename VT<R>::c2 C2;
    const Geo& g = c->geo;
    // Few vectors on a large lattice; by Nv, V and Vb alone, as the order of the sums goes with it.  With up to 131072
    // sites the matrix cores win (65536, 4^4 blocks, 5 vectors, 5 right-hand sides, FP16 basis: 14 against 21 us), and
    // with seven vectors on some of the larger ones (294912 sites, FP16: 8 %).
    const int nbw = 255 / g.Vb + 2;           // blocks that 256 sites can touch
    const size_t shb = (size_t)nbw * c->nc * PS_RHS * sizeof(C2);
    if (c->Nv <= 6 && g.V > 131072 && shb <= 64 * 1024) {
        hipLaunchKernelGGL((k_prolong_site<R, BS>), dim3((g.V + 255) / 256), dim3(256), shb, c->stream, g, c->Nv, B,
                           (const C2*)coarse, (C2*)fine, nrhs, nbw);
        HIP_TRY(hipGetLastError());
        return MGLMA_OK;
    }
    const int ng = (nrhs + 15) / 16, nt = (6 * g.Vb + 16 * W - 1) / (16 * W);
    // few blocks: ns workgroups share a block's columns, at least four tiles (one a wavefront) each
    long long ns = (1024 + 2LL * g.V1 * ng - 1) / (2LL * g.V1 * ng);
    if (ns > (nt + 3) / 4) ns = (nt + 3) / 4;
    const dim3 grid(g.V1, 2, (unsigned)(ng * ns));
#define LAUNCH(NS)                                                                                              \
    hipLaunchKernelGGL((k_prolong<R, BS, NS, W>), grid, dim3(256), 0, c->stream, g, c->Nv, B, (const C2*)coarse, \
                       (C2*)fine, nrhs, (int)ns)
    switch ((c->Nv + 3) / 4) {
        case 1: LAUNCH(1); break;
        case 2: LAUNCH(2); break;
        case 3: LAUNCH(3); break;
        case 4: LAUNCH(4); break;
        case 5: LAUNCH(5); break;
        case 6: LAUNCH(6); break;
        case 7: LAUNCH(7); break;
        case 8: LAUNCH(8); break;
        case 9: LAUNCH(9); break;
        case 10: LAUNCH(10); break;
        case 11: LAUNCH(11); break;
        case 12: LAUNCH(12); break;
        case 13: LAUNCH(13); break;
        case 14: LAUNCH(14); break;
        case 15: LAUNCH(15); break;
        case 16: LAUNCH(16); break;
        default: return MGLMA_ERR_SHAPE;
    }
#undef LAUNCH
    HIP_TRY(hipGetLastError());
    return MGLMA_OK;
}

int mg_prolong(mglma_ctx* c, int prec, const void* coarse, void* fine, int nrhs) {
    if (nrhs <= 0) return MGLMA_OK;
    const Geo& g = c->geo;
    // Blocks of few sites with many vectors are refused: the coarse vectors of the blocks that 256 sites touch, past 48
    // KB.  No kernel here needs that; the shapes that T takes do not change with its kernels.
    const size_t cb = prec == MGLMA_F64 ? sizeof(cx<double>) : sizeof(cx<float>);
    if ((size_t)(255 / g.Vb + 2) * c->nc * cb > 48 * 1024) return MGLMA_ERR_SHAPE;
    const bool v = cols4(g, fine);
    switch (prec) {
        case MGLMA_F64: return prolong_launch<double, double2, 1>(c, c->B64, coarse, fine, nrhs);
        case MGLMA_F32:
            MG_TRY(mg_need_b32(c));
            if (v) return prolong_launch<float, float2, 4>(c, c->B32, coarse, fine, nrhs);
            return prolong_launch<float, float2, 1>(c, c->B32, coarse, fine, nrhs);
        case MGLMA_F16:   // FP32 fields, FP16 basis
            if (v) return prolong_launch<float, __half2, 4>(c, c->B16, coarse, fine, nrhs);
            return prolong_launch<float, __half2, 1>(c, c->B16, coarse, fine, nrhs);
        default: return MGLMA_ERR_ARG;
    }
}

extern "C" int mglma_restrict(mglma_ctx* c, int prec, const void* fine, void* coarse, int nrhs) {
    if (!c || !fine || !coarse || nrhs < 0) return MGLMA_ERR_ARG;
    if (!c->have_subspace) return MGLMA_ERR_NO_SUBSPACE;
    return mg_restrict(c, prec, fine, coarse, nrhs);
}

extern "C" int mglma_prolong(mglma_ctx* c, int prec, const void* coarse, void* fine, int nrhs) {
    if (!c || !fine || !coarse || nrhs < 0) return MGLMA_ERR_ARG;
    if (!c->have_subspace) return MGLMA_ERR_NO_SUBSPACE;
    return mg_prolong(c, prec, coarse, fine, nrhs);
}

// ---------------------------------------------------------------------------
// Galerkin operator
// ---------------------------------------------------------------------------
__global__ void k_op_copies(size_t nblk, int nc, const double2* __restrict__ D, double* __restrict__ D64p,
                            float* __restrict__ D32p, bf16_t* __restrict__ Dbf) {
    // planar copies [blk][0 = re, 1 = im][i][j] in FP64, FP32 and BF16
    size_t n = nblk * nc * nc;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x) {
        double2 v = D[e];
        size_t blk = e / ((size_t)nc * nc), ij = e % ((size_t)nc * nc);
        const size_t er = (blk * 2 + 0) * nc * nc + ij, ei = er + (size_t)nc * nc;
        if (D64p) {
            D64p[er] = v.x;
            D64p[ei] = v.y;
        }
        float fr = (float)v.x, fi = (float)v.y;
        if (D32p) {
            D32p[er] = fr;
            D32p[ei] = fi;
        }
        if (Dbf) {
            // round to nearest even
            uint32_t ur = __float_as_uint(fr), ui = __float_as_uint(fi);
            ur += 0x7fff + ((ur >> 16) & 1);
            ui += 0x7fff + ((ui >> 16) & 1);
            Dbf[er] = (bf16_t)(ur >> 16);
            Dbf[ei] = (bf16_t)(ui >> 16);
        }
    }
}

// ---------------------------------------------------------------------------
// coarse gamma matrices (gamma5 gamma_k)_1(y, t): alpha=0 rows c, alpha=1 cols d
//   sum_{x in B_y, x0 = t} sum_col sum_{s',t'} conj(phi_{0c}(s',col)) m_k[s'][t'] phi_{1d}(t',col)
// with m_k = -i sigma_k (the upper-right block of gamma5 gamma_k).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_coarse_gamma(Geo g, int Nv, const double2* __restrict__ B,
                                                      double2* __restrict__ G1) {
    const int y = blockIdx.x / g.b[0], t = blockIdx.x % g.b[0];
    const int Vb = g.Vb, ns = Vb / g.b[0];   // spatial sites per block slice
    const size_t K = (size_t)6 * Vb;
    const double2* P0 = B + ((size_t)y * 2 + 0) * Nv * K;
    const double2* P1 = B + ((size_t)y * 2 + 1) * Nv * K;
    const int nout = 3 * Nv * Nv;
    for (int o = threadIdx.x; o < nout; o += blockDim.x) {
        int k = o / (Nv * Nv), cd = o % (Nv * Nv), cc = cd / Nv, d = cd % Nv;
        cx<double> acc = cmk(0.0, 0.0);
        for (int col = 0; col < 3; ++col) {
            for (int ls = 0; ls < ns; ++ls) {
                int l = t * ns + ls;
                cx<double> a0 = ldc<double2, double>(P0 + ((size_t)cc * 6 + 0 + col) * Vb + l);
                cx<double> a1 = ldc<double2, double>(P0 + ((size_t)cc * 6 + 3 + col) * Vb + l);
                cx<double> b0 = ldc<double2, double>(P1 + ((size_t)d * 6 + 0 + col) * Vb + l);
                cx<double> b1 = ldc<double2, double>(P1 + ((size_t)d * 6 + 3 + col) * Vb + l);
                // (gamma5 gamma_k psi)(s') for the upper spins s' = 0, 1 reads spin tc in {2, 3}
                cx<double> u0, u1;
                {
                    int tc;
                    double cr, ci;
                    gk_row(k + 1, 0, &tc, &cr, &ci);
                    u0 = cmk(cr, ci) * (tc == 2 ? b0 : b1);
                    gk_row(k + 1, 1, &tc, &cr, &ci);
                    u1 = cmk(cr, ci) * (tc == 2 ? b0 : b1);
                }
                cjmac(acc, a0, u0);
                cjmac(acc, a1, u1);
            }
        }
        G1[(((size_t)y * g.b[0] + t) * 3 + k) * Nv * Nv + cd] = make_double2(acc.re, acc.im);
    }
}

// Matrix-core version (v_mfma_f64_16x16x4), one workgroup per (block, time
// slice).  With O_{s s'}[c][d] = sum_{col, l in slice} conj(phi_{0c}(s, col))
// phi_{1d}(s', col) for the four spin pairs (one per wavefront, a GEMM of
// Nv x 3 n_s by 3 n_s x Nv), gamma5 gamma_k being monomial gives
// G_k = sum_s coef_k(s) O_{s, pi_k(s) - 2}.  Lane (lr, lq) takes k runs of
// four consecutive sites, so its operand loads are contiguous (needs the slice
// size n_s % 4 == 0, Nv <= 32).
__global__ __launch_bounds__(256) void k_coarse_gamma_mfma(Geo g, int Nv, const double2* __restrict__ B,
                                                           double2* __restrict__ G1) {
    typedef Mfma<double>::v4 V4;
    extern __shared__ double2 Os[];                    // [4 spin pairs][Nv][Nv]
    const int y = blockIdx.x / g.b[0], t = blockIdx.x % g.b[0];
    const int Vb = g.Vb, ns = Vb / g.b[0];
    const size_t K6 = (size_t)6 * Vb;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 15, lq = lane >> 4;
    const int s0 = w >> 1, s1 = w & 1;                 // spin inside chirality 0 / 1
    const int ntr = (Nv + 15) / 16;
    const double2* P0 = B + ((size_t)y * 2 + 0) * Nv * K6 + (size_t)t * ns;
    const double2* P1 = B + ((size_t)y * 2 + 1) * Nv * K6 + (size_t)t * ns;
    V4 cr[2][2], ci[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            cr[a][b] = V4{0, 0, 0, 0};
            ci[a][b] = V4{0, 0, 0, 0};
        }
    const int K = 3 * ns;
    for (int kc = 0; kc < K; kc += 16) {
        const int kb = kc + 4 * lq;
        const bool kok = kb < K;
        const int col = kok ? kb / ns : 0, ls = kok ? kb - col * ns : 0;
        double ar[2][4], ai[2][4], br[2][4], bi[2][4];
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
            const int c = 16 * tt + lr;
            if (tt < ntr && kok && c < Nv) {
                ld4c(P0 + ((size_t)c * 6 + 3 * s0 + col) * Vb + ls, ar[tt], ai[tt]);
                ld4c(P1 + ((size_t)c * 6 + 3 * s1 + col) * Vb + ls, br[tt], bi[tt]);
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) ar[tt][q] = ai[tt][q] = br[tt][q] = bi[tt][q] = 0.0;
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                for (int ct = 0; ct < 2; ++ct) {
                    if (rt < ntr && ct < ntr) {
                        // conj(a) b
                        cr[rt][ct] = Mfma<double>::mac(ar[rt][q], br[ct][q], cr[rt][ct]);
                        cr[rt][ct] = Mfma<double>::mac(ai[rt][q], bi[ct][q], cr[rt][ct]);
                        ci[rt][ct] = Mfma<double>::mac(ar[rt][q], bi[ct][q], ci[rt][ct]);
                        ci[rt][ct] = Mfma<double>::mac(-ai[rt][q], br[ct][q], ci[rt][ct]);
                    }
                }
    }
    const int nn = Nv * Nv;
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) {
            if (rt < ntr && ct < ntr) {
                const int d = 16 * ct + lr;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int c = 16 * rt + Mfma<double>::row(lq, r);
                    if (c < Nv && d < Nv) Os[(size_t)w * nn + c * Nv + d] = make_double2(cr[rt][ct][r], ci[rt][ct][r]);
                }
            }
        }
    __syncthreads();
    for (int o = threadIdx.x; o < 3 * nn; o += blockDim.x) {
        const int k = o / nn, cd = o - k * nn;
        cx<double> acc = cmk(0.0, 0.0);
#pragma unroll
        for (int sp = 0; sp < 2; ++sp) {
            int tc;
            double cre, cim;
            gk_row(k + 1, sp, &tc, &cre, &cim);
            const double2 v = Os[(size_t)(sp * 2 + (tc - 2)) * nn + cd];
            acc = acc + cmk(cre, cim) * cmk(v.x, v.y);
        }
        G1[(((size_t)y * g.b[0] + t) * 3 + k) * nn + cd] = make_double2(acc.re, acc.im);
    }
}

// ---------------------------------------------------------------------------
// ABI: build the subspace
// ---------------------------------------------------------------------------
template <int NTR, bool APPLY, bool GRAM, bool TV>
static int qr_pass(mglma_ctx* c, double2* B, int nsets, int Nv, int K, const double2* tv, const double2* X, double2* G,
                   float2* B32, __half2* B16) {
    const size_t shb = ((APPLY ? 2 * NTR * (NTR + 1) * 64 : 0) + (GRAM ? 4 * NTR * 256 : 0)) * sizeof(double2);
    hipLaunchKernelGGL((k_qr_pass<NTR, APPLY, GRAM, TV>), dim3(nsets), dim3(256), shb, c->stream, c->geo, Nv, K, tv, B,
                       X, G, B32, B16);
    HIP_TRY(hipGetLastError());
    return MGLMA_OK;
}

// Cholesky QR twice, B [nsets][Nv][K]: Gram of the source; apply and Gram of the
// result; apply.  TV: the source is the test vectors, else B itself.
template <int NTR, bool TV>
static int cholqr(mglma_ctx* c, double2* B, int nsets, int Nv, int K, const double2* tv, float2* B32, __half2* B16) {
    const size_t gsz = (size_t)nsets * Nv * Nv * sizeof(double2);
    double2 *Gb, *Rb;
    int* bad;
    MG_TRY(mg_scratch(c, 0, gsz, (void**)&Gb));
    MG_TRY(mg_scratch(c, 1, gsz, (void**)&Rb));
    MG_TRY(mg_scratch(c, 7, 64, (void**)&bad));
    HIP_TRY(hipMemsetAsync(bad, 0, sizeof(int), c->stream));
    const size_t shr = (size_t)Nv * Nv * sizeof(double2);
    MG_TRY((qr_pass<NTR, false, true, TV>(c, B, nsets, Nv, K, tv, nullptr, Gb, nullptr, nullptr)));
    hipLaunchKernelGGL(k_chol_inv, dim3(nsets), dim3(64), shr, c->stream, Nv, (const double2*)Gb, Rb, 3e-7, bad);
    MG_TRY((qr_pass<NTR, true, true, TV>(c, B, nsets, Nv, K, tv, Rb, Gb, nullptr, nullptr)));
    hipLaunchKernelGGL(k_chol_inv, dim3(nsets), dim3(64), shr, c->stream, Nv, (const double2*)Gb, Rb, 3e-7, bad);
    MG_TRY((qr_pass<NTR, true, false, false>(c, B, nsets, Nv, K, nullptr, Rb, nullptr, B32, B16)));
    int hbad = 0;
    HIP_TRY(hipMemcpyAsync(&hbad, bad, sizeof(int), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    return hbad ? MGLMA_ERR_RANK : MGLMA_OK;
}
template <bool TV>
static int cholqr_n(mglma_ctx* c, double2* B, int nsets, int Nv, int K, const double2* tv, float2* B32, __half2* B16) {
    switch ((Nv + 15) / 16) {
        case 1: return cholqr<1, TV>(c, B, nsets, Nv, K, tv, B32, B16);
        case 2: return cholqr<2, TV>(c, B, nsets, Nv, K, tv, B32, B16);
        case 3: return cholqr<3, TV>(c, B, nsets, Nv, K, tv, B32, B16);
        case 4: return cholqr<4, TV>(c, B, nsets, Nv, K, tv, B32, B16);
        default: return MGLMA_ERR_SHAPE;
    }
}

// Cholesky QR, twice, of nsets sets of Nv vectors of K complex each (B
// [nsets][Nv][K], in place, FP64): each set orthonormalised in order with a
// positive real diagonal.  Errors: RANK.
int mg_cholqr_sets(mglma_ctx* c, double2* B, int nsets, int Nv, int K) {
    return cholqr_n<false>(c, B, nsets, Nv, K, nullptr, nullptr, nullptr);
}

extern "C" int mglma_build_subspace(mglma_ctx* c, int Nv, const double* tv) {
    if (!c || !tv) return MGLMA_ERR_ARG;
    if (!c->have_gauge) return MGLMA_ERR_NO_GAUGE;
    const Geo& g = c->geo;
    if (Nv < 1 || Nv > 64 || Nv > 6 * g.Vb) return MGLMA_ERR_ARG;
    mg_free_subspace(c);
    c->Nv = Nv;
    c->nc = 2 * Nv;
    const int nc = c->nc;
    size_t nb = (size_t)g.V * 12 * Nv;
    size_t nd = (size_t)g.V1 * 9 * nc * nc;
    // resident: the FP64 basis (R, T of the FP64 path, the Galerkin build, the
    // coarse gammas), its FP16 copy (the preconditioner's transfers), D_1 and
    // its BF16 copy; the FP32 basis and FP32 D_1 are formed when first used
    MG_TRY(mg_malloc(c, (void**)&c->B64, nb * 16));
    MG_TRY(mg_malloc(c, (void**)&c->B16, nb * 4));
    MG_TRY(mg_malloc(c, (void**)&c->D64, nd * 16));
    MG_TRY(mg_malloc(c, (void**)&c->Dbf, nd * 4));
    MG_TRY(mg_malloc(c, (void**)&c->G1, (size_t)g.V1 * g.b[0] * 3 * Nv * Nv * 16));

    // 1. block-project and chirally split the test vectors and orthonormalise
    //    each (block, chirality) set: Cholesky QR twice (also writes the FP16 copy)
    const int qrc = cholqr_n<true>(c, c->B64, g.V1 * 2, Nv, 6 * g.Vb, (const double2*)tv, c->B32, c->B16);
    if (qrc == MGLMA_ERR_RANK) mg_free_subspace(c);
    MG_TRY(qrc);

    // 2. Galerkin operator, block by block; the forward pieces go to a
    //    temporary of the operator's size, released after the build
    double2* gtmp;
    MG_TRY(mg_malloc(c, (void**)&gtmp, nd * 16));
    int grc = mg_galerkin(c, gtmp);
    if (grc == MGLMA_OK) grc = mg_op_copies(c, (size_t)g.V1 * 9, nc, c->D64, nullptr, nullptr, c->Dbf);
    if (grc == MGLMA_OK && hipStreamSynchronize(c->stream) != hipSuccess) grc = MGLMA_ERR_HIP;
    mg_free(c, gtmp, nd * 16);
    if (grc != MGLMA_OK) { mg_free_subspace(c); return grc; }

    // 3. coarse gamma matrices
    if ((g.Vb / g.b[0]) % 4 == 0 && Nv <= 32)
        hipLaunchKernelGGL(k_coarse_gamma_mfma, dim3(g.V1 * g.b[0]), dim3(256), (size_t)4 * Nv * Nv * sizeof(double2),
                           c->stream, g, Nv, c->B64, c->G1);
    else
        hipLaunchKernelGGL(k_coarse_gamma, dim3(g.V1 * g.b[0]), dim3(256), 0, c->stream, g, Nv, c->B64, c->G1);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(c->stream));

    // 4. even-odd reduced form of D_1 where the coarse lattice allows it
    MG_TRY(mg_eo_setup(c));
    c->have_subspace = true;
    return MGLMA_OK;
}

int mg_op_copies(mglma_ctx* c, size_t nblk, int nc, const double2* D, double* D64p, float* D32p, bf16_t* Dbf) {
    hipLaunchKernelGGL(k_op_copies, dim3(2048), dim3(256), 0, c->stream, nblk, nc, D, D64p, D32p, Dbf);
    HIP_TRY(hipGetLastError());
    return MGLMA_OK;
}

int mg_need_b32(mglma_ctx* c) {
    if (c->B32) return MGLMA_OK;
    const size_t nb = (size_t)c->geo.V * 12 * c->Nv;
    MG_TRY(mg_malloc(c, (void**)&c->B32, nb * 8));
    return mg_convert(c, MGLMA_F64, c->B64, MGLMA_F32, c->B32, nb, 1, nullptr, 0);
}

int mg_need_d32(mglma_ctx* c) {
    if (c->D32p) return MGLMA_OK;
    const size_t nd = (size_t)c->geo.V1 * 9 * c->nc * c->nc;
    MG_TRY(mg_malloc(c, (void**)&c->D32p, nd * 8));
    return mg_op_copies(c, (size_t)c->geo.V1 * 9, c->nc, c->D64, nullptr, c->D32p, nullptr);
}

// ---------------------------------------------------------------------------
// exports (tests)
// ---------------------------------------------------------------------------
__global__ void k_export_basis(Geo g, int Nv, const double2* __restrict__ B, double2* __restrict__ out) {
    // out[y][j][l][s][col]
    const int nc = 2 * Nv;
    size_t n = (size_t)g.V1 * nc * g.Vb * 12;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x) {
        int sc = (int)(e % 12);
        size_t t = e / 12;
        int l = (int)(t % g.Vb);
        t /= g.Vb;
        int j = (int)(t % nc);
        int y = (int)(t / nc);
        int a = j / Nv, s = sc / 3, col = sc % 3;
        double2 v = make_double2(0.0, 0.0);
        if (s / 2 == a) v = B[(((size_t)y * nc + j) * 6 + (s % 2) * 3 + col) * g.Vb + l];
        out[e] = v;
    }
}

extern "C" int mglma_export_basis(mglma_ctx* c, double* out) {
    if (!c || !out) return MGLMA_ERR_ARG;
    if (!c->have_subspace) return MGLMA_ERR_NO_SUBSPACE;
    hipLaunchKernelGGL(k_export_basis, dim3(2048), dim3(256), 0, c->stream, c->geo, c->Nv, c->B64, (double2*)out);
    HIP_TRY(hipGetLastError());
    return MGLMA_OK;
}

extern "C" int mglma_export_coarse_op(mglma_ctx* c, double* out) {
    if (!c || !out) return MGLMA_ERR_ARG;
    if (!c->have_subspace) return MGLMA_ERR_NO_SUBSPACE;
    size_t nd = (size_t)c->geo.V1 * 9 * c->nc * c->nc;
    return mg_copy(c, out, c->D64, nd * 16);
}

extern "C" int mglma_export_coarse_gammas(mglma_ctx* c, double* out) {
    if (!c || !out) return MGLMA_ERR_ARG;
    if (!c->have_subspace) return MGLMA_ERR_NO_SUBSPACE;
    size_t n = (size_t)c->geo.V1 * c->geo.b[0] * 3 * c->Nv * c->Nv;
    return mg_copy(c, out, c->G1, n * 16);
}
