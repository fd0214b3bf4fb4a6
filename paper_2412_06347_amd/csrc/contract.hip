// Contractions of the isovector vector correlator.
//
// All of them are sums over a time slice of bilinears psi_b(x)^+ G_k psi_a(x)
// with G_k = gamma5 gamma_k (k = 1..3), weighted by a source-side spin factor:
//  * point source (eq:tmr with one source position y):
//      C(y0+t, y0) = -1/3 sum_k sum_{a,b} (gamma_k gamma5)_{ab} sum_x psi^j_b(x)^+ G_k psi^i_a(x),
//    a, b = (spin, colour) source indices with equal colour, using
//    S(y,x) = gamma5 S(x,y)^+ gamma5;
//  * stochastic spin-diluted wall source (eq:C_stoch2):
//      G^n(t_n+t, t_n) = -1/(3 L^3) sum_k sum_s conj((gamma5 gamma_k^+)_{s's}) sum_x
//                        (S_j eta^{(s')})^+ G_k (S_i eta^{(s)}),  s' the row of column s;
//  * the same on coarse vectors through (gamma5 gamma_k)_1 per block time
//    slice (eq:coarse:gamma), so fields T c are never formed.
// In the chiral basis G_k = [[0, m_k], [m_k, 0]] with m_k = -i sigma_k, one
// entry per row and column.
//
// Each workgroup writes one partial sum per time slice; a second pass adds the
// partials of every time slice in a fixed order, so the result does not depend
// on launch or batch composition.
#include "mglma_internal.h"

#include <mutex>

// Both kinds have the same form: with columns (source spin sa, source colour c;
// c = 0 alone for the wall source) and sb the column of row sa of G_k,
//   scale * sum_k sum_{sa, c} G_k[sa][sb] psi^j_{(sb,c)}(x)^+ G_k psi^i_{(sa,c)}(x),
// scale = 1/3 (point: (gamma_k gamma5)_{ab} = -G_k[a][b]) or 1/(3 L^3) (wall:
// G_k is anti-Hermitian, -conj(G_k[s'][s]) = G_k[s][s']).
// G_k[s][t] is non-zero at t = gk_col(k, s) only; the products of two entries
// of one G_k are real: G_k[s][.] G_k[s'][.] = gk_sign(k, s, s').
__device__ constexpr int gk_col(int k, int s) { return k < 3 ? 3 - s : s ^ 2; }
__device__ constexpr double gk_sign(int k, int s, int t) {
    return k == 1 ? -1.0 : ((k == 2) == ((s ^ t) & 1) ? -1.0 : 1.0);
}

// ---------------------------------------------------------------------------
// Source-averaged two-point functions and level terms (eq:C_ij level sums,
// eq:cdecomp, eq:C_stoch, eq:timetrans).
//
// Stage 1 (one launch per route): workgroup (x0, chunk, source n, pair p)
// adds the weighted densities of the sites of time slice x0 in its chunk
// and writes one partial sum part[p][n][x0][chunk].  The chunking depends on
// the lattice only, so a source's partials do not depend on which other
// sources share the launch.
// Stage 2: one thread per (row, t) adds the partials of every source in
// source order at x0 = (t_src[n] + t) mod L0, forms the level difference
// G(P_row) - G(P_row+1) where asked, and scales by 1/nsrc.
// ---------------------------------------------------------------------------
#define LV_MAXPAIR 8
#define LV_MAXCHUNK 32
#define LV_MAXSRC 512

struct PairSet {
    const double2* pi[LV_MAXPAIR];
    const double2* pj[LV_MAXPAIR];
};
struct SrcTimes {
    int t[LV_MAXSRC];
};

// chunks per time slice (at most LV_MAXCHUNK): whole passes of 256 threads over
// the fine sites of a slice, single coarse sites where there are that few
static int fine_chunks(const Geo& g) {
    const int n = (g.V3 + 255) / 256, per = (n + LV_MAXCHUNK - 1) / LV_MAXCHUNK;
    return (n + per - 1) / per;
}
static int coarse_chunks(const Geo& g) {
    const int n = g.V1 / g.L1[0];
    return n > LV_MAXCHUNK ? LV_MAXCHUNK : n;
}

// workgroup sum of one complex per thread (256 threads), fixed order
__device__ __forceinline__ double2 wg_sum256(double re, double im) {
    __shared__ double sre[256], sim[256];
    sre[threadIdx.x] = re;
    sim[threadIdx.x] = im;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            sre[threadIdx.x] += sre[threadIdx.x + o];
            sim[threadIdx.x] += sim[threadIdx.x + o];
        }
        __syncthreads();
    }
    return make_double2(sre[0], sim[0]);
}

// grid (L0 * nchunk, nsrc, npair), block 256; fields of source n start at
// column n * 4 NCS of each piece (column sa * NCS + c, NCS source colours);
// part index ((pair0 + p) * nsrc + n) * L0 + x0, times LV_MAXCHUNK, plus the
// chunk.  SAME: psi_i = psi_j (the level rows), each field read once.
//
// Bound: HBM, the 4 NCS fields of a source read once (1.53 GB for the 12
// columns on 48 x 24^3).  For one source colour c and one sink colour the sum
// only couples the 4 x 4 matrix of (source spin, sink spin) entries, so a
// thread loads those 16 values of its site in one run of independent
// coalesced loads and forms all 3 x 4 x 4 products from registers.  (Walking
// the 36 (k, sa, c) terms and loading both fields of each re-read every value
// six times through the caches: 1.34 ms; this form 0.26 ms,
// 5.8 TB/s.)  Sums of their own for every weight, colour pair, site and chunk, the
// scale last: the error of a slice (Gaussian fields, 24^3 sites, against long
// double, per sqrt(number of products)) is 4.9e-16, with one running sum a thread
// over weights, colours and sites 1.1e-15, of the 36 terms' form 8.5e-16; same time.
template <int NCS, bool SAME>
__global__ __launch_bounds__(256) void k_fine_slice_part(Geo g, int nchunk, int nsrc, int pair0, PairSet P,
                                                         double scale, double2* __restrict__ part) {
    const int x0 = blockIdx.x / nchunk, ch = blockIdx.x - x0 * nchunk;
    const int n = blockIdx.y, p = blockIdx.z;
    const int b0 = g.b[0], y0 = x0 / b0, l0 = x0 - y0 * b0;
    const int b123 = g.b[1] * g.b[2] * g.b[3], rowsz = g.V1 / g.L1[0];
    const long tot = (long)rowsz * b123;
    const int e0 = (int)(tot * ch / nchunk), e1 = (int)(tot * (ch + 1) / nchunk);
    const size_t V = g.V;
    const double2* pi = P.pi[p] + (size_t)n * 4 * NCS * 12 * V;
    const double2* pj = P.pj[p] + (size_t)n * 4 * NCS * 12 * V;
    double re = 0.0, im = 0.0;
    for (int e = e0 + (int)threadIdx.x; e < e1; e += 256) {
        const int kb = e / b123, lo = e - kb * b123;
        const int i = (y0 * rowsz + kb) * g.Vb + l0 * b123 + lo;
        double sr = 0.0, si = 0.0;
#pragma unroll 1
        for (int q = 0; q < 3 * NCS; ++q) {
            const int c = q / 3, col = q - 3 * c;
            const size_t off = ((size_t)c * 12 + col) * V + i;
            double2 A[4][4], B[4][4];
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int sp = 0; sp < 4; ++sp) A[s][sp] = pi[off + (size_t)(s * NCS * 12 + 3 * sp) * V];
            if (!SAME) {
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int sp = 0; sp < 4; ++sp) B[s][sp] = pj[off + (size_t)(s * NCS * 12 + 3 * sp) * V];
            }
            double qr = 0.0, qi = 0.0;
#pragma unroll
            for (int k = 1; k <= 3; ++k)
#pragma unroll
                for (int sa = 0; sa < 4; ++sa) {
                    double kr = 0.0, ki = 0.0;
#pragma unroll
                    for (int sp = 0; sp < 4; ++sp) {
                        const double2 b = SAME ? A[gk_col(k, sa)][sp] : B[gk_col(k, sa)][sp];
                        const double2 a = A[sa][gk_col(k, sp)];
                        const double sg = gk_sign(k, sa, sp);
                        kr = fma(sg * b.x, a.x, kr);
                        kr = fma(sg * b.y, a.y, kr);
                        if (!SAME) {
                            ki = fma(sg * b.x, a.y, ki);
                            ki = fma(-sg * b.y, a.x, ki);
                        }
                    }
                    qr += kr;
                    qi += ki;
                }
            sr += qr;
            si += qi;
        }
        re += sr;
        im += si;
    }
    // (SAME: the sum is real; the product carries NaN and infinity into both parts)
    const double2 v = wg_sum256(re, SAME ? 0.0 * re : im);
    if (threadIdx.x == 0)
        part[((((size_t)(pair0 + p) * nsrc + n) * g.L[0] + x0) * LV_MAXCHUNK) + ch] =
            make_double2(scale * v.x, scale * v.y);
}

// Coarse pieces on the FP64 matrix cores (v_mfma_f64_16x16x4): with Gb the
// stored alpha = 0 x alpha = 1 block of (gamma5 gamma_k)_1(y, t),
//   u^+ Gamma v = u_0^+ Gb v_1 - conj(v_0^+ Gb u_1),
// and S = [u_0 of 16 columns]^+ Gb is a GEMM whose rows are 16 / (4 NCS)
// (piece, source) groups.  One workgroup per (block row y0, chunk of its
// coarse sites, row tile), the tiles of a chunk back to back on one XCD;
// wavefront w takes the block time slice w % b0 (every ns-th site of the
// chunk when b0 <= 2).  MFMA lane (lr, lq) supplies A[row lr][4 s + lq] and
// B[4 s + lq][col lr], so a step of NS reads four rows of Gb whole; the lane
// then weights its own columns of S with v_1.  SAME (u = v): the second
// product is minus the conjugate of the first one with the columns exchanged,
// so the sum is twice the real part of the first.
//
// Bound: HBM, 3 b0 Nv^2 complex of Gb per coarse site (287 MB on 48 x 24^3,
// Nv = 24), and about as long in the matrix cores for two row tiles.  NS >= Nv
// / 4 steps are unrolled, so that the loads of a whole Gb are in flight.  Two
// pieces of 12 columns there: 1.14 ms with the Nv x Nv products spread over
// lanes and summed by shuffles per term, 0.51 ms with T = Gb v_1 (16 rows of Gb
// in 64-byte runs, two steps in flight), 0.18 ms here.
template <int NCS, bool SAME, int NS>
__global__ __launch_bounds__(256) void k_coarse_slice_part(Geo g, int Nv, int nchunk, int nsrc, int npn, int pair0,
                                                           const double2* __restrict__ G1, PairSet P, double scale,
                                                           double2* __restrict__ part) {
    typedef Mfma<double>::v4 V4;
    constexpr int NCOL = 4 * NCS, GPT = 16 / NCOL, RT = (NS + 3) / 4, GS = NS <= 8 ? NS : 4;
    __shared__ double2 red[4][GPT];
    int item, tile;
    if (!site_tile(g.L1[0] * nchunk, (npn + GPT - 1) / GPT, &item, &tile)) return;
    const int y0 = item / nchunk, ch = item - y0 * nchunk;
    const int b0 = g.b[0], rowsz = g.V1 / g.L1[0];
    const int ys0 = (int)((long)rowsz * ch / nchunk), ys1 = (int)((long)rowsz * (ch + 1) / nchunk);
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 15, lq = lane >> 4;
    const int nc = 2 * Nv;
    const size_t cs = (size_t)g.V1 * nc, nn = (size_t)Nv * Nv;
    const int nsub = b0 >= 4 ? 1 : 4 / b0;       // wavefronts per time slice
    const int sub = b0 >= 4 ? 0 : w / b0;
    // row lr of the tile: group (piece, source) tile * GPT + lr / NCOL, source column lr % NCOL
    const int pl = tile * GPT + lr / NCOL;
    const bool con = lr < GPT * NCOL && pl < npn;
    const size_t ao = con ? (size_t)(pl % nsrc * NCOL + lr % NCOL) * cs : 0;
    const double2* uj = P.pj[con ? pl / nsrc : 0] + ao;
    const double2* vi = P.pi[con ? pl / nsrc : 0] + ao;
    // result register r: row lq + 4 r, of group r / NCS and source column lq + 4 (r % NCS)
    const double2 *wi_[GPT], *wj_[GPT];
#pragma unroll
    for (int q = 0; q < GPT; ++q) {
        const int pn = tile * GPT + q < npn ? tile * GPT + q : npn - 1;
        wi_[q] = P.pi[pn / nsrc] + (size_t)(pn % nsrc) * NCOL * cs + Nv;
        wj_[q] = P.pj[pn / nsrc] + (size_t)(pn % nsrc) * NCOL * cs + Nv;
    }
    for (int t0 = 0; t0 < b0; t0 += 4) {
        const int t = b0 >= 4 ? t0 + w : w % b0;
        double re[GPT], im[GPT];
#pragma unroll
        for (int q = 0; q < GPT; ++q) re[q] = im[q] = 0.0;
        if (t < b0 && sub < nsub) {
            for (int ys = ys0 + sub; ys < ys1; ys += nsub) {
                const int y = y0 * rowsz + ys;
                double ar[NS], ai[NS], br[SAME ? 1 : NS], bi[SAME ? 1 : NS];
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    const int c = 4 * s + lq;
                    const bool cok = con && c < Nv;
                    const uint32_t o = (uint32_t)y * (uint32_t)nc + (cok ? c : 0);
                    const double2 u = uj[o];
                    ar[s] = cok ? u.x : 0.0;
                    ai[s] = cok ? u.y : 0.0;
                    if (!SAME) {
                        const double2 v = vi[o];
                        br[s] = cok ? v.x : 0.0;
                        bi[s] = cok ? v.y : 0.0;
                    }
                }
#pragma unroll 1
                for (int k = 1; k <= 3; ++k) {
                    const double2* Gb = G1 + (((size_t)y * b0 + t) * 3 + (k - 1)) * nn;
                    V4 cr[RT], ci[RT], dr[SAME ? 1 : RT], di[SAME ? 1 : RT];
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) {
                        cr[rt] = ci[rt] = V4{0, 0, 0, 0};
                        if (!SAME) dr[rt] = di[rt] = V4{0, 0, 0, 0};
                    }
#pragma unroll
                    for (int s0 = 0; s0 < NS; s0 += GS) {
                        double2 gv[GS][RT];
#pragma unroll
                        for (int s = 0; s < GS; ++s)
#pragma unroll
                            for (int rt = 0; rt < RT; ++rt) {
                                const int c = 4 * (s0 + s) + lq, d = 16 * rt + lr;
                                gv[s][rt] = Gb[(c < Nv ? c : Nv - 1) * Nv + (d < Nv ? d : Nv - 1)];
                            }
#pragma unroll
                        for (int s = 0; s < GS; ++s)
#pragma unroll
                            for (int rt = 0; rt < RT; ++rt) {
                                const double2 b = gv[s][rt];
                                cr[rt] = Mfma<double>::mac(ar[s0 + s], b.x, cr[rt]);
                                cr[rt] = Mfma<double>::mac(ai[s0 + s], b.y, cr[rt]);
                                ci[rt] = Mfma<double>::mac(ar[s0 + s], b.y, ci[rt]);
                                ci[rt] = Mfma<double>::mac(-ai[s0 + s], b.x, ci[rt]);
                                if (!SAME) {
                                    dr[rt] = Mfma<double>::mac(br[s0 + s], b.x, dr[rt]);
                                    dr[rt] = Mfma<double>::mac(bi[s0 + s], b.y, dr[rt]);
                                    di[rt] = Mfma<double>::mac(br[s0 + s], b.y, di[rt]);
                                    di[rt] = Mfma<double>::mac(-bi[s0 + s], b.x, di[rt]);
                                }
                            }
                        if (GS < NS) __builtin_amdgcn_sched_barrier(0);   // bounded register use
                    }
                    // row of spin s, partner of spin sp: S v_1 (partner's v for u_0, partner's u for v_0)
#pragma unroll
                    for (int r = 0; r < GPT * NCS; ++r) {
                        const int q = r / NCS, col = lq + 4 * (r % NCS), sp = col / NCS, sc = col - sp * NCS;
                        const int pt = gk_col(k, sp);
                        const uint32_t o = (uint32_t)y * (uint32_t)nc;
                        const double2* pv = wi_[q] + (size_t)(pt * NCS + sc) * cs + o;
                        const double2* pu = wj_[q] + (size_t)(pt * NCS + sc) * cs + o;
                        cx<double> x = cmk(0.0, 0.0), x2 = cmk(0.0, 0.0);
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt) {
                            const int d = 16 * rt + lr;
                            if (d < Nv) {
                                cmac(x, cmk(cr[rt][r], ci[rt][r]), ldc<double2, double>(pv + d));
                                if (!SAME) cmac(x2, cmk(dr[rt][r], di[rt][r]), ldc<double2, double>(pu + d));
                            }
                        }
                        int tc;
                        double wr, wi;
                        gk_row(k, pt, &tc, &wr, &wi);    // u_0 in row sp: G_k[pt][sp]
                        if (SAME) {
                            re[q] += 2.0 * (wr * x.re - wi * x.im);
                        } else {
                            cx<double> f = cmk(wr, wi) * x;
                            gk_row(k, sp, &tc, &wr, &wi);   // v_0 in row sp: G_k[sp][pt]
                            f = f - cmk(wr, wi) * conj(x2);
                            re[q] += f.re;
                            im[q] += f.im;
                        }
                    }
                }
            }
        }
        // the wavefront's lanes, then the wavefronts of a time slice, all in a fixed order
#pragma unroll
        for (int q = 0; q < GPT; ++q) {
            if (SAME) im[q] = 0.0 * re[q];
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                re[q] += __shfl_xor(re[q], o, 64);
                im[q] += __shfl_xor(im[q], o, 64);
            }
            if (lane == 0) red[w][q] = make_double2(re[q], im[q]);
        }
        __syncthreads();
        const int nt = b0 - t0 < 4 ? b0 - t0 : 4;
        if ((int)threadIdx.x < nt * GPT) {
            const int tt = threadIdx.x / GPT, gq = threadIdx.x - tt * GPT, pg = tile * GPT + gq;
            if (pg < npn) {
                double sr = 0.0, si = 0.0;
                for (int s = 0; s < nsub; ++s) {
                    const double2 v = red[tt + s * b0][gq];
                    sr += v.x;
                    si += v.y;
                }
                const int pp = pg / nsrc, ns = pg - pp * nsrc, x0 = y0 * b0 + t0 + tt;
                part[((((size_t)(pair0 + pp) * nsrc + ns) * g.L[0] + x0) * LV_MAXCHUNK) + ch] =
                    make_double2(scale * sr, scale * si);
            }
        }
        __syncthreads();
    }
}

// out[row][t] (+)= (1/ntot) sum_n [S(row, n, x_n) - diff * S(row + 1, n, x_n)],
// S(p, n, x) = sum_{c < nch[p]} part[p][n][x][c], x_n = (t_src[n] + t) mod L0
struct PairChunks {
    int nch[LV_MAXPAIR];
};
__global__ void k_levels_finish(int L0, int nrow, int npair, int nsrc, int diff, SrcTimes ts, PairChunks pc,
                                const double2* __restrict__ part, double scale, int accumulate,
                                double2* __restrict__ out) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nrow * L0) return;
    const int row = e / L0, t = e - row * L0;
    double re = 0.0, im = 0.0;
    for (int n = 0; n < nsrc; ++n) {
        int x = ts.t[n] + t;
        x = x >= L0 ? x - L0 : x;
        for (int q = 0; q < 2; ++q) {
            const int p = row + q;
            if (q == 1 && (!diff || p >= npair)) break;
            const double sg = q == 0 ? 1.0 : -1.0;
            const double2* pp = part + (((size_t)p * nsrc + n) * L0 + x) * LV_MAXCHUNK;
            // chunks in four sums of their own (chunk c in sum c % 4), then those
            double2 s[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) s[u] = make_double2(0.0, 0.0);
            for (int c = 0; c < pc.nch[p]; c += 4) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (c + u < pc.nch[p]) {
                        s[u].x += pp[c + u].x;
                        s[u].y += pp[c + u].y;
                    }
                }
            }
            re += sg * ((s[0].x + s[1].x) + (s[2].x + s[3].x));
            im += sg * ((s[0].y + s[1].y) + (s[2].y + s[3].y));
        }
    }
    double2 o = make_double2(scale * re, scale * im);
    if (accumulate) {
        o.x += out[e].x;
        o.y += out[e].y;
    }
    out[e] = o;
}

struct SrcKind {
    int ncs;        // source colours: 3 (point) or 1 (wall)
    double scale;
};

template <int NCS, bool SAME>
static int slice_partials_k(mglma_ctx* c, double scale, int nsrc, int nfine, int npair, const PairSet& P,
                            double2* part, PairChunks* pc) {
    const Geo& g = c->geo;
    const int nchf = fine_chunks(g), nchc = coarse_chunks(g);
    for (int p = 0; p < npair; ++p) pc->nch[p] = p < nfine ? nchf : nchc;
    if (nfine > 0) {
        hipLaunchKernelGGL((k_fine_slice_part<NCS, SAME>), dim3(g.L[0] * nchf, nsrc, nfine), dim3(256), 0, c->stream,
                           g, nchf, nsrc, 0, P, scale, part);
        HIP_TRY(hipGetLastError());
    }
    if (npair > nfine) {
        PairSet Q;
        for (int p = 0; p < LV_MAXPAIR; ++p) {
            Q.pi[p] = p + nfine < LV_MAXPAIR ? P.pi[p + nfine] : nullptr;
            Q.pj[p] = p + nfine < LV_MAXPAIR ? P.pj[p + nfine] : nullptr;
        }
        constexpr int GPT = 16 / (4 * NCS);
        const int npn = (npair - nfine) * nsrc;
        const dim3 grid(site_tile_grid((long)g.L1[0] * nchc, (npn + GPT - 1) / GPT));
#define LV_COARSE(NS)                                                                                          \
    hipLaunchKernelGGL((k_coarse_slice_part<NCS, SAME, NS>), grid, dim3(256), 0, c->stream, g, c->Nv, nchc, nsrc, \
                       npn, nfine, (const double2*)c->G1, Q, scale, part)
        const int ns = (c->Nv + 3) / 4;
        if (ns <= 2) LV_COARSE(2);
        else if (ns <= 4) LV_COARSE(4);
        else if (ns <= 6) LV_COARSE(6);
        else if (ns <= 8) LV_COARSE(8);
        else if (ns <= 12) LV_COARSE(12);
        else LV_COARSE(16);
#undef LV_COARSE
        HIP_TRY(hipGetLastError());
    }
    return MGLMA_OK;
}

// Partials of every pair for sources [0, nsrc) of the given pieces into part
// (npair * nsrc * L0 * LV_MAXCHUNK complex) and the chunk counts.
static int slice_partials(mglma_ctx* c, const SrcKind& K, int nsrc, int nfine, int npair, const PairSet& P,
                          double2* part, PairChunks* pc) {
    bool same = true;
    for (int p = 0; p < npair; ++p) same = same && P.pi[p] == P.pj[p];
    if (K.ncs == 3)
        return same ? slice_partials_k<3, true>(c, K.scale, nsrc, nfine, npair, P, part, pc)
                    : slice_partials_k<3, false>(c, K.scale, nsrc, nfine, npair, P, part, pc);
    return same ? slice_partials_k<1, true>(c, K.scale, nsrc, nfine, npair, P, part, pc)
                : slice_partials_k<1, false>(c, K.scale, nsrc, nfine, npair, P, part, pc);
}

static int check_sources(mglma_ctx* c, int kind, int nsrc, const int* t_src, SrcKind* K) {
    if (kind != MGLMA_SRC_POINT && kind != MGLMA_SRC_STOCH) return MGLMA_ERR_ARG;
    if (nsrc < 1 || nsrc > LV_MAXSRC || !t_src) return MGLMA_ERR_ARG;
    for (int n = 0; n < nsrc; ++n)
        if (t_src[n] < 0 || t_src[n] >= c->L[0]) return MGLMA_ERR_ARG;
    K->ncs = kind == MGLMA_SRC_POINT ? 3 : 1;
    K->scale = kind == MGLMA_SRC_POINT ? 1.0 / 3.0 : 1.0 / (3.0 * c->geo.V3);
    return MGLMA_OK;
}

// Shared body of mglma_contract_levels and its allocation-free variant:
// part holds at least npair * nsb * L0 * LV_MAXCHUNK complex, out_dev the
// nrow * L0 result; sources are processed nsb at a time.
static int levels_body(mglma_ctx* c, const SrcKind& K, int nsrc, const int* t_src, int nfine, int npair,
                       const PairSet& P, int diff, int nrow, int nsb, double2* part, double2* out_dev,
                       double scale = 0.0, int accumulate = 0) {
    if (scale == 0.0) scale = 1.0 / nsrc;
    const int L0 = c->L[0], ncol = 4 * K.ncs;
    for (int n0 = 0; n0 < nsrc; n0 += nsb) {
        const int nb = nsrc - n0 < nsb ? nsrc - n0 : nsb;
        PairSet Pn;
        const size_t fstride = (size_t)ncol * 12 * c->geo.V, cstride = (size_t)ncol * c->geo.V1 * c->nc;
        for (int p = 0; p < LV_MAXPAIR; ++p) {
            const size_t off = (size_t)n0 * (p < nfine ? fstride : cstride);
            Pn.pi[p] = p < npair ? P.pi[p] + off : nullptr;
            Pn.pj[p] = p < npair ? P.pj[p] + off : nullptr;
        }
        PairChunks pc;
        MG_TRY(slice_partials(c, K, nb, nfine, npair, Pn, part, &pc));
        SrcTimes ts;
        for (int n = 0; n < nb; ++n) ts.t[n] = t_src[n0 + n];
        hipLaunchKernelGGL(k_levels_finish, dim3((nrow * L0 + 127) / 128), dim3(128), 0, c->stream, L0, nrow, npair,
                           nb, diff, ts, pc, (const double2*)part, scale, (n0 > 0 || accumulate) ? 1 : 0,
                           out_dev);
        HIP_TRY(hipGetLastError());
    }
    return MGLMA_OK;
}

static int levels_args(mglma_ctx* c, int kind, int nsrc, const int* t_src, const double* fine, int ncoarse,
                       const double* const* coarse, int exact_top, double* G_host, SrcKind* K,
                       PairSet* P, int* nfine, int* npair) {
    if (!c || !G_host || ncoarse < 0 || (ncoarse > 0 && !coarse)) return MGLMA_ERR_ARG;
    MG_TRY(check_sources(c, kind, nsrc, t_src, K));
    *nfine = fine ? 1 : 0;
    *npair = *nfine + ncoarse;
    if (*npair < 1 || *npair > LV_MAXPAIR) return MGLMA_ERR_ARG;
    if (ncoarse > 0 && !c->have_subspace) return MGLMA_ERR_NO_SUBSPACE;
    if (exact_top && !c->have_top) return MGLMA_ERR_NO_TOP;
    for (int k = 0; k < ncoarse; ++k)
        if (!coarse[k]) return MGLMA_ERR_ARG;
    for (int p = 0; p < LV_MAXPAIR; ++p) {
        const double* f = p < *nfine ? fine : (p < *npair ? coarse[p - *nfine] : nullptr);
        P->pi[p] = P->pj[p] = (const double2*)f;
    }
    return MGLMA_OK;
}

extern "C" int mglma_contract_levels(mglma_ctx* c, int kind, int nsrc, const int* t_src, const double* fine,
                                     int ncoarse, const double* const* coarse, int exact_top, double* G_host) {
    SrcKind K;
    PairSet P;
    int nfine, npair;
    MG_TRY(levels_args(c, kind, nsrc, t_src, fine, ncoarse, coarse, exact_top, G_host, &K, &P, &nfine, &npair));
    const int L0 = c->L[0], nrow = npair + (exact_top ? 1 : 0);
    double2 *part, *out;
    MG_TRY(mg_scratch(c, 28, (size_t)npair * nsrc * L0 * LV_MAXCHUNK * 16, (void**)&part));
    MG_TRY(mg_scratch(c, 29, (size_t)nrow * L0 * 16 + 256, (void**)&out));
    MG_TRY(levels_body(c, K, nsrc, t_src, nfine, npair, P, 1, npair, nsrc, part, out));
    if (exact_top) MG_TRY(mg_top_corr(c, out + (size_t)npair * L0));
    HIP_TRY(hipMemcpyAsync(G_host, out, (size_t)nrow * L0 * 16, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    return MGLMA_OK;
}

extern "C" int mglma_contract_levels_acc(mglma_ctx* c, int kind, int nsrc, const int* t_src, const double* fine,
                                         int ncoarse, const double* const* coarse, double weight, int accumulate,
                                         double* G_dev) {
    if (!G_dev || !(weight == weight)) return MGLMA_ERR_ARG;
    SrcKind K;
    PairSet P;
    int nfine, npair;
    double dummy;
    MG_TRY(levels_args(c, kind, nsrc, t_src, fine, ncoarse, coarse, 0, &dummy, &K, &P, &nfine, &npair));
    if (weight == 0.0) return MGLMA_ERR_ARG;
    const int L0 = c->L[0];
    double2* part;
    MG_TRY(mg_scratch(c, 28, (size_t)npair * nsrc * L0 * LV_MAXCHUNK * 16, (void**)&part));
    return levels_body(c, K, nsrc, t_src, nfine, npair, P, 1, npair, nsrc, part, (double2*)G_dev, weight,
                       accumulate ? 1 : 0);
}

extern "C" int mglma_contract_pair(mglma_ctx* c, int kind, int nsrc, const int* t_src, int coarse,
                                   const double* psi_i, const double* psi_j, double* G_host) {
    if (!c || !psi_i || !psi_j || !G_host || (coarse != 0 && coarse != 1)) return MGLMA_ERR_ARG;
    SrcKind K;
    MG_TRY(check_sources(c, kind, nsrc, t_src, &K));
    if (coarse && !c->have_subspace) return MGLMA_ERR_NO_SUBSPACE;
    PairSet P;
    for (int p = 0; p < LV_MAXPAIR; ++p) P.pi[p] = P.pj[p] = nullptr;
    P.pi[0] = (const double2*)psi_i;
    P.pj[0] = (const double2*)psi_j;
    const int L0 = c->L[0];
    double2 *part, *out;
    MG_TRY(mg_scratch(c, 28, (size_t)nsrc * L0 * LV_MAXCHUNK * 16, (void**)&part));
    MG_TRY(mg_scratch(c, 29, (size_t)L0 * 16 + 256, (void**)&out));
    MG_TRY(levels_body(c, K, nsrc, t_src, coarse ? 0 : 1, 1, P, 0, 1, nsrc, part, out));
    HIP_TRY(hipMemcpyAsync(G_host, out, (size_t)L0 * 16, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    return MGLMA_OK;
}

// one source: the same two-point function (entry t of its row is C(t0 + t, t0))
static int contract_one(mglma_ctx* c, int kind, int coarse, const double* pi, const double* pj, int t0, double* C) {
    if (!c || !pi || !pj || !C || t0 < 0 || t0 >= c->L[0]) return MGLMA_ERR_ARG;
    return mglma_contract_pair(c, kind, 1, &t0, coarse, pi, pj, C);
}

extern "C" int mglma_contract_point(mglma_ctx* c, const double* pi, const double* pj, int y0, double* C) {
    return contract_one(c, MGLMA_SRC_POINT, 0, pi, pj, y0, C);
}

extern "C" int mglma_contract_point_coarse(mglma_ctx* c, const double* ci, const double* cj, int y0, double* C) {
    return contract_one(c, MGLMA_SRC_POINT, 1, ci, cj, y0, C);
}

extern "C" int mglma_contract_stoch(mglma_ctx* c, const double* pi, const double* pj, int tn, double* C) {
    return contract_one(c, MGLMA_SRC_STOCH, 0, pi, pj, tn, C);
}

extern "C" int mglma_contract_stoch_coarse(mglma_ctx* c, const double* ci, const double* cj, int tn, double* C) {
    return contract_one(c, MGLMA_SRC_STOCH, 1, ci, cj, tn, C);
}

// ---------------------------------------------------------------------------
// Allocation-free level assembly: the partial sums and the result live in a
// fixed device array (each device that the library runs on holds its own
// copy for the life of the process).  Its device address is looked up once
// per device when the first context on that device is created; host code
// uses only that address, never the array's name.
// ---------------------------------------------------------------------------
#define NOALLOC_BYTES ((size_t)8 << 20)
#define NOALLOC_MAXDEV 64
static __device__ __align__(256) double2 scratch[NOALLOC_BYTES / sizeof(double2)];
static double2* noalloc_ptr[NOALLOC_MAXDEV];
static std::mutex noalloc_mu;

int mg_noalloc_init(int device) {
    if (device < 0 || device >= NOALLOC_MAXDEV) return MGLMA_ERR_ARG;
    std::lock_guard<std::mutex> lk(noalloc_mu);
    if (noalloc_ptr[device]) return MGLMA_OK;
    void* p = nullptr;
    HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return MGLMA_ERR_HIP;
    noalloc_ptr[device] = (double2*)p;
    return MGLMA_OK;
}

extern "C" int mglma_contract_levels_noalloc(mglma_ctx* c, int kind, int nsrc, const int* t_src,
                                             const double* fine, int ncoarse, const double* const* coarse,
                                             double* G_host) {
    SrcKind K;
    PairSet P;
    int nfine, npair;
    MG_TRY(levels_args(c, kind, nsrc, t_src, fine, ncoarse, coarse, 0, G_host, &K, &P, &nfine, &npair));
    if (c->device < 0 || c->device >= NOALLOC_MAXDEV) return MGLMA_ERR_ARG;
    double2* base;
    {
        std::lock_guard<std::mutex> lk(noalloc_mu);
        base = noalloc_ptr[c->device];
    }
    if (!base) return MGLMA_ERR_HIP;
    const int L0 = c->L[0], nrow = npair;
    const size_t cap = NOALLOC_BYTES / sizeof(double2);
    const size_t out_n = ((size_t)nrow * L0 + 15) / 16 * 16;    // result first, 256-byte aligned partials
    const size_t per_src = (size_t)npair * L0 * LV_MAXCHUNK;
    if (out_n + per_src > cap) return MGLMA_ERR_SHAPE;            // L0 too long for the fixed workspace
    size_t nsb = (cap - out_n) / per_src;
    if (nsb > (size_t)nsrc) nsb = (size_t)nsrc;
    double2* out = base;
    double2* part = base + out_n;
    MG_TRY(levels_body(c, K, nsrc, t_src, nfine, npair, P, 1, nrow, (int)nsb, part, out));
    HIP_TRY(hipMemcpyAsync(G_host, out, (size_t)nrow * L0 * 16, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    return MGLMA_OK;
}
