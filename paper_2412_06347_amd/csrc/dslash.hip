// Wilson-clover operator M = (1 + A) - kappa H on the blocked device layout.
//
//   (M psi)(x) = (1 + A(x)) psi(x)
//                - kappa sum_mu [ (1 - gamma_mu) U_mu(x) psi(x+mu)
//                                 + (1 + gamma_mu) U_mu(x-mu)^+ psi(x-mu) ]
// (kappa-normalised O(a)-improved Wilson operator of tab:ensembles; Q = gamma5 M
// is the Hermitian operator of section "Variance reduction using deflation").
//
// One thread per site (and direction, k_dslash).  Spinor, link and clover components
// are stored site-innermost, so every load of a wavefront is one contiguous
// run.  Each hop is spin-projected to a half spinor (rank-2 projector
// 1 -/+ gamma_mu in the chiral basis), multiplied by the link and expanded.
// Storage is FP64, FP32 or FP16; FP32 computes in FP32.  FP16 computes in
// FP32 for one right-hand side and on the packed FP16 data with FP32
// accumulation for batches (k_dslash_h).
#include "tile.h"
#include "wilson_h.h"

// o = link times the projected neighbour spinor of one hop
template <int MU, bool FWD, typename S, typename G, typename R>
__device__ __forceinline__ void hop_half(const Geo& g, int i, const int lc[4], const int yc[4],
                                         const S* __restrict__ pin, const G* __restrict__ U, cx<R> o[6]) {
    const size_t V = g.V;
    bool wrap;
    int j = FWD ? geo_fwd(g, i, MU, lc, yc, &wrap) : geo_bwd(g, i, MU, lc, yc, &wrap);
    cx<R> p[12];
#pragma unroll
    for (int sc = 0; sc < 12; ++sc) p[sc] = ldc<S, R>(pin + (size_t)sc * V + j);
    cx<R> h[6];
    project<MU, FWD, R>(p, h);
    if (wrap && g.bcneg[MU]) {
#pragma unroll
        for (int k = 0; k < 6; ++k) h[k] = -h[k];
    }
    // link U_mu(x) for the forward hop, U_mu(x-mu)^+ for the backward hop
    const G* ul = U + (size_t)(MU * 9) * V + (FWD ? i : j);
    cx<R> u[9];
#pragma unroll
    for (int e = 0; e < 9; ++e) u[e] = ldc<G, R>(ul + (size_t)e * V);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            cx<R> t = cmk((R)0, (R)0);
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                if (FWD) cmac(t, u[a * 3 + b], h[s * 3 + b]);
                else cjmac(t, u[b * 3 + a], h[s * 3 + b]);
            }
            o[s * 3 + a] = t;
        }
}

// Workgroup -> (site tile, rhs) mapping.  Workgroups are dealt to the eight
// XCDs round robin (workgroup b runs on XCD b % 8), each XCD with its own L2.
// XCD x gets the contiguous tile range [x*ntp/8, (x+1)*ntp/8), so the
// neighbour spinors and links a tile reads were mostly brought into that
// XCD's L2 by the adjacent tiles, and the nrhs workgroups of one tile are
// dealt to the same XCD back to back so its links and clover are read from
// HBM once for the whole batch.
//
// One right-hand side (or fields past tile_fits): 64 sites per workgroup and a
// wavefront per direction, so that a site is a chain of two hops instead of
// eight, in 140 registers (FP64) instead of 486.  The half spinors meet in LDS
// and are added in a fixed order, that of the tile kernel below (the same bits in
// FP64 and FP32); wavefronts 2 and 3 have a chirality's clover term ready by then.
// Against a thread per site: 16 x 8^3 FP64 10.4 -> 5.3 us, FP32 9.3 -> 4.8, FP16
// 7.5 -> 4.3 (the latency of the loads); 48 x 24^3 FP64 271 -> 257 us (4.0 TB/s),
// FP32 136 -> 135, FP16 66 -> 51 (5.0 TB/s).
template <typename S, typename G, typename R>
__global__ __launch_bounds__(256) void k_dslash(Geo g, const S* __restrict__ in, S* __restrict__ out,
                                                const G* __restrict__ U, const G* __restrict__ C, R kappa,
                                                int gamma5, int nrhs, int ntp) {
    __shared__ cx<R> ho[8][6][64];
    const int b = blockIdx.x, pos = b >> 3, tl = pos / nrhs;
    const int tile = (b & 7) * (ntp >> 3) + tl;
    if (tile * 64 >= g.V) return;        // uniform over the workgroup
    in += (size_t)(pos - tl * nrhs) * 12 * g.V;
    out += (size_t)(pos - tl * nrhs) * 12 * g.V;
    const int w = wave_id(), lane = threadIdx.x & 63;
    // the last tile's idle lanes repeat the last site, stores included (the same values)
    const int i = tile * 64 + lane < g.V ? tile * 64 + lane : g.V - 1;
    const size_t V = g.V;
    int lc[4], yc[4];
    geo_coords(g, i, lc, yc);
    const int ch = w & 1;
    cx<R> o[2][6], res[6];
    switch (w) {
        case 0: hop_half<0, true, S, G, R>(g, i, lc, yc, in, U, o[0]); hop_half<0, false, S, G, R>(g, i, lc, yc, in, U, o[1]); break;
        case 1: hop_half<1, true, S, G, R>(g, i, lc, yc, in, U, o[0]); hop_half<1, false, S, G, R>(g, i, lc, yc, in, U, o[1]); break;
        case 2: hop_half<2, true, S, G, R>(g, i, lc, yc, in, U, o[0]); hop_half<2, false, S, G, R>(g, i, lc, yc, in, U, o[1]); break;
        default: hop_half<3, true, S, G, R>(g, i, lc, yc, in, U, o[0]); hop_half<3, false, S, G, R>(g, i, lc, yc, in, U, o[1]); break;
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        ho[2 * w][k][lane] = o[0][k];
        ho[2 * w + 1][k][lane] = o[1][k];
    }
    if (w >= 2) {
        cx<R> p[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) p[k] = ldc<S, R>(in + (size_t)(6 * ch + k) * V + i);
        clover_block<G, R>(C + (size_t)ch * 18 * V, V, i, p, res);
    }
    __syncthreads();
    if (w < 2) return;
    cx<R> acc[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = cmk((R)0, (R)0);
    auto get = [&](int d) {
#pragma unroll
        for (int k = 0; k < 6; ++k) o[0][k] = ho[d][k][lane];
    };
    get(0); reconstruct_add<0, true, R>(acc, o[0]);
    get(1); reconstruct_add<0, false, R>(acc, o[0]);
    get(2); reconstruct_add<1, true, R>(acc, o[0]);
    get(3); reconstruct_add<1, false, R>(acc, o[0]);
    get(4); reconstruct_add<2, true, R>(acc, o[0]);
    get(5); reconstruct_add<2, false, R>(acc, o[0]);
    get(6); reconstruct_add<3, true, R>(acc, o[0]);
    get(7); reconstruct_add<3, false, R>(acc, o[0]);
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        cx<R> v = res[k] - kappa * (ch ? acc[6 + k] : acc[k]);
        if (gamma5 && ch) v = -v;
        stc<S, R>(out + (size_t)(6 * ch + k) * V + i, v);
    }
}

// Batches: a tile of 64 sites per workgroup, its links (CL: and clover term) in
// LDS, one right-hand side per wavefront at a time, neighbours inside the tile
// by lane exchange (tile.h).  Bound: the L1 caches' outstanding misses (about
// 390 lines per 64 sites and right-hand side; the faces along x_2 and x_3 use a
// quarter of each line they touch), not HBM.  48 x 24^3, 12 right-hand sides,
// against a thread per site with two right-hand sides and all eight neighbours
// read through the caches: FP64 2.38 -> 1.51 ms, FP32 1.11 -> 0.83 ms (2.3 TB/s
// of the fields, links and clover term once), FP16 0.51 -> 0.41 ms.  Tried: the
// links in LDS alone without the lane exchange 1.10 ms (FP32), two or three
// wavefronts per tile 0.83-0.88, groups of right-hand sides over a plane of
// blocks (fewer L2 misses, links staged again) 0.93-1.08 ms.
//
// SO: output storage.  RESID: the output is (rsub - M in) / scale[rhs] (the
// residual of an approximate solution, stored rescaled in SO).
template <typename S, typename G, typename R, bool CL, int W, typename SO = S, bool RESID = false>
__global__ __launch_bounds__(256, W) void k_dslash_tile(Geo g, const S* __restrict__ in, SO* __restrict__ out,
                                                        const G* __restrict__ U, const G* __restrict__ C, R kappa,
                                                        int gamma5, int nrhs, int ntp, int ng,
                                                        const S* __restrict__ rsub = nullptr,
                                                        const double* __restrict__ scale = nullptr) {
    __shared__ G ul[tile_gauge(CL)];
    const int bid = blockIdx.x, pos = bid >> 3, tl = pos / ng;
    const int tile = (bid & 7) * (ntp >> 3) + tl;
    if (tile * TILE >= g.V) return;      // uniform over the workgroup
    const int w = wave_id(), nw = blockDim.x >> 6, lane = threadIdx.x & 63;
    // the last tile's idle lanes repeat the last site, stores included (the same values)
    const int i = tile * TILE + lane < g.V ? tile * TILE + lane : g.V - 1;
    const size_t V = g.V;
    int lc[4], yc[4];
    geo_coords(g, i, lc, yc);
    tile_stage_gauge<CL, G>(g, i, lc, yc, U, C, ul, w, nw, lane);
    __syncthreads();
    const uint32_t vc = g.V;
    const int i0 = tile * TILE;
    for (int q = (pos - tl * ng) * nw + w; q < nrhs; q += ng * nw) {
        const FieldRsrc pr = field_rsrc(in + q * 12 * V, vc);
        const uint32_t io = opaque_v((uint32_t)i);
        cx<R> acc[12], own[12];
        tile_own<S, R>(pr, io, vc, own);
        const int lo = (int)opaque_v(lane);
        tile_hops<S, G, R>(g, i, i0, lc, yc, pr, own, ul, lo, acc);
        const R isc = RESID ? (R)(1.0 / scale[q]) : (R)1;
#pragma unroll
        for (int ch = 0; ch < 2; ++ch) {
            cx<R> res[6];
            tile_clover<CL, G, R>(ul, lo, C, vc, io, ch, own + 6 * ch, res);
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                cx<R> v = res[k] - kappa * acc[6 * ch + k];
                if (gamma5 && ch == 1) v = -v;
                if (RESID) v = isc * (buf_ldc<S, R>(comp_rsrc<1>(rsub + q * 12 * V, 6 * ch + k, vc), io, 0) - v);
                buf_stc<SO, R>(out + q * 12 * V, vc, io, 6 * ch + k, v);
            }
        }
    }
}

// FP16 storage computed on the packed FP16 data: the helpers of wilson_h.h.
// One hop on packed FP16 data: as tile_hop, the half spinor h = p0 + SG (i) q
// (form FZ) formed by its owner; the other forms of it that the link products
// need are exact, so they follow after the change of lanes.
template <int MU, bool FWD>
__device__ __forceinline__ void hop_h(const Geo& g, int i, int i0, const int lc[4], const int yc[4],
                                      const FieldRsrc& pin, const h2 own[12], const h2* ul, int lane,
                                      cx<float> acc[12]) {
    const uint32_t V = g.V;
    const Nbr n = tile_nbr<MU, FWD>(g, i, i0, lc, yc, 4u);
    h2 p[12], h[6], hl[6];
#pragma unroll
    for (int sc = 0; sc < 12; ++sc) p[sc] = buf_ld<h2>(pin.part[sc / 2], n.off, (sc % 2) * V * 4u);
    proj_h<MU, FWD, FZ>(own, h);
#pragma unroll
    for (int k = 0; k < 6; ++k) h[k] = __builtin_bit_cast(h2, lane_get(__builtin_bit_cast(int, h[k]), n.src));
    proj_h<MU, FWD, FZ>(p, hl);
    h2 hre[6], him[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const h2 z = n.in ? h[k] : hl[k];
        hre[k] = form<FWD ? FN : FZ>(z);
        him[k] = form<FWD ? FS : FSN>(z);
    }
    const h2* u = ul + (2 * MU + (FWD ? 0 : 1)) * 9 * TILE + lane;
    cx<float> o[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) o[k] = cmk(0.f, 0.f);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int c2 = 0; c2 < 3; ++c2) {
            const h2 uu = u[(FWD ? a * 3 + c2 : c2 * 3 + a) * TILE];
#pragma unroll
            for (int sp = 0; sp < 2; ++sp) {
                o[sp * 3 + a].re = dot2(uu, hre[sp * 3 + c2], o[sp * 3 + a].re);
                o[sp * 3 + a].im = dot2(uu, him[sp * 3 + c2], o[sp * 3 + a].im);
            }
        }
    reconstruct_sg<MU, FWD, float>(acc, o, n.neg ? -1.f : 1.f);
    __builtin_amdgcn_sched_barrier(0);
}

// Batches in FP16: the tile kernel on packed FP16 data.
template <bool CL>
__global__ __launch_bounds__(256, 4) void k_dslash_h(Geo g, const h2* __restrict__ in, h2* __restrict__ out,
                                                     const h2* __restrict__ U, const h2* __restrict__ C, float kappa,
                                                     int gamma5, int nrhs, int ntp, int ng) {
    __shared__ h2 ul[tile_gauge(CL)];
    const int bid = blockIdx.x, pos = bid >> 3, tl = pos / ng;
    const int tile = (bid & 7) * (ntp >> 3) + tl;
    if (tile * TILE >= g.V) return;
    const int w = wave_id(), nw = blockDim.x >> 6, lane = threadIdx.x & 63;
    const int i = tile * TILE + lane < g.V ? tile * TILE + lane : g.V - 1;
    const int i0 = tile * TILE;
    const uint32_t V = g.V;
    int lc[4], yc[4];
    geo_coords(g, i, lc, yc);
    tile_stage_gauge<CL, h2>(g, i, lc, yc, U, C, ul, w, nw, lane);
    __syncthreads();
    for (int q = (pos - tl * ng) * nw + w; q < nrhs; q += ng * nw) {
        const FieldRsrc pin = field_rsrc(in + (size_t)q * 12 * V, V);
        const int lo = (int)opaque_v(lane);
        const uint32_t io = opaque_v((uint32_t)i) * 4u;
        cx<float> acc[12];
        h2 own[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            own[k] = buf_ld<h2>(pin.part[k / 2], io, k % 2 * V * 4u);
            acc[k] = cmk(0.f, 0.f);
        }
        hop_h<0, true>(g, i, i0, lc, yc, pin, own, ul, lo, acc);
        hop_h<0, false>(g, i, i0, lc, yc, pin, own, ul, lo, acc);
        hop_h<1, true>(g, i, i0, lc, yc, pin, own, ul, lo, acc);
        hop_h<1, false>(g, i, i0, lc, yc, pin, own, ul, lo, acc);
        hop_h<2, true>(g, i, i0, lc, yc, pin, own, ul, lo, acc);
        hop_h<2, false>(g, i, i0, lc, yc, pin, own, ul, lo, acc);
        hop_h<3, true>(g, i, i0, lc, yc, pin, own, ul, lo, acc);
        hop_h<3, false>(g, i, i0, lc, yc, pin, own, ul, lo, acc);
#pragma unroll
        for (int ch = 0; ch < 2; ++ch) {
            h2 p[1][6];
            cx<float> res[1][6];
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                p[0][k] = own[6 * ch + k];
                res[0][k] = -kappa * acc[6 * ch + k];
            }
            clover_dot2<1>([&](int k) { return CL ? ul[(72 + ch * 18 + k) * TILE + lo]
                                                  : buf_ld<h2>(comp_rsrc<TILE_COMPS>(C, ch * 18 + k / TILE_COMPS * TILE_COMPS, V),
                                                               io, k % TILE_COMPS * V * 4u); },
                           p, res);
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                cx<float> v = res[0][k];
                if (gamma5 && ch == 1) v = -v;
                buf_st<h2>(out + (size_t)q * 12 * V, V, (uint32_t)i, 6 * ch + k, h2{(_Float16)v.re, (_Float16)v.im});
            }
        }
    }
}

int mg_dslash(mglma_ctx* c, int prec, int gamma5, const void* in, void* out, int nrhs) {
    if (nrhs == 0) return MGLMA_OK;
    const Geo& g = c->geo;
    // refused: more than 2^31 - 1 tiles of 256 sites, padded as below (2^39 sites of all right-hand sides)
    if ((size_t)((g.V + 255) / 256 + 7) / 8 * 8 * nrhs > 0x7fffffffu) return MGLMA_ERR_SHAPE;
    if (nrhs >= 2 && tile_fits(g.V, prec_cbytes(prec))) {
        const TileGrid t(g.V, nrhs);
        switch (prec) {
            case MGLMA_F64:
                // links alone in LDS (74 KB, two workgroups on a compute unit; with the clover term one:
                // 2 rhs 570 instead of 365 us, 12 rhs the same)
                hipLaunchKernelGGL((k_dslash_tile<double2, double2, double, false, 2>), t.grid, t.block, 0, c->stream, g,
                                   (const double2*)in, (double2*)out, c->U64, c->C64, c->kappa, gamma5, nrhs, t.nt, t.ng);
                break;
            case MGLMA_F32:
                // the clover term in LDS as well from four right-hand sides on: 55 instead of 37 KB a
                // workgroup, so two instead of four on a compute unit, which costs batches of two or three
                // (48 x 24^3: 2 rhs 204 against 264 us, 3: 271 / 281, 4: 342 / 323, 12: 948 / 828), and not where two on
                // a compute unit leave up to half as many for a second round (24 x 12^3, 648 workgroups: 5 rhs 24 against
                // 33 us, 9: 38 / 47, 16: 63 / 62; 32 x 12^3, 864: 5 rhs 31 / 34, 9: 49 / 49, 16: 84 / 71)
                if (nrhs < 4 || (t.nt * t.ng > 512 && t.nt * t.ng <= 768))
                    hipLaunchKernelGGL((k_dslash_tile<float2, float2, float, false, 4>), t.grid, t.block, 0, c->stream,
                                       g, (const float2*)in, (float2*)out, c->U32, c->C32, (float)c->kappa, gamma5,
                                       nrhs, t.nt, t.ng);
                else
                    hipLaunchKernelGGL((k_dslash_tile<float2, float2, float, true, 2>), t.grid, t.block, 0, c->stream,
                                       g, (const float2*)in, (float2*)out, c->U32, c->C32, (float)c->kappa, gamma5,
                                       nrhs, t.nt, t.ng);
                break;
            case MGLMA_F16:
                // as for FP32, at half the LDS (48 x 24^3: 2 rhs 96 against 113 us, 3: 130 / 126, 12: 447 / 409)
                if (nrhs < 3)
                    hipLaunchKernelGGL(k_dslash_h<false>, t.grid, t.block, 0, c->stream, g, (const h2*)in, (h2*)out,
                                       (const h2*)c->U16, (const h2*)c->C16, (float)c->kappa, gamma5, nrhs, t.nt, t.ng);
                else
                    hipLaunchKernelGGL(k_dslash_h<true>, t.grid, t.block, 0, c->stream, g, (const h2*)in, (h2*)out,
                                       (const h2*)c->U16, (const h2*)c->C16, (float)c->kappa, gamma5, nrhs, t.nt, t.ng);
                break;
            default: return MGLMA_ERR_ARG;
        }
        HIP_TRY(hipGetLastError());
        return MGLMA_OK;
    }
    const int ntp = ((g.V + 63) / 64 + 7) / 8 * 8;   // tiles, padded to a multiple of the XCD count
    if ((size_t)ntp * nrhs > 0x7fffffffu) return MGLMA_ERR_SHAPE;
    dim3 grid(ntp * nrhs);
    switch (prec) {
        case MGLMA_F64:
            hipLaunchKernelGGL((k_dslash<double2, double2, double>), grid, dim3(256), 0, c->stream, g,
                               (const double2*)in, (double2*)out, c->U64, c->C64, c->kappa, gamma5, nrhs, ntp);
            break;
        case MGLMA_F32:
            hipLaunchKernelGGL((k_dslash<float2, float2, float>), grid, dim3(256), 0, c->stream, g,
                               (const float2*)in, (float2*)out, c->U32, c->C32, (float)c->kappa, gamma5, nrhs, ntp);
            break;
        case MGLMA_F16:
            hipLaunchKernelGGL((k_dslash<__half2, __half2, float>), grid, dim3(256), 0, c->stream, g,
                               (const __half2*)in, (__half2*)out, c->U16, c->C16, (float)c->kappa, gamma5, nrhs, ntp);
            break;
        default: return MGLMA_ERR_ARG;
    }
    HIP_TRY(hipGetLastError());
    return MGLMA_OK;
}

// p16 = (r - M z) / scale[rhs] in FP16, from FP32 z and r (the rescaled
// residual that starts the FP16 smoother), one launch.
int mg_dslash_resid16(mglma_ctx* c, const void* z, const void* r, void* p16, const double* scale, int nrhs) {
    if (nrhs <= 0) return MGLMA_OK;
    const Geo& g = c->geo;
    if (!tile_fits(g.V, sizeof(float2))) return MGLMA_ERR_SHAPE;   // links alone past the device's memory
    const TileGrid t(g.V, nrhs);
    hipLaunchKernelGGL((k_dslash_tile<float2, float2, float, true, 2, __half2, true>), t.grid, t.block, 0, c->stream,
                       g, (const float2*)z, (__half2*)p16, c->U32, c->C32, (float)c->kappa, 0, nrhs, t.nt, t.ng,
                       (const float2*)r, scale);
    HIP_TRY(hipGetLastError());
    return MGLMA_OK;
}

extern "C" int mglma_apply_D(mglma_ctx* c, int prec, int gamma5, const void* in, void* out, int nrhs) {
    if (!c || !in || !out || in == out || nrhs < 0 || nrhs > 65535) return MGLMA_ERR_ARG;
    if (!c->have_gauge) return MGLMA_ERR_NO_GAUGE;
    return mg_dslash(c, prec, gamma5 ? 1 : 0, in, out, nrhs);
}
