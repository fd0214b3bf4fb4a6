// Schwarz alternating procedure (SAP) smoother on M z = r (the paper's fine
// solver is SAP-preconditioned GCR, section "Comparison of the cost", after
// Luscher 2003).  The aggregation blocks are coloured like a chessboard
// (colour = parity of y_0 + y_1 + y_2 + y_3); a cycle updates the blocks of
// colour 0, then those of colour 1.  A block update forms the residual
// rho = r - M z on the block's sites, makes nmr minimal-residual steps on
// M_BB d = rho_B (M_BB: all couplings between two sites of the block,
// including the hop that wraps around the lattice when the block spans a
// whole extent) and adds d to z.
//
// One workgroup per (block, right-hand side), one thread per block site.  The
// block's z is staged in LDS for the residual (hops inside the block read LDS)
// and then accumulates z + d there, written back once at the end; the
// minimal-residual vector s lives in LDS for the block operator's neighbour
// reads (FP32, or FP16 with FP16 links, where the block steps compute on packed
// FP16 data with FP32 sums) and in FP32 registers for the site's own arithmetic.
// Links and clover come from the FP16 or FP32 copies (L2-resident while the
// right-hand sides of a block run back to back), vectors are FP32.  Blocks of
// one colour do not couple when every block-grid extent is even or one, so one
// launch per colour updates them all without ordering between workgroups.
//
// Bound: vector instructions (about 1640 a site for the residual and 1330 a
// block step, which alone issue at 85-90 % of the rate), then the L1 misses of
// links and faces.  Hence no branches in the hops, neighbours outside the block
// from a zero column or past the end of a buffer, sums by row operations, and
// each hop's loads tied after the hop before it: 128 registers without spills,
// four wavefronts per SIMD.  Half-sweep of 12 right-hand sides, 4 steps, on
// 48 x 24^3 with 4^4 blocks: 1.16 -> 0.99 ms (FP16 links), 1.51 -> 1.42 ms
// (FP32); 32 x 16^3, 2^4 blocks, 4 right-hand sides: 0.66 -> 0.25 ms (a
// workgroup has as many threads as its block needs, not 256).  Tried: the
// residual in a tile kernel of its own and the block solves in another, 0.49 +
// 0.66 ms, and both kinds of workgroups interleaved in one launch over two
// halves of the batch, 0.57 ms per half and step.  A grid that leaves the chip idle
// takes 26 us a half-sweep, one wavefront's own rate of issue: links and clover
// term kept in registers over the steps there save 5 %.
#include "tile.h"
#include "wilson_h.h"

#include <type_traits>
#include <vector>

namespace {

constexpr int SAP_MAXVB = 256;

// A hop of the block operator M_BB: neighbours inside the block; hops that leave
// it are dropped (weight 0), a hop that wraps back into the block (block-grid
// extent one) keeps its boundary phase.  No branches: a lane without a
// neighbour reads its own site with weight 0.
struct BlockHop {
    int jl, ls;     // neighbour and link site inside the block
    float sg;       // +-1, or 0
};
template <int MU, bool FWD>
__device__ __forceinline__ BlockHop block_hop(const Geo& g, int l, const int lc[4]) {
    const bool in = FWD ? lc[MU] + 1 < g.b[MU] : lc[MU] > 0, wraps = g.L1[MU] == 1;
    const int step = FWD ? g.sl[MU] : -g.sl[MU], back = wraps ? -(g.b[MU] - 1) * step : 0;
    const float outside = wraps ? (g.bcneg[MU] ? -1.f : 1.f) : 0.f;
    BlockHop h;
    h.jl = l + (in ? step : back);
    h.ls = FWD ? l : h.jl;
    h.sg = in ? 1.f : outside;
    return h;
}

// links of one direction at block-local site ls (base: the block's first site)
template <typename G, typename F>
__device__ __forceinline__ void block_links(const G* __restrict__ U, int mu, uint32_t V, uint32_t site, F use) {
    rsrc_t r[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) r[a] = comp_rsrc<SAP_COMPS>(U, mu * 9 + 3 * a, V);
#pragma unroll
    for (int e = 0; e < 9; ++e) use(e, buf_ld<G>(r[e / 3], site * (uint32_t)sizeof(G), e % 3 * V * (uint32_t)sizeof(G)));
}

template <int LD, int MU, bool FWD>
__device__ __forceinline__ void sap_hop(const Geo& g, uint32_t lo, int l, const int lc[4], const float2* sh,
                                        const float2* __restrict__ U, cx<float> acc[12]) {
    const BlockHop b = block_hop<MU, FWD>(g, l, lc);
    cx<float> u[9], p[12], h[6];
    block_links<float2>(U, MU, g.V, lo + b.ls, [&](int e, float2 v) { u[e] = cmk(v.x, v.y); });
#pragma unroll
    for (int sc = 0; sc < 12; ++sc) p[sc] = ldc<float2, float>(sh + sc * LD + b.jl);
    project<MU, FWD, float>(p, h);
    cx<float> o[6];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            cx<float> t = cmk(0.f, 0.f);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                if (FWD) cmac(t, u[a * 3 + c], h[s * 3 + c]);
                else cjmac(t, u[c * 3 + a], h[s * 3 + c]);
            }
            o[s * 3 + a] = t;
        }
    reconstruct_sg<MU, FWD, float>(acc, o, b.sg);
    // keep the next hop's loads after this one (bounded register use)
    __builtin_amdgcn_sched_barrier(0);
}

// The same on packed FP16 data (FP16 links): the link products as v_dot2_f32_f16
// with FP32 sums.  A lane without a neighbour in the block reads the zero column
// LD - 64; only where a hop can wrap back into the block (WRAP: a block-grid
// extent of one) does the sum carry a boundary phase.
template <int LD, int MU, bool FWD, bool WRAP>
__device__ __forceinline__ void sap_hop(const Geo& g, uint32_t lo, int l, const int lc[4], const h2* sh,
                                        const h2* __restrict__ U, cx<float> acc[12]) {
    BlockHop b = block_hop<MU, FWD>(g, l, lc);
    h2 u[9], p[12], hre[6], him[6];
    block_links<h2>(U, MU, g.V, lo + b.ls, [&](int e, h2 v) { u[e] = v; });
    if (b.sg == 0.f) b.jl = LD - 64;
#pragma unroll
    for (int sc = 0; sc < 12; ++sc) p[sc] = sh[sc * LD + b.jl];
    proj_h<MU, FWD, FWD ? FN : FZ>(p, hre);
    proj_h<MU, FWD, FWD ? FS : FSN>(p, him);
    cx<float> o[6];
#pragma unroll
    for (int sp = 0; sp < 2; ++sp)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            float re = 0.f, im = 0.f;
#pragma unroll
            for (int c2 = 0; c2 < 3; ++c2) {
                const h2 uu = FWD ? u[a * 3 + c2] : u[c2 * 3 + a];
                re = dot2(uu, hre[sp * 3 + c2], re);
                im = dot2(uu, him[sp * 3 + c2], im);
            }
            o[sp * 3 + a] = cmk(re, im);
        }
    if (WRAP) reconstruct_sg<MU, FWD, float>(acc, o, b.sg);
    else reconstruct_add<MU, FWD, float>(acc, o);
    __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ h2 to_h2(cx<float> v) { return h2{(_Float16)v.re, (_Float16)v.im}; }

// scale of the FP16 copy of a block vector: sigma = the root mean square
// entry (|s|^2 / nent)^(1/2), formed as |s| / nent^(1/2) so that nothing
// underflows, when |s|^2 is a normal FP32 number in [1e-36, 1e36]; else
// sigma = 1 (a block with entries this small drops out of FP16 and is left
// as it is; NaN and infinity also take this branch)
__device__ __forceinline__ void sap_sigma(float ss, float rnent, float& sig, float& isig) {
    if (ss >= 1e-36f && ss <= 1e36f) {
        sig = sqrtf(ss) * rnent;
        isig = 1.f / sig;
    } else {
        sig = 1.f;
        isig = 1.f;
    }
}

// v + v of the lane whose number differs in bit BIT: the sums of a butterfly, by
// register swaps and row operations instead of LDS round trips (a row rotation
// by 4 pairs the same sums as an exchange of bit 2 once bit 3 is summed)
template <int BIT> __device__ __forceinline__ float lane_add(float v) {
    const int x = __float_as_int(v);
    if constexpr (BIT == 32) {
        const auto p = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        return __int_as_float(p[0]) + __int_as_float(p[1]);
    } else if constexpr (BIT == 16) {
        const auto p = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        return __int_as_float(p[0]) + __int_as_float(p[1]);
    } else {
        // row_ror:8, row_ror:4, quad_perm [2,3,0,1], quad_perm [1,0,3,2]
        constexpr int ctrl = BIT == 8 ? 0x128 : BIT == 4 ? 0x124 : BIT == 2 ? 0x4e : 0xb1;
        return v + __int_as_float(__builtin_amdgcn_update_dpp(0, x, ctrl, 0xf, 0xf, true));
    }
}

// sum of N values over the workgroup (every thread gets the totals)
template <int NT, int N>
__device__ __forceinline__ void sap_reduce(float (&v)[N], float* red) {
#pragma unroll
    for (int n = 0; n < N; ++n) {
        v[n] = lane_add<32>(v[n]);
        v[n] = lane_add<16>(v[n]);
        v[n] = lane_add<8>(v[n]);
        v[n] = lane_add<4>(v[n]);
        v[n] = lane_add<2>(v[n]);
        v[n] = lane_add<1>(v[n]);
    }
    constexpr int nw = NT / 64;
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int n = 0; n < N; ++n) red[N * w + n] = v[n];
    }
    __syncthreads();
#pragma unroll
    for (int n = 0; n < N; ++n) v[n] = 0.f;
#pragma unroll
    for (int k = 0; k < nw; ++k)
#pragma unroll
        for (int n = 0; n < N; ++n) v[n] += red[N * k + n];
}

// nmr minimal-residual steps on M_BB d = rho_B and z += d: one workgroup per
// (block, right-hand side), one thread per block site.  The vector s lives in
// LDS for the block operator's neighbour reads (FP32, or FP16 with FP16 links,
// where the block steps compute on packed FP16 data with FP32 sums) and in FP32
// registers for the site's own arithmetic; z waits in LDS.
//
// FP16 links: the FP16 copy holds s / sigma, sigma the root mean square entry
// over the block of the previous step's s (of rho_B for the first step), so
// that the block's values sit in FP16's normal range whatever the scale of the
// right-hand side (solutions of point sources fall off by orders of magnitude
// across the lattice) and never overflow it (a minimal-residual step does not
// increase |s|); t = sigma M_BB (s / sigma).  |s|^2 is summed afresh in every
// step's reduction: tracking it by |s'|^2 = |s|^2 - |<t,s>|^2 / |t|^2 cancels
// when a step removes nearly all of a block's residual, and the scale then
// overflowed FP16.
// LDS of a workgroup of NT threads (the sites of a block, rounded up to
// wavefronts): z, the copy of s (column NT: zero) and the reduction's partials.
template <typename G, int NT> struct SapLds {
    static constexpr bool PK = std::is_same<G, h2>::value;
    static constexpr int LD = PK ? NT + 64 : NT;
    typedef typename std::conditional<PK, h2, float2>::type SH;
    float2 zs[12 * NT];
    SH sh[12 * LD];
    float red[4 * (NT / 64)];
};
// s: rho on entry; WRAP: some block-grid extent is one
template <typename G, int NT, bool WRAP>
__device__ __forceinline__ void sap_block_solve(const Geo& g, uint32_t lo, int l, bool on, const int lc[4],
                                                const G* __restrict__ U, const G* __restrict__ C, float kappa, int nmr,
                                                cx<float> s[12], SapLds<G, NT>& L) {
    constexpr bool PK = SapLds<G, NT>::PK;
    constexpr int LD = SapLds<G, NT>::LD;
    const uint32_t V = g.V;
    const int lt = threadIdx.x;
    auto* sh = L.sh;
    float2* zs = L.zs;
    float* red = L.red;
    if constexpr (PK) {
        if (lt < 12) sh[lt * LD + NT] = h2{(_Float16)0, (_Float16)0};
    }
    float sig = 1.f, isig = 1.f;
    const float rnent = 1.f / sqrtf(12.f * (float)g.Vb);
    if (PK) {
        float v[1] = {0.f};
#pragma unroll
        for (int k = 0; k < 12; ++k) v[0] += s[k].re * s[k].re + s[k].im * s[k].im;
        if (g.Vb < NT) v[0] = on ? v[0] : 0.f;
        sap_reduce<NT, 1>(v, red);
        sap_sigma(v[0], rnent, sig, isig);
    }
    for (int it = 0; it < nmr; ++it) {
        // the previous step's neighbour reads ended before its reduction
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            if constexpr (PK) {
                sh[k * LD + lt] = to_h2(isig * s[k]);
            } else {
                sh[k * LD + lt] = make_float2(s[k].re, s[k].im);
            }
        }
        __syncthreads();
        // links and clover are re-read every step: an offset opaque to the
        // compiler keeps their loads inside the loop instead of holding all
        // of them in registers across the steps
        const uint32_t lo_o = opaque_v(lo), io = lo_o + (uint32_t)l;
        cx<float> t[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) t[k] = cmk(0.f, 0.f);
        if constexpr (PK) {
            sap_hop<LD, 0, true, WRAP>(g, lo_o, l, lc, sh, U, t);
            sap_hop<LD, 0, false, WRAP>(g, lo_o, l, lc, sh, U, t);
            sap_hop<LD, 1, true, WRAP>(g, lo_o, l, lc, sh, U, t);
            sap_hop<LD, 1, false, WRAP>(g, lo_o, l, lc, sh, U, t);
            sap_hop<LD, 2, true, WRAP>(g, lo_o, l, lc, sh, U, t);
            sap_hop<LD, 2, false, WRAP>(g, lo_o, l, lc, sh, U, t);
            sap_hop<LD, 3, true, WRAP>(g, lo_o, l, lc, sh, U, t);
            sap_hop<LD, 3, false, WRAP>(g, lo_o, l, lc, sh, U, t);
        } else {
            sap_hop<LD, 0, true>(g, lo_o, l, lc, sh, U, t);
            sap_hop<LD, 0, false>(g, lo_o, l, lc, sh, U, t);
            sap_hop<LD, 1, true>(g, lo_o, l, lc, sh, U, t);
            sap_hop<LD, 1, false>(g, lo_o, l, lc, sh, U, t);
            sap_hop<LD, 2, true>(g, lo_o, l, lc, sh, U, t);
            sap_hop<LD, 2, false>(g, lo_o, l, lc, sh, U, t);
            sap_hop<LD, 3, true>(g, lo_o, l, lc, sh, U, t);
            sap_hop<LD, 3, false>(g, lo_o, l, lc, sh, U, t);
        }
#pragma unroll
        for (int ch = 0; ch < 2; ++ch) {
            if constexpr (PK) {
                // Rounded from the FP32 registers again (once, in v_fma_mixlo, for
                // the negated forms), component 5 as the neighbours read it; a
                // scale opaque to the compiler keeps the copy in LDS out of it.
                // Nothing singles component 5 out: these are the roundings of the
                // results so far.  The four steps amplify one unit in the last
                // place, so any single rule (the copy in LDS for all twelve, or
                // these rounded alike, and one form of the update below) moves z by
                // 1.3e-5 to 3.9e-5 of its norm, at the same error of 2.86e-4
                // against 64-bit values; the copy takes 1 % less time.
                const float isc = __int_as_float((int)opaque_v((uint32_t)__float_as_int(isig)));
                h2 own[1][6];
                cx<float> res[1][6];
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    own[0][k] = 6 * ch + k == 5 ? sh[5 * LD + lt] : to_h2(isc * s[6 * ch + k]);
                    res[0][k] = -kappa * t[6 * ch + k];
                }
                clover_dot2<1>([&](int k) { return buf_ld<h2>(comp_rsrc<SAP_COMPS>(C, ch * 18 + k / 3 * 3, V), io * 4u,
                                                              k % 3 * V * 4u); },
                               own, res);
#pragma unroll
                for (int k = 0; k < 6; ++k) t[6 * ch + k] = sig * res[0][k];
            } else {
                cx<float> res[6];
                clover_apply<float>([&](int k) { return buf_ldc<G, float>(comp_rsrc<SAP_COMPS>(C, ch * 18 + k / 3 * 3, V), io,
                                                                          k % 3 * V); },
                                    s + 6 * ch, res);
#pragma unroll
                for (int k = 0; k < 6; ++k) t[6 * ch + k] = res[k] - kappa * t[6 * ch + k];
            }
        }
        // <t,s>, <t,t> and (FP16 links) |s|^2; the reduction also orders this
        // step's LDS reads before the next step's writes
        float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            v[0] += t[k].re * s[k].re + t[k].im * s[k].im;
            v[1] += t[k].re * s[k].im - t[k].im * s[k].re;
            v[2] += t[k].re * t[k].re + t[k].im * t[k].im;
            if (PK) v[3] += s[k].re * s[k].re + s[k].im * s[k].im;
        }
        // idle threads repeat the last site: they take no part in the sums
        if (g.Vb < NT) {
#pragma unroll
            for (int n = 0; n < 4; ++n) v[n] = on ? v[n] : 0.f;
        }
        if constexpr (PK) {
            sap_reduce<NT, 4>(v, red);
        } else {
            float w[3] = {v[0], v[1], v[2]};
            sap_reduce<NT, 3>(w, red);
            v[0] = w[0];
            v[1] = w[1];
            v[2] = w[2];
        }
        const float tt = v[2];
        const cx<float> om = tt > 0.f ? cmk(v[0] / tt, v[1] / tt) : cmk(0.f, 0.f);
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            cx<float> zk = ldc<float2, float>(zs + k * NT + lt);
            cmac(zk, om, s[k]);
            zs[k * NT + lt] = make_float2(zk.re, zk.im);
        }
        if (it + 1 == nmr) break;
        if (PK) sap_sigma(v[3], rnent, sig, isig);   // the scale of the next copy
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            if constexpr (PK) {   // fused by hand, so that the source says where the roundings fall
                s[k].re -= __builtin_fmaf(t[k].re, om.re, -(t[k].im * om.im));
                s[k].im -= k == 5 ? __builtin_fmaf(t[k].im, om.re, t[k].re * om.im)
                                  : __builtin_fmaf(t[k].re, om.im, t[k].im * om.re);
            } else {
                s[k] = s[k] - om * t[k];
            }
        }
    }
}

// x, in an order after all of v
__device__ __forceinline__ uint32_t after_v(uint32_t x, const cx<float> v[12]) {
    asm volatile("" : "+v"(x)
                 : "v"(v[0].re), "v"(v[0].im), "v"(v[1].re), "v"(v[1].im), "v"(v[2].re), "v"(v[2].im), "v"(v[3].re),
                   "v"(v[3].im), "v"(v[4].re), "v"(v[4].im), "v"(v[5].re), "v"(v[5].im), "v"(v[6].re), "v"(v[6].im),
                   "v"(v[7].re), "v"(v[7].im), "v"(v[8].re), "v"(v[8].im), "v"(v[9].re), "v"(v[9].im), "v"(v[10].re),
                   "v"(v[10].im), "v"(v[11].re), "v"(v[11].im));
    return x;
}

// hop of the full operator for the residual: the neighbour's spinor from the
// LDS copy of the block's z when it lies inside the block (not across a lattice
// wrap), else from the global field; no branches (tile_nbr's offsets)
template <int NT, int MU, bool FWD, typename G>
__device__ __forceinline__ void sap_hop_res(const Geo& g, int i, int l, const int lc[4], const int yc[4],
                                            const FieldRsrc& pz, const float2* zs, const G* __restrict__ U,
                                            cx<float> acc[12]) {
    const uint32_t V = g.V;
    bool wrap;
    const int j = FWD ? geo_fwd(g, i, MU, lc, yc, &wrap) : geo_bwd(g, i, MU, lc, yc, &wrap);
    const bool in = FWD ? (lc[MU] + 1 < g.b[MU]) : (lc[MU] > 0);
    // this hop's loads after the sums of the hop before it (bounded register use)
    const uint32_t off = after_v(in ? 0xfffffff0u : (uint32_t)j * 8u, acc);
    const uint32_t us = after_v((uint32_t)(FWD ? i : j) * (uint32_t)sizeof(G), acc);
    const int jl = in ? (FWD ? l + g.sl[MU] : l - g.sl[MU]) : l;
    cx<float> p[12], h[6];
#pragma unroll
    for (int sc = 0; sc < 12; ++sc) {
        const float2 a = buf_ld<float2>(pz.part[sc / 2], off, sc % 2 * V * 8u), b = zs[sc * NT + jl];
        p[sc] = cmk(in ? b.x : a.x, in ? b.y : a.y);
    }
    project<MU, FWD, float>(p, h);
    cx<float> o[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) o[k] = cmk(0.f, 0.f);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const rsrc_t ru = comp_rsrc<SAP_COMPS>(U, MU * 9 + 3 * a, V);
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const G w = buf_ld<G>(ru, us, b * V * (uint32_t)sizeof(G));
            const cx<float> v = ldc<G, float>(&w);      // link entry (a, b)
#pragma unroll
            for (int sp = 0; sp < 2; ++sp) {
                if (FWD) cmac(o[sp * 3 + a], v, h[sp * 3 + b]);
                else cjmac(o[sp * 3 + b], v, h[sp * 3 + a]);
            }
        }
    }
    reconstruct_sg<MU, FWD, float>(acc, o, wrap && g.bcneg[MU] ? -1.f : 1.f);
    // keep the next hop's loads after this one (bounded register use)
    __builtin_amdgcn_sched_barrier(0);
}

// The residual and the block solve of one (block, right-hand side).
template <typename G, typename GP, int W, int NT, bool WRAP>
__global__ __launch_bounds__(NT, W) void k_sap_half(Geo g, const float2* __restrict__ rhs, float2* __restrict__ z,
                                                           const G* __restrict__ U, const G* __restrict__ C,
                                                           float kappa, const int* __restrict__ blist, int nblk,
                                                           int nrhs, int npad, int nmr) {
    __shared__ SapLds<GP, NT> L;
    const int item = (blockIdx.x & 7) * (npad >> 3) + (blockIdx.x >> 3);
    if (item >= nblk * nrhs) return;   // uniform over the workgroup
    const int kb = item / nrhs, q = item - kb * nrhs;
    const uint32_t V = g.V, lo = (uint32_t)blist[kb] * (uint32_t)g.Vb;
    const bool on = (int)threadIdx.x < g.Vb;
    const int lt = threadIdx.x, l = on ? lt : g.Vb - 1, i = (int)lo + l;
    int lc[4], yc[4];
    geo_coords(g, i, lc, yc);
    const FieldRsrc pz = field_rsrc(z + (size_t)q * 12 * V, V), pr = field_rsrc(rhs + (size_t)q * 12 * V, V);
#pragma unroll
    for (int k = 0; k < 12; ++k) L.zs[k * NT + lt] = buf_ld<float2>(pz.part[k / 2], (uint32_t)i * 8u, k % 2 * V * 8u);
    __syncthreads();
    cx<float> s[12];
    {
        cx<float> acc[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = cmk(0.f, 0.f);
        sap_hop_res<NT, 0, true, G>(g, i, l, lc, yc, pz, L.zs, U, acc);
        sap_hop_res<NT, 0, false, G>(g, i, l, lc, yc, pz, L.zs, U, acc);
        sap_hop_res<NT, 1, true, G>(g, i, l, lc, yc, pz, L.zs, U, acc);
        sap_hop_res<NT, 1, false, G>(g, i, l, lc, yc, pz, L.zs, U, acc);
        sap_hop_res<NT, 2, true, G>(g, i, l, lc, yc, pz, L.zs, U, acc);
        sap_hop_res<NT, 2, false, G>(g, i, l, lc, yc, pz, L.zs, U, acc);
        sap_hop_res<NT, 3, true, G>(g, i, l, lc, yc, pz, L.zs, U, acc);
        sap_hop_res<NT, 3, false, G>(g, i, l, lc, yc, pz, L.zs, U, acc);
#pragma unroll
        for (int ch = 0; ch < 2; ++ch) {
            cx<float> p[6], res[6];
#pragma unroll
            for (int k = 0; k < 6; ++k) p[k] = ldc<float2, float>(L.zs + (6 * ch + k) * NT + lt);
            const uint32_t io = after_v((uint32_t)i, acc);
            tile_clover<false, G, float>(nullptr, 0, C, V, io, ch, p, res);
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                const int sc = 6 * ch + k;
                s[sc] = buf_ldc<float2, float>(pr.part[sc / 2], io, sc % 2 * V) - (res[k] - kappa * acc[sc]);
            }
        }
    }
    sap_block_solve<GP, NT, WRAP>(g, lo, l, on, lc, (const GP*)U, (const GP*)C, kappa, nmr, s, L);
    if (on) {
#pragma unroll
        for (int k = 0; k < 12; ++k) buf_st<float2>(z + (size_t)q * 12 * V, V, (uint32_t)i, k, L.zs[k * NT + lt]);
    }
}

}  // namespace

// Block order by colour (lazy; depends on the geometry only).  SAP needs
// every block-grid extent even or one (then blocks of one colour never
// couple) and at most 256 sites per block.
int mg_sap_setup(mglma_ctx* c) {
    if (c->sap_blk) return MGLMA_OK;
    const Geo& g = c->geo;
    for (int mu = 0; mu < 4; ++mu)
        if (g.L1[mu] != 1 && g.L1[mu] % 2) return MGLMA_ERR_SHAPE;
    if (g.Vb > SAP_MAXVB) return MGLMA_ERR_SHAPE;
    std::vector<int> order;
    order.reserve(g.V1);
    int n0 = 0;
    for (int colour = 0; colour < 2; ++colour) {
        if (colour == 1) n0 = (int)order.size();
        for (int y = 0; y < g.V1; ++y) {
            int k = y, par = 0;
            for (int mu = 3; mu >= 0; --mu) {
                par += k % g.L1[mu];
                k /= g.L1[mu];
            }
            if (par % 2 == colour) order.push_back(y);
        }
    }
    int* d = nullptr;
    MG_TRY(mg_malloc(c, (void**)&d, (size_t)g.V1 * sizeof(int)));
    HIP_TRY(hipMemcpyAsync(d, order.data(), (size_t)g.V1 * sizeof(int), hipMemcpyHostToDevice, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    c->sap_blk = d;
    c->sap_n0 = n0;
    return MGLMA_OK;
}

// one half-sweep: the blocks bl[0..nblk) of one colour (GP: the links' type in
// the packed arithmetic of the block steps)
template <typename G, typename GP, int W, int NT>
static int sap_half_nt(mglma_ctx* c, const int* bl, int nblk, const float2* r, float2* z, const G* U, const G* C,
                       int nrhs, int nmr) {
    const Geo& g = c->geo;
    const long long npad = ((long long)nblk * nrhs + 7) / 8 * 8;
    if (npad > 0x7fffffffLL) return MGLMA_ERR_SHAPE;
    if (g.L1[0] == 1 || g.L1[1] == 1 || g.L1[2] == 1 || g.L1[3] == 1)
        hipLaunchKernelGGL((k_sap_half<G, GP, W, NT, true>), dim3((unsigned)npad), dim3(NT), 0, c->stream, g, r, z, U, C,
                           (float)c->kappa, bl, nblk, nrhs, (int)npad, nmr);
    else
        hipLaunchKernelGGL((k_sap_half<G, GP, W, NT, false>), dim3((unsigned)npad), dim3(NT), 0, c->stream, g, r, z, U,
                           C, (float)c->kappa, bl, nblk, nrhs, (int)npad, nmr);
    HIP_TRY(hipGetLastError());
    return MGLMA_OK;
}
template <typename G, typename GP, int W>
static int sap_half(mglma_ctx* c, const int* bl, int nblk, const float2* r, float2* z, const G* U, const G* C,
                    int nrhs, int nmr) {
    switch ((c->geo.Vb + 63) / 64) {
        case 1: return sap_half_nt<G, GP, W, 64>(c, bl, nblk, r, z, U, C, nrhs, nmr);
        case 2: return sap_half_nt<G, GP, W, 128>(c, bl, nblk, r, z, U, C, nrhs, nmr);
        case 3: return sap_half_nt<G, GP, W, 192>(c, bl, nblk, r, z, U, C, nrhs, nmr);
        default: return sap_half_nt<G, GP, W, 256>(c, bl, nblk, r, z, U, C, nrhs, nmr);
    }
}

// ncycle SAP cycles on M z = r (FP32 vectors, z updated in place); links and
// clover from the FP16 (prec F16) or FP32 (prec F32) copies
#define SAP_EV_MAX 4096
static int sap_fold_events(mglma_ctx* c);

int mg_sap(mglma_ctx* c, int prec, const void* r, void* z, int nrhs, int ncycle, int nmr) {
    if (nrhs == 0 || ncycle == 0) return MGLMA_OK;
    MG_TRY(mg_sap_setup(c));
    const Geo& g = c->geo;
    if (!sap_fits(g.V)) return MGLMA_ERR_SHAPE;   // 179 million sites: links and clover term are 361 GB there
    for (int h = 0; h < 2 * ncycle; ++h) {
        const int nblk = h % 2 == 0 ? c->sap_n0 : g.V1 - c->sap_n0;
        if (nblk == 0) continue;
        const int* bl = c->sap_blk + (h % 2 == 0 ? 0 : c->sap_n0);
        hipEvent_t ev[2] = {nullptr, nullptr};
        if (c->sap_timing) {
            // at most SAP_EV_MAX recorded pairs: fold the finished ones
            // into the running sum before reusing their events
            if (c->sap_ev_used + 2 > 2 * SAP_EV_MAX) MG_TRY(sap_fold_events(c));
            while (c->sap_ev.size() < c->sap_ev_used + 2) {
                hipEvent_t e;
                HIP_TRY(hipEventCreate(&e));
                c->sap_ev.push_back(e);
            }
            ev[0] = c->sap_ev[c->sap_ev_used];
            ev[1] = c->sap_ev[c->sap_ev_used + 1];
            HIP_TRY(hipEventRecord(ev[0], c->stream));
        }
        if (prec == MGLMA_F16)
            MG_TRY((sap_half<__half2, h2, 4>(c, bl, nblk, (const float2*)r, (float2*)z, c->U16, c->C16, nrhs, nmr)));
        else
            MG_TRY((sap_half<float2, float2, 3>(c, bl, nblk, (const float2*)r, (float2*)z, c->U32, c->C32, nrhs, nmr)));
        if (ev[1]) {
            HIP_TRY(hipEventRecord(ev[1], c->stream));
            c->sap_ev_used += 2;   // counted once both events are recorded
        }
    }
    return MGLMA_OK;
}

static void sap_clear_timing(mglma_ctx* c) {
    c->sap_ev_used = 0;
    c->sap_ms_acc = 0.0;
    c->sap_n_acc = 0;
}

// add the durations of the recorded pairs to the running sum and free the pairs
static int sap_fold_events(mglma_ctx* c) {
    hipError_t e = hipStreamSynchronize(c->stream);
    for (size_t k = 0; e == hipSuccess && k + 1 < c->sap_ev_used; k += 2) {
        float t = 0.f;
        e = hipEventElapsedTime(&t, c->sap_ev[k], c->sap_ev[k + 1]);
        c->sap_ms_acc += t;
        c->sap_n_acc += 1;
    }
    c->sap_ev_used = 0;
    if (e != hipSuccess) {
        sap_clear_timing(c);
        mg_last_hip_error(e, "SAP launch timing", __FILE__, __LINE__);
        return MGLMA_ERR_HIP;
    }
    return MGLMA_OK;
}

extern "C" int mglma_sap_timing(mglma_ctx* c, int enable) {
    if (!c) return MGLMA_ERR_ARG;
    sap_clear_timing(c);
    HIP_TRY(hipStreamSynchronize(c->stream));
    c->sap_timing = enable != 0;
    return MGLMA_OK;
}

extern "C" int mglma_sap_elapsed(mglma_ctx* c, double* ms, int* launches) {
    if (!c || !ms || !launches) return MGLMA_ERR_ARG;
    MG_TRY(sap_fold_events(c));
    *ms = c->sap_ms_acc;
    *launches = (int)c->sap_n_acc;
    sap_clear_timing(c);
    return MGLMA_OK;
}

extern "C" int mglma_sap_smooth(mglma_ctx* c, int prec, int ncycle, int nmr, const float* r_dev, float* z_dev,
                                int nrhs) {
    if (!c || !r_dev || !z_dev || nrhs < 0 || nrhs > 65535 || ncycle < 0 || nmr < 0 || nmr > 64)
        return MGLMA_ERR_ARG;
    if (prec != MGLMA_F16 && prec != MGLMA_F32) return MGLMA_ERR_ARG;
    if (!c->have_gauge) return MGLMA_ERR_NO_GAUGE;
    return mg_sap(c, prec, r_dev, z_dev, nrhs, ncycle, nmr);
}
