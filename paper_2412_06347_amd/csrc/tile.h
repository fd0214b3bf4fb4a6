// Wilson hops of a tile of 64 sites for a batch of right-hand sides, and the
// buffer accesses they share with the SAP kernel.
//
// A workgroup owns 64 consecutive sites (lane = site) and its wavefronts walk
// the right-hand sides, one per wavefront at a time.  The tile's eight links
// per site are staged in LDS once for the whole batch; the spinors of
// neighbours inside the tile come from the lane that owns them, so only the
// faces of the tile (a time slice of a 4^4 block) are read through the caches.
#pragma once
#include "mglma_internal.h"
#include "wilson.h"

#define TILE 64                     // sites of a workgroup
// staged entries: links [direction 2 mu + backward][9][TILE] and, CL, the clover term [2][18][TILE]
__host__ __device__ constexpr int tile_gauge(bool CL) { return (CL ? 108 : 72) * TILE; }

// the wavefront's index as a scalar (uniform addresses for its right-hand side)
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

// Launch shape of a batch of nrhs right-hand sides: tiles padded to a multiple
// of the XCD count, and ng workgroups per tile, back to back on one XCD, that
// share the right-hand sides.  One workgroup stages a tile's links once for
// the whole batch; where the tiles alone leave the chip idle (fewer than two
// workgroups per compute unit) the rounds of four right-hand sides are dealt
// to several.
struct TileGrid {
    int nt, ng;
    dim3 grid, block;
    TileGrid(int V, int nrhs) {
        const int rounds = (nrhs + 3) / 4;
        nt = ((V + TILE - 1) / TILE + 7) / 8 * 8;
        ng = nt >= 512 ? 1 : (512 + nt - 1) / nt;
        if (ng > rounds) ng = rounds;
        grid = dim3((unsigned)nt * ng);
        block = dim3(64 * ((nrhs + rounds - 1) / rounds));
    }
};

// every wavefront copies its share of the tile's links U_mu(x), U_mu(x - mu) and clover term
template <bool CL, typename G>
__device__ __forceinline__ void tile_stage_gauge(const Geo& g, int i, const int lc[4], const int yc[4],
                                                 const G* __restrict__ U, const G* __restrict__ C, G* ul, int w,
                                                 int nw, int lane) {
    const size_t V = g.V;
    for (int d = w; d < (CL ? 12 : 8); d += nw) {
        const int mu = d >> 1;
        int j = i;
        bool wrap;
        // static indices for the coordinate arrays
        if (d < 8 && (d & 1)) j = mu == 0 ? geo_bwd(g, i, 0, lc, yc, &wrap)
                       : mu == 1 ? geo_bwd(g, i, 1, lc, yc, &wrap)
                       : mu == 2 ? geo_bwd(g, i, 2, lc, yc, &wrap) : geo_bwd(g, i, 3, lc, yc, &wrap);
        const G* src = d < 8 ? U + (size_t)(mu * 9) * V : C + (size_t)((d - 8) * 9) * V;
        G v[9];
#pragma unroll
        for (int e = 0; e < 9; ++e) v[e] = src[(size_t)e * V + (uint32_t)j];
#pragma unroll
        for (int e = 0; e < 9; ++e) ul[(d * 9 + e) * TILE + lane] = v[e];
    }
}

// Links and clover do not change between the right-hand sides; offsets that the
// compiler cannot see through keep their loads inside the loop over the
// right-hand sides instead of in registers across it.
__device__ __forceinline__ uint32_t opaque_v(uint32_t x) {
    asm volatile("" : "+v"(x));
    return x;
}
// Buffer loads and stores: the per-component offset (component x V) is uniform
// and goes in a scalar register, the site offset is the only vector operand.
// A resource's bytes stay below 2^32: it spans at most TILE_COMPS components of
// the fields, links and clover term here, SAP_COMPS in the SAP kernel, and larger
// lattices take another path (tile_fits) or are refused (sap_fits).
constexpr int TILE_COMPS = 2, SAP_COMPS = 3;
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t mk_rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
typedef uint32_t u2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u4_t __attribute__((ext_vector_type(4)));
template <typename S> __device__ __forceinline__ S buf_ld(rsrc_t r, uint32_t off, uint32_t soff) {
    if constexpr (sizeof(S) == 4) return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b32(r, off, soff, 0));
    else if constexpr (sizeof(S) == 8) return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, 0));
    else return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, 0));
}
// Stores take component `comp` V + `site` of a field with the component in the
// resource's address and no scalar offset: a 16-byte buffer store whose scalar
// offset is a register gets no wait state before a later write of its data
// registers, and on gfx950 that write has reached the last four lanes of each
// row of 16 first (FP64 batches: a few wrong values per 10^8).  With a constant
// offset the compiler places the wait state.
template <typename S> __device__ __forceinline__ void buf_st(S* f, uint32_t V, uint32_t site, int comp, S v) {
    const rsrc_t r = mk_rsrc(f + (size_t)comp * V, V * (uint32_t)sizeof(S));
    const uint32_t off = site * (uint32_t)sizeof(S);
    if constexpr (sizeof(S) == 4) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, off, 0, 0);
    else if constexpr (sizeof(S) == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2_t, v), r, off, 0, 0);
    else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4_t, v), r, off, 0, 0);
}
// components [c0, c0 + n) of a field (n: 1, TILE_COMPS or SAP_COMPS)
template <int n, typename S> __device__ __forceinline__ rsrc_t comp_rsrc(S* f, int c0, uint32_t V) {
    return mk_rsrc(f + (size_t)c0 * V, n * V * (uint32_t)sizeof(S));
}
// one right-hand side
struct FieldRsrc {
    rsrc_t part[6];
};
template <typename S> __device__ __forceinline__ FieldRsrc field_rsrc(S* f, uint32_t V) {
    return {{comp_rsrc<TILE_COMPS>(f, 0, V), comp_rsrc<TILE_COMPS>(f, 2, V), comp_rsrc<TILE_COMPS>(f, 4, V),
             comp_rsrc<TILE_COMPS>(f, 6, V), comp_rsrc<TILE_COMPS>(f, 8, V), comp_rsrc<TILE_COMPS>(f, 10, V)}};
}
static inline bool rsrc_fits(size_t V, size_t sbytes, int comps) { return comps * V * sbytes < ((size_t)1 << 32); }
static inline bool tile_fits(size_t V, size_t sbytes) { return rsrc_fits(V, sbytes, TILE_COMPS); }
static inline bool sap_fits(size_t V) { return rsrc_fits(V, sizeof(float2), SAP_COMPS); }
// entry `comp` V + `site` of a resource, as complex R
template <typename S, typename R> __device__ __forceinline__ cx<R> buf_ldc(rsrc_t r, uint32_t site, uint32_t comp) {
    const S v = buf_ld<S>(r, site * (uint32_t)sizeof(S), comp * (uint32_t)sizeof(S));
    return ldc<S, R>(&v);
}
template <typename S, typename R>
__device__ __forceinline__ void buf_stc(S* f, uint32_t V, uint32_t site, int comp, cx<R> x) {
    S v;
    stc<S, R>(&v, x);
    buf_st<S>(f, V, site, comp, v);
}

template <typename S, typename R>
__device__ __forceinline__ void tile_own(const FieldRsrc& pr, uint32_t io, uint32_t V, cx<R> own[12]) {
#pragma unroll
    for (int k = 0; k < 12; ++k) own[k] = buf_ldc<S, R>(pr.part[k / 2], io, k % 2 * V);
}

// value of another lane of the wavefront; src = 4 * lane
__device__ __forceinline__ int lane_get(int v, int src) { return __builtin_amdgcn_ds_bpermute(src, v); }
__device__ __forceinline__ float lane_get(float v, int src) { return __int_as_float(lane_get(__float_as_int(v), src)); }
__device__ __forceinline__ double lane_get(double v, int src) {
    return __hiloint2double(lane_get(__double2hiint(v), src), lane_get(__double2loint(v), src));
}
template <typename R> __device__ __forceinline__ cx<R> lane_get(cx<R> v, int src) {
    return cmk(lane_get(v.re, src), lane_get(v.im, src));
}

// Where a hop's neighbour spinor comes from: from lane src / 4 when the
// neighbour lies in the tile, else from memory.  Lanes that need no load carry
// an offset past the resource, for which a buffer load returns 0 without an
// access.
struct Nbr {
    uint32_t off;    // byte offset of the neighbour site
    int src;
    bool in, neg;    // inside the tile; the boundary phase applies
};
template <int MU, bool FWD>
__device__ __forceinline__ Nbr tile_nbr(const Geo& g, int i, int i0, const int lc[4], const int yc[4], uint32_t size) {
    bool wrap;
    const int j = FWD ? geo_fwd(g, i, MU, lc, yc, &wrap) : geo_bwd(g, i, MU, lc, yc, &wrap);
    const uint32_t k = (uint32_t)(j - i0);
    Nbr n;
    n.in = k < TILE;
    n.off = n.in ? 0xfffffff0u : (uint32_t)j * size;
    n.src = 4 * (int)(k & (TILE - 1));
    n.neg = wrap && g.bcneg[MU];
    return n;
}

// acc += (1 -/+ gamma_mu) U psi of one hop for the right-hand side in pr, own =
// the spinor of the lane's own site
template <int MU, bool FWD, typename S, typename G, typename R>
__device__ __forceinline__ void tile_hop(const Geo& g, int i, int i0, const int lc[4], const int yc[4],
                                         const FieldRsrc& pr, const cx<R> own[12], const G* ul, int lane,
                                         cx<R> acc[12]) {
    const uint32_t V = g.V;
    const Nbr n = tile_nbr<MU, FWD>(g, i, i0, lc, yc, sizeof(S));
    cx<R> p[12], h[6], hl[6];
#pragma unroll
    for (int sc = 0; sc < 12; ++sc) {
        const S v = buf_ld<S>(pr.part[sc / 2], n.off, (sc % 2) * V * (uint32_t)sizeof(S));
        p[sc] = ldc<S, R>(&v);
    }
    // the projection is the same on every lane: the owner of a neighbour inside
    // the tile projects, and six components instead of twelve change lanes
    project<MU, FWD, R>(own, h);
#pragma unroll
    for (int k = 0; k < 6; ++k) h[k] = lane_get(h[k], n.src);
    project<MU, FWD, R>(p, hl);
#pragma unroll
    for (int k = 0; k < 6; ++k) h[k] = cmk(n.in ? h[k].re : hl[k].re, n.in ? h[k].im : hl[k].im);
    const G* u = ul + (2 * MU + (FWD ? 0 : 1)) * 9 * TILE + lane;
    cx<R> o[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) o[k] = cmk((R)0, (R)0);
    // one link entry at a time: few live registers next to the accumulators
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const cx<R> v = ldc<G, R>(u + (FWD ? a * 3 + b : b * 3 + a) * TILE);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                if (FWD) cmac(o[s * 3 + a], v, h[s * 3 + b]);
                else cjmac(o[s * 3 + a], v, h[s * 3 + b]);
            }
        }
    reconstruct_sg<MU, FWD, R>(acc, o, n.neg ? (R)-1 : (R)1);
    // keep the next hop's loads after this one (bounded register use)
    __builtin_amdgcn_sched_barrier(0);
}

template <typename S, typename G, typename R>
__device__ __forceinline__ void tile_hops(const Geo& g, int i, int i0, const int lc[4], const int yc[4],
                                          const FieldRsrc& pr, const cx<R> own[12], const G* ul, int lane,
                                          cx<R> acc[12]) {
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = cmk((R)0, (R)0);
    tile_hop<0, true, S, G, R>(g, i, i0, lc, yc, pr, own, ul, lane, acc);
    tile_hop<0, false, S, G, R>(g, i, i0, lc, yc, pr, own, ul, lane, acc);
    tile_hop<1, true, S, G, R>(g, i, i0, lc, yc, pr, own, ul, lane, acc);
    tile_hop<1, false, S, G, R>(g, i, i0, lc, yc, pr, own, ul, lane, acc);
    tile_hop<2, true, S, G, R>(g, i, i0, lc, yc, pr, own, ul, lane, acc);
    tile_hop<2, false, S, G, R>(g, i, i0, lc, yc, pr, own, ul, lane, acc);
    tile_hop<3, true, S, G, R>(g, i, i0, lc, yc, pr, own, ul, lane, acc);
    tile_hop<3, false, S, G, R>(g, i, i0, lc, yc, pr, own, ul, lane, acc);
}

// res[6] = C_ch p[6] at site io
template <bool CL, typename G, typename R>
__device__ __forceinline__ void tile_clover(const G* ul, int lane, const G* C, uint32_t V, uint32_t io, int ch,
                                            const cx<R> p[6], cx<R> res[6]) {
    if (CL)
        clover_apply<R>([&](int k) { return ldc<G, R>(ul + (72 + ch * 18 + k) * TILE + lane); }, p, res);
    else
        clover_apply<R>([&](int k) {
            return buf_ldc<G, R>(comp_rsrc<TILE_COMPS>(C, ch * 18 + k / TILE_COMPS * TILE_COMPS, V), io,
                                 k % TILE_COMPS * V);
        }, p, res);
}
