// Coarse-grid operator application (fig:A): nearest-neighbour stencil of
// nine dense nc x nc complex blocks per coarse site,
//   out[r][y] = sum_dir D_1[y][dir] in[r][nbr(y, dir)],
// with gamma5 = 1 giving Q_1 = (gamma5)_1 D_1 (rows of the alpha = 1
// chirality negated).
//
// * FP64 / FP32 (matrix cores, v_mfma_f64_16x16x4 / v_mfma_f32_16x16x4):
//   same tiling as BF16 below, operator in the working precision (FP32: from a
//   planar copy), vectors loaded as they are.
// * BF16 (matrix cores): each wavefront owns a 16-row x 16-rhs output tile and
//   runs v_mfma_f32_16x16x16_bf16 over (direction, 16-column) steps.  The
//   complex product uses the planar real form
//   Re = Dr Br - Di Bi, Im = Dr Bi + Di Br (four real MFMAs per step); the
//   FP32 vectors are rounded to bfloat16 on load and accumulation is FP32.
#include "mglma_internal.h"

// FP64 / FP32 on the matrix cores (v_mfma_*_16x16x4).
// grid: the (coarse site, 16-rhs tile) items (site_tile); block: 64 *
// ceil(nc/16) * DG threads, wave w owns output rows 16w..16w+15 and the 16
// right-hand sides of the item's tile; with DG = 3 three waves take three of a row
// tile's directions each and their sums are added in LDS.  A wave that has all nine
// sums the same groups of three and adds them in the same order, so that a
// right-hand side's bits do not depend on the batch (1-4 % of the time; FP32 error
// against exact values, 48 columns, 7.2e-7 -> 3.9e-7).  FP64 reads the interleaved
// complex operator [y][dir][i][j] (the library's D_1 itself), FP32 the planar copy
// [y][dir][0 = re, 1 = im][i][j].
//
// In an MFMA lane (lr, lq) supplies A[row lr][k] and B[k][col lr]: neighbouring
// lanes hold different rows.  Loaded that way every lane is an L1 access of its
// own (65 a load; the caches' tags then take 90 % of the time, whatever the
// matrix cores do), so a wave loads its 16 x 16 tiles of operator and vectors
// along the rows, 64 or 256 bytes a row, and changes lanes in LDS (its own
// part of it, no barrier).  Slots are exchanged within a row (xor with the row)
// so that neither side has bank conflicts.  FP64 folds the sums of each direction
// into the result: against long double the error is 3.7e-16 of the result's norm
// (48 columns; 1.35e-15 with one sum through all nine directions).  Three real
// products per complex one (im = (ar + ai)(br + bi) - ar br - ai bi) take 10 % less
// time, but the smaller part of a result then carries the rounding of the larger
// one, and an infinite entry makes it NaN.
// 48 x 24^3, 24 vectors: FP64, 32 right-hand sides 398 -> 335 us, 12: 223 -> 204,
// 1: 169 -> 183 (the operator's bytes); FP32, 32: 208 -> 188; 32 x 16^3, 20
// right-hand sides FP64: 78 -> 66.  Tried for 32 / 20: the row tiles of a site
// sharing vectors that the workgroup brings in once, a barrier a step, 326 / 67-73;
// two tiles of right-hand sides a wave, 307 / 67, but half the wavefronts cover the
// loads of small grids; a sum for each of the four products, the same times.
template <typename R> struct CoarseTile;
template <> struct CoarseTile<double> {
    static constexpr int LDS = 2 * 256;      // 16-byte units a wave: operator, vectors
    typedef double2 U;
    double2 a[4], b[4];
    // row i of the tile, column j: lane (j, i % 4), register i / 4
    template <bool FULL>
    __device__ __forceinline__ void load(const double* P, size_t, const double2* const* v, const int* m, int nc, int k0,
                                         int lr, int, size_t zo) {
        const int k = k0 + lr;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (!FULL) a[i] = b[i] = make_double2(0.0, 0.0);
            if (FULL || k < nc) {
                a[i] = ((const double2*)P)[(uint32_t)(m[i] * nc + k)];
                b[i] = v[i][zo + k];
            }
        }
    }
    __device__ __forceinline__ void put(double2* sh, int lr, int lq) const {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 4 * i + lq;
            sh[r * 16 + (lr ^ r)] = a[i];
            sh[256 + r * 16 + (lr ^ r)] = b[i];
        }
    }
    static __device__ __forceinline__ void get(const double2* sh, int lr, int lq, double (&ar)[4], double (&ai)[4],
                                               double (&br)[4], double (&bi)[4]) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const double2 x = sh[lr * 16 + ((4 * s + lq) ^ lr)], z = sh[256 + lr * 16 + ((4 * s + lq) ^ lr)];
            ar[s] = x.x; ai[s] = x.y;
            br[s] = z.x; bi[s] = z.y;
        }
    }
    static __device__ __forceinline__ int row(int i, int lane) { return 4 * i + (lane >> 4); }      // of a[i], b[i]
    static __device__ __forceinline__ int vrow(int i, int lane) { return row(i, lane); }
};
template <> struct CoarseTile<float> {
    static constexpr int LDS = 2 * 64 + 128;
    typedef float4 U;
    float4 a[2], b[2];
    // four columns of the operator's planes (lane: row lane / 4), two of a vector (row lane / 8 + 8 i)
    template <bool FULL>
    __device__ __forceinline__ void load(const float* P, size_t nn, const float2* const* v, const int* m, int nc,
                                         int k0, int, int lane, size_t zo) {
        const int k = k0 + 4 * (lane & 3), kv = k0 + 2 * (lane & 7);
        const float* p = P + (uint32_t)(m[0] * nc + k);
        if (!FULL) a[0] = a[1] = b[0] = b[1] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (FULL || k < nc) {
            a[0] = *(const float4*)p;
            a[1] = *(const float4*)(p + nn);
        }
        if (FULL || kv < nc) {
            b[0] = *(const float4*)(v[0] + zo + kv);
            b[1] = *(const float4*)(v[1] + zo + kv);
        }
    }
    __device__ __forceinline__ void put(float4* sh, int, int lane) const {
        const int r = lane >> 2, u = r * 4 + ((lane & 3) ^ (r >> 2));
        sh[u] = a[0];
        sh[64 + u] = a[1];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int q = (lane >> 3) + 8 * i;
            sh[128 + q * 8 + ((lane & 7) ^ (q >> 1))] = b[i];
        }
    }
    static __device__ __forceinline__ void get(const float4* sh, int lr, int lq, float (&ar)[4], float (&ai)[4],
                                               float (&br)[4], float (&bi)[4]) {
        const int u = lr * 4 + (lq ^ (lr >> 2));
        const float4 x = sh[u], z = sh[64 + u];
        const float4 p = sh[128 + lr * 8 + ((2 * lq) ^ (lr >> 1))], q = sh[128 + lr * 8 + ((2 * lq + 1) ^ (lr >> 1))];
        ar[0] = x.x; ar[1] = x.y; ar[2] = x.z; ar[3] = x.w;
        ai[0] = z.x; ai[1] = z.y; ai[2] = z.z; ai[3] = z.w;
        br[0] = p.x; bi[0] = p.y; br[1] = p.z; bi[1] = p.w;
        br[2] = q.x; bi[2] = q.y; br[3] = q.z; bi[3] = q.w;
    }
    static __device__ __forceinline__ int row(int, int lane) { return lane >> 2; }
    static __device__ __forceinline__ int vrow(int i, int lane) { return (lane >> 3) + 8 * (i & 1); }
};

// VEC = false (FP32 with nc not a multiple of four): entries loaded one by one,
// straight into the lanes that multiply them
template <typename R, bool VEC, int DG>
__global__ __launch_bounds__(DG == 1 ? 512 : 768) void k_coarse_mfma(Geo g, int nc, const R* __restrict__ P,
                                                     const typename VT<R>::c2* __restrict__ in,
                                                     typename VT<R>::c2* __restrict__ out, int nrhs, int gamma5) {
    typedef typename VT<R>::c2 C2;
    typedef typename Mfma<R>::v4 V4;
    typedef CoarseTile<R> T;
    extern __shared__ char shraw[];
    int y, tile;
    if (!site_tile(g.V1, (nrhs + 15) / 16, &y, &tile)) return;
    const int ntr = (nc + 15) / 16;
    const int wall = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int w = DG > 1 ? wall % ntr : wall, dg = DG > 1 ? wall / ntr : 0;
    const int m0 = w * 16, n0 = tile * 16;
    const int lr = lane & 15, lq = lane >> 4;
    const size_t V1 = g.V1, nn = (size_t)nc * nc;
    // groups of three directions, all of them or (DG = 3) one a wave: summed one by one and added in order either way
    static_assert(DG == 1 || DG == 3, "");
    const int nk = (nc + 15) / 16, it0 = 3 * nk * dg, it1 = DG == 1 ? 9 * nk : it0 + 3 * nk;
    V4 cr = {0, 0, 0, 0}, ci = {0, 0, 0, 0}, gr = {0, 0, 0, 0}, gi = {0, 0, 0, 0}, re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
    // FP64: the sums of one direction into those of its group
    auto flush = [&]() {
        gr += cr;
        gi += ci;
        cr = ci = V4{0, 0, 0, 0};
    };
    // a group's sums into those of all (DG = 3: left in cr, ci)
    auto flush_group = [&](bool first) {
        if constexpr (sizeof(R) == 8) {
            cr = gr;
            ci = gi;
            gr = gi = V4{0, 0, 0, 0};
        }
        if constexpr (DG == 1) {
            re = first ? cr : re + cr;
            im = first ? ci : im + ci;
            cr = ci = V4{0, 0, 0, 0};
        }
    };
    auto mac = [&](const R (&ar)[4], const R (&ai)[4], const R (&br)[4], const R (&bi)[4]) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            cr = Mfma<R>::mac(ar[s], br[s], cr);
            ci = Mfma<R>::mac(ar[s], bi[s], ci);
            cr = Mfma<R>::mac(-ai[s], bi[s], cr);
            ci = Mfma<R>::mac(ai[s], br[s], ci);
        }
    };
    // rows past nc and right-hand sides past nrhs repeat the last one: their results are not written
    if constexpr (VEC) {
        typename T::U* sh = (typename T::U*)shraw + wall * T::LDS;
        int m[4];
        const C2* v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            m[i] = m0 + T::row(i, lane) < nc ? m0 + T::row(i, lane) : nc - 1;
            const int n = n0 + T::vrow(i, lane);
            v[i] = in + (size_t)(n < nrhs ? n : nrhs - 1) * V1 * nc;
        }
        T f;
        auto load = [&](int it) {
            const int dir = it / nk, k0 = (it - dir * nk) * 16;
            const R* Pr = P + ((size_t)y * 9 + dir) * 2 * nn;
            const size_t zo = (size_t)coarse_nbr(g, y, dir) * nc;
            if (k0 + 16 <= nc) f.template load<true>(Pr, nn, v, m, nc, k0, lr, lane, zo);
            else f.template load<false>(Pr, nn, v, m, nc, k0, lr, lane, zo);
        };
        load(it0);
        for (int it = it0; it < it1;) {
            const int g0 = it, g1 = it + 3 * nk;
            for (int d1 = it + nk; it < g1; ++it) {
                f.put(sh, lr, sizeof(R) == 8 ? lq : lane);
                if (it + 1 < it1) load(it + 1);
                wave_lds_fence();
                R ar[4], ai[4], br[4], bi[4];
                T::get(sh, lr, lq, ar, ai, br, bi);
                wave_lds_fence();
                mac(ar, ai, br, bi);
                if (sizeof(R) == 8 && it + 1 == d1) {
                    flush();
                    d1 += nk;
                }
            }
            flush_group(g0 == 0);
        }
    } else {
        const size_t mo = (size_t)(m0 + lr < nc ? m0 + lr : nc - 1) * nc;
        const C2* v = in + (size_t)(n0 + lr < nrhs ? n0 + lr : nrhs - 1) * V1 * nc;
        for (int it = it0; it < it1; ++it) {
            const int dir = it / nk, k0 = (it - dir * nk) * 16;
            const R* Pr = P + ((size_t)y * 9 + dir) * 2 * nn + mo;
            const size_t zo = (size_t)coarse_nbr(g, y, dir) * nc;
            R ar[4], ai[4], br[4], bi[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int k = k0 + lq + 4 * s;
                const bool ok = k < nc;
                const C2 x = ok ? v[zo + k] : C2{0, 0};
                ar[s] = ok ? Pr[k] : (R)0;
                ai[s] = ok ? Pr[nn + k] : (R)0;
                br[s] = x.x;
                bi[s] = x.y;
            }
            mac(ar, ai, br, bi);
            if ((it + 1) % (3 * nk) == 0) flush_group(dir == 2);
        }
    }
    if constexpr (DG == 1) {
        cr = re;
        ci = im;
    } else {
        __syncthreads();
        V4* part = (V4*)shraw;
        if (dg > 0) {
            part[((dg - 1) * ntr + w) * 2 * 64 + lane] = cr;
            part[((dg - 1) * ntr + w) * 2 * 64 + 64 + lane] = ci;
        }
        __syncthreads();
        if (dg > 0) return;
#pragma unroll
        for (int q = 1; q < DG; ++q) {
            cr += part[((q - 1) * ntr + w) * 2 * 64 + lane];
            ci += part[((q - 1) * ntr + w) * 2 * 64 + 64 + lane];
        }
    }
    // register t of this lane holds C[row(lq, t)][col lr]
    if (n0 + lr < nrhs) {
        C2* o = out + ((size_t)(n0 + lr) * V1 + y) * nc;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int row = m0 + Mfma<R>::row(lq, t);
            if (row < nc) {
                const R sg = (gamma5 && row >= nc / 2) ? (R)-1 : (R)1;
                o[row] = C2{sg * cr[t], sg * ci[t]};
            }
        }
    }
}

#ifndef COARSE_DG
#define COARSE_DG 3
#endif
typedef short bf4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ short f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7fff + ((u >> 16) & 1);
    return (short)(u >> 16);
}

// grid: the (coarse site, 16-rhs tile) items; block: 64 * ceil(nc/16) * DG threads.  Wave w
// owns row tile w % ntr and the directions dir = w / ntr + DG * k of the nine
// stencil entries; with DG > 1 the DG partial sums of a row tile are added in
// LDS in a fixed order.  FULL: nc is a multiple of 16, so every fragment load
// is in range and can be one 8-byte (operator) / two 16-byte (vector) load
// per lane.
template <bool FULL, int DG>
__global__ void k_coarse_bf16(Geo g, int nc, const bf16_t* __restrict__ Dbf, const float2* __restrict__ in,
                              float2* __restrict__ out, int nrhs, int gamma5) {
    __shared__ f4_t part[DG > 1 ? 2 * 4 * 64 * (DG - 1) : 1];   // DG > 1 only with <= 4 row tiles
    int y, tile;
    if (!site_tile(g.V1, (nrhs + 15) / 16, &y, &tile)) return;
    const int n0 = tile * 16;
    const int ntr = (nc + 15) / 16;
    const int wall = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int w = wall % ntr, dg = wall / ntr;
    const int m0 = w * 16;
    const int lr = lane & 15, lq = lane >> 4;          // row/col within the tile, k quarter
    const size_t V1 = g.V1, nn = (size_t)nc * nc;
    f4_t cr = {0.f, 0.f, 0.f, 0.f}, ci = {0.f, 0.f, 0.f, 0.f};
    const int n = n0 + lr;                            // rhs of this lane's B column
    const int m = m0 + lr;                            // row of this lane's A fragment
    const bool nok = n < nrhs;
    for (int dir = dg; dir < 9; dir += DG) {
        const int z = coarse_nbr(g, y, dir);
        const bf16_t* Dr = Dbf + ((size_t)y * 9 + dir) * 2 * nn;
        const bf16_t* Di = Dr + nn;
        const float2* v = in + ((size_t)(nok ? n : 0) * V1 + z) * nc;
        for (int k0 = 0; k0 < nc; k0 += 16) {
            const int kb = k0 + 4 * lq;
            bf4_t ar, ai, br, bi, bn;
            if (FULL) {
                ar = *(const bf4_t*)(Dr + (size_t)m * nc + kb);
                ai = *(const bf4_t*)(Di + (size_t)m * nc + kb);
                float4 x01 = nok ? *(const float4*)(v + kb) : make_float4(0.f, 0.f, 0.f, 0.f);
                float4 x23 = nok ? *(const float4*)(v + kb + 2) : make_float4(0.f, 0.f, 0.f, 0.f);
                br[0] = f2bf(x01.x); bi[0] = f2bf(x01.y); bn[0] = f2bf(-x01.y);
                br[1] = f2bf(x01.z); bi[1] = f2bf(x01.w); bn[1] = f2bf(-x01.w);
                br[2] = f2bf(x23.x); bi[2] = f2bf(x23.y); bn[2] = f2bf(-x23.y);
                br[3] = f2bf(x23.z); bi[3] = f2bf(x23.w); bn[3] = f2bf(-x23.w);
            } else {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    int k = kb + t;
                    bool ok = k < nc;
                    ar[t] = (ok && m < nc) ? (short)Dr[(size_t)m * nc + k] : (short)0;
                    ai[t] = (ok && m < nc) ? (short)Di[(size_t)m * nc + k] : (short)0;
                    float2 x = (ok && nok) ? v[k] : make_float2(0.f, 0.f);
                    br[t] = f2bf(x.x);
                    bi[t] = f2bf(x.y);
                    bn[t] = f2bf(-x.y);
                }
            }
            cr = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ar, br, cr, 0, 0, 0);
            cr = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ai, bn, cr, 0, 0, 0);
            ci = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ar, bi, ci, 0, 0, 0);
            ci = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ai, br, ci, 0, 0, 0);
        }
    }
    if (DG > 1) {
        // partial sums of direction groups 1..DG-1 to LDS, group 0 adds them in order
        if (dg > 0) {
            part[((dg - 1) * 4 + w) * 2 * 64 + lane] = cr;
            part[((dg - 1) * 4 + w) * 2 * 64 + 64 + lane] = ci;
        }
        __syncthreads();
        if (dg > 0) return;
#pragma unroll
        for (int q = 1; q < DG; ++q) {
            cr += part[((q - 1) * 4 + w) * 2 * 64 + lane];
            ci += part[((q - 1) * 4 + w) * 2 * 64 + 64 + lane];
        }
    }
    // C[row = 4*lq + t][col = lr]
    if (nok) {
        const int row0 = m0 + 4 * lq;
        float2* o = out + ((size_t)n * V1 + y) * nc + row0;
        if (FULL) {
            float s[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) s[t] = (gamma5 && row0 + t >= nc / 2) ? -1.f : 1.f;
            *(float4*)o = make_float4(s[0] * cr[0], s[0] * ci[0], s[1] * cr[1], s[1] * ci[1]);
            *(float4*)(o + 2) = make_float4(s[2] * cr[2], s[2] * ci[2], s[3] * cr[3], s[3] * ci[3]);
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                int row = row0 + t;
                if (row < nc) {
                    float sg = (gamma5 && row >= nc / 2) ? -1.f : 1.f;
                    o[t] = make_float2(sg * cr[t], sg * ci[t]);
                }
            }
        }
    }
}

template <typename R, bool VEC>
static int coarse_launch(const Geo& g, int nc, const R* P, const void* in, void* out, int nrhs, int gamma5,
                         hipStream_t stream) {
    typedef typename VT<R>::c2 C2;
    const int ntr = (nc + 15) / 16;
    const dim3 grid(site_tile_grid(g.V1, (nrhs + 15) / 16));
    // few waves: the directions of a row tile over three of them (16 sites, nc = 16, one right-hand side: 10.3 ->
    // 5.6 us; 512 sites, nc = 32, 48 right-hand sides 66 us, 52 with one).  With three or four row tiles, nine or
    // twelve waves, up to one workgroup a compute unit (4 sites, FP64, nc = 48: 29 -> 23 us, nc = 64: 38 -> 31; 324 sites,
    // nc = 64: 2-7 % slower).  The sums have the same order either way.
    const long items = (long)g.V1 * ((nrhs + 15) / 16);
    const int dg = ntr <= 2 ? (items * ntr < 2048 ? 3 : 1) : ntr <= 4 && items <= 256 ? 3 : 1;
    const size_t shb = (size_t)ntr * dg * CoarseTile<R>::LDS * 16;
    if (dg > 1)
        hipLaunchKernelGGL((k_coarse_mfma<R, VEC, 3>), grid, dim3(64 * ntr * dg), shb, stream, g, nc, P, (const C2*)in,
                           (C2*)out, nrhs, gamma5);
    else
        hipLaunchKernelGGL((k_coarse_mfma<R, VEC, 1>), grid, dim3(64 * ntr), shb, stream, g, nc, P, (const C2*)in,
                           (C2*)out, nrhs, gamma5);
    HIP_TRY(hipGetLastError());
    return MGLMA_OK;
}

int mg_coarse_apply(mglma_ctx* c, int prec, int gamma5, const void* in, void* out, int nrhs) {
    if (prec == MGLMA_F32) MG_TRY(mg_need_d32(c));
    return mg_stencil_apply(c, c->geo, c->nc, (const double*)c->D64, c->D32p, c->Dbf, prec, gamma5, in, out, nrhs);
}

// any level: the stencil of the grid g.L1 (block grid of a Geo): FP64 from
// the interleaved operator P64 [V][9][nc][nc] complex, FP32 / BF16 from the
// planar copies P32 / Pbf [V][9][re/im][nc][nc]
int mg_stencil_apply(mglma_ctx* c, const Geo& g, int nc, const double* P64, const float* P32, const bf16_t* Pbf,
                     int prec, int gamma5, const void* in, void* out, int nrhs) {
    if (nrhs <= 0) return MGLMA_OK;
    if (prec == MGLMA_BF16) {
        // up to four row tiles: three direction groups, three times the wavefronts
        // in flight per coarse site
        constexpr int DG = COARSE_DG;
        const int ntr = (nc + 15) / 16;
        dim3 grid(site_tile_grid(g.V1, (nrhs + 15) / 16));
        if (ntr <= 4) {
            dim3 block(64 * ntr * DG);
            if (nc % 16 == 0)
                hipLaunchKernelGGL((k_coarse_bf16<true, DG>), grid, block, 0, c->stream, g, nc, Pbf,
                                   (const float2*)in, (float2*)out, nrhs, gamma5);
            else
                hipLaunchKernelGGL((k_coarse_bf16<false, DG>), grid, block, 0, c->stream, g, nc, Pbf,
                                   (const float2*)in, (float2*)out, nrhs, gamma5);
        } else {
            dim3 block(64 * ntr);
            if (nc % 16 == 0)
                hipLaunchKernelGGL((k_coarse_bf16<true, 1>), grid, block, 0, c->stream, g, nc, Pbf,
                                   (const float2*)in, (float2*)out, nrhs, gamma5);
            else
                hipLaunchKernelGGL((k_coarse_bf16<false, 1>), grid, block, 0, c->stream, g, nc, Pbf,
                                   (const float2*)in, (float2*)out, nrhs, gamma5);
        }
        HIP_TRY(hipGetLastError());
        return MGLMA_OK;
    }
    if (prec == MGLMA_F64) return coarse_launch<double, true>(g, nc, P64, in, out, nrhs, gamma5, c->stream);
    if (prec != MGLMA_F32) return MGLMA_ERR_ARG;
    if (nc % 4 == 0) return coarse_launch<float, true>(g, nc, P32, in, out, nrhs, gamma5, c->stream);
    return coarse_launch<float, false>(g, nc, P32, in, out, nrhs, gamma5, c->stream);
}

extern "C" int mglma_coarse_apply(mglma_ctx* c, int prec, int gamma5, const void* in, void* out, int nrhs) {
    if (!c || !in || !out || in == out || nrhs < 0 || nrhs > 65535 * 16) return MGLMA_ERR_ARG;
    if (!c->have_subspace) return MGLMA_ERR_NO_SUBSPACE;
    if (prec != MGLMA_F64 && prec != MGLMA_F32 && prec != MGLMA_BF16) return MGLMA_ERR_ARG;
    return mg_coarse_apply(c, prec, gamma5 ? 1 : 0, in, out, nrhs);
}
