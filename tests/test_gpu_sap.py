"""GPU parity of the SAP smoother (the smoother of the paper's fine solver,
sec. "Comparison of the cost") against the oracle's SAP cycles, and the
multigrid solve with SAP smoothing against the oracle's operator."""
import numpy as np
import pytest

from oracle import dirac, subspace, sap
from paper_2412_06347_amd import synth
from tests.gpu_util import relerr
from tests.gpu_setup import Pair

pytestmark = pytest.mark.gpu

CASES = [
    # L, block: block grids (2,1,1,2) with 2^4 blocks, (2,2,2,4), and (2,1,1,2) with 4^4 blocks
    ((4, 2, 2, 4), (2, 2, 2, 2)),
    ((4, 4, 4, 8), (2, 2, 2, 2)),
    ((8, 4, 4, 8), (4, 4, 4, 4)),
]


@pytest.fixture(scope="module", params=CASES, ids=["2^4_ext1", "2^4", "4^4_ext1"])
def pair(request):
    L, b = request.param
    return Pair(L, b, 2, kappa=0.124, oracle_galerkin=False)


@pytest.mark.parametrize("prec,tol", [(1, 2e-6), (2, 5e-3)], ids=["f32", "f16"])
def test_sap_cycles_parity(pair, prec, tol):
    from paper_2412_06347_amd import mglma
    nrhs, ncycle, nmr = 2, 2, 4
    r = synth.gaussian_fields(nrhs, pair.L, 51)
    z0 = 0.1 * synth.gaussian_fields(nrhs, pair.L, 52)
    rd, zd = pair.fine_dev(r, mglma.F32), pair.fine_dev(z0, mglma.F32)
    pair.ctx.sap_smooth(rd, zd, ncycle=ncycle, nmr=nmr, prec=prec)
    got = pair.fine_host(zd, mglma.F32)
    bl = subspace.Blocking(pair.L, pair.b)
    ref = []
    for q in range(nrhs):
        z = pair.lat(z0)[q]
        for _ in range(ncycle):
            z = sap.sap_cycle(pair.D, bl, pair.lat(r)[q], z, nmr)
        ref.append(z)
    ref = pair.canon(np.stack(ref))
    e = relerr(got, ref)
    print("SAP %d cycles, %d MR steps, prec %d: rel. error %.2e" % (ncycle, nmr, prec, e))
    assert e < tol


# block sizes of 36, 81 and 192 sites: part of one wavefront, two and three wavefronts, with and without wrap-around
SIZES = [((6, 6, 4, 4), (3, 3, 2, 2)), ((6, 6, 6, 6), (3, 3, 3, 3)), ((8, 4, 4, 6), (4, 4, 4, 3))]


@pytest.mark.parametrize("L,b", SIZES, ids=["36", "81", "192_ext1"])
@pytest.mark.parametrize("prec,tol", [(1, 2e-6), (2, 5e-3)], ids=["f32", "f16"])
def test_sap_block_sizes(L, b, prec, tol):
    """A workgroup has as many wavefronts as the block needs; its idle threads stay out of the block's sums."""
    test_sap_cycles_parity(Pair(L, b, 2, kappa=0.124, oracle_galerkin=False), prec, tol)


@pytest.mark.parametrize("scale", [1e-7, 1e3])
def test_sap_cycles_parity_scaled(pair, scale):
    """FP16 links at right-hand sides far from unit scale (entries around
    1e-7 lie below FP16's normal range): the FP16 block vectors are scaled
    per block, so the relative error stays that of unit-scale inputs."""
    from paper_2412_06347_amd import mglma
    nrhs, ncycle, nmr = 2, 2, 4
    r = scale * synth.gaussian_fields(nrhs, pair.L, 61)
    z0 = 0.1 * scale * synth.gaussian_fields(nrhs, pair.L, 62)
    rd, zd = pair.fine_dev(r, mglma.F32), pair.fine_dev(z0, mglma.F32)
    pair.ctx.sap_smooth(rd, zd, ncycle=ncycle, nmr=nmr, prec=mglma.F16)
    got = pair.fine_host(zd, mglma.F32)
    bl = subspace.Blocking(pair.L, pair.b)
    ref = []
    for q in range(nrhs):
        z = pair.lat(z0)[q]
        for _ in range(ncycle):
            z = sap.sap_cycle(pair.D, bl, pair.lat(r)[q], z, nmr)
        ref.append(z)
    ref = pair.canon(np.stack(ref))
    e = relerr(got, ref)
    print("SAP FP16, inputs scaled by %g: rel. error %.2e" % (scale, e))
    assert e < 5e-3


def test_sap_cycles_tiny_blocks(pair):
    """FP16 links with blocks whose entries are far below the rest (a source
    on one time slice, 1e-21 elsewhere: the block norms there underflow
    FP32): those blocks drop out of the FP16 block steps instead of turning
    the result non-finite, and the rest matches the oracle's cycles."""
    from paper_2412_06347_amd import mglma
    nrhs, ncycle, nmr = 2, 2, 4
    r = synth.gaussian_fields(nrhs, pair.L, 71)
    t = np.arange(int(np.prod(pair.L))) // int(np.prod(pair.L[1:]))
    r = r * np.where(t == 0, 1.0, 1e-21)[None, :, None, None]
    z0 = np.zeros_like(r)
    rd, zd = pair.fine_dev(r, mglma.F32), pair.fine_dev(z0, mglma.F32)
    pair.ctx.sap_smooth(rd, zd, ncycle=ncycle, nmr=nmr, prec=mglma.F16)
    got = pair.fine_host(zd, mglma.F32)
    assert np.isfinite(got).all()
    bl = subspace.Blocking(pair.L, pair.b)
    ref = []
    for q in range(nrhs):
        z = pair.lat(z0)[q]
        for _ in range(ncycle):
            z = sap.sap_cycle(pair.D, bl, pair.lat(r)[q], z, nmr)
        ref.append(z)
    ref = pair.canon(np.stack(ref))
    e = relerr(got, ref)
    print("SAP FP16, source on one time slice, 1e-21 elsewhere: rel. error %.2e" % e)
    assert e < 5e-3


def test_sap_block_eigenvector(pair):
    """FP16 links where a block step removes nearly all of a block's residual:
    r on one colour-0 block is an eigenvector of that block's M_BB, so the
    first minimal-residual step leaves only rounding in s.  The FP16 copy's
    scale comes from |s|^2 summed afresh (a running |s|^2 - |<t,s>|^2/|t|^2
    cancels here and its scale overflowed FP16); the result stays finite
    and matches the oracle's cycles."""
    from paper_2412_06347_amd import mglma
    if int(np.prod(pair.b)) > 16:
        pytest.skip("dense block operator built for 2^4 blocks only")
    bl = subspace.Blocking(pair.L, pair.b)
    y0 = next(y for y in range(bl.V1) if sap.block_colour(bl, y) == 0)
    mask = sap.block_mask(bl, y0)
    idx = np.flatnonzero(np.broadcast_to(mask[..., None, None], tuple(pair.L) + (4, 3)))
    n = idx.size
    Mbb = np.zeros((n, n), dtype=complex)
    for k in range(n):
        e = np.zeros(tuple(pair.L) + (4, 3), dtype=complex)
        e.flat[idx[k]] = 1.0
        Mbb[:, k] = sap.block_apply(pair.D, mask, e).flat[idx]
    lam, vec = np.linalg.eig(Mbb)
    k = int(np.argsort(np.abs(lam))[n // 2])
    f = np.zeros(tuple(pair.L) + (4, 3), dtype=complex)
    f.flat[idx] = vec[:, k]
    r = pair.canon(f[None])
    z0 = np.zeros_like(r)
    rd, zd = pair.fine_dev(r, mglma.F32), pair.fine_dev(z0, mglma.F32)
    ncycle, nmr = 2, 4
    pair.ctx.sap_smooth(rd, zd, ncycle=ncycle, nmr=nmr, prec=mglma.F16)
    got = pair.fine_host(zd, mglma.F32)
    assert np.isfinite(got).all()
    z = pair.lat(z0)[0]
    for _ in range(ncycle):
        z = sap.sap_cycle(pair.D, bl, f, z, nmr)
    e = relerr(got, pair.canon(z[None]))
    print("SAP FP16, r an eigenvector of one block's M_BB: rel. error %.2e" % e)
    assert e < 5e-3


def test_sap_smoothed_solve(pair):
    from paper_2412_06347_amd import mglma
    b = synth.gaussian_fields(2, pair.L, 53)
    for sm in (mglma.F32, mglma.F16):
        x = pair.ctx.fine(2)
        p = mglma.default_params(tol=1e-10, inner=mglma.F32, coarse=mglma.BF16, smoother=sm,
                                 smoother_alg=mglma.SMOOTH_SAP, nu_post=1, sap_mr=4)
        rc, st = pair.ctx.solve(pair.fine_dev(b), x, p)
        xs = pair.fine_host(x)
        r = pair.canon(pair.D.M(pair.lat(xs))) - b
        res = (np.linalg.norm(r.reshape(2, -1), axis=1) / np.linalg.norm(b.reshape(2, -1), axis=1)).max()
        print("SAP-smoothed MG solve (smoother prec %d): %d iterations, oracle residual %.2e"
              % (sm, st[0]["inner"], res))
        assert rc == 0 and res < 1.05e-10


def test_sap_arguments():
    import torch
    from paper_2412_06347_amd import mglma
    P = Pair((6, 4, 4, 4), (2, 2, 2, 2), 2, oracle_galerkin=False)   # block grid (3,2,2,2): odd extent
    r = P.ctx.fine(1, mglma.F32)
    z = P.ctx.fine(1, mglma.F32)
    with pytest.raises(mglma.MglmaError) as e:
        P.ctx.sap_smooth(r, z)
    assert e.value.code == -2
    with pytest.raises(mglma.MglmaError) as e:
        P.ctx.solve(P.ctx.fine(1), P.ctx.fine(1), mglma.default_params(smoother_alg=mglma.SMOOTH_SAP))
    assert e.value.code == -2
    Q = Pair((4, 4, 4, 4), (2, 2, 2, 2), 2, oracle_galerkin=False)
    r = Q.ctx.fine(1, mglma.F32)
    z = Q.ctx.fine(1, mglma.F32)
    for kw in (dict(prec=mglma.F64), dict(nmr=65), dict(ncycle=-1)):
        with pytest.raises(mglma.MglmaError) as e:
            Q.ctx.sap_smooth(r, z, **kw)
        assert e.value.code == -1
    for kw in (dict(inner=mglma.F64), dict(sap_mr=0)):
        with pytest.raises(mglma.MglmaError) as e:
            Q.ctx.solve(Q.ctx.fine(1), Q.ctx.fine(1), mglma.default_params(smoother_alg=mglma.SMOOTH_SAP, **kw))
        assert e.value.code == -1
    # no right-hand sides: nothing to do (pointers still valid)
    assert mglma.lib().mglma_sap_smooth(Q.ctx._ctx, mglma.F16, 1, 4, mglma._ptr(r), mglma._ptr(z), 0) == 0


def test_sap_launch_timing():
    """The launch timing records one event pair per half-sweep while enabled."""
    from paper_2412_06347_amd import mglma
    P = Pair((4, 4, 4, 4), (2, 2, 2, 2), 2, oracle_galerkin=False)
    r, z = P.ctx.fine(3, mglma.F32), P.ctx.fine(3, mglma.F32)
    r.normal_()
    z.zero_()
    P.ctx.sap_timing(True)
    P.ctx.sap_smooth(r, z, ncycle=2, nmr=4)
    ms, n = P.ctx.sap_elapsed()
    assert n == 4 and ms > 0.0
    assert P.ctx.sap_elapsed() == (0.0, 0)          # cleared by the previous call
    P.ctx.sap_timing(False)
    P.ctx.sap_smooth(r, z, ncycle=1, nmr=4)
    assert P.ctx.sap_elapsed()[1] == 0
