"""GPU parity of the block basis, R/T, the Galerkin operator and the coarse
apply against the oracle (FP64 to 1e-12 relative; FP32 and BF16 bounded)."""
import numpy as np
import pytest

from paper_2412_06347_amd import synth
from tests.gpu_util import to_dev, from_dev, relerr
from tests.gpu_setup import Pair

pytestmark = pytest.mark.gpu

CASES = [
    ((4, 4, 4, 4), (2, 2, 2, 2), 8),        # the 4^4 workload: 2^4 blocks, 8 test vectors
    ((6, 4, 6, 2), (3, 2, 3, 1), 3),        # odd blocks, coarse extents 2/3, nc = 6
    ((8, 8, 4, 4), (4, 4, 4, 4), 8),        # 4^4 blocks, coarse extent 1 in space
    ((4, 4, 4, 8), (2, 2, 2, 4), 20),       # nc = 40: partial 16-row / 16-column matrix-core tiles
    ((4, 4, 4, 4), (2, 2, 2, 2), 40),       # nc = 80: the VALU Galerkin kernel (n_c > 64)
]


@pytest.fixture(scope="module", params=CASES, ids=["4^4", "odd", "b4", "nc40", "nc80"])
def pair(request):
    L, b, Nv = request.param
    return Pair(L, b, Nv)


def test_basis_parity(pair):
    import torch
    bl, Nv = pair.bl, pair.Nv
    out = torch.empty((bl.V1, 2 * Nv, bl.Vb, 4, 3, 2), dtype=torch.float64, device="cuda")
    pair.ctx.export_basis(out)
    got = from_dev(out)
    E = np.zeros((bl.V1, 2, Nv, bl.Vb, 4, 3), dtype=complex)
    for a in range(2):
        E[:, a, :, :, 2 * a:2 * a + 2, :] = pair.B.phi[:, a].reshape(bl.V1, Nv, bl.Vb, 2, 3)
    E = E.reshape(bl.V1, 2 * Nv, bl.Vb, 4, 3)
    assert np.abs(got - E).max() < 1e-12


def test_coarse_operator_parity(pair):
    import torch
    bl, nc = pair.bl, 2 * pair.Nv
    out = torch.empty((bl.V1, 9, nc, nc, 2), dtype=torch.float64, device="cuda")
    pair.ctx.export_coarse_op(out)
    got = from_dev(out)
    assert relerr(got, pair.D1) < 1e-12


def test_coarse_gammas_parity(pair):
    import torch
    from oracle import coarse
    bl, Nv = pair.bl, pair.Nv
    out = torch.empty((bl.V1, bl.b[0], 3, Nv, Nv, 2), dtype=torch.float64, device="cuda")
    pair.ctx.export_coarse_gammas(out)
    ref = coarse.coarse_gammas(pair.B)[:, :, :, :Nv, Nv:]
    assert relerr(from_dev(out), ref) < 1e-12


# prec 2: FP32 fields with the FP16 copy of the basis (bound: the FP16
# rounding of the basis, 2^-11 relative per entry)
@pytest.mark.parametrize("prec,tol", [(0, 1e-12), (1, 2e-6), (2, 1e-3)])
def test_restrict_prolong_parity(pair, prec, tol):
    import torch
    from paper_2412_06347_amd import mglma
    n = 19    # more than one 16-wide tile of right-hand sides
    fp = 1 if prec == 2 else prec
    psi = synth.gaussian_fields(n, pair.L, 77)
    ref_c = pair.B.restrict(pair.lat(psi))
    x = pair.fine_dev(psi, fp)
    cdt = torch.float64 if prec == 0 else torch.float32
    c = torch.empty((n, pair.bl.V1, 2 * pair.Nv, 2), dtype=cdt, device="cuda")
    pair.ctx.restrict(x, c, prec)
    e_r = relerr(from_dev(c), ref_c)
    assert e_r < tol
    cv = synth.gaussian_coarse(n, pair.bl.V1, 2 * pair.Nv, 78)
    ref_f = pair.canon(pair.B.prolong(cv))
    ct = to_dev(cv).to(cdt)
    y = pair.ctx.fine(n, fp)
    pair.ctx.prolong(ct, y, prec)
    e_p = relerr(pair.fine_host(y, fp), ref_f)
    print("prec %d: restrict %.2e prolong %.2e" % (prec, e_r, e_p))
    assert e_p < tol


# block, vectors, right-hand sides: every number of 16-row tiles and of four-vector steps, columns in
# and out of fours and of whole chunks, one block (several workgroups or wavefronts for it), and
# fields off the 16-byte alignment that four columns at once need
@pytest.mark.parametrize("b,Nv,n,shift", [((2, 2, 2, 2), 13, 1, 0), ((2, 2, 2, 2), 24, 8, 1), ((3, 3, 3, 3), 33, 17, 0),
                                          ((3, 2, 1, 1), 20, 5, 0), ((4, 4, 4, 4), 64, 16, 0), ((4, 4, 4, 4), 1, 2, 1)])
@pytest.mark.parametrize("prec,tol", [(0, 1e-12), (1, 2e-6), (2, 1e-3)])
def test_transfer_shapes(b, Nv, n, shift, prec, tol):
    import torch
    L = b if b[0] == 4 else tuple(2 * m for m in b)
    pair = Pair(L, b, Nv, oracle_galerkin=False)
    fp = 1 if prec == 2 else prec
    cdt = torch.float64 if prec == 0 else torch.float32
    psi = synth.gaussian_fields(n, L, 79)
    src = pair.fine_dev(psi, fp)
    buf = torch.zeros(src.numel() + 2, dtype=src.dtype, device="cuda")
    x = buf[2 * shift:2 * shift + src.numel()].view(src.shape)
    x.copy_(src)
    c = torch.empty((n, pair.bl.V1, 2 * Nv, 2), dtype=cdt, device="cuda")
    pair.ctx.restrict(x, c, prec)
    assert relerr(from_dev(c), pair.B.restrict(pair.lat(psi))) < tol
    cv = synth.gaussian_coarse(n, pair.bl.V1, 2 * Nv, 80)
    pair.ctx.prolong(to_dev(cv).to(cdt), x, prec)
    torch.cuda.synchronize()
    assert relerr(pair.fine_host(x.clone(), fp), pair.canon(pair.B.prolong(cv))) < tol
    assert float(buf[:2 * shift].abs().sum()) == 0 and float(buf[2 * shift + src.numel():].abs().sum()) == 0


# 256 and 511 blocks of 48 sites, 1022 of 24, 256 of 42 and 512 of 48: eight or four wavefronts a block
@pytest.mark.parametrize("L,b", [((8, 16, 8, 12), (2, 4, 2, 3)), ((14, 292, 2, 3), (2, 4, 2, 3)),
                                 ((14, 292, 2, 3), (2, 4, 1, 3)), ((8, 28, 12, 4), (2, 7, 3, 1)),
                                 ((16, 16, 8, 12), (2, 4, 2, 3))])
@pytest.mark.parametrize("prec,tol", [(0, 1e-12), (1, 2e-6), (2, 1e-3)])
def test_restrict_many_blocks(L, b, prec, tol):
    """R x against sums over the exported basis, and the same bits for a column alone."""
    import torch
    from paper_2412_06347_amd import mglma
    ctx = mglma.Context(L, b, 0.124, 1.0)
    g = torch.Generator(device="cuda").manual_seed(23)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda", dtype=torch.float64)   # noqa: E731
    Nv, n, Vb = 5, 17, int(np.prod(b))
    V1, dt = ctx.V // Vb, torch.float64 if prec == 0 else torch.float32
    ctx.load_gauge(0.4 * rnd(ctx.V, 4, 3, 3, 2))
    ctx.build_subspace(rnd(Nv, 12, ctx.V, 2))
    B = torch.empty((V1, 2 * Nv, Vb, 4, 3, 2), dtype=torch.float64, device="cuda")
    ctx.export_basis(B)
    B = torch.view_as_complex(B)
    x = rnd(n, 12, ctx.V, 2).to(dt)
    y, z = torch.empty((n, V1, 2 * Nv, 2), dtype=dt, device="cuda"), torch.empty((1, V1, 2 * Nv, 2), dtype=dt, device="cuda")
    ctx.restrict(x, y, prec)
    for k in range(n):
        f = torch.view_as_complex(x[k].double()).reshape(4, 3, V1, Vb).permute(2, 3, 0, 1)
        ref = (B.conj() * f[:, None]).sum((2, 3, 4))
        assert relerr(from_dev(y[k]), ref.cpu().numpy()) < tol
        ctx.restrict(x[k:k + 1], z, prec)
        assert torch.equal(z[0], y[k])
    ctx.close()


@pytest.mark.parametrize("prec,tol", [(0, 1e-12), (1, 2e-6), (3, 2e-2)])
@pytest.mark.parametrize("gamma5", [0, 1])
def test_coarse_apply_parity(pair, prec, tol, gamma5):
    import torch
    from oracle import coarse, subspace
    n = 19    # more than one 16-wide tile of right-hand sides
    v = synth.gaussian_coarse(n, pair.bl.V1, 2 * pair.Nv, 91)
    ref = coarse.coarse_apply(pair.D1, pair.nbr, v)
    if gamma5:
        ref = ref * subspace.coarse_gamma5(pair.Nv)[None, None, :]
    cdt = torch.float64 if prec == 0 else torch.float32
    x = to_dev(v).to(cdt)
    y = torch.empty_like(x)
    pair.ctx.coarse_apply(x, y, prec, gamma5)
    err = relerr(from_dev(y), ref)
    print("coarse apply prec=%d gamma5=%d rel err %.3e" % (prec, gamma5, err))
    assert err < tol


# vectors and right-hand sides: columns in and out of fours and sixteens, one and several row tiles, and
# full, partial and several tiles of right-hand sides
@pytest.mark.parametrize("Nv,n", [(1, 3), (8, 16), (13, 17), (22, 33)])
@pytest.mark.parametrize("prec,tol", [(0, 1e-12), (1, 2e-6)])
def test_coarse_apply_shapes(Nv, n, prec, tol):
    import torch
    from oracle import coarse
    P = Pair((4, 4, 2, 4), (2, 2, 2, 2), Nv)
    x = synth.gaussian_coarse(n, P.bl.V1, 2 * Nv, 81)
    xd = to_dev(x).to(torch.float64 if prec == 0 else torch.float32)
    y = torch.empty_like(xd)
    P.ctx.coarse_apply(xd, y, prec)
    ref = (coarse.coarse_dense(P.D1, P.nbr) @ x.reshape(n, -1).T).T.reshape(x.shape)
    assert relerr(from_dev(y), ref) < tol


# the transfers and the coarse operator share out a small grid among more wavefronts: 192 blocks, 1296 blocks
# with 16 and 10 columns (FP32: in and out of fours), 768 blocks with two row tiles, 192 with three and four
@pytest.mark.parametrize("L,Nv", [((8, 8, 8, 6), 12), ((12, 12, 12, 12), 8), ((12, 12, 12, 12), 5), ((12, 8, 8, 16), 12),
                                  ((8, 8, 8, 6), 21), ((8, 8, 8, 6), 32)])
def test_column_bits_do_not_depend_on_batch(L, Nv):
    """A right-hand side gives the same bits alone, in a batch of one tile of 16
    and in one of several."""
    import torch
    from paper_2412_06347_amd import mglma
    ctx = mglma.Context(L, (2, 2, 2, 2), 0.124, 1.0)
    g = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda", dtype=torch.float64)   # noqa: E731
    ctx.load_gauge(0.4 * rnd(ctx.V, 4, 3, 3, 2))      # any 3 x 3 matrices do as links here
    ctx.build_subspace(rnd(Nv, 12, ctx.V, 2))
    n, V1, nc = 40, ctx.V // 16, 2 * Nv
    fine, coarse = rnd(n, 12, ctx.V, 2), rnd(n, V1, nc, 2)
    calls = [("R", fine, coarse, lambda x, y, p: ctx.restrict(x, y, p)), ("T", coarse, fine, lambda x, y, p: ctx.prolong(x, y, p)),
             ("D", coarse, coarse, lambda x, y, p: ctx.coarse_apply(x, y, p))]
    for name, src, dst, call in calls:
        for prec in (mglma.F64, mglma.F32, mglma.F16 if name != "D" else mglma.BF16):
            dt = torch.float64 if prec == mglma.F64 else torch.float32
            x, y = src.to(dt), torch.empty_like(dst, dtype=dt)
            call(x, y, prec)
            for k in (1, 16, 17):
                z = torch.empty_like(y[:k])
                call(x[:k], z, prec)
                assert torch.equal(z, y[:k]), (name, prec, k)


# few vectors on lattices past 131072 sites, one thread a site: 4^4, 3^4 and 2^4 blocks, a part of a workgroup at the
# end, one tile of 16 right-hand sides and more; the first sizes past that on the matrix cores (131072 sites, seven vectors)
@pytest.mark.parametrize("L,b,Nv,n", [((24, 24, 16, 16), (4, 4, 4, 4), 1, 17), ((30, 18, 18, 15), (3, 3, 3, 3), 5, 3),
                                      ((26, 18, 18, 16), (2, 2, 2, 2), 6, 33), ((32, 16, 16, 16), (4, 4, 4, 4), 6, 2),
                                      ((30, 18, 18, 15), (3, 3, 3, 3), 7, 2)])
def test_prolong_few_vectors(L, b, Nv, n):
    """T c of few vectors against sums over the exported basis in FP64, and the
    same bits for a column in the batch and alone.  A part of the result is a sum of 2 Nv products with a rounding
    each of at most half a spacing of the sum of their sizes, the reference has three for two products: (5 Nv) / 2
    spacings for a part, 4 Nv for both."""
    import torch
    from paper_2412_06347_amd import mglma
    ctx = mglma.Context(L, b, 0.124, 1.0)
    g = torch.Generator(device="cuda").manual_seed(17)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda", dtype=torch.float64)   # noqa: E731
    ctx.load_gauge(0.4 * rnd(ctx.V, 4, 3, 3, 2))
    ctx.build_subspace(rnd(Nv, 12, ctx.V, 2))
    Vb = int(np.prod(b))
    V1, nc = ctx.V // Vb, 2 * Nv
    B = torch.empty((V1, nc, Vb, 4, 3, 2), dtype=torch.float64, device="cuda")
    ctx.export_basis(B)
    c = rnd(n, V1, nc, 2)
    B = torch.view_as_complex(B)
    unit = torch.zeros((nc, V1, nc, 2), dtype=torch.float32, device="cuda")
    unit[range(nc), :, range(nc), 0] = 1.0
    for prec, dt in ((mglma.F64, torch.float64), (mglma.F32, torch.float32), (mglma.F16, torch.float32)):
        x = c.to(dt)
        y = torch.empty((n, 12, ctx.V, 2), dtype=dt, device="cuda")
        ctx.prolong(x, y, prec)
        Bc = torch.view_as_complex(torch.view_as_real(B).to(dt).double())
        if prec == mglma.F16:   # the FP16 basis itself: rounded by half a spacing, from FP64 or (another 2^-24) FP32
            e = torch.empty((nc, 12, ctx.V, 2), dtype=dt, device="cuda")
            ctx.prolong(unit, e, prec)
            Bc = torch.view_as_complex(e.double()).reshape(nc, 4, 3, V1, Vb).permute(3, 0, 4, 1, 2)
            d, m = torch.view_as_real(Bc - B).abs(), torch.view_as_real(B).abs()
            assert bool((d <= (2.0 ** -11 + 2.0 ** -23) * m + 2.0 ** -25).all())
        eps = 4 * Nv * torch.finfo(dt).eps
        for k in range(0, n, 2):
            ref, size = 0, 0
            xk = torch.view_as_complex(x[k].double())
            for j in range(nc):
                ref = ref + Bc[:, j] * xk[:, j, None, None, None]
                size = size + Bc[:, j].abs() * xk[:, j, None, None, None].abs()
            got = torch.view_as_complex(y[k].double()).reshape(4, 3, V1, Vb).permute(2, 3, 0, 1)
            far = int(((got - ref).abs() > eps * size).sum())
            assert far == 0, (prec, k, far)
            z = torch.empty_like(y[:1])
            ctx.prolong(x[k:k + 1], z, prec)
            assert torch.equal(z[0], y[k]), (prec, k)
    ctx.close()


def coarse_op(pair):
    import torch
    nc = 2 * pair.Nv
    out = torch.empty((pair.bl.V1, 9, nc, nc, 2), dtype=torch.float64, device="cuda")
    pair.ctx.export_coarse_op(out)
    return from_dev(out)


def test_coarse_apply_small_part():
    """FP64: the real and the imaginary part of the result each carry the rounding
    of their own products, also where one is 1e10 times the other.  At a tiny kappa
    D_1 is the identity to 1e-12, so the imaginary part of the result is that of
    the vector; the bound is that of a sum of 2 * 9 * 16 products and 9 partial
    sums in any order, u = 2^-53 a term."""
    import torch
    P = Pair((4, 4, 2, 4), (2, 2, 2, 2), 8, kappa=1e-12, oracle_galerkin=False)
    D = coarse_op(P)
    x = synth.gaussian_coarse(17, P.bl.V1, 16, 83)
    x = x.real + 1e-10j * x.imag
    xd = to_dev(x)
    y = torch.empty_like(xd)
    P.ctx.coarse_apply(xd, y)
    g = x[:, P.nbr]                                              # [n][y][dir][j]
    s = lambda a, b: np.einsum("ydij,nydj->nyi", a.astype(np.longdouble), b.astype(np.longdouble))   # noqa: E731
    ref = s(D.real, g.imag) + s(D.imag, g.real)
    mag = s(np.abs(D.real), np.abs(g.imag)) + s(np.abs(D.imag), np.abs(g.real))
    err = np.abs(from_dev(y).imag - ref) / mag
    print("largest error of the small part: %.1f u" % (err.max() * 2 ** 53))
    assert err.max() <= 300 * 2.0 ** -53


def test_coarse_apply_infinite_entry():
    """An infinite real entry makes both parts of what it multiplies infinite, as
    re = ar br - ai bi, im = ar bi + ai br do, and nothing else (grid extents of
    three: every site meets it through one direction only)."""
    import torch
    P = Pair((6, 6, 6, 6), (2, 2, 2, 2), 5, oracle_galerkin=False)
    D = coarse_op(P)
    n, y0, j = 3, 40, 7
    x = synth.gaussian_coarse(n, P.bl.V1, 10, 84)
    xr = torch.from_numpy(np.stack([x.real, x.imag], -1)).cuda()
    xr[1, y0, j, 0], xr[1, y0, j, 1] = float("inf"), 0.0
    out = torch.empty_like(xr)
    P.ctx.coarse_apply(xr, out)
    got = out.cpu().numpy()
    want = np.zeros(got.shape)
    for y, d in zip(*np.nonzero(P.nbr == y0)):
        want[1, y, :, 0], want[1, y, :, 1] = np.sign(D[y, d, :, j].real), np.sign(D[y, d, :, j].imag)
    assert not np.isnan(got).any()
    assert np.array_equal(np.where(np.isinf(got), np.sign(got), 0.0), want)


def test_rank_deficient_basis_is_an_error():
    import torch
    from paper_2412_06347_amd import mglma
    L, b = (4, 4, 4, 4), (2, 2, 2, 2)
    U = synth.gauge_field(L, 0.3, 1)
    ctx = mglma.Context(L, b, 0.12, 1.0)
    ctx.load_gauge(to_dev(U))
    tv = synth.gaussian_fields(3, L, 5)
    tv[2] = (1 - 2j) * tv[0]
    x = ctx.fine(3)
    ctx.import_fields(to_dev(tv), x)
    with pytest.raises(mglma.MglmaError) as e:
        ctx.build_subspace(x)
    assert e.value.code == -5
