"""GPU parity of the clover term and the Wilson-clover apply against the
oracle (FP64 to 1e-12 relative; FP32 / FP16 errors bounded and reported)."""
import numpy as np
import pytest

from oracle import dirac
from paper_2412_06347_amd import synth
from tests.gpu_util import to_dev, from_dev, relerr

pytestmark = pytest.mark.gpu

CASES = [
    # L, block, kappa, csw, eps
    ((4, 4, 4, 4), (2, 2, 2, 2), 0.120, 1.0, 0.3),      # the 4^4 workload
    ((6, 4, 6, 2), (3, 2, 3, 1), 0.124, 1.3, 0.3),      # odd blocks, extent-2 direction
    ((8, 2, 4, 6), (8, 1, 2, 3), 0.125, 1.0, 0.25),     # block = L in time, b = 1
]


def _ctx(L, b, kappa, csw, eps, seed=1):
    import torch
    from paper_2412_06347_amd import mglma
    U = synth.gauge_field(L, eps, seed)
    ctx = mglma.Context(L, b, kappa, csw)
    ctx.load_gauge(to_dev(U))
    torch.cuda.synchronize()
    return ctx, U


@pytest.mark.parametrize("case", CASES)
def test_clover_parity(case):
    import torch
    L, b, kappa, csw, eps = case
    ctx, U = _ctx(*case)
    out = torch.empty((ctx.V, 2, 6, 6, 2), dtype=torch.float64, device="cuda")
    ctx.export_clover(out)
    got = from_dev(out)
    Cl = dirac.clover(U, L, kappa, csw).reshape(-1, 12, 12)
    ref = np.stack([Cl[:, :6, :6], Cl[:, 6:, 6:]], axis=1)
    assert np.abs(got - ref).max() < 1e-13


@pytest.mark.parametrize("L", [(3, 1, 2, 5), (2, 2, 2, 2), (5, 13, 1, 2)])
def test_clover_small_extents(L):
    """Less than a workgroup of sites, a partial second one, and extents of one and two."""
    test_clover_parity((L, L, 0.12, 1.1, 0.3))


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("gamma5", [0, 1])
def test_apply_parity(case, gamma5):
    import torch
    from paper_2412_06347_amd import mglma
    L, b, kappa, csw, eps = case
    ctx, U = _ctx(*case)
    D = dirac.WilsonClover(U, L, kappa, csw)
    nrhs = 3
    psi = synth.gaussian_fields(nrhs, L, seed=7)
    ref = D.M(dirac.fields_to_lattice(psi, L))
    if gamma5:
        ref = dirac.gamma5_field(ref)
    ref = dirac.fields_to_canonical(ref)
    for prec, tol in [(mglma.F64, 1e-12), (mglma.F32, 2e-6), (mglma.F16, 2e-3)]:
        x = ctx.fine(nrhs, prec)
        y = ctx.fine(nrhs, prec)
        ctx.import_fields(to_dev(psi), x, prec)
        ctx.apply_D(x, y, prec, gamma5)
        out = torch.empty((nrhs, ctx.V, 4, 3, 2), dtype=torch.float64, device="cuda")
        ctx.export_fields(y, out, prec)
        got = from_dev(out)
        err = relerr(got, ref)
        print("L=%s prec=%d gamma5=%d rel err %.3e" % (L, prec, gamma5, err))
        assert err < tol


@pytest.mark.parametrize("nrhs", [2, 4, 7])
def test_apply_f16_batches(nrhs):
    """FP16 batches go through the packed kernel in groups of three right-hand
    sides; ragged last groups (4 = 3 + 1, 7 = 3 + 3 + 1) and a lattice whose
    volume is not a multiple of the 256-site tile (6 x 4 x 6 x 2 = 288)."""
    import torch
    from paper_2412_06347_amd import mglma
    case = CASES[1]
    L = case[0]
    ctx, U = _ctx(*case)
    D = dirac.WilsonClover(U, L, case[2], case[3])
    psi = synth.gaussian_fields(nrhs, L, seed=70 + nrhs)
    for gamma5 in (0, 1):
        ref = D.M(dirac.fields_to_lattice(psi, L))
        if gamma5:
            ref = dirac.gamma5_field(ref)
        ref = dirac.fields_to_canonical(ref)
        x = ctx.fine(nrhs, mglma.F16)
        y = ctx.fine(nrhs, mglma.F16)
        ctx.import_fields(to_dev(psi), x, mglma.F16)
        ctx.apply_D(x, y, mglma.F16, gamma5)
        out = torch.empty((nrhs, ctx.V, 4, 3, 2), dtype=torch.float64, device="cuda")
        ctx.export_fields(y, out, mglma.F16)
        got = from_dev(out)
        for r in range(nrhs):
            err = relerr(got[r], ref[r])
            print("nrhs=%d rhs=%d gamma5=%d rel err %.3e" % (nrhs, r, gamma5, err))
            assert err < 2e-3


@pytest.mark.parametrize("nrhs", [2, 3, 4, 5, 9, 13])
@pytest.mark.parametrize("L,b", [((4, 3, 3, 3), (2, 3, 3, 1)), ((8, 4, 4, 4), (4, 4, 4, 4)), ((3, 5, 3, 3), (3, 5, 3, 3))],
                         ids=["tail_tile", "tile_is_slice", "one_block"])
def test_apply_batch_tiles(L, b, nrhs):
    """Batches run in tiles of 64 sites with the neighbours inside a tile taken
    from its lanes: a ragged last tile, tiles that are whole block slices, tiles
    across slices of a block that spans the lattice; batches around the rounds
    of four right-hand sides.  Tolerances: those of test_apply_parity."""
    import torch
    from paper_2412_06347_amd import mglma
    ctx, U = _ctx(L, b, 0.124, 1.0, 0.3, seed=5)
    D = dirac.WilsonClover(U, L, 0.124, 1.0)
    psi = synth.gaussian_fields(nrhs, L, seed=31)
    ref = D.M_canon(dirac.fields_to_lattice(psi, L))
    for prec, tol in [(mglma.F64, 1e-12), (mglma.F32, 2e-6), (mglma.F16, 2e-3)]:
        x, y = ctx.fine(nrhs, prec), ctx.fine(nrhs, prec)
        ctx.import_fields(to_dev(psi), x, prec)
        ctx.apply_D(x, y, prec)
        out = torch.empty((nrhs, ctx.V, 4, 3, 2), dtype=torch.float64, device="cuda")
        ctx.export_fields(y, out, prec)
        assert relerr(from_dev(out), ref) < tol


@pytest.mark.parametrize("gamma5", [0, 1])
@pytest.mark.parametrize("L,b", [((2, 2, 2, 2), (2, 2, 2, 2)), ((4, 4, 4, 4), (4, 4, 4, 4)), ((9, 5, 3, 7), (3, 5, 3, 1))],
                         ids=["part_of_a_tile", "whole_tiles", "tail_tile"])
def test_apply_single_tiles(L, b, gamma5):
    """One right-hand side: 64 sites per workgroup, a wavefront per direction,
    with less than a tile, whole tiles and a ragged last one.  Tolerances: those
    of test_apply_parity; FP64 and FP32 sum as a batch does."""
    import torch
    from paper_2412_06347_amd import mglma
    ctx, U = _ctx(L, b, 0.124, 1.0, 0.3, seed=6)
    D = dirac.WilsonClover(U, L, 0.124, 1.0)
    psi = synth.gaussian_fields(2, L, seed=32)
    ref = D.M_canon(dirac.fields_to_lattice(psi, L))
    if gamma5:
        ref = ref * np.array([1, 1, -1, -1]).reshape(4, 1)
    for prec, tol in [(mglma.F64, 1e-12), (mglma.F32, 2e-6), (mglma.F16, 2e-3)]:
        x, y, z = (ctx.fine(2, prec) for _ in range(3))
        ctx.import_fields(to_dev(psi), x, prec)
        for q in range(2):
            ctx.apply_D(x[q:q + 1], y[q:q + 1], prec, gamma5)
        ctx.apply_D(x, z, prec, gamma5)
        out = torch.empty((2, ctx.V, 4, 3, 2), dtype=torch.float64, device="cuda")
        ctx.export_fields(y, out, prec)
        assert relerr(from_dev(out), ref) < tol
        if prec != mglma.F16:
            assert float((y - z).abs().max()) <= 8 * torch.finfo(y.dtype).eps * float(z.abs().max())


@pytest.mark.parametrize("prec", [0, 1, 2], ids=["f64", "f32", "f16"])
def test_apply_batch_repeats(prec):
    """A full-size batch gives the values of one right-hand side at a time in
    every pass (FP64 and FP32 sum in the same order: equal to a few rounding
    errors; FP16 batches compute on packed data), and the same bits each time."""
    import torch
    from paper_2412_06347_amd import mglma
    L, nrhs = (48, 24, 24, 24), 12
    ctx = mglma.Context(L, (4, 4, 4, 4), 0.124, 1.0)
    g = torch.Generator(device="cuda").manual_seed(9)
    # any 3 x 3 matrices do as links here
    ctx.load_gauge(0.4 * torch.randn((ctx.V, 4, 3, 3, 2), generator=g, device="cuda", dtype=torch.float64))
    x, y, ref = ctx.fine(nrhs, prec), ctx.fine(nrhs, prec), ctx.fine(nrhs, prec)
    x.copy_(torch.randn(x.shape, generator=g, device="cuda", dtype=torch.float32))
    for q in range(nrhs):
        ctx.apply_D(x[q:q + 1], ref[q:q + 1], prec)
    first = None
    for _ in range(8):
        y.zero_()
        ctx.apply_D(x, y, prec)
        err = float((y.float() - ref.float()).abs().max())
        assert err <= (1e-5, 1e-4, 0.25)[prec], err
        first = y.clone() if first is None else first
        assert torch.equal(y, first)


@pytest.mark.parametrize("L,b,nrhs", [((48, 24, 24, 24), (4, 4, 4, 4), 12), ((8, 4, 6, 5), (2, 4, 3, 5), 5), ((4, 4, 4, 4), (4, 4, 4, 4), 2),
                                      ((24, 12, 12, 12), (4, 4, 4, 4), 5)], ids=["full_size", "tail_tile", "one_block", "second_round"])
@pytest.mark.parametrize("prec", [0, 1, 2], ids=["f64", "f32", "f16"])
def test_apply_column_bits(prec, L, b, nrhs):
    """FP64 and FP32: a right-hand side has the same bits alone and in a batch (the
    hops, the clover term and their sums in one order), at every site.  FP16 batches
    also round the projected half spinors, at most 2 max|x|, to FP16: 2^-11 max|x|
    in each of the 2 * 3 products of eight hops, times kappa max|U|; both results
    are rounded, 2^-12 max|y| each; 1 % for the FP32 sums."""
    import torch
    from paper_2412_06347_amd import mglma
    ctx = mglma.Context(L, b, 0.124, 1.0)
    g = torch.Generator(device="cuda").manual_seed(11)
    U = 0.4 * torch.randn((ctx.V, 4, 3, 3, 2), generator=g, device="cuda", dtype=torch.float64)
    ctx.load_gauge(U)
    x, y = ctx.fine(nrhs, prec), ctx.fine(nrhs, prec)
    x.copy_(torch.randn(x.shape, generator=g, device="cuda", dtype=torch.float32))
    ctx.apply_D(x, y, prec)
    z = ctx.fine(1, prec)
    for q in range(nrhs):
        ctx.apply_D(x[q:q + 1], z, prec)
        if prec != mglma.F16:
            assert torch.equal(z[0], y[q]), q
        else:
            most = 0.124 * 48 * float(U.abs().max()) * float(x[q].abs().max()) + float(z.abs().max())
            assert float((z[0].float() - y[q].float()).abs().max()) <= 1.01 * 2.0 ** -11 * most, q


def test_apply_refuses_too_many_sites():
    """Sites times right-hand sides past the largest grid: an error, and no launch."""
    import torch
    from paper_2412_06347_amd import mglma
    ctx = mglma.Context((72, 64, 64, 32), (4, 4, 4, 4), 0.124, 1.0)
    ctx.load_gauge(torch.zeros((ctx.V, 4, 3, 3, 2), dtype=torch.float64, device="cuda"))
    x, y = torch.zeros(2, device="cuda"), torch.zeros(2, device="cuda")
    for prec in (mglma.F64, mglma.F32, mglma.F16):
        assert mglma.lib().mglma_apply_D(ctx._ctx, prec, 0, mglma._ptr(x), mglma._ptr(y), 65535) == -2


def test_import_export_roundtrip():
    import torch
    from paper_2412_06347_amd import mglma
    ctx, U = _ctx(*CASES[1])
    psi = synth.gaussian_fields(2, CASES[1][0], seed=3)
    x = ctx.fine(2, mglma.F64)
    ctx.import_fields(to_dev(psi), x)
    out = torch.empty((2, ctx.V, 4, 3, 2), dtype=torch.float64, device="cuda")
    ctx.export_fields(x, out)
    assert np.array_equal(from_dev(out), psi)


@pytest.mark.parametrize("L,b", [((32, 16, 16, 16), (4, 4, 4, 4))])
def test_apply_parity_full_size(L, b):
    """The 16^3 x 32 workload at full size, FP64, in the launch configuration
    the benchmark times."""
    import torch
    from paper_2412_06347_amd import mglma
    ctx, U = _ctx(L, b, 0.124, 1.0, 0.3, seed=2)
    D = dirac.WilsonClover(U, L, 0.124, 1.0)
    psi = synth.gaussian_fields(1, L, seed=9)
    ref = dirac.fields_to_canonical(D.M(dirac.fields_to_lattice(psi, L)))
    x = ctx.fine(1, mglma.F64)
    y = ctx.fine(1, mglma.F64)
    ctx.import_fields(to_dev(psi), x)
    ctx.apply_D(x, y)
    out = torch.empty((1, ctx.V, 4, 3, 2), dtype=torch.float64, device="cuda")
    ctx.export_fields(y, out)
    assert relerr(from_dev(out), ref) < 1e-12
