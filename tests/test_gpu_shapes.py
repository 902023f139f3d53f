"""Image and scene sizes at the edges of the kernels' tiles, through the C ABI,
against the FP64 oracle.

Tolerances are those of the dedicated tests: float32 entries 1e-6 relative
(bilinear, non-negative terms; 2e-6 with the flux rescale, one more rounding of
the scale and of the product) or of the column bound (cubic).
"""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


def _inputs(n, N, K, seed):
    rng = np.random.default_rng([n, N, K, seed])
    radii = np.linspace(0.0, 0.3 * N, K)
    return (rng.random((K, n, n)) ** 3).astype(np.float32), radii, rng


def _fill(lib, torch):
    """Poison a library's buffer and build it again: an entry the build does
    not write stays NaN."""
    from paper_2106_09122_amd import psflib
    lib.buf.fill_(0xFF)
    h = psflib.build(lib.desc, lib.cube.data_ptr(), lib.radii, lib.buf.data_ptr(), lib.nbytes,
                     torch.cuda.current_stream().cuda_stream)
    psflib.destroy(lib.h)
    lib.h = h


# ------------------------------------------------ float32 orbit builds ----
# one block, one tile and several; every remainder of 4 and sides around
# multiples of 32 (whole lines) and 4; beyond 141 the pair no longer fits the LDS
SIDES = [1, 2, 3, 4, 5, 6, 31, 32, 33, 34, 63, 64, 65, 67, 95, 97, 100, 127, 141, 142, 143, 161, 164]


@pytest.mark.parametrize("n", SIDES)
@pytest.mark.parametrize("rotate,flux", [("bilinear", "none"), ("bilinear", "preserve"), ("cubic", "none"),
                                         ("cubic", "preserve")])
def test_orbit_build_sides(torch, n, rotate, flux):
    from paper_2106_09122_amd import psflib
    for N in (5, 6):
        cube, radii, _ = _inputs(n, N, 4, 1)
        mode = dict(rotate=rotate, flux=flux, oob="zero")
        A = O.build_library(cube, radii, N, 1.0, **mode)
        lib = psflib.Library(torch.from_numpy(cube).cuda(), radii, N, 1.0, **mode)
        _fill(lib, torch)
        got = lib.get_columns(np.arange(N * N)).cpu().numpy().T.astype(np.float64)
        if rotate == "bilinear":
            tol = (2e-6 if flux == "preserve" else 1e-6) * A
        else:
            b = O.column_max_bound(cube, radii, N, 1.0, oob="zero", rotate="cubic")
            if flux == "preserve":
                A0 = O.build_library(cube, radii, N, 1.0, rotate=rotate, oob="zero")
                t0, t1 = A0.sum(axis=0), A.sum(axis=0)
                b = 2 * b * np.abs(np.where(t0 != 0, t1 / np.where(t0 != 0, t0, 1.0), 1.0))
            tol = 1e-6 * b[None, :]
        assert np.all(np.abs(got - A) <= tol + 1e-300), (n, N)
        tau = lib.column_sums().cpu().numpy()
        assert np.all(np.abs(tau - A.sum(axis=0)) <= np.sum(np.broadcast_to(tol, A.shape), axis=0) + 1e-300)
        lib.close()


# ------------------------------------------------------------ products ----
# The products against float64 products with the library's own columns (which
# the tests above and the dedicated ones compare with the oracle): what is
# tested is the streaming and summation, float32 sums of rounded products over
# blocked chains: 1e-5 of the sum of magnitudes, as the dedicated tests.
def _library(torch, n, N, storage, seed=3, **mode):
    from paper_2106_09122_amd import psflib
    cube, radii, rng = _inputs(n, N, 3, seed)
    lib = psflib.Library(torch.from_numpy(cube).cuda(), radii, N, 1.0, storage=storage, **mode)
    A = torch.cat([lib.get_columns(np.arange(j, min(j + 4096, N * N))) for j in range(0, N * N, 4096)])
    return lib, A.double(), rng  # A: [columns][pixels]


# rows: one pixel, below and at one step of 256 (64) rows, ragged steps, one
# full row block (128), just over it and several; columns: fewer than waves,
# ragged groups, enough for 2, 4 and 8 at a time and for every split rule
ADJOINT = [(1, 1), (1, 5), (2, 3), (3, 130), (8, 33), (16, 130), (17, 130), (22, 70), (23, 91), (32, 47),
           (33, 46), (45, 65), (64, 64), (67, 33), (96, 11), (100, 47), (127, 7), (128, 3), (128, 48),
           (129, 2), (131, 48), (181, 9), (182, 40)]


@pytest.mark.parametrize("storage", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("n,N", ADJOINT)
def test_adjoint_shapes(torch, n, N, storage):
    print("adjoint", n, N, storage, flush=True)
    lib, A, rng = _library(torch, n, N, storage)
    g = torch.from_numpy(rng.standard_normal(n * n).astype(np.float32)).cuda()
    out = torch.full((N * N,), float("nan"), device="cuda")
    lib.apply_adjoint(g, out=out)
    ref, mag = A @ g.double(), A.abs() @ g.double().abs()
    assert torch.all((out.double() - ref).abs() <= 1e-5 * mag + 1e-300)
    assert torch.equal(out, lib.apply_adjoint(g))  # fixed order: bitwise reproducible
    lib.close()


# one launch (few columns) and split; one pixel, images smaller than a
# workgroup, rows that end inside a thread's four, every row-block width, up to
# just past 16384 rows; columns that fill no block of 16, one, and several chunks
APPLY = [(1, 1), (1, 40), (2, 3), (3, 33), (5, 46), (8, 32), (16, 7), (17, 33), (22, 47), (32, 32), (33, 46),
         (45, 48), (64, 33), (80, 33), (91, 40), (96, 34), (101, 35), (127, 33), (128, 32), (128, 35),
         (129, 5), (129, 34), (182, 33)]


@pytest.mark.parametrize("storage", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("n,N", APPLY)
def test_apply_shapes(torch, n, N, storage):
    print("apply", n, N, storage, flush=True)
    lib, A, rng = _library(torch, n, N, storage)
    Z = torch.from_numpy(rng.random(N * N).astype(np.float32)).cuda()
    out = torch.full((n * n,), float("nan"), device="cuda")
    lib.apply(Z, out=out)
    ref = Z.double() @ A
    assert torch.all((out.double() - ref).abs() <= 1e-5 * ref.abs() + 1e-300)
    assert torch.equal(out, lib.apply(Z))
    lib.close()


# grouped plans: images of 1 to 4 pixels, rows that end 1 to 3 past a wave's or
# an item's first row, whole and chunked columns, 1 to 17 scenes of a library
@pytest.mark.parametrize("storage,chunks", [("fp32", (0, 16, 64)), ("bf16", (0, 8))])
def test_grouped_shapes(torch, storage, chunks):
    from paper_2106_09122_amd import psflib
    sizes = [(1, 3), (2, 5), (3, 4), (7, 9), (9, 9), (17, 8), (23, 9), (33, 5), (45, 6), (15, 12)]
    built = [_library(torch, n, N, storage) for n, N in sizes]
    libs, As = [b[0] for b in built], [b[1] for b in built]
    rng = np.random.default_rng(7)
    which = [L for L in range(len(libs)) for _ in range((1, 3, 17)[L % 3])]
    scenes = [torch.from_numpy(rng.random(libs[L].ncols).astype(np.float32)).cuda() for L in which]
    plan = psflib.Grouped(libs, which, scenes, autotune=False)
    for chunk in chunks:
        plan.set_shape(chunk, 256)
        for im in plan.images:
            im.fill_(float("nan"))
        plan.run()
        torch.cuda.synchronize()
        for b, L in enumerate(which):
            ref = scenes[b].double() @ As[L]
            err = (plan.images[b].double() - ref).abs()
            # 16 bits: hi + lo parts of the scene, u^2 = 2^-16 of each value
            assert torch.all(err <= (1e-5 if storage == "fp32" else 2.0**-15) * ref + 1e-300), (chunk, sizes[L])
    plan.close()
    for lib in libs:
        lib.close()


# ------------------------------------------------- 16-bit orbit builds ----
# scenes whose base columns fill, exceed or miss blocks of 8 and windows of 16,
# an odd scene's centre column, more than one block of the sort; images with the
# pair whole in LDS (up to 131), with staged boxes, sides not a multiple of 8
BUILD16 = [(1, 1), (5, 2), (8, 3), (7, 6), (33, 7), (16, 8), (31, 9), (6, 10), (100, 5), (127, 11), (128, 12),
           (131, 5), (132, 5), (133, 6), (134, 7), (136, 8), (141, 9), (142, 3), (167, 10), (9, 46), (4, 67)]


@pytest.mark.parametrize("storage", ["bf16", "fp16"])
@pytest.mark.parametrize("rotate,flux", [("bilinear", "none"), ("bilinear", "preserve"), ("cubic", "none"),
                                         ("cubic", "preserve")])
def test_build16_sides(torch, storage, rotate, flux):
    """Columns against the float32 library's: the 16-bit rounding of a value within
    a float32 rounding (2^-21 of the column's bound) of it.  Slots without a column
    are zero: the products of a poisoned buffer are those of its columns."""
    from paper_2106_09122_amd import psflib
    t16 = torch.bfloat16 if storage == "bf16" else torch.float16
    for n, N in BUILD16:
        print("build16", n, N, storage, rotate, flux, flush=True)
        cube, radii, rng = _inputs(n, N, 4, 5)
        mode = dict(rotate=rotate, flux=flux, oob="zero")
        d = torch.from_numpy(cube).cuda()
        full = psflib.Library(d, radii, N, 1.0, **mode)
        lib = psflib.Library(d, radii, N, 1.0, storage=storage, **mode)
        _fill(lib, torch)
        want = full.get_columns(np.arange(N * N)).double()
        got = lib.get_columns(np.arange(N * N)).double()
        e = lib.exponents().cpu().numpy()[:, None]
        unit = torch.from_numpy(np.where(e < -1000, 1.0, np.ldexp(1.0, e))).cuda()
        top = torch.from_numpy(np.where(e < -1000, 0.0, np.ldexp(1.0, e + 15))).cuda()  # at least the column's bound
        low, high = [((want + d * 2.0 ** -21 * top) / unit).float().to(t16).double() * unit for d in (-1, 1)]
        assert torch.all((low <= got) & (got <= high)), (n, N)
        sums = (lib.column_sums() - full.column_sums()).abs()
        assert torch.all(sums <= 2.0 ** -21 * n * n * top[:, 0]), (n, N)
        z = torch.from_numpy(rng.random(N * N).astype(np.float32)).cuda()
        err = (lib.apply(z).double() - z.double() @ got).abs()
        assert torch.all(err <= 1e-5 * (z.double() @ got.abs())), (n, N)
        g = torch.from_numpy(rng.random(n * n).astype(np.float32)).cuda()
        err = (lib.apply_adjoint(g).double() - got @ g.double()).abs()
        assert torch.all(err <= 1e-5 * (got.abs() @ g.double())), (n, N)
        lib.close()
        full.close()


# a library whose base columns (over 512 MiB) are not kept between the passes of a
# flux-preserving build, beside the sizes above whose are: both forms, the pair
# staged whole and in boxes
@pytest.mark.parametrize("n,N,rotate", [(128, 193, "bilinear"), (193, 128, "bilinear"), (193, 128, "cubic")])
def test_build16_flux_large(torch, n, N, rotate):
    from paper_2106_09122_amd import psflib
    cube, radii, _ = _inputs(n, N, 4, 6)
    mode = dict(rotate=rotate, flux="preserve")
    d = torch.from_numpy(cube).cuda()
    full, lib = psflib.Library(d, radii, N, 1.0, **mode), psflib.Library(d, radii, N, 1.0, storage="bf16", **mode)
    cols = np.concatenate([[0, N - 1, N * N // 2, N * N - 1], np.arange(5, N * N, N * N // 200)])
    want, got = full.get_columns(cols).double(), lib.get_columns(cols).double()
    e = lib.exponents().cpu().numpy()[cols][:, None]
    unit, top = (torch.from_numpy(np.ldexp(1.0, e + k)).cuda() for k in (0, 15))
    low, high = [((want + k * 2.0 ** -21 * top) / unit).float().bfloat16().double() * unit for k in (-1, 1)]
    assert torch.all((low <= got) & (got <= high))
    lib.close()
    full.close()


# ---------------------------------------------------- spline coefficients ----
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_spline_keeps_what_is_not_finite(torch, value):
    """One sample that is not finite: every column that samples its PSF with a
    weight has no finite entry under the image's centre, wherever the sample lies;
    columns of the other PSFs are untouched (n above the filter's reach of 32)."""
    from paper_2106_09122_amd import psflib
    n, N = 121, 9
    cube, radii, _ = _inputs(n, N, 5, 7)
    clean = psflib.Library(torch.from_numpy(cube).cuda(), radii, N, 1.0, rotate="cubic")
    cube[4, 2, 3] = value
    lib = psflib.Library(torch.from_numpy(cube).cuda(), radii, N, 1.0, rotate="cubic")
    far = (np.hypot(*np.meshgrid(np.arange(N) - 4.0, np.arange(N) - 4.0)) > radii[3]).ravel()
    mid = (n // 2) * n + n // 2
    got, want = lib.get_columns(np.arange(N * N)).cpu().numpy(), clean.get_columns(np.arange(N * N)).cpu().numpy()
    assert not np.isfinite(got[far][:, mid]).any()
    assert np.array_equal(got[~far], want[~far])
    lib.close()
    clean.close()


# ------------------------------------------------------- orbit ordering ----
# base columns below, at and above one sort block and the one-workgroup sort
# (4096: 128 x 128), one bracket to more than the sort's threads, brackets left
# empty, wide ones (many items each); the column of a PSF that is all k + 1 tells
# its radial sample, so a column taken for another bracket's shows
@pytest.mark.parametrize("N,K", [(2, 2), (63, 3), (64, 40), (65, 12), (127, 2), (128, 128), (128, 300), (129, 5),
                                 (130, 1400), (200, 12)])
@pytest.mark.parametrize("storage", ["fp32", "bf16"])
def test_orbit_order(torch, N, K, storage):
    from paper_2106_09122_amd import psflib
    cube = np.broadcast_to(np.arange(1, K + 1, dtype=np.float32)[:, None, None], (K, 1, 1)).copy()
    radii = np.linspace(0.1, 0.6 * N, K)
    lib = psflib.Library(torch.from_numpy(cube).cuda(), radii, N, 1.0, storage=storage)
    _fill(lib, torch)
    c = np.arange(N) - 0.5 * (N - 1)
    want = np.interp(np.hypot(*np.meshgrid(c, c)).ravel(), radii, np.arange(1, K + 1))
    got = lib.get_columns(np.arange(N * N)).cpu().numpy()[:, 0]
    unit = 1e-6 if storage == "fp32" else 2.0 ** -8  # float32 blend; bf16 rounding
    assert np.all(np.abs(got - want) <= unit * want * 1.001)
    z = torch.from_numpy(np.random.default_rng(N).random(N * N).astype(np.float32)).cuda()
    ref = float(z.double() @ torch.from_numpy(got).cuda().double())
    assert abs(float(lib.apply(z)[0]) - ref) <= 1e-5 * ref
    assert np.allclose(lib.column_sums().cpu().numpy(), want, rtol=1e-6)
    lib.close()


# ------------------------------------------------------------ batched ----
# scenes at the edges of every tile (32, 64, 128, 256) and of the kernels' ranges;
# images of an odd number of pixels, smaller and larger than a tile of 256; one
# slice of columns, several, and more than 16 (a narrow image, a wide scene)
@pytest.mark.parametrize("storage", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("n,N", [(1, 3), (3, 150), (16, 16), (17, 100), (31, 33), (33, 90), (64, 31)])
def test_batched_shapes(torch, n, N, storage):
    """Non-negative terms: 1e-5 relative for the float32 sums, and for the 16-bit
    forms a rounding of each scene value (half a unit of its mantissa: 2^-8, 2^-11)."""
    lib, A, rng = _library(torch, n, N, storage)
    tol = 1e-5 + {"fp32": 0.0, "bf16": 2.0 ** -8, "fp16": 2.0 ** -11}[storage]
    for B in (1, 7, 32, 33, 64, 65, 128, 129, 257):
        print("batched", n, N, storage, B, flush=True)
        Z = torch.from_numpy(rng.uniform(0.5, 1.0, (B, N * N)).astype(np.float32)).cuda()
        out = torch.full((B, n * n), float("nan"), device="cuda")
        lib.apply_batched(Z, out=out)
        ref = Z.double() @ A
        assert torch.all((out.double() - ref).abs() <= tol * ref + 1e-300), B
        assert torch.equal(out, lib.apply_batched(Z))
    lib.close()
