"""Builds beyond the bounds of the orbits' sort, which take the other kernels:

 * more than 8192 PSFs: the bilinear and cubic gathers from pair-interleaved
   copies, the flux rescale of float32 columns, the packing pass and the natural
   order of the 16-bit slots;
 * blocks of 1024 base columns times brackets above 2^24: columns in bracket order
   with the pair in LDS (the bucket sort), packed for the 16-bit forms.
"""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu


def _natural_order(torch, lib):
    """The slot -> column map of a 16-bit library (the second int32 array after the
    column sums, each part 256-byte aligned) lists the columns in order."""
    def up(x):
        return (x + 255) // 256 * 256
    pad = (lib.ncols + 63) // 64 * 64
    off = up(up(up(lib.M * pad * 2) + lib.ncols * 8) + pad * 4)
    perm = lib.buf[off:off + pad * 4].view(torch.int32)
    return torch.equal(perm[:lib.ncols], torch.arange(lib.ncols, dtype=torch.int32, device="cuda")) and bool(
        torch.all(perm[lib.ncols:] == -1))


def _rounded(torch, A32, e, storage):
    """RN16(A32 2^-e) 2^e, exact but for the one rounding (A32: [columns][pixels])."""
    x = np.ldexp(A32.astype(np.float64), -e[:, None]).astype(np.float32)
    r = torch.from_numpy(x).to(torch.bfloat16 if storage == "bf16" else torch.float16).double().numpy()
    return np.ldexp(r, e[:, None])


@pytest.mark.parametrize("rotate,flux", [("bilinear", "none"), ("bilinear", "preserve"), ("cubic", "none"),
                                         ("cubic", "preserve")])
@pytest.mark.parametrize("n,N,oob", [(1, 3, "clamp"), (5, 6, "zero"), (18, 5, "zero")])
def test_gathers(n, N, oob, rotate, flux):
    """Entries against the FP64 oracle with the tolerances of the orbit builds'
    tests (bilinear 1e-6 relative, 2e-6 rescaled; cubic 1e-6 of the column's bound,
    twice that rescaled), the 16-bit forms exactly the rounded float32 entries."""
    import torch
    from paper_2106_09122_amd import psflib
    K = 8200
    rng = np.random.default_rng([n, N])
    cube = (rng.random((K, n, n)) ** 3).astype(np.float32)
    radii = np.linspace(0.0, 0.6 * N, K)
    mode = dict(rotate=rotate, flux=flux, oob=oob)
    print("gathers", n, N, mode, flush=True)
    A = O.build_library(cube, radii, N, 1.0, **mode)
    d = torch.from_numpy(cube).cuda()
    libs = {}
    for storage in ("fp32", "bf16", "fp16"):
        lib = libs[storage] = psflib.Library(d, radii, N, 1.0, storage=storage, **mode)
        lib.buf.fill_(0xFF)  # built again over a poisoned buffer: an entry not written stays
        h = psflib.build(lib.desc, lib.cube.data_ptr(), lib.radii, lib.buf.data_ptr(), lib.nbytes,
                         torch.cuda.current_stream().cuda_stream)
        psflib.destroy(lib.h)
        lib.h = h
    got = libs["fp32"].get_columns(np.arange(N * N)).cpu().numpy()
    if rotate == "bilinear":
        tol = (2e-6 if flux == "preserve" else 1e-6) * A
    else:
        _, _, r, ct, st = O.scene_geometry(N, 1.0)
        b = np.zeros(N * N)
        for j in range(N * N):
            k, w, zero = O.radial_bracket(r[j], radii, "linear", oob)
            if not zero:
                m = [np.abs(O.spline_coefficients(cube[q].astype(np.float64))).max() for q in (k, k + 1)]
                b[j] = (1.0 - w) * m[0] + w * m[1]
        if flux == "preserve":
            t0 = O.build_library(cube, radii, N, 1.0, rotate=rotate, oob=oob).sum(axis=0)
            t1 = A.sum(axis=0)
            b = 2 * b * np.abs(np.where(t0 != 0, t1 / np.where(t0 != 0, t0, 1.0), 1.0))
        tol = 1e-6 * b[None, :]
    assert np.all(np.abs(got.T - A) <= tol + 1e-300)
    z = torch.from_numpy(rng.random(N * N).astype(np.float32)).cuda()
    g = torch.from_numpy(rng.random(n * n).astype(np.float32)).cuda()
    for storage, lib in libs.items():
        cols = lib.get_columns(np.arange(N * N))
        if storage != "fp32":
            e = lib.exponents().cpu().numpy().astype(np.int64)
            assert np.array_equal(cols.cpu().numpy().astype(np.float64), _rounded(torch, got, e, storage)), storage
            assert _natural_order(torch, lib)
        sums = lib.column_sums().cpu().numpy()
        assert np.all(np.abs(sums - A.sum(axis=0)) <= np.sum(np.broadcast_to(tol, A.shape), axis=0) + 1e-300)
        cols = cols.double()
        err = (lib.apply(z).double() - z.double() @ cols).abs()
        assert torch.all(err <= 1e-5 * (z.double() @ cols.abs()) + 1e-300), storage
        err = (lib.apply_adjoint(g).double() - cols @ g.double()).abs()
        assert torch.all(err <= 1e-5 * (cols.abs() @ g.double()) + 1e-300), storage
        lib.close()


@pytest.mark.parametrize("n", [1, 3])
def test_columns_in_bracket_order(n):
    """8192 PSFs and a scene just beyond the sort's bound (2051 blocks of base columns,
    8192 brackets): sampled columns against the oracle (1e-6 relative), the bf16 form
    exactly the rounded float32 entries of all columns, the sums of all columns."""
    import torch
    from paper_2106_09122_amd import psflib
    N, K = 2898, 8192
    rng = np.random.default_rng(n)
    cube = (0.1 + rng.random((K, n, n))).astype(np.float32)
    radii = np.linspace(0.0, 0.5 * N, K)  # the corners lie beyond: identically zero
    print("bracket order", n, flush=True)
    d = torch.from_numpy(cube).cuda()
    full = psflib.Library(d, radii, N, 1.0, oob="zero")
    A = full.buf[:full.ncols * full.M * 4].view(torch.float32).view(full.ncols, full.M)
    cols = np.concatenate([[0, N - 1, N * N - 1], rng.choice(N * N, 600, replace=False)])
    want = O.build_library(cube, radii, N, 1.0, oob="zero", columns=cols).T
    got = A[torch.from_numpy(cols).cuda()].cpu().numpy()
    assert np.all(np.abs(got - want) <= 1e-6 * want)
    sums = A.double().sum(dim=1)
    assert torch.all((full.column_sums() - sums).abs() <= 1e-6 * sums)
    lib = psflib.Library(d, radii, N, 1.0, oob="zero", storage="bf16")
    assert _natural_order(torch, lib)
    e = lib.exponents().cpu().numpy()
    pad = (lib.ncols + 63) // 64 * 64
    M16 = lib.buf[:lib.M * pad * 2].view(torch.bfloat16).view(pad // 8, lib.M, 8).transpose(1, 2).reshape(pad, lib.M)
    scaled = np.ldexp(A.cpu().numpy(), np.where(e < -1000, 0, -e)[:, None])  # exact; a zero column stays zero
    assert torch.equal(M16[:lib.ncols].cpu(), torch.from_numpy(scaled).bfloat16())
    assert torch.all(M16[lib.ncols:] == 0)
    assert torch.equal(lib.column_sums(), full.column_sums())
    lib.close()
    full.close()
