"""Rounding errors of the 16-bit adjoint: no larger than those of sums whose chains are
64 products long (256 threads of a workgroup with every 256th row each, their sums in
pairs over the wave, the four waves' in order).

The library is exact in 16 bits and float32 here, so the error against float64 is the
summation's alone.  Both errors are the root mean square over thousands of columns,
each with a relative spread of one part in a hundred: 8% above counts as larger."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _chains(A, g):
    """float32 sums in the order above; A: [columns][pixels], fused products."""
    C, M = A.shape
    U = -(-M // 256)
    A = np.pad(A, ((0, 0), (0, U * 256 - M))).reshape(C, U, 256)
    g = np.pad(g, (0, U * 256 - M)).reshape(U, 256)
    acc = np.zeros((C, 256), np.float32)
    for u in range(U):
        acc = (A[:, u].astype(np.float64) * g[u] + acc).astype(np.float32)
    v = acc.reshape(C, 4, 64)
    while v.shape[2] > 1:
        h = v.shape[2] // 2
        v = v[..., :h] + v[..., h:]
    return ((v[:, 0, 0] + v[:, 1, 0]) + v[:, 2, 0]) + v[:, 3, 0]


# each wave a column of its own (many columns), and the waves of a workgroup on one
@pytest.mark.parametrize("n,N", [(64, 112), (96, 112), (101, 112), (128, 111), (64, 90), (96, 90), (101, 90),
                                 (128, 90)])
@pytest.mark.parametrize("signed", [True, False])
def test_adjoint_rounding(n, N, signed):
    import torch
    from paper_2106_09122_amd import psflib
    rng = np.random.default_rng([n, N])
    cube = torch.from_numpy((rng.random((3, n, n)) ** 3).astype(np.float32)).cuda()
    lib = psflib.Library(cube, np.linspace(0.0, 0.3 * N, 3), N, 1.0, storage="bf16")
    gh = (rng.standard_normal(lib.M) if signed else rng.random(lib.M)).astype(np.float32)
    got = lib.apply_adjoint(torch.from_numpy(gh).cuda()).cpu().numpy()
    cols = rng.permutation(N * N)[:5000]
    A = np.concatenate([lib.get_columns(c).cpu().numpy() for c in np.array_split(cols, 10)])
    ref = A.astype(np.float64) @ gh.astype(np.float64)
    mag = A.astype(np.float64) @ np.abs(gh.astype(np.float64))
    err, bound = (float(np.sqrt(np.mean(((x - ref) / mag) ** 2))) for x in (got[cols], _chains(A, gh)))
    print("adjoint rounding", n, N, signed, err, bound, err / bound, flush=True)
    assert err <= 1.08 * bound
    lib.close()
