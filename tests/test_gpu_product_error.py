"""Rounding errors of the float32 products' sums over slices (chunks) of columns.

Non-negative terms: the sum over the slices is the last and largest part of every
output's sum, and with slices added in pairs or in float64 the whole root mean square
error stays below half a float32 unit (2^-24), the bound of a single rounding; a chain
through 16 or more slices exceeds it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

UNIT = 2.0 ** -24


def _rms(x, ref):
    keep = ref > 0
    return float((((x.double() - ref)[keep] / ref[keep]) ** 2).mean().sqrt())


# narrow images (many slices, up to 64), and wider ones
@pytest.mark.parametrize("n,N", [(16, 250), (33, 150), (20, 60), (64, 112)])
@pytest.mark.parametrize("B", [7, 20])
def test_batched_slices(n, N, B):
    import torch
    from paper_2106_09122_amd import psflib
    rng = np.random.default_rng([n, N])
    cube = torch.from_numpy((rng.random((3, n, n)) ** 3).astype(np.float32)).cuda()
    lib = psflib.Library(cube, np.linspace(0.0, 0.3 * N, 3), N, 1.0)
    A = torch.cat([lib.get_columns(np.arange(j, min(j + 4096, N * N))) for j in range(0, N * N, 4096)])
    Z = torch.from_numpy(rng.random((B, N * N)).astype(np.float32)).cuda()
    err = _rms(lib.apply_batched(Z), Z.double() @ A.double())
    print("batched rounding", n, N, B, err / UNIT, flush=True)
    assert err <= UNIT
    lib.close()


# chunk counts just above one block of 16, several blocks
@pytest.mark.parametrize("n,N", [(80, 33), (96, 40), (64, 112), (20, 60)])
def test_matvec_chunks(n, N):
    import torch
    from paper_2106_09122_amd import psflib
    rng = np.random.default_rng([n, N])
    cube = torch.from_numpy((rng.random((3, n, n)) ** 3).astype(np.float32)).cuda()
    lib = psflib.Library(cube, np.linspace(0.0, 0.3 * N, 3), N, 1.0)
    A = torch.cat([lib.get_columns(np.arange(j, min(j + 4096, N * N))) for j in range(0, N * N, 4096)])
    Z = [torch.from_numpy(rng.random(N * N).astype(np.float32)).cuda() for _ in range(20)]
    err = _rms(torch.stack([lib.apply(z) for z in Z]), torch.stack(Z).double() @ A.double())
    print("matvec rounding", n, N, err / UNIT, flush=True)
    assert err <= UNIT
    lib.close()


# Slices of many blocks of 128 columns (wide batches, whose tiles fill the GPU): the
# rounding of a chain of k near equal non-negative terms is 0.42 sqrt(k / 3) of a unit
# in the mean, for 128 blocks in runs of 16, then 8 runs, 0.8 units in all; 2.8 in one chain
@pytest.mark.parametrize("n,N,B", [(128, 128, 200), (96, 96, 400), (64, 181, 256), (101, 101, 100), (45, 128, 1024)])
def test_batched_long_slices(n, N, B):
    import torch
    from paper_2106_09122_amd import psflib
    rng = np.random.default_rng([n, N, B])
    cube = torch.from_numpy((rng.random((3, n, n)) ** 3).astype(np.float32)).cuda()
    lib = psflib.Library(cube, np.linspace(0.0, 0.3 * N, 3), N, 1.0)
    A = torch.cat([lib.get_columns(np.arange(j, min(j + 4096, N * N))) for j in range(0, N * N, 4096)])
    Z = torch.from_numpy(rng.random((B, N * N)).astype(np.float32)).cuda()
    out = lib.apply_batched(Z)
    pick = [0, 31, 32, B - 1]
    err = _rms(out[pick], Z[pick].double() @ A.double())
    print("batched rounding", n, N, B, err / UNIT, flush=True)
    assert err <= UNIT
    lib.close()
