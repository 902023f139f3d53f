"""Infinite library entries in the products (a flux-preserving rescale of a column
whose sum all but cancels can overflow float32): an infinite entry reaches the
sums that its row and column belong to, as an infinity, and no other.  Reference:
the same products in float64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# one pixel, less than a step of rows, steps that the image does not fill, steps
# that do not fill a round (96^2: 36 steps of 256 rows), columns that start at any
# float, several row blocks (from 129^2), few columns (waves share one) and many
CASES = [(1, 5), (2, 3), (3, 40), (17, 40), (33, 50), (64, 20), (96, 9), (96, 56), (101, 20), (127, 12),
         (129, 8), (150, 46), (182, 6)]


def _built(n, N, storage):
    import torch
    from paper_2106_09122_amd import psflib
    rng = np.random.default_rng([n, N])
    cube = torch.from_numpy(rng.uniform(0.5, 1.0, (3, n, n)).astype(np.float32)).cuda()
    lib = psflib.Library(cube, np.linspace(0.0, 0.3 * N, 3), N, 1.0, storage=storage)
    return torch, lib, rng


def _poke(torch, lib, storage, cells):
    """Make the entries (column, row; in 16 bits group of 8 slots, row[, slot]) infinite."""
    M = lib.M
    if storage == "fp32":
        A = lib.buf[:lib.ncols * M * 4].view(torch.float32).view(lib.ncols, M)
    else:
        pad = (lib.ncols + 63) // 64 * 64
        A = lib.buf[:pad * M * 2].view(torch.bfloat16 if storage == "bf16" else torch.float16).view(pad // 8, M, 8)
    for c in cells:
        A[c] = float("inf")


@pytest.mark.parametrize("storage", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("n,N", CASES)
def test_adjoint_of_infinite_entries(n, N, storage):
    print("infinite entries", n, N, storage, flush=True)
    torch, lib, rng = _built(n, N, storage)
    g = torch.from_numpy(rng.uniform(0.5, 1.0, lib.M).astype(np.float32)).cuda()
    units = lib.ncols if storage == "fp32" else (lib.ncols + 63) // 64 * 8
    # one in every column, their rows spread over the image, its last row among them
    rows = np.arange(units) * (lib.M - 1) // max(units - 1, 1)
    rows[-1] = lib.M - 1
    _poke(torch, lib, storage, zip(range(units), rows))
    assert torch.all(lib.apply_adjoint(g) == float("inf"))
    lib.close()


@pytest.mark.parametrize("storage", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("n,N", CASES)
def test_one_infinite_entry(n, N, storage):
    print("one infinite entry", n, N, storage, flush=True)
    torch, lib, rng = _built(n, N, storage)
    g = torch.from_numpy(rng.uniform(0.5, 1.0, lib.M).astype(np.float32)).cuda()
    z = torch.from_numpy(rng.uniform(0.5, 1.0, (3, lib.ncols)).astype(np.float32)).cuda()
    before = [lib.apply_adjoint(g), lib.apply(z[0]), lib.apply_batched(z)]
    row = lib.M - 1
    _poke(torch, lib, storage, [(0, row) if storage == "fp32" else (0, row, 0)])  # slot 0 holds a column
    A = torch.cat([lib.get_columns(np.arange(j, min(j + 512, lib.ncols)))[:, row] for j in range(0, lib.ncols, 512)])
    hit = torch.isinf(A)
    assert int(hit.sum()) == 1
    got = lib.apply_adjoint(g)
    assert torch.all(got[hit] == float("inf")) and torch.equal(got[~hit], before[0][~hit])
    got = lib.apply(z[0])
    assert got[row] == float("inf") and torch.equal(got[:row], before[1][:row])
    got = lib.apply_batched(z)
    assert torch.all(got[:, row] == float("inf")) and torch.equal(got[:, :row], before[2][:, :row])
    lib.close()
