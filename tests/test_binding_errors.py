"""Arguments that the differentiable operations refuse before any device call (so
these run without a GPU)."""
import numpy as np
import pytest

fit = pytest.importorskip("paper_2106_09122_amd.fit")
torch = pytest.importorskip("torch")


def test_chi2_arguments_that_are_not_tensors():
    S, V = torch.ones(4), torch.ones(4, dtype=torch.float64)
    for counts in (np.ones(4), None, [1.0] * 4):
        with pytest.raises(ValueError, match="counts must be a float64 tensor of 4 elements on cpu"):
            fit.chi2(S, counts, V, 1.0)
    with pytest.raises(ValueError, match="var must be a float64 tensor of 4 elements on cpu"):
        fit.chi2(S, V, np.ones(4), 1.0)
    with pytest.raises(ValueError, match="model must be a float32 image"):
        fit.chi2(S.double(), None, None, 1.0)  # the model is looked at first
    with pytest.raises(AttributeError):
        fit.chi2(np.ones(4, np.float32), V, V, 1.0)


def test_disk_parameters_that_are_not_tensors():
    with pytest.raises(AttributeError):
        fit.render_disk(np.ones(5), 4, 1.0, 8.0)


@pytest.mark.parametrize("numel", [0, 1, 4])
def test_fewer_parameters_than_the_disk_has(numel):
    """The renderer reads five values: fewer are refused."""
    with pytest.raises(ValueError, match="theta must have 5 elements"):
        fit.render_disk(torch.ones(numel, dtype=torch.float64), 4, 1.0, 8.0)

    class Grid:
        N, S = 4, 1.0

    with pytest.raises(ValueError, match="theta must have 5 elements"):
        fit.loss_and_grad(Grid(), torch.ones(numel), torch.ones(4).double(), torch.ones(4).double(), 1.0, 8.0)
