"""The natively marshalled calls refuse what they cannot take before anything reaches the library."""
import pytest
import torch

from paper_2603_06938_amd import binding as sw


@pytest.mark.parametrize("x,kind", [
    (torch.zeros(1, 2, 3, 4), ValueError),                          # not on a GPU
    (torch.zeros(2, 3, 4), ValueError),                             # a dimension short
    (torch.zeros(1, 2, 3, 4, dtype=torch.float64), TypeError),
    ([[1.0]], TypeError),
], ids=["cpu", "rank", "dtype", "list"])
def test_forward_refuses(x, kind):
    t = torch.zeros(1, 2, 3, 1, 4)
    with pytest.raises(kind):
        sw.swimba_mixer_fwd(x, t, t, None, t, t, t, 2, 64)
    with pytest.raises((TypeError, ValueError)):
        sw.swimba_step_multi(t, x, t, t, None, t, t, t, 2)
