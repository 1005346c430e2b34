"""What the natively marshalled calls raise on the GPU is what torch and the library raise by themselves."""
import pytest
import torch

from paper_2603_06938_amd import binding as sw

pytestmark = pytest.mark.gpu


def test_out_of_memory_keeps_its_type():
    """A program that catches torch.OutOfMemoryError (and retries with less) sees it from these calls too."""
    u = torch.zeros(1 << 20, 1, device="cuda:0")
    W = torch.zeros(256, 1, device="cuda:0")          # 1 GiB of logits
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (64 << 20)) / total)
    try:
        with pytest.raises(torch.OutOfMemoryError):
            sw.swimba_router_linear(u, W)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)


@pytest.mark.parametrize("k,status", [(-1, 2), (0, 2), (5, 2), (17, 4)])
def test_refused_sizes_raise_their_status(k, status):
    """Before any output of that size is asked for."""
    E = 4 if k < 17 else 32
    x, dt = torch.zeros(1, 2, 3, 4, device="cuda:0"), torch.zeros(1, 2, 3, device="cuda:0")
    A, Be, lg = torch.zeros(3, device="cuda:0"), torch.zeros(1, 2, E, 1, 4, device="cuda:0"), torch.zeros(1, 2, E, device="cuda:0")
    W = torch.zeros(E, 1, 4, 8, device="cuda:0")
    with pytest.raises(sw.SwimbaError) as e:
        sw.swimba_mixer_fwd(x, dt, A, None, Be, Be, lg, k, 64, want_topk=True)
    assert e.value.status == status
    with pytest.raises(sw.SwimbaError) as e:
        sw.swimba_mixer_fwd_proj(torch.zeros(1, 2, 8, device="cuda:0"), W, W, x, dt, A, None, lg, k, 64, want_topk=True)
    assert e.value.status == status
