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
