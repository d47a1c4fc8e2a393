"""Device memory that builds take beside what they hand out, against what their lists need."""
import pytest
import torch

from recording_allocator import RecordingAllocator

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rg():
    from paper_2509_05207_amd import binding
    binding.lib()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return binding


def test_scratch_of_the_shuffle(rg):
    """16 bytes per train node (its key and position) beside the 4 of the seeds, 12 per bucket of 64 to 128, and a bit per node of the graph."""
    n, d = 3_000_000, "cuda"
    indptr, indices = torch.zeros(n + 1, dtype=torch.int64, device=d), torch.zeros(0, dtype=torch.int32, device=d)
    a = RecordingAllocator(rg)
    s = rg.rg_build_schedule(indptr, indices, torch.arange(n, dtype=torch.int32, device=d), 100_000, [], 5, 0, 0, allocator=a.struct)
    assert a.peak < 20 * n + 12 * n // 64 + n // 8 + (1 << 18)
    del s
