"""Device memory that builds take beside what they hand out, against what their lists need."""
import numpy as np
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


@pytest.mark.parametrize("look", ["1", "0"])
@pytest.mark.parametrize("codes", ["1", "0"])
def test_scratch_of_a_plan(rg, look, codes, monkeypatch):
    """Beside its codes (4 bytes a position; 8 where they have to be entries) a plan takes 4 bytes per 512 positions while it is made; looking whether
    row_of is ranks takes nothing.  The selection's scratch is 8 bytes per 2,048 nodes and 0.13 MB."""
    monkeypatch.setenv("RAPIDGNN_ROW_RANKS", look)
    monkeypatch.setenv("RAPIDGNN_PLAN_CODES", codes)
    rng = np.random.default_rng(1)
    n, d = 4_000_000, "cuda"
    indptr, indices = torch.zeros(n + 1, dtype=torch.int64, device=d), torch.zeros(0, dtype=torch.int32, device=d)
    s = rg.rg_build_schedule(indptr, indices, torch.arange(n, dtype=torch.int32, device=d), 100_000, [], 5, 0, 0)
    is_local = (rng.random(n) < 0.99).astype(np.uint8)
    row_of = np.where(is_local, np.cumsum(is_local) - 1, np.cumsum(1 - is_local) - 1).astype(np.int32)
    table = torch.zeros((n, 4), dtype=torch.int32, device=d)
    feat = rg.make_features(torch.from_numpy(is_local).to(d), torch.from_numpy(row_of).to(d), table, table, 16)
    a = RecordingAllocator(rg)
    c = rg.rg_build_cache([s], feat, 0, allocator=a.struct)
    route = 4 if codes == "1" else 8
    assert a.live < route * n + n + n // 2 + (1 << 18)                       # routes; the tally's byte and the slot map's half per node
    assert a.peak - a.live < n // 128 + n // 256 + (1 << 18)
    del c
