"""Sample offsets and tile jobs at the edges of their chunks of 1,024 nodes and of the scan of the chunks (8,192 of them a
round): frontiers of those sizes, rows of several tiles first, last and between empty rows; against numpy and the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rg():
    from paper_2509_05207_amd import binding
    binding.lib()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return binding


@pytest.mark.parametrize("nodes", [1, 3, 4, 5, 255, 1023, 1024, 1025, 4097, 8192 * 1024 + 3])
def test_offsets_of_frontiers_of_every_size(rg, nodes):
    d = "cuda"
    deg = torch.from_numpy(np.random.default_rng(nodes).integers(0, 4, size=nodes)).to(d)
    indptr = torch.zeros(nodes + 1, dtype=torch.int64, device=d)
    indptr[1:] = torch.cumsum(deg, 0)
    start = torch.arange(int(indptr[-1]), device=d) - torch.repeat_interleave(indptr[:-1], deg)
    indices = ((torch.repeat_interleave(torch.arange(nodes, device=d), deg) % max(nodes - 3, 1)) + start).clamp_(max=nodes - 1).to(torch.int32)
    train = torch.randperm(nodes, device=d, dtype=torch.int32)
    s = rg.rg_build_schedule(indptr, indices, train, nodes, [2], 1, 0, 0)
    ids = rg.rg_schedule_frontier(s, 0)[0].long()
    off, nbr = rg.rg_schedule_samples(s, 0)
    want = torch.zeros(nodes + 1, dtype=torch.int64, device=d)
    want[1:] = torch.cumsum(deg[ids].clamp(max=2), 0)
    assert torch.equal(off, want) and nbr.numel() == int(want[-1])


@pytest.mark.parametrize("nodes", [1024, 1025, 2050])
def test_tile_jobs_at_the_chunks_edges(rg, orc, nodes):
    rng = np.random.default_rng(nodes)
    n = 140_000
    deg = np.zeros(n, np.int64)
    train = np.sort(rng.permutation(n)[:nodes]).astype(np.int32)
    o = orc.epoch_seeds(train, 5, 1, 2)                                  # the order the nodes come in
    for k in (0, 1, 1023, nodes - 1, nodes // 2):
        deg[o[k]] = [70_000, 16_385, 131_073, 66_000, 16_384][k % 5]
    indptr = np.zeros(n + 1, np.int64)
    indptr[1:] = np.cumsum(deg)
    indices = np.concatenate([np.sort(rng.permutation(n)[:x]) for x in deg if x]).astype(np.int32)
    a = orc.Schedule(indptr, indices, train, nodes, [7], 5, 1, 2, n_threads=4)
    b = rg.rg_build_schedule(torch.from_numpy(indptr).cuda(), torch.from_numpy(indices).cuda(), torch.from_numpy(train).cuda(), nodes, [7], 5, 1, 2)
    for x, y in zip(a.samples(0), rg.rg_schedule_samples(b, 0)):
        assert np.array_equal(y.cpu().numpy(), x)
