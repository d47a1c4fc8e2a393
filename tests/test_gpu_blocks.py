"""Computation blocks where the workgroup map changes shape: numbers of batches around the eight XCDs, groups of batches of
every size, batches with few edges and none; and the O(f) sampler's samples marked in every way; against the oracle."""
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


def graph(rng, n, most):
    deg = rng.integers(0, most + 1, size=n)
    deg[rng.random(n) < 0.2] = 0
    indptr = np.zeros(n + 1, np.int64)
    rows = []
    for v in range(n):
        r = np.unique(rng.integers(0, n, size=deg[v]))
        rows.append(r.astype(np.int32))
        indptr[v + 1] = indptr[v] + r.size
    return indptr, np.concatenate(rows)


@pytest.mark.parametrize("n_batches", [1, 7, 8, 9, 17])
@pytest.mark.parametrize("group", [1, 3, 8, 100])
def test_blocks_of_every_group(rg, orc, n_batches, group):
    rng = np.random.default_rng(n_batches)
    n, batch = 3000, 40
    indptr, indices = graph(rng, n, 12)
    train = rng.permutation(n)[: n_batches * batch - 3].astype(np.int32)
    o = orc.Schedule(indptr, indices, train, batch, [5, 1, 3], 1, 0, 0)
    s = rg.rg_build_schedule(torch.from_numpy(indptr).cuda(), torch.from_numpy(indices).cuda(), torch.from_numpy(train).cuda(), batch, [5, 1, 3], 1, 0, 0)
    rg.rg_schedule_build_blocks(s, workspace_limit_bytes=4 * n * group)
    for hop in range(3):
        assert np.array_equal(rg.rg_schedule_block(s, hop).cpu().numpy(), o.block(hop)), hop


@pytest.mark.parametrize("mark_pass", ["0", "1", None])
@pytest.mark.parametrize("fanout", [[2, 3], [40, 40], [255, 2], [256, 3], [300, 1]])
def test_positions_sampler_in_every_marking(rg, orc, mark_pass, fanout, monkeypatch):
    if mark_pass is not None:
        monkeypatch.setenv("RAPIDGNN_MARK_PASS", mark_pass)
    rng = np.random.default_rng(len(fanout) + fanout[0])
    n = 2000
    indptr, indices = graph(rng, n, 700)
    train = rng.permutation(n)[:500].astype(np.int32)
    o = orc.Schedule(indptr, indices, train, 60, fanout, 1, 0, 0, sampler="positions")
    s = rg.rg_build_schedule_with(torch.from_numpy(indptr).cuda(), torch.from_numpy(indices).cuda(), torch.from_numpy(train).cuda(), 60, fanout, 1, 0, 0,
                                  sampler=rg.RG_SAMPLER_POSITIONS)
    for hop in range(3):
        assert np.array_equal(rg.rg_schedule_frontier(s, hop)[0].cpu().numpy(), o.frontier(hop)[0]), hop
    for hop in range(2):
        assert np.array_equal(rg.rg_schedule_samples(s, hop)[1].cpu().numpy(), o.samples(hop)[1]), hop


@pytest.mark.parametrize("batch,n_batches,rest", [(64, 3, 0), (65, 3, 2), (8200, 2, 1), (9000, 9, 8999), (120_000, 1, 0), (500, 17, 499)])
def test_blocks_of_batches_of_every_size(rg, batch, n_batches, rest):
    """From one workgroup per batch (1,024 edges on average) to the most there are (128) and several rounds of them; a last batch
    much smaller than the average; every edge's place against the input nodes themselves."""
    n, deg = 150_000, 20
    g = torch.Generator("cuda").manual_seed(batch)
    steps = torch.randint(0, n // deg, (n, deg), device="cuda", generator=g, dtype=torch.int32)
    indices = (steps + torch.arange(deg, device="cuda", dtype=torch.int32) * (n // deg)).reshape(-1).contiguous()
    indptr = torch.arange(0, n * deg + 1, deg, device="cuda", dtype=torch.int64)
    train = torch.randperm(n, device="cuda", generator=g)[: batch * n_batches - rest].to(torch.int32)
    s = rg.rg_build_schedule(indptr, indices, train, batch, [16, 3], 1, 0, 0)
    rg.rg_schedule_build_blocks(s)
    ids, _, off = rg.rg_schedule_frontier(s, 2)
    for hop in range(2):
        _, _, at = rg.rg_schedule_frontier(s, hop)
        samp_off, nbr = rg.rg_schedule_samples(s, hop)
        src = rg.rg_schedule_block(s, hop).to(torch.int64)
        ends = samp_off[torch.from_numpy(np.asarray(at)).to("cuda")]
        first = torch.from_numpy(np.asarray(off[:-1])).to("cuda")
        assert torch.equal(ids[src + torch.repeat_interleave(first, ends[1:] - ends[:-1])], nbr), hop


@pytest.mark.parametrize("force", ["1", "0"])
@pytest.mark.parametrize("n,batch,fanout", [(33, 5, [3]), (64, 64, [2, 2]), (65, 7, [4, 4]), (2047, 300, [5, 1, 3]), (2049, 1, [40, 2]), (4100, 4100, [3, 3, 3, 3]),
                                            (60_000, 900, [6, 5]), (150_000, 2000, [4, 2, 2])])
def test_blocks_by_ranks_and_by_tables(rg, orc, n, batch, fanout, force, monkeypatch):
    """Positions from bitmaps in LDS and from tables: graphs around whole words and pairs of words, one to five bitmaps, batches of one seed and
    of all nodes, one batch shared out among all workgroups and many."""
    monkeypatch.setenv("RAPIDGNN_BLOCK_RANKS", force)
    rng = np.random.default_rng(n)
    indptr, indices = graph(rng, n, 12)
    train = rng.permutation(n)[: max(batch, min(n, 3 * batch + 1))].astype(np.int32)
    o = orc.Schedule(indptr, indices, train, batch, fanout, 1, 0, 0)
    s = rg.rg_build_schedule(torch.from_numpy(indptr).cuda(), torch.from_numpy(indices).cuda(), torch.from_numpy(train).cuda(), batch, fanout, 1, 0, 0)
    rg.rg_schedule_build_blocks(s)
    for hop in range(len(fanout)):
        assert np.array_equal(rg.rg_schedule_block(s, hop).cpu().numpy(), o.block(hop)), hop
