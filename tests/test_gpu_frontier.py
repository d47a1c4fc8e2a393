"""Frontiers written lane by lane (fewer than 64 new IDs in a wave's 16,384 on average), through LDS and group by group (more
than 4,096), for both ways of marking what was reached: batches that reach next to nothing, a little, about a quarter and
most of the graph, at sizes around a wave's and a workgroup's span; against the oracle."""
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


@pytest.mark.parametrize("mark_pass", ["0", "1"])
@pytest.mark.parametrize("n", [300, 16_383, 16_385, 65_537, 140_001])
@pytest.mark.parametrize("share", [0.002, 0.02, 0.29, 2.0])
def test_new_ids_of_every_density(rg, orc, n, share, mark_pass, monkeypatch):
    monkeypatch.setenv("RAPIDGNN_MARK_PASS", mark_pass)
    rng = np.random.default_rng(n)
    deg = 20
    indices = np.sort((rng.integers(0, n, size=(n, 1)) + np.arange(deg) * (n // deg) + rng.integers(0, n // deg, size=(n, deg))) % n, axis=1)
    keep = np.concatenate([np.ones((n, 1), bool), np.diff(indices, axis=1) > 0], axis=1)
    indptr = np.zeros(n + 1, np.int64)
    indptr[1:] = np.cumsum(keep.sum(axis=1))
    indices = indices[keep].astype(np.int32)
    batch = max(1, int(n * share / 16))
    train = rng.permutation(n)[: min(n, 3 * batch - 1)].astype(np.int32)
    o = orc.Schedule(indptr, indices, train, batch, [16, 2], 3, 0, 0, n_threads=4)
    s = rg.rg_build_schedule(torch.from_numpy(indptr).cuda(), torch.from_numpy(indices).cuda(), torch.from_numpy(train).cuda(), batch, [16, 2], 3, 0, 0)
    for hop in range(3):
        ids, off = o.frontier(hop)
        gids, _, goff = rg.rg_schedule_frontier(s, hop)
        assert np.array_equal(goff, off) and np.array_equal(gids.cpu().numpy(), ids), hop


@pytest.mark.parametrize("n", [1_048_575, 1_048_577, 1_228_800, 1_228_801, 2_200_000])
@pytest.mark.parametrize("n_train,batch", [(40_000, 40_000), (41_000, 20_480), (300, 20), (360, 20), (180, 20)])
@pytest.mark.parametrize("mark_pass", ["1", "0"])
def test_marks_in_pieces_and_parts(rg, orc, n, n_train, batch, mark_pass, monkeypatch):
    """Bitmaps on both sides of the 1,048,576 IDs from which on they go in two pieces and of the 1,228,800 that fit one, and of three pieces; batches whose samples are marked in several parts, and in one; one,
    two, fifteen, eighteen and nine batches, of which the pass sends whole eights to an XCD each."""
    monkeypatch.setenv("RAPIDGNN_MARK_PASS", mark_pass)
    rng = np.random.default_rng(n + n_train)
    deg = 18
    step = n // deg
    indices = ((np.arange(deg) * step)[None, :] + rng.integers(0, step, size=(n, deg))).astype(np.int32)       # ascending: one ID per stretch
    indptr = np.arange(0, n * deg + 1, deg, dtype=np.int64)
    train = rng.permutation(n)[:n_train].astype(np.int32)
    o = orc.Schedule(indptr, indices.ravel(), train, batch, [16], 3, 0, 0, n_threads=4)
    s = rg.rg_build_schedule(torch.from_numpy(indptr).cuda(), torch.from_numpy(indices.ravel()).cuda(), torch.from_numpy(train).cuda(), batch, [16], 3, 0, 0)
    ids, off = o.frontier(1)
    gids, _, goff = rg.rg_schedule_frontier(s, 1)
    assert np.array_equal(goff, off) and np.array_equal(gids.cpu().numpy(), ids)


@pytest.mark.parametrize("n", [40, 2047, 2048, 2049, 4100])
@pytest.mark.parametrize("beta", [1, 7, 9, 64, 65, 255, 256, 300])
def test_frequencies_from_the_bitmaps(rg, n, beta):
    """The epoch's frequencies as column sums of the batches' bitmaps: batches fewer than the waves that share them out, as many as
    a round takes and more, up to and past what eight planes count; nodes up to, at and past a workgroup's; some nodes in
    every batch (the hubs that every row ends with)."""
    rng = np.random.default_rng(n + beta)
    deg, hubs = min(n // 2, 60), 3
    rows = np.sort(np.stack([np.concatenate([rng.permutation(n - hubs)[:deg], np.arange(n - hubs, n)]) for _ in range(n)]), axis=1).astype(np.int32)
    indptr = torch.arange(0, n * (deg + hubs) + 1, deg + hubs, dtype=torch.int64, device="cuda")
    per_batch = max(1, min(n // beta, 40))
    train = torch.from_numpy(rng.permutation(n)[: per_batch * beta].astype(np.int32)).cuda()
    s = rg.rg_build_schedule(indptr, torch.from_numpy(rows.ravel()).cuda(), train, per_batch, [64, 64], 3, 0, 0)
    ids = rg.rg_schedule_frontier(s, 2)[0].cpu().numpy()
    feat = rg.make_features(torch.zeros(n, dtype=torch.uint8, device="cuda"), torch.arange(n, dtype=torch.int32, device="cuda"),
                            torch.zeros((1, 4), dtype=torch.int32, device="cuda"), torch.zeros((n, 4), dtype=torch.int32, device="cuda"), 16)
    cache = rg.rg_build_cache([s], feat, n // 3)
    assert np.array_equal(rg.rg_cache_view(cache, n)["freq"].cpu().numpy().view(np.uint32), np.bincount(ids, minlength=n).astype(np.uint32))
