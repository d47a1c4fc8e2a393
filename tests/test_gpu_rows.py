"""GPU parity of the sampling of rows above 64 IDs at fan-outs up to 64, where a row is streamed against a guessed cut:
row lengths around the blocks' and chunks' ends, row starts at every distance from a 128-byte boundary (and at the start of
the array), first cuts that let through too few, too many and the usual number of candidates -- against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

LENGTHS = [65, 66, 67, 68, 96, 97, 127, 128, 129, 130, 191, 192, 193, 254, 255, 256, 257, 258, 260, 285, 287, 288, 289, 511, 512, 513, 515, 543, 544, 767, 768, 769,
           1023, 1024, 1025, 1056, 1300, 2047, 2049, 4099]


@pytest.fixture(scope="module")
def rg():
    from paper_2509_05207_amd import binding
    binding.lib()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return binding


@pytest.fixture(scope="module")
def graph():
    rng = np.random.default_rng(9)
    n = 4800
    deg = np.where(rng.random(n) < 0.25, rng.integers(0, 65, size=n), rng.choice(LENGTHS, size=n))
    rows = [np.sort(rng.choice(n, size=int(d), replace=False)).astype(np.int32) for d in deg]
    indptr = np.zeros(n + 1, np.int64)
    indptr[1:] = np.cumsum(deg)
    return n, indptr, np.concatenate(rows), rng.permutation(n)[:1500].astype(np.int32)


@pytest.mark.parametrize("shift", [0, 1, 30])
@pytest.mark.parametrize("scale", [None, "0.05", "0.6", "30"])
@pytest.mark.parametrize("fanout", [(1, 2), (5, 16), (17, 32), (33, 48), (63, 64)])
def test_rows_against_a_guessed_cut(rg, orc, graph, fanout, scale, shift, monkeypatch):
    n, indptr, indices, train = graph
    if scale is not None:
        monkeypatch.setenv("RAPIDGNN_GUESS_SCALE", scale)
    o = orc.Schedule(indptr, indices, train, 200, list(fanout), 3, 1, 2, n_threads=8)
    dx = torch.zeros(indices.size + shift, dtype=torch.int32, device="cuda")[shift:]          # rows at every distance from a boundary
    dx.copy_(torch.from_numpy(indices))
    g = rg.rg_build_schedule(torch.from_numpy(indptr).cuda(), dx, torch.from_numpy(train).cuda(), 200, list(fanout), 3, 1, 2)
    for hop in range(o.L + 1):
        ids, off = o.frontier(hop)
        gids, _, goff = rg.rg_schedule_frontier(g, hop)
        assert np.array_equal(goff, off) and np.array_equal(gids.cpu().numpy(), ids), f"frontier {hop}"
    for hop in range(o.L):
        so, nb = o.samples(hop)
        gso, gnb = rg.rg_schedule_samples(g, hop)
        assert np.array_equal(gso.cpu().numpy(), so) and np.array_equal(gnb.cpu().numpy(), nb), f"samples {hop}"


@pytest.mark.parametrize("fanout,scales", [(40, ("0.1", "1", "10")), (64, ("0.6", "1", "1.5", "1.8", "3"))])
def test_tiles_against_other_cuts(rg, orc, fanout, scales, monkeypatch):
    """The pieces of rows above 16,384 IDs, when the first cut misses; lists of one to three candidates per lane and longer ones (the safe
    guess lets 104 through at a fan-out of 64)."""
    rng = np.random.default_rng(10)
    n = 60_000
    deg = np.full(n, 3)
    deg[:6] = [16385, 20000, 40000, 59999, 16384, 30011]
    indptr = np.zeros(n + 1, np.int64)
    indptr[1:] = np.cumsum(deg)
    indices = np.concatenate([np.sort(rng.choice(n, size=int(d), replace=False)).astype(np.int32) for d in deg])
    train = np.arange(40, dtype=np.int32)
    o = orc.Schedule(indptr, indices, train, 10, [fanout], 0, 0, 0, n_threads=8)
    for scale in scales:
        monkeypatch.setenv("RAPIDGNN_GUESS_SCALE", scale)
        g = rg.rg_build_schedule(torch.from_numpy(indptr).cuda(), torch.from_numpy(indices).cuda(), torch.from_numpy(train).cuda(), 10, [fanout], 0, 0, 0)
        assert np.array_equal(rg.rg_schedule_samples(g, 0)[1].cpu().numpy(), o.samples(0)[1]), scale


@pytest.mark.parametrize("more", [0, 1])
@pytest.mark.parametrize("deg", [16_385, 33_000])
def test_pieces_of_few_and_of_many_long_rows(rg, orc, deg, more):
    """A first hop's rows above 16,384 IDs go in small pieces up to six large ones per compute unit, in large ones beyond: on the line and past it."""
    rows = 6 * torch.cuda.get_device_properties(0).multi_processor_count + more
    n, small = 2 * deg, 50
    rng = np.random.default_rng(deg)
    long_rows = 2 * np.arange(deg, dtype=np.int32) + rng.integers(0, 2, size=(rows, deg), dtype=np.int32)
    short_rows = np.sort(rng.integers(0, n // 8, size=(small, 8), dtype=np.int32) + np.arange(8, dtype=np.int32) * (n // 8), axis=1)
    indptr = np.concatenate([np.arange(rows + 1, dtype=np.int64) * deg, rows * deg + 8 * np.arange(1, small + 1), np.full(n - rows - small, rows * deg + 8 * small)])
    indices = np.concatenate([long_rows.ravel(), short_rows.ravel()])
    train = rng.permutation(rows + small).astype(np.int32)
    batch = -(-train.size // 20)
    o = orc.Schedule(indptr, indices, train, batch, [7], 1, 0, 0, n_threads=8)
    s = rg.rg_build_schedule(torch.from_numpy(indptr).cuda(), torch.from_numpy(indices).cuda(), torch.from_numpy(train).cuda(), batch, [7], 1, 0, 0)
    so, nb = o.samples(0)
    gso, gnb = rg.rg_schedule_samples(s, 0)
    assert np.array_equal(gso.cpu().numpy(), so) and np.array_equal(gnb.cpu().numpy(), nb)
    assert np.array_equal(rg.rg_schedule_frontier(s, 1)[0].cpu().numpy(), o.frontier(1)[0])


def test_more_pieces_than_waves_and_few_nodes(rg, orc):
    """A second hop whose frontiers, 20 times the same 400 rows above 16,384 IDs, make more pieces than the chip runs waves (no more than 28
    per compute unit) but no more units of nodes: every wave has a piece, or two, and a unit of its own behind them."""
    n, deg, hubs, seeds = 36_000, 17_500, 400, 600
    rng = np.random.default_rng(2)
    hub_ids = np.sort(rng.choice(n, size=hubs, replace=False)).astype(np.int32)
    train = rng.choice(np.setdiff1d(np.arange(n), hub_ids), size=seeds, replace=False).astype(np.int32)
    degs = rng.integers(0, 30, size=n)
    degs[hub_ids] = deg
    degs[train] = hubs
    indptr = np.concatenate([[0], np.cumsum(degs)]).astype(np.int64)
    is_hub, is_seed = np.zeros(n, bool), np.zeros(n, bool)
    is_hub[hub_ids], is_seed[train] = True, True
    rows = [2 * np.arange(deg) + rng.integers(0, 2, size=deg) if is_hub[v] else hub_ids if is_seed[v] else np.sort(rng.choice(n, size=degs[v], replace=False)) for v in range(n)]
    indices = np.concatenate(rows).astype(np.int32)
    o = orc.Schedule(indptr, indices, train, 30, [60, 9], 1, 0, 0, n_threads=8)
    nodes, off = o.frontier(1)
    waves = 28 * torch.cuda.get_device_properties(0).multi_processor_count
    assert is_hub[nodes].sum() > waves >= nodes.size // 4
    s = rg.rg_build_schedule(torch.from_numpy(indptr).cuda(), torch.from_numpy(indices).cuda(), torch.from_numpy(train).cuda(), 30, [60, 9], 1, 0, 0)
    for hop in range(2):
        so, nb = o.samples(hop)
        gso, gnb = rg.rg_schedule_samples(s, hop)
        assert np.array_equal(gso.cpu().numpy(), so) and np.array_equal(gnb.cpu().numpy(), nb), hop
    assert np.array_equal(rg.rg_schedule_frontier(s, 2)[0].cpu().numpy(), o.frontier(2)[0])


@pytest.mark.parametrize("batch,rest", [(1000, 0), (2000, 0), (2000, 1999), (40_000, 1)])
def test_small_frontiers_of_more_units_than_waves(rg, orc, batch, rest):
    """40,000 nodes of 300 IDs each, in units of four: more units than waves run at once, each wave's by index; in frontier order, and by the batches'
    like places with a last batch of one node."""
    n, deg = 40_000, 300
    rng = np.random.default_rng(4)
    indices = (rng.integers(0, n // deg, size=(n, deg), dtype=np.int32) + np.arange(deg, dtype=np.int32) * (n // deg)).ravel()
    indptr = np.arange(0, n * deg + 1, deg, dtype=np.int64)
    train = rng.permutation(n)[: n - rest].astype(np.int32)
    o = orc.Schedule(indptr, indices, train, batch, [6], 1, 0, 0, n_threads=8)
    s = rg.rg_build_schedule(torch.from_numpy(indptr).cuda(), torch.from_numpy(indices).cuda(), torch.from_numpy(train).cuda(), batch, [6], 1, 0, 0)
    assert np.array_equal(rg.rg_schedule_samples(s, 0)[1].cpu().numpy(), o.samples(0)[1])
    assert np.array_equal(rg.rg_schedule_frontier(s, 1)[0].cpu().numpy(), o.frontier(1)[0])
