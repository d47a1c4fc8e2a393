"""Hub rows sampled from the keys' side (key values undone and looked up) against the oracle, which reads the rows: rows
at the shortest length the path takes and below it, fan-outs to the largest it takes and above, first ranges of key values
that hold too few and too many; and where rows go to the tile jobs instead: out of order, without memory for their tables,
too few of them."""
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


def hub_graph(rng, n, hub_deg, shuffled=()):
    """Short rows, three in ten of which point to a hub, and the hubs; rows ascend but for those of the hubs in `shuffled`."""
    hubs = rng.permutation(n)[:len(hub_deg)]
    picks = rng.integers(0, n, size=(n, 4))
    picks[:, 3] = np.where(rng.random(n) < 0.3, hubs[rng.integers(0, len(hubs), size=n)], picks[:, 2])
    picks.sort(axis=1)
    keep = np.concatenate([np.ones((n, 1), bool), np.diff(picks, axis=1) > 0], axis=1)
    keep[hubs] = False
    deg = keep.sum(axis=1)
    deg[hubs] = hub_deg
    indptr = np.zeros(n + 1, np.int64)
    indptr[1:] = np.cumsum(deg)
    indices = np.empty(indptr[-1], np.int32)
    is_hub = np.zeros(n, bool)
    is_hub[hubs] = True
    indices[np.repeat(~is_hub, deg)] = picks[keep]
    for k, (h, d) in enumerate(zip(hubs, hub_deg)):
        row = rng.permutation(n)[:d]
        indices[indptr[h]:indptr[h + 1]] = row if k in shuffled else np.sort(row)
    return indptr, indices, hubs


def check(rg, orc, indptr, indices, train, batch, fanout, allocator=None):
    o = orc.Schedule(indptr, indices, train, batch, fanout, 5, 1, 2, n_threads=8)
    g = rg.rg_build_schedule(torch.from_numpy(indptr).cuda(), torch.from_numpy(indices).cuda(), torch.from_numpy(train).cuda(), batch, fanout, 5, 1, 2,
                             allocator=allocator)
    assert g.n_batches == o.n_batches
    for hop in range(o.L + 1):
        ids, off = o.frontier(hop)
        gids, _, goff = rg.rg_schedule_frontier(g, hop)
        assert np.array_equal(goff, off) and np.array_equal(gids.cpu().numpy(), ids), f"frontier {hop}"
    for hop in range(o.L):
        so, nb = o.samples(hop)
        gso, gnb = rg.rg_schedule_samples(g, hop)
        assert np.array_equal(gso.cpu().numpy(), so) and np.array_equal(gnb.cpu().numpy(), nb), f"samples {hop}"


HUB_DEGREES = [16384, 16385, 20011, 65536, 131073, 199_999, 30_000, 150_000]


@pytest.mark.parametrize("shuffled,mark_pass", [((), "1"), ((), "0"), ((6, 7), "1")])
@pytest.mark.parametrize("fanout", [[1, 1], [12, 4], [60, 20], [200, 3], [448], [449]])
def test_hub_rows_equal_the_oracle(rg, orc, fanout, shuffled, mark_pass, monkeypatch):
    """Every row in order: all from 16,385 IDs on are sampled from the keys' side, and marked by the pass or as they are
    sampled.  Two that are not in order: the hop's rows are read."""
    monkeypatch.setenv("RAPIDGNN_HUB_ROWS", "16385")
    monkeypatch.setenv("RAPIDGNN_MARK_PASS", mark_pass)
    rng = np.random.default_rng(sum(fanout))
    n = 200_000
    indptr, indices, hubs = hub_graph(rng, n, HUB_DEGREES, shuffled)
    train = np.unique(np.concatenate([hubs, rng.permutation(n)[:300]])).astype(np.int32)
    check(rg, orc, indptr, indices, train, 64, fanout)


@pytest.mark.parametrize("first_range", ["0.01", "0.4", "9"])
@pytest.mark.parametrize("fanout", [[5, 2], [200, 3]])
def test_first_ranges_that_hold_too_few_or_too_many(rg, orc, fanout, first_range, monkeypatch):
    """Of the guessed range of key values, a hundredth, less than half and nine times as much: rounds that go on behind what they
    looked through, and (fan-out 200: 245 expected, 1,024 in the list) ones that start again with half of it."""
    monkeypatch.setenv("RAPIDGNN_HUB_ROWS", "16385")
    monkeypatch.setenv("RAPIDGNN_HUB_RANGE", first_range)
    rng = np.random.default_rng(sum(fanout))
    n = 200_000
    indptr, indices, hubs = hub_graph(rng, n, HUB_DEGREES)
    train = np.unique(np.concatenate([hubs, rng.permutation(n)[:300]])).astype(np.int32)
    check(rg, orc, indptr, indices, train, 64, fanout)


def requested_bytes(rg, monkeypatch, *args, hub_rows=None):
    if hub_rows:
        monkeypatch.setenv("RAPIDGNN_HUB_ROWS", hub_rows)
    else:
        monkeypatch.delenv("RAPIDGNN_HUB_ROWS", raising=False)
    a = RecordingAllocator(rg)
    check(rg, *args, allocator=a.struct)
    return a.requested


@pytest.mark.parametrize("sparse", ["0", "1"])
@pytest.mark.parametrize("n_train,worth_it", [(800, False), (64 * 110, True)])
def test_hub_rows_without_being_forced(rg, orc, n_train, worth_it, sparse, monkeypatch):
    """13 batches that share five hub rows make 806 tile jobs of them in a hop, 110 batches 6,820: only those are worth tables
    (24 tile jobs per compute unit, 256 of them), which the device memory asked for shows."""
    monkeypatch.setenv("RAPIDGNN_SPARSE_FRONTIER", sparse)
    rng = np.random.default_rng(11)
    n = 900_000
    indptr, indices, hubs = hub_graph(rng, n, [899_999, 880_000, 700_000, 800_000, 600_000])
    train = rng.permutation(n)[:n_train].astype(np.int32)
    args = (orc, indptr, indices, train, 64, [3, 2, 5])
    by_rule = requested_bytes(rg, monkeypatch, *args)
    never = requested_bytes(rg, monkeypatch, *args, hub_rows="2e9")
    tables = 5 * 32 * n // 8                                  # per hop: five rows, a bucket of 32 bytes per eight IDs
    if worth_it:
        assert by_rule > never + tables
    else:
        assert by_rule < never + tables / 10


def test_hub_rows_without_memory_for_their_tables(rg, orc, monkeypatch):
    monkeypatch.setenv("RAPIDGNN_HUB_ROWS", "16385")
    rng = np.random.default_rng(4)
    n = 200_000
    indptr, indices, hubs = hub_graph(rng, n, [150_000, 199_999, 180_000])
    train = np.unique(np.concatenate([hubs, rng.permutation(n)[:100]])).astype(np.int32)
    a = rg.TorchAllocator(limit_bytes=1 << 20)
    check(rg, orc, indptr, indices, train, 64, [12, 4], allocator=a.struct)
    assert a.n_refused == 2                                  # the tables of either hop, nothing else


@pytest.mark.parametrize("fanout", [[12, 4], [3, 2, 2]])
def test_hub_rows_take_no_memory_that_the_build_needs(rg, orc, fanout, monkeypatch):
    """An allocator with just what the build takes without tables suffices; and where there is more, one hop's tables are
    the most that is ever held."""
    rng = np.random.default_rng(4)
    n = 200_000
    indptr, indices, hubs = hub_graph(rng, n, [150_000, 199_999, 180_000, 190_000])
    train = np.unique(np.concatenate([hubs, rng.permutation(n)[:100]])).astype(np.int32)
    args = (rg, orc, indptr, indices, train, 64, fanout)
    monkeypatch.setenv("RAPIDGNN_HUB_ROWS", "2e9")
    without = RecordingAllocator(rg)
    check(*args, allocator=without.struct)
    monkeypatch.setenv("RAPIDGNN_HUB_ROWS", "16385")
    tight = RecordingAllocator(rg, total_bytes=without.peak)
    check(*args, allocator=tight.struct)
    assert tight.n_refused > 0 and tight.peak <= without.peak
    free = RecordingAllocator(rg)
    check(*args, allocator=free.struct)
    tables = 4 * 32 * n // 8                                 # four rows, a bucket of 32 bytes per eight IDs
    assert tables / 2 < free.peak - without.peak < tables + (1 << 19)
