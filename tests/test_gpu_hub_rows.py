"""Hub rows sampled from the keys' side (key values undone and looked up) against the oracle, which reads the rows: rows
at the shortest length the path takes and below it, fan-outs to the largest it takes and above, rows that are not in
order, and a graph where the path is taken without being forced."""
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


@pytest.mark.parametrize("fanout", [[1, 1], [12, 4], [60, 20], [200, 3], [448], [449]])
def test_hub_rows_equal_the_oracle(rg, orc, fanout, monkeypatch):
    monkeypatch.setenv("RAPIDGNN_HUB_ROWS", "16385")
    rng = np.random.default_rng(sum(fanout))
    n = 200_000
    indptr, indices, hubs = hub_graph(rng, n, [16384, 16385, 20011, 65536, 131073, 199_999, 30_000, 150_000], shuffled=(6, 7))
    train = np.unique(np.concatenate([hubs, rng.permutation(n)[:300]])).astype(np.int32)
    check(rg, orc, indptr, indices, train, 64, fanout)


@pytest.mark.parametrize("sparse", ["0", "1"])
def test_hub_rows_without_being_forced(rg, orc, sparse, monkeypatch):
    monkeypatch.setenv("RAPIDGNN_SPARSE_FRONTIER", sparse)
    rng = np.random.default_rng(11)
    n = 900_000
    indptr, indices, hubs = hub_graph(rng, n, [899_999, 880_000, 300_000, 500_000, 600_000])
    train = rng.permutation(n)[:800].astype(np.int32)
    check(rg, orc, indptr, indices, train, 64, [3, 2, 5])


def test_hub_rows_without_memory_for_their_tables(rg, orc, monkeypatch):
    monkeypatch.setenv("RAPIDGNN_HUB_ROWS", "16385")
    rng = np.random.default_rng(4)
    n = 200_000
    indptr, indices, hubs = hub_graph(rng, n, [150_000, 199_999, 180_000])
    train = np.unique(np.concatenate([hubs, rng.permutation(n)[:100]])).astype(np.int32)
    a = rg.TorchAllocator(limit_bytes=1 << 20)
    check(rg, orc, indptr, indices, train, 64, [12, 4], allocator=a.struct)
    assert a.n_refused == 2                                  # the tables of either hop, nothing else
