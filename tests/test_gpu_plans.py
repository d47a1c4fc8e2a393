"""A cache's plans where batches and the plan kernel's tiles of 2,048 positions meet: batches that begin and end inside a
tile, on its edge, span several, are many to a tile; counts and rows against numpy."""
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


@pytest.mark.parametrize("n_train,batch", [(1, 1), (300, 7), (2047, 2047), (2048, 2048), (2049, 2048), (4096, 64), (6145, 2049), (10_000, 5000), (30_000, 4096)])
@pytest.mark.parametrize("K", [0, 900, 60_000])
def test_counts_and_rows_of_every_batch(rg, n_train, batch, K):
    rng = np.random.default_rng(n_train + K)
    n = 60_000
    d = "cuda"
    indptr, indices = torch.zeros(n + 1, dtype=torch.int64, device=d), torch.zeros(0, dtype=torch.int32, device=d)
    train = torch.from_numpy(rng.permutation(n)[:n_train].astype(np.int32)).to(d)
    scheds = [rg.rg_build_schedule(indptr, indices, train, batch, [], 5, 0, e) for e in (0, 1)]
    is_local = (rng.random(n) < 0.25).astype(np.uint8)
    row_of = np.where(is_local, np.cumsum(is_local) - 1, np.cumsum(1 - is_local) - 1).astype(np.int32)
    table = rng.integers(0, 2**31, size=(n, 4)).astype(np.int32)
    remote = torch.from_numpy(table[is_local == 0]).pin_memory()          # misses are copied by a launch of their own
    feat = rg.make_features(torch.from_numpy(is_local).to(d), torch.from_numpy(row_of).to(d), torch.from_numpy(table[is_local == 1]).to(d), remote, 16)
    cache = rg.rg_build_cache(scheds, feat, K)
    cached = np.zeros(n, bool)
    cached[rg.rg_cache_view(cache, n)["cache_ids"].cpu().numpy()] = True
    for s in scheds:
        ids, _, off = rg.rg_schedule_frontier(s, 0)
        ids = ids.cpu().numpy()
        want = []
        for b in range(s.n_batches):
            v = ids[off[b]:off[b + 1]]
            local, hit = int(is_local[v].sum()), int((cached[v] & (is_local[v] == 0)).sum())
            want.append(dict(n_rows=v.size, n_local=local, n_hit=hit, n_miss=v.size - local - hit))
        out = torch.full((n_train, 4), -7, dtype=torch.int32, device=d)
        assert rg.rg_gather_batches(s, cache, feat, 0, s.n_batches, out) == want
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), table[ids])


@pytest.mark.parametrize("n", [1, 31, 33, 1000, 4096])
@pytest.mark.parametrize("order", ["ranks", "last two swapped", "shuffled", "all local", "all remote"])
@pytest.mark.parametrize("look", ["1", "0"])
def test_rows_whatever_order_the_tables_are_in(rg, n, order, look, monkeypatch):
    """Ten epochs over all nodes whose plans look whether row_of is the ranks the slot map knows -- where it is, where it is
    but for two nodes, and where it is any order -- and plans that do not look."""
    monkeypatch.setenv("RAPIDGNN_ROW_RANKS", look)
    rng = np.random.default_rng(n)
    d = "cuda"
    indptr, indices = torch.zeros(n + 1, dtype=torch.int64, device=d), torch.zeros(0, dtype=torch.int32, device=d)
    scheds = [rg.rg_build_schedule(indptr, indices, torch.arange(n, dtype=torch.int32, device=d), 700, [], 5, 0, e) for e in range(10)]
    is_local = (rng.random(n) < {"all local": 2.0, "all remote": -1.0}.get(order, 0.4)).astype(np.uint8)
    rows = {}
    row_of = np.zeros(n, np.int32)
    for side in (0, 1):
        nodes = np.flatnonzero(is_local == side)
        at = np.arange(nodes.size)
        if order == "shuffled":
            at = rng.permutation(nodes.size)
        elif order == "last two swapped" and side == 0 and nodes.size > 1:
            at[-2:] = at[-2:][::-1]
        row_of[nodes] = at
        t = np.zeros((max(nodes.size, 1), 4), np.int32)
        t[at] = np.stack([nodes, nodes * 3, nodes ^ 5, -nodes], axis=1)
        rows[side] = torch.from_numpy(t).to(d)
    feat = rg.make_features(torch.from_numpy(is_local).to(d), torch.from_numpy(row_of).to(d), rows[1], rows[0], 16)
    cache = rg.rg_build_cache(scheds, feat, n // 5)
    for s in scheds[::4]:
        ids = rg.rg_schedule_frontier(s, 0)[0].cpu().numpy()
        out = torch.full((n, 4), -7, dtype=torch.int32, device=d)
        rg.rg_gather_batches(s, cache, feat, 0, s.n_batches, out)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), np.stack([ids, ids * 3, ids ^ 5, -ids], axis=1))


@pytest.mark.parametrize("codes", ["1", "0"])
@pytest.mark.parametrize("K,at", [(0, None), (50, None), (0, 0), (50, 0), (50, 1), (700, 0), (700, 1)])
@pytest.mark.parametrize("place", ["hbm", "pinned"])
def test_rows_at_the_end_of_what_a_code_holds(rg, codes, K, at, place, monkeypatch):
    """Plans of codes and of entries.  A remote table of one-byte rows, two billion of them: the last row that a code holds beside K
    slots (at = 0) and the first that none does (at = 1) are some node's, in the second epoch's plan alone; batches of one epoch
    are served from its plan whatever the other's is made of.  at = None: every row small."""
    if place == "pinned" and at is not None:
        pytest.skip("two billion rows in HBM alone")
    monkeypatch.setenv("RAPIDGNN_PLAN_CODES", codes)
    n, far_node, d = 5000, 4321, "cuda"
    rng = np.random.default_rng(K)
    indptr, indices = torch.zeros(n + 1, dtype=torch.int64, device=d), torch.zeros(0, dtype=torch.int32, device=d)
    others = np.setdiff1d(np.arange(n), [far_node]).astype(np.int32)
    # the far node is listed in one batch, the others below it in every epoch: it is the last candidate of a tie and never cached
    trains = [others, np.append(others, np.int32(far_node))]
    scheds = [rg.rg_build_schedule(indptr, indices, torch.from_numpy(rng.permutation(t)).to(d), 333, [], 5, 0, e) for e, t in enumerate(trains)]
    is_local = (np.arange(n) % 3 == 0).astype(np.uint8)
    is_local[far_node] = 0
    row_of = np.where(is_local, np.cumsum(is_local) - 1, np.cumsum(1 - is_local) - 1).astype(np.int32)
    value = rng.integers(0, 256, size=n).astype(np.uint8)
    if at is not None:
        row_of[far_node] = 2**31 - 1 - K + at if K or at == 0 else 2**31 - 1
    local = np.zeros(n, np.uint8)
    local[row_of[is_local == 1]] = value[is_local == 1]
    remote = torch.zeros(2**31 if at is not None else n, dtype=torch.uint8, device=d if place == "hbm" else "cpu")
    if place == "pinned":
        remote = remote.pin_memory()
    far = np.flatnonzero(is_local == 0)
    remote[torch.from_numpy(row_of[far].astype(np.int64)).to(remote.device)] = torch.from_numpy(value[far]).to(remote.device)
    feat = rg.make_features(torch.from_numpy(is_local).to(d), torch.from_numpy(row_of).to(d), torch.from_numpy(local).to(d), remote, 1)
    cache = rg.rg_build_cache(scheds, feat, K)
    cached = np.zeros(n, bool)
    cached[rg.rg_cache_view(cache, n)["cache_ids"].cpu().numpy()] = True
    assert cached.sum() == K and not cached[far_node]
    for s in scheds:
        ids, _, off = rg.rg_schedule_frontier(s, 0)
        ids = ids.cpu().numpy()
        want = []
        for b in range(s.n_batches):
            v = ids[off[b]:off[b + 1]]
            loc, hit = int(is_local[v].sum()), int((cached[v] & (is_local[v] == 0)).sum())
            want.append(dict(n_rows=v.size, n_local=loc, n_hit=hit, n_miss=v.size - loc - hit))
        out = torch.zeros((ids.size, 1), dtype=torch.uint8, device=d)
        assert rg.rg_gather_batches(s, cache, feat, 0, s.n_batches, out) == want
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy()[:, 0], value[ids])


@pytest.mark.parametrize("row_bytes", [1, 3, 16, 30, 100, 2408, 4100])
@pytest.mark.parametrize("n,missing", [(1, 1.0), (63, 0.5), (65, 0.0), (5000, 0.01), (5000, 0.5), (40_000, 1.0), (600_000, 0.3)])
def test_misses_of_a_pinned_table(rg, n, missing, row_bytes):
    """The launch that finds a batch's misses and copies them: one row to a wave and many, rows of one piece and of several rounds of a
    wave's pieces, vectors, overlapping last vectors and odd tails; a block per batch and one for all."""
    if n * row_bytes > 64 << 20:
        pytest.skip("wide rows at the smaller counts")
    d = "cuda"
    rng = np.random.default_rng(n + row_bytes)
    indptr, indices = torch.zeros(n + 1, dtype=torch.int64, device=d), torch.zeros(0, dtype=torch.int32, device=d)
    s = rg.rg_build_schedule(indptr, indices, torch.arange(n, dtype=torch.int32, device=d), max(1, n - n // 3), [], 5, 0, 0)
    is_local = (rng.random(n) >= missing).astype(np.uint8)
    row_of = np.where(is_local, np.cumsum(is_local) - 1, np.cumsum(1 - is_local) - 1).astype(np.int32)
    stride = (row_bytes + 15) // 16 * 16 if row_bytes % 4 == 0 else row_bytes
    table = rng.integers(0, 256, size=(n, stride)).astype(np.uint8)
    local = torch.from_numpy(np.concatenate([table[is_local == 1], table[:1]])).to(d)
    remote = torch.from_numpy(np.concatenate([table[is_local == 0], table[:1]])).pin_memory()
    feat = rg.make_features(torch.from_numpy(is_local).to(d), torch.from_numpy(row_of).to(d), local, remote, row_bytes)
    cache = rg.rg_build_cache([s], feat, int(0.2 * n))
    ids, _, off = rg.rg_schedule_frontier(s, 0)
    ids = ids.cpu().numpy()
    side = torch.cuda.Stream()
    for whole in (True, False):
        out = torch.full((n, stride), 7, dtype=torch.uint8, device=d)
        if whole:
            rg.rg_gather_batches(s, cache, feat, 0, s.n_batches, out, side_stream=side)
        else:
            for b in range(s.n_batches):
                rg.rg_gather_batch(s, cache, feat, b, out[off[b]:], out_stride=stride)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        assert np.array_equal(got[:, :row_bytes], table[ids][:, :row_bytes])
        assert (got[:, row_bytes:] == 7).all()


@pytest.mark.parametrize("row_bytes", [255, 257, 1202, 16383, 16384, 16400, 30_002, 100_004, (1 << 20) + 4])
@pytest.mark.parametrize("n,missing", [(1, 1.0), (7, 1.0), (40, 0.5), (600, 0.01)])
def test_few_misses_of_wide_rows(rg, n, missing, row_bytes):
    """Rows whose pieces are shared out among waves: one part and many, widths that the parts do not divide, vectors, overlapping last vectors and odd tails."""
    if n * row_bytes > 64 << 20:
        pytest.skip("wide rows at the smaller counts")
    d = "cuda"
    rng = np.random.default_rng(n + row_bytes)
    indptr, indices = torch.zeros(n + 1, dtype=torch.int64, device=d), torch.zeros(0, dtype=torch.int32, device=d)
    s = rg.rg_build_schedule(indptr, indices, torch.arange(n, dtype=torch.int32, device=d), n, [], 5, 0, 0)
    is_local = np.ones(n, np.uint8)
    is_local[rng.permutation(n)[: max(1, int(n * missing))]] = 0
    row_of = np.where(is_local, np.cumsum(is_local) - 1, np.cumsum(1 - is_local) - 1).astype(np.int32)
    table = rng.integers(0, 256, size=(n, row_bytes + 5)).astype(np.uint8)
    for pad in sorted({0, 4, -row_bytes % 4}):                   # strides of the tables and of the block; the last: vectors whatever the width
        rows = np.ascontiguousarray(table[:, : row_bytes + pad])
        local = torch.from_numpy(np.concatenate([rows[is_local == 1], rows[:1]])).to(d)
        remote = torch.from_numpy(np.concatenate([rows[is_local == 0], rows[:1]])).pin_memory()
        feat = rg.make_features(torch.from_numpy(is_local).to(d), torch.from_numpy(row_of).to(d), local, remote, row_bytes)
        cache = rg.rg_build_cache([s], feat, 0)
        out = torch.full((n, row_bytes + pad), 7, dtype=torch.uint8, device=d)
        rg.rg_gather_batch(s, cache, feat, 0, out, out_stride=row_bytes + pad)
        torch.cuda.synchronize()
        got, ids = out.cpu().numpy(), rg.rg_schedule_frontier(s, 0)[0].cpu().numpy()
        assert np.array_equal(got[:, :row_bytes], rows[ids][:, :row_bytes])
        assert (got[:, row_bytes:] == 7).all()


@pytest.mark.parametrize("n", [1, 15, 16, 1039, 2047, 2048, 2049, 2064, 50_000])
@pytest.mark.parametrize("shift", [0, 1])
def test_candidates_counted_by_the_histogram(rg, n, shift):
    """The byte histogram leaves the candidates of every 2,048 nodes: caches that hold all candidates, one less, and none, with is_local at an aligned address
    and not, and last tiles of one node, of sixteen and of parts of both."""
    d = "cuda"
    rng = np.random.default_rng(n)
    indptr, indices = torch.zeros(n + 1, dtype=torch.int64, device=d), torch.zeros(0, dtype=torch.int32, device=d)
    scheds = [rg.rg_build_schedule(indptr, indices, torch.from_numpy(rng.permutation(n)[: max(1, n * k // 4)].astype(np.int32)).to(d), max(1, n // 5), [], 5, 0, k) for k in (1, 2, 4)]
    is_local = np.zeros(n + shift, np.uint8)
    is_local[shift:] = rng.random(n) < 0.3
    local = torch.from_numpy(is_local).to(d)[shift:]
    feat = rg.make_features(local, torch.arange(n, dtype=torch.int32, device=d), torch.zeros((n, 4), device=d), torch.zeros((n, 4), device=d), 16)
    freq = np.zeros(n, np.int64)
    for s in scheds:
        np.add.at(freq, rg.rg_schedule_frontier(s, 0)[0].cpu().numpy(), 1)
    cand = np.flatnonzero((freq > 0) & (is_local[shift:] == 0))
    for K in sorted({0, max(0, cand.size - 1), cand.size, n + 5}):
        want = np.sort(cand[np.lexsort((cand, -freq[cand]))[:K]])
        assert np.array_equal(rg.rg_cache_view(rg.rg_build_cache(scheds, feat, K), n)["cache_ids"].cpu().numpy(), want)
