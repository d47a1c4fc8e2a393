"""Batches classified on the fly at the sizes where the routing kernel changes shape (waves, tiles of 1,024 rows, the
sixteen counter pairs), against indexing in numpy."""
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


@pytest.mark.parametrize("rows", [1, 63, 64, 65, 255, 257, 1023, 1024, 1025, 16 * 1024 - 1, 16 * 1024 + 1, 40_000])
def test_rows_and_counts_of_batches_of_every_size(rg, rows):
    rng = np.random.default_rng(rows)
    n = 50_000
    d = "cuda"
    indptr, indices = torch.zeros(n + 1, dtype=torch.int64, device=d), torch.zeros(0, dtype=torch.int32, device=d)
    train = torch.from_numpy(rng.permutation(n)[:rows].astype(np.int32)).to(d)
    s = rg.rg_build_schedule(indptr, indices, train, rows, [], 5, 0, 0)            # no hop: the input set is the seeds
    hot = rg.rg_build_schedule(indptr, indices, train[: (rows + 1) // 2], rows, [], 5, 0, 1)
    is_local = (rng.random(n) < 0.3).astype(np.uint8)
    row_of = np.where(is_local, np.cumsum(is_local) - 1, np.cumsum(1 - is_local) - 1).astype(np.int32)
    table = rng.integers(0, 2**31, size=(n, 4)).astype(np.int32)
    feat = rg.make_features(torch.from_numpy(is_local).to(d), torch.from_numpy(row_of).to(d), torch.from_numpy(table[is_local == 1]).to(d),
                            torch.from_numpy(table[is_local == 0]).to(d), 16)
    cache = rg.rg_build_cache([hot], feat, rows)                                    # caches the remote half it was built from, no plan for s
    ids = rg.rg_schedule_frontier(s, 0)[0].cpu().numpy()
    cached = np.zeros(n, bool)
    cached[rg.rg_cache_view(cache, n)["cache_ids"].cpu().numpy()] = True
    want = table[ids]
    for c in (None, cache):
        n_local = int(is_local[ids].sum())
        n_hit = 0 if c is None else int(cached[ids].sum())
        stats = dict(n_rows=rows, n_local=n_local, n_hit=n_hit, n_miss=rows - n_local - n_hit)
        for call in (rg.rg_gather_batch, rg.rg_gather_batch_noalloc):
            for want_stats in (True, False):
                out = torch.full((rows + 1, 4), -7, dtype=torch.int32, device=d)
                st = call(s, c, feat, 0, out, want_stats=want_stats)
                torch.cuda.synchronize()
                assert np.array_equal(out[:rows].cpu().numpy(), want) and bool((out[rows] == -7).all())
                assert st == (stats if want_stats else None)
        assert rg.rg_classify_batch(s, c, feat, 0) == stats
