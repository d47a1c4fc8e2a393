"""rg_graph_validate's count against a count row by row in numpy: sizes around the vectors, waves and tiles of the flat
pass, indices at every 4-byte phase, IDs and rows damaged in every way the check names."""
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


def count_row_by_row(indptr, indices):
    n, bad = indptr.size - 1, 0
    for v in range(n):
        b, e = int(indptr[v]), int(indptr[v + 1])
        if e < b or (v == 0 and b != 0):
            bad += 1
            continue
        for j in range(b, e):
            u = int(indices[j])
            if u < 0 or u >= n or (j > b and indices[j - 1] >= u):
                bad += 1
    return bad


def check(rg, indptr, indices, phase):
    pad = torch.zeros(indices.size + phase, dtype=torch.int32, device="cuda")
    pad[phase:] = torch.from_numpy(indices).cuda()
    assert rg.rg_graph_validate(torch.from_numpy(indptr).cuda(), pad[phase:]) == count_row_by_row(indptr, indices)


@pytest.mark.parametrize("edges", [0, 1, 3, 4, 5, 7, 255, 256, 257, 1023, 1025, 4099, 20_011])
@pytest.mark.parametrize("phase", [0, 1, 2, 3])
def test_violations_are_counted_at_every_size_and_phase(rg, edges, phase):
    rng = np.random.default_rng(7 * edges + phase)
    n = 500
    cuts = np.sort(rng.integers(0, edges + 1, size=n - 1))
    indptr = np.concatenate([[0], cuts, [edges]]).astype(np.int64)                 # empty rows among them
    rows = [np.sort(rng.choice(n, size=int(d), replace=d > n)) for d in np.diff(indptr)]
    indices = np.concatenate(rows).astype(np.int32) if edges else np.zeros(0, np.int32)
    check(rg, indptr, indices, phase)
    if edges:
        hit = rng.integers(0, edges, size=1 + edges // 50)
        indices[hit] = rng.choice(np.array([-1, n, n + 5, 0, n - 1, -2**31, 2**31 - 1], np.int64), size=hit.size).astype(np.int32)
        check(rg, indptr, indices, phase)


@pytest.mark.parametrize("n", [3000, 16_384, 16_385])
def test_rows_out_of_order_are_counted_row_by_row(rg, n):
    """Up to 16 workgroups of four rows per compute unit (256 of them) the rows are counted behind the first look at indptr
    without a word from the host, beyond on its request."""
    rng = np.random.default_rng(3)
    deg = 8
    indptr = np.arange(0, deg * n + 1, deg).astype(np.int64)
    indices = np.sort(rng.integers(0, n, size=(n, deg)), axis=1).astype(np.int32).ravel()
    for damage in ({5: 5 * deg - 11}, {0: 3}, {n // 2: 0, 17: 19 * deg}, {n: 0}):
        bad = indptr.copy()
        for k, x in damage.items():
            bad[k] = x
        check(rg, bad, indices, 0)


@pytest.mark.parametrize("edges", [2_100_003, 34_000_001])
@pytest.mark.parametrize("rows", [40, 300_000])
def test_violations_over_many_waves(rg, edges, rows):
    """Waves of one round of 1,024 IDs and of several; rows that span many waves (a row, or empty ones, beginning on the edges
    between two) and rows that are many to a round; damage at the starts of rows, where it may be none, and inside."""
    rng = np.random.default_rng(edges + rows)
    indptr = np.sort(np.concatenate([[0, 0, edges], [edges // 3] * 200, rng.integers(0, edges + 1, size=rows), np.arange(1, edges, edges // 64 // 1024 * 1024), np.arange(1, edges, edges // 64 // 1024 * 1024)])).astype(np.int64)
    n = indptr.size - 1
    first = np.zeros(edges + 1, bool)
    first[indptr[:-1]] = True
    first = first[:edges]
    at = np.arange(edges)
    indices = ((at - np.maximum.accumulate(np.where(first, at, 0))) % n).astype(np.int32)      # falls back to 0 within rows of more than n IDs too
    hit = rng.integers(0, edges, size=1000)
    indices[hit] = rng.choice(np.array([-1, n, 0, n - 1, 2**31 - 1]), size=hit.size)
    bad = (indices < 0) | (indices >= n)
    bad[1:] |= ~first[1:] & (indices[:-1] >= indices[1:])
    pad = torch.zeros(edges + 3, dtype=torch.int32, device="cuda")
    pad[3:] = torch.from_numpy(indices).cuda()
    assert rg.rg_graph_validate(torch.from_numpy(indptr).cuda(), pad[3:]) == int(bad.sum())


@pytest.mark.parametrize("light", ["one each", "one in 64", "one in 64, elsewhere", "none", "six each", "sixteen each", "every third block", "mixed"])
@pytest.mark.parametrize("heavy_first", [True, False])
def test_violations_where_few_rows_hold_most_ids(rg, light, heavy_first):
    """Graphs whose rows hold 16 IDs and more on average, most of them in a few rows: blocks of 64 rows with few IDs together, in runs of
    every kind, next to blocks with many; repeated IDs on the starts of rows, where they are no fault, and behind them, where they are."""
    rng = np.random.default_rng(len(light))
    rows, heavy = 400_000, 24
    deg = {"one each": lambda: np.ones(rows, np.int64),
           "one in 64": lambda: (np.arange(rows) % 64 == 0).astype(np.int64),
           "one in 64, elsewhere": lambda: (np.arange(rows) % 64 == 37).astype(np.int64) * rng.integers(1, 40, size=rows),
           "none": lambda: np.zeros(rows, np.int64),
           "six each": lambda: np.full(rows, 6) - (rng.random(rows) < 0.008),                   # blocks of 384 IDs and of fewer
           "sixteen each": lambda: np.full(rows, 16),
           "every third block": lambda: np.where(np.arange(rows) // 64 % 3 == 0, 60, 1),
           "mixed": lambda: np.repeat(rng.choice([0, 1, 5, 6, 7, 16, 200], size=rows // 500), 500)}[light]()
    big = np.full(heavy, 800_001)
    deg = np.concatenate([big, deg] if heavy_first else [deg[: rows // 2], big[::2], deg[rows // 2:], big[1::2]])
    indptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    n, edges = indptr.size - 1, int(indptr[-1])
    assert edges >= 16 * n and edges >= 1 << 24
    first = np.zeros(edges + 1, bool)
    first[indptr[:-1]] = True
    first = first[:edges]
    at = np.arange(edges)
    indices = ((at - np.maximum.accumulate(np.where(first, at, 0))) % n).astype(np.int32)
    hit = rng.integers(0, edges, size=5000)
    indices[hit] = rng.choice(np.array([-1, n, 0, n - 1, 2**31 - 1]), size=hit.size)
    bad = (indices < 0) | (indices >= n)
    bad[1:] |= ~first[1:] & (indices[:-1] >= indices[1:])
    for phase in (0, 3):
        pad = torch.zeros(edges + phase, dtype=torch.int32, device="cuda")
        pad[phase:] = torch.from_numpy(indices).cuda()
        assert rg.rg_graph_validate(torch.from_numpy(indptr).cuda(), pad[phase:]) == int(bad.sum())
