"""Launch shapes computed on the host, compiled by themselves: what a launch may have at most, and that its units cover the work."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_05207_amd", "csrc")
DRIVER = r"""
#include "rg_launch.h"
#include <cstdio>
#include <cstring>
int main()
{
    char what[32];
    long long a[8];
    while (scanf("%31s %lld %lld %lld %lld %lld %lld %lld %lld", what, a, a + 1, a + 2, a + 3, a + 4, a + 5, a + 6, a + 7) == 9) {
        if (!strcmp(what, "positions")) {
            const rg::PositionUnits u = rg::position_units(a[0], a[1], (uint32_t)a[2], a[3] != 0, a[4], (uint32_t)a[5], (int)a[6], a[7] != 0);
            printf("%u %lld %u\n", u.nodes, (long long)u.n, u.grid);
        }
        if (!strcmp(what, "remote")) {
            const rg::RemoteShape r = rg::remote_shape(a[0], a[1], a[2], (int)a[3], (int)a[4]);
            printf("%d %lld %lld\n", r.per_wave, (long long)r.parts, (long long)r.waves);
        }
        if (!strcmp(what, "ranks")) printf("%d\n", rg::blocks_by_ranks(a[0], (uint32_t)a[1], a[2], a[3], (int)a[4]) ? 1 : 0);
    }
}
"""


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    d = tmp_path_factory.mktemp("shapes")
    (d / "driver.cpp").write_text(DRIVER)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, "-o", str(d / "driver"), str(d / "driver.cpp")])

    def ask(what, *args):
        line = " ".join([what] + [str(int(x)) for x in args] + ["0"] * (8 - len(args)))
        return [int(x) for x in subprocess.run([str(d / "driver")], input=line + "\n", capture_output=True, text=True, check=True).stdout.split()]
    return ask


@pytest.mark.parametrize("fanout", [1, 3, 25, 50, 64, 85, 86, 128, 129, 256, 1984])
@pytest.mark.parametrize("scattered", [False, True])
@pytest.mark.parametrize("n_cur", [1, 64, 40_000, 2**26, 2**27 + 1, 2**30 - 1, 2**31 - 1, 80 * 10**9])
@pytest.mark.parametrize("beta", [0, 1, 147, 65_535])
def test_units_of_the_position_sampler(shapes, n_cur, fanout, beta, scattered):
    """beta > 0: batches of equal length by place, which frontiers of up to 2^30 nodes go by."""
    if beta and n_cur >= 2**30:
        pytest.skip("by position")
    longest = -(-n_cur // max(beta, 1))
    nodes, n_units, grid = shapes("positions", n_cur, n_cur * min(fanout, 40), fanout, beta > 0, longest, beta, 256, scattered)
    assert 1 <= nodes <= 64 and (nodes == 1 or nodes * fanout <= 256)
    assert n_units == (-(-longest // nodes) * beta if beta else -(-n_cur // nodes))
    assert 1 <= grid and grid * 256 < 2**32                      # what a launch may have
    assert grid * 4 >= min(n_units, 2**26 - 4)                   # a wave per unit, as far as that goes


@pytest.mark.parametrize("n_cur,row,fanout,scattered,nodes", [
    # measured, us with 64 / 128 / 256 draws to a unit
    (3_700_000, 500, 10, False, 25),     # 468 / 346 / 292, the walks
    (150_000, 30, 16, True, 4),          # 115 / 119 / 130, marks all over a map of 15 M IDs
    (150_000, 30, 30, True, 2),          # 189 / 198 / 212
    (150_000, 100, 50, True, 1),         # 309 / 315 / 339
    (1_000_000, 30, 4, True, 16),        # 179 / 187 / 198
    (1_000_000, 30, 23, True, 5),        # 917 / 872 / 871
    (1_000_000, 8, 10, True, 6),         # 401 / 417 / 440
    (1_000_000, 8, 50, True, 5),         # 482 / 403 / 406
])
def test_units_by_what_bounds_them(shapes, n_cur, row, fanout, scattered, nodes):
    assert shapes("positions", n_cur, n_cur * min(row, fanout), fanout, 0, 0, 0, 256, scattered)[0] == nodes


@pytest.mark.parametrize("n,hops,batches,per_batch,by_ranks", [
    # measured, us by tables / by ranks
    (233_000, 2, 147, 199_000, True),       # 250 / 176
    (233_000, 2, 2_000, 1_400, False),      # 137 / 163
    (233_000, 2, 1, 199_000, False),        # 32 / 64
    (160_000, 3, 700, 3_750, True),         # 111 / 81
    (80_000, 8, 64, 613_000, True),         # 273 / 201
    (64_000, 4, 4_000, 2_000, True),        # 460 / 169
    (32_000, 3, 1_000, 500, False),         # 40 / 44
    (32_000, 3, 1_000, 1_000, True),        # 54 / 46
    (20_000, 1, 700, 320, False),           # 25 / 30
    (20_000, 3, 700, 1_860, True),          # 51 / 44
    (16_000, 2, 500, 256, False),           # 26 / 28
    (16_000, 2, 500, 1_114, True),          # 33 / 29
    (16_000, 3, 1_000, 552, False),         # 41 / 49
    (8_000, 3, 4_000, 1_003, False),        # 89 / 127
    (4_000, 2, 1_000, 140, False),          # 27 / 36
    (4_000, 3, 1_000, 138, False),          # 30 / 42
])
def test_blocks_by_ranks_where_they_are_faster(shapes, n, hops, batches, per_batch, by_ranks):
    assert shapes("ranks", n, hops, batches, batches * per_batch, 256) == [int(by_ranks)]


@pytest.mark.parametrize("rows,misses,row_bytes,vec,least,most", [
    # waves; measured, us with 256 / 512 to 1,024 / all of them, a wave to 64 rows and fewer
    (1_000, 1_000, 16_384, 16, 256, 256),            # 315 / - / 346
    (3_000, 3_000, 4_096, 16, 400, 700),             # 240 / 244 / 285
    (3_000, 600, 4_096, 16, 2_000, 3_000),           # a fifth: 79 / - / 70
    (30_000, 30_000, 400, 16, 500, 1_000),           # 294 / 300 / 324
    (20_000, 20_000, 1_202, 1, 20_000, 20_000),      # 1,643 / - / 641
    (20_000, 10_000, 1_202, 1, 20_000, 20_000),      # 1,045 / - / 357
    (2_000, 2_000, 16, 16, 2_000, 2_000),            # 38 / - / 24
    (5_000, 5_000, 17, 1, 1_250, 5_000),             # 48 / - / 32
    (8, 8, 1 << 20, 16, 64, 64),                     # shared out in parts: 440 / - / 171
    (500, 250, 9_602, 1, 16_000, 32_000),            # so too, a wave a row 189, so 89
    (300, 300, 3_001, 1, 2_400, 4_800),              # 76, so 45
    (3_000, 300, 1_202, 1, 12_000, 24_000),          # 48, so 37
    (100, 100, 255, 1, 100, 100),
    (100_000, 100_000, 2_408, 16, 32_768, 32_768),
])
def test_waves_that_ask_the_link(shapes, rows, misses, row_bytes, vec, least, most):
    pieces = -(-row_bytes // vec)
    per_wave, parts, waves = shapes("remote", rows, misses, pieces, vec, 256)
    assert least <= waves <= most


@pytest.mark.parametrize("rows", [1, 7, 64, 2_047, 4_096, 100_000, 2**31 - 1])
@pytest.mark.parametrize("pieces", [1, 2, 63, 64, 128, 1_024, 65_537, 2**28, 2**32 - 1])
@pytest.mark.parametrize("one_in", [1, 2, 30])
@pytest.mark.parametrize("vec", [1, 16])
def test_remote_rows_have_waves(shapes, rows, pieces, one_in, vec):
    per_wave, parts, waves = shapes("remote", rows, max(1, rows // one_in), pieces, vec, 256)
    assert 1 <= per_wave <= 64 and parts >= 1 and (per_wave == 1 or parts == 1)
    assert 1 <= waves <= 32_768
    assert rows * parts < 2**40                                  # the kernel counts units in 64 bits
    if parts > 1:
        assert pieces // parts >= (512 if vec == 16 else 128)    # of a part
