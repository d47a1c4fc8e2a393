// Launch shapes that follow from sizes alone.  Nothing of HIP is used here, so that they can be compiled and tested by themselves.
#pragma once
#include <algorithm>
#include <stdint.h>

namespace rg {

// HIP documents that a launch has fewer than 2^32 work-items along x (the runtime this was tested on also ran 2^32 + 512 of them rightly; nothing promises it).
constexpr uint64_t MAX_WORK_ITEMS = 0xFFFFFFFFull;
// Workgroups for n_groups shares of work, for kernels whose workgroups take a further share where there are more shares than workgroups.
inline uint32_t grid_for(int64_t n_groups, uint32_t threads) { return (uint32_t)std::max<int64_t>(1, std::min<int64_t>(n_groups, (int64_t)(MAX_WORK_ITEMS / threads))); }

// ---------------------------------------------------------------- the O(f) sampler (sample_positions_kernel)
constexpr int POS_THREADS = 256;
constexpr int POS_WAVES = POS_THREADS / 64;
constexpr int POS_DRAWS = 256;           // positions of a wave in LDS (the launch of 25 M draws with 64 / 128 / 256 / 384 / 512: 468 / 346 / 292 / 318 / 328 us)
constexpr int POS_LEAST = 64;            // draws per unit, at least, where there are few
struct PositionUnits {
    uint32_t nodes;                      // of a unit
    int64_t n;
    uint32_t grid;
};
// As many draws to a unit as a wave has room for, or as few as give every wave that the chip holds a unit.  by_place: the units of each of beta batches
// are counted as those of the longest (see ByPlace).  A wave per unit: waves that walk over the units by turns drift apart, and with them what they read (292
// us, so 312); only where a launch cannot have that many waves do they.
// scattered: the waves mark their n_samples in maps of 8.4 M IDs and more.  Every mark is then a line of its own, which the launch waits for, and fewer draws to a
// unit pay up to POS_SCATTERED rounds of waves, as long as a unit has POS_SAMPLES of the samples (15 M nodes, rows of 30 IDs, units of 256 / 128 / 64 draws, us: 150,000 nodes of fan-out 16
// 130 / 119 / 115, 30 212 / 198 / 189; 1,000,000 of 4 198 / 187 / 179, of 10 397 / 388 / 388, of 23 871 / 872 / 917; rows of 100, 150,000 of 50 339 / 315 / 309; 60 M nodes, rows of 8 IDs,
// 1,000,000 of 10 440 / 417 / 401, of 50 406 / 403 / 482).
constexpr int64_t POS_SCATTERED = 16, POS_SAMPLES = 32;
inline PositionUnits position_units(int64_t n_cur, int64_t n_samples, uint32_t fanout, bool by_place, int64_t longest, uint32_t beta, int n_cu, bool scattered)
{
    const int64_t waves = (int64_t)n_cu * 32, all = n_cur * (int64_t)fanout;
    const auto nodes_of = [&](int64_t draws) { return std::max<int64_t>(1, std::min<int64_t>(64, draws / fanout)); };
    int64_t draws = POS_DRAWS;
    while (draws > POS_LEAST && (all < draws * waves || (scattered && all < draws * waves * POS_SCATTERED && nodes_of(draws / 2) * n_samples >= POS_SAMPLES * n_cur))) draws /= 2;
    const int64_t nodes = nodes_of(draws);
    const int64_t n = by_place ? (longest + nodes - 1) / nodes * beta : (n_cur + nodes - 1) / nodes;
    return PositionUnits{(uint32_t)nodes, n, grid_for((n + POS_WAVES - 1) / POS_WAVES, POS_THREADS)};
}

// ---------------------------------------------------------------- remote rows out of pinned memory (gather_remote_kernel)
constexpr int CHUNKS_IN_FLIGHT = 8;      // loads a lane has under way (of both gather kernels)
constexpr int64_t LINK_BYTES = 2 << 20;
struct RemoteShape {
    int per_wave;                        // consecutive rows of a wave's round
    int64_t parts;                       // waves to a row (then per_wave is 1)
    int64_t waves;
};
// n_remote of n_rows rows are remote, pieces to a row, vec bytes to a piece.
inline RemoteShape remote_shape(int64_t n_rows, int64_t n_remote, uint64_t pieces, int vec, int n_cu)
{
    // Two pieces a lane, or a single row, fewer rows where that leaves compute units without waves (rows of 2,408 bytes, 1,971 us at one row a wave
    // and the link's rate, 1,979 at 32; a list of the misses 1,974).
    RemoteShape r{1, 1, 0};
    while (r.per_wave < 64 && r.per_wave * pieces < 128 && n_rows / (2 * r.per_wave) >= (int64_t)n_cu * 8) r.per_wave <<= 1;
    // Few misses of wide rows: a row's pieces are shared out among waves, a round of them (8 KB) or more each (8 rows of 1 MB 440 us with a wave a row, 171 so,
    // 181 with a list of the misses; one 352 / 32 / 39; with parts for 512 waves, not 64, 64 rows of 64 KB 104 us for 88).  Where pieces are single bytes a
    // round has little under way, and more waves of two pieces a lane are the better (500 rows of 9,602 bytes, half of them misses, a wave a row / so / a list 189 / 89 / 93 us;
    // 300 of 3,001, misses alone 76 / 45 / 56; 3,000 of 1,202, a tenth 48 / 37 / 43).
    const uint64_t least = vec == 16 ? 64 * CHUNKS_IN_FLIGHT : 128;
    const int64_t busy = vec == 16 ? 64 : (int64_t)n_cu * 64;
    if (r.per_wave == 1)
        while (n_remote * r.parts < busy && pieces >= (uint64_t)r.parts * 2 * least && n_rows * r.parts <= (int64_t)n_cu * 64) r.parts *= 2;
    // Where all rows would be asked for at once the link is at its best with LINK_BYTES on it, so that the more of its pieces a wave has under way, the fewer
    // waves (a list of misses / all waves / so, us: 1,000 rows of 16 KB, misses alone 326 / 346 / 313; 3,000 of 4 KB 250 / 285 / 244, half of them misses 144 / 160 / 137,
    // a fifth 79 / 70 / 71; 30,000 of 400 bytes 312 / 324 / 300; 20,000 of 2,408 930 / 930 / 922). Where pieces are single bytes fewer waves are slower
    // (20,000 rows of 1,202 bytes, half of them misses 381 / 357 / 390); more rows than the chip holds waves take further rounds anyway.
    const int64_t n_units = (n_rows * r.parts + r.per_wave - 1) / r.per_wave, all_waves = (int64_t)n_cu * 128;
    r.waves = std::min(n_units, all_waves);
    if (vec == 16 && n_units <= all_waves) {
        const double under_way = (double)r.per_wave * (double)pieces / (double)r.parts * (double)n_remote / (double)n_rows;
        r.waves = std::min(r.waves, (int64_t)((double)LINK_BYTES / (16.0 * std::min(64.0 * CHUNKS_IN_FLIGHT, std::max(1.0, under_way)))));
    }
    return r;
}

// ---------------------------------------------------------------- computation blocks
// By ranks (block_ranks_kernel) rather than by tables of positions: where the batches are so many that each has few workgroups to make bitmaps for, and where a
// batch has samples enough to pay for clearing and counting them, some 18 us a round of workgroups at 233,000 nodes (edges: samples of all hops and batches).
// By tables / by ranks, us: 233,000 nodes, 147 batches of 199,000 samples 250 / 176, 31,000 95 / 60, 7,700 53 / 42; 500 of 3,400 74 / 58; 2,000 of 1,400 137 / 163,
// of 300 50 / 157; 100 batches of 200,000 179 / 120, 64 123 / 94, 64 of 7,700 35 / 37; 40 of 200,000 86 / 83, 40 of 31,000 42 / 44, 20 of 200,000 62 / 73, one 32 / 64;
// 30,000 nodes, 64 of 6,000 31 / 26.  Two to eight hops on 20,000 to 160,000 nodes, 64 to 700 batches: 0.34 to 1.05 of the tables' time.
// Behind the first round of workgroups a batch costs 17 ns (two hops) to 28 (four), while the tables of small graphs stay in the L2s, so that there the batch
// has to have the more samples the smaller the graph: 1,000 batches, three hops, 8,000 nodes, 1,000 samples 40 / 45, 2,000 48 / 46; 32,000 nodes, 500
// 40 / 44, 1,000 54 / 46; one hop, 16,000 nodes, 320 27 / 31, 640 34 / 33; 4,000 batches, 8,000 nodes, 1,000 samples 89 / 127, 32,000 nodes 161 / 129;
// 500 batches, two hops, 16,000 nodes, 256 26 / 28, 1,100 33 / 29.
constexpr uint64_t RANK_NODE_SAMPLES = 6000000;          // nodes times samples per batch and bitmap, from which on
inline bool blocks_by_ranks(uint64_t n_nodes, uint32_t L, uint64_t beta, uint64_t edges, int n_cu)
{
    const uint64_t cus = (uint64_t)n_cu, nodes_per_edge = beta * 2 >= cus ? 64 : 16;
    if (beta * 4 < cus || edges * nodes_per_edge < n_nodes * beta) return false;
    const uint64_t least = beta <= cus ? 0 : beta <= 2 * cus ? RANK_NODE_SAMPLES / 4 : RANK_NODE_SAMPLES;
    return edges * n_nodes >= least * (L + 1) * beta;
}

}  // namespace rg
