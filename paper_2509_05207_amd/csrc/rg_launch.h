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
inline PositionUnits position_units(int64_t n_cur, uint32_t fanout, bool by_place, int64_t longest, uint32_t beta, int n_cu)
{
    const int64_t waves = (int64_t)n_cu * 32;
    int64_t draws = POS_DRAWS;
    while (draws > POS_LEAST && n_cur * fanout < draws * waves) draws /= 2;
    const int64_t nodes = std::max<int64_t>(1, std::min<int64_t>(64, draws / fanout));
    const int64_t n = by_place ? (longest + nodes - 1) / nodes * beta : (n_cur + nodes - 1) / nodes;
    return PositionUnits{(uint32_t)nodes, n, grid_for((n + POS_WAVES - 1) / POS_WAVES, POS_THREADS)};
}

}  // namespace rg
