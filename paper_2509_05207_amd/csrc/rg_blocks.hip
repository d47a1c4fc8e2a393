// Computation blocks (Sec. 4 par. (8): the sampled subgraph handed to the trainer).
//
// Block of hop l, batch b: destinations U_l of the batch, sources U_{l+1} of the batch (destination j is
// source j, since U_{l+1} starts with U_l), edges = the hop's samples.  What is computed here is the
// relabelling src_pos[k] = position of samp_nbr[k] in the batch's U_{l+1}; with samp_off it is the
// block's CSR in block-local indices, and the gathered feature block is already in source order.
//
// Method, in small graphs with many batches: ranks in bitmaps (block_ranks_kernel).  Elsewhere a position table of n_nodes int32 per batch, filled by scattering j -> table[U_L[j]] and read back once per
// sampled edge.  U_{l+1} is the beginning of U_L, so the one table gives every hop's positions.  Only entries written for
// the same batch are ever read (every sampled ID is in U_L), so the table is never cleared.  Batches are processed
// in groups sized to a workspace limit: with 288 GB of HBM one group usually covers the epoch.
//
// The tables are bound by their scattered reads.  All workgroups of a batch run on one XCD (workgroup g runs on XCD g mod
// 8), so that a batch's table is in one L2 and not read by all eight, and a thread keeps four edges in flight: 233 k nodes, 147
// batches, 29 M edges: positions and edges 616 us, 302 so.  With up to 128 workgroups per batch instead of 32, so that an XCD is at two
// batches at a time and their tables (0.9 MB each) stay in its 4 MB of L2, and four positions in flight too: 252.
#include "rg_internal.h"
#include "rg_launch.h"

#include <algorithm>

namespace rg {

constexpr int BLK_THREADS = 256;
constexpr int BLK_PER_BATCH = 128;      // workgroups per batch at most; each walks its share with a stride
constexpr int BLK_IN_FLIGHT = 4;
constexpr int BLK_XCDS = 8;

// Workgroup g's batch within a group of batches, and its number among the batch's workgroups: batches go round the XCDs.
__device__ __forceinline__ uint32_t batch_of_workgroup(uint32_t g, uint32_t per_batch, uint32_t *part)
{
    const uint32_t r = g / BLK_XCDS;
    *part = r % per_batch;
    return r / per_batch * BLK_XCDS + g % BLK_XCDS;
}
static unsigned workgroups_for(uint32_t n_batches, uint32_t per_batch) { return (n_batches + BLK_XCDS - 1) / BLK_XCDS * BLK_XCDS * per_batch; }
// Workgroups of a batch, of nb that a launch holds: one round of its threads for an average batch's entries, up to half of what
// an XCD holds, so that two batches' tables are in its L2 and not eight.  A launch of few batches (the workspace holds nine tables of
// 111 M nodes) or of small ones would leave the chip idle with that, and there each access is a wait for memory: as many as fill
// the chip, down to one entry per thread.  Positions and edges of an epoch, 32 workgroups for every batch / by the entries alone / so: 111 M nodes, 147
// batches 529 / 541 / 525 us, 30 M nodes 340 / 333 / 322, 2.45 M nodes, 196 batches 3,927 / 2,980 / 2,944, 1 M nodes 1,097 / 850 / 843,
// 233,000 nodes 292 / 260 / 252, 60,000 nodes, 18 small batches 23 / 23 / 22.
static uint32_t workgroups_per_batch(int64_t n, uint32_t beta, uint32_t nb, int n_cu)
{
    const int64_t each = n / beta, round = each / (BLK_THREADS * BLK_IN_FLIGHT) + 1, most = each / BLK_THREADS + 1;
    const int64_t fill = (int64_t)n_cu * (2048 / BLK_THREADS) / ((nb + BLK_XCDS - 1) / BLK_XCDS * BLK_XCDS);
    return (uint32_t)std::min<int64_t>(std::max(round, std::min(most, fill)), BLK_PER_BATCH);
}

// table[k][U_{L,b}[j]] = j for batch b = b_lo + k
__global__ void __launch_bounds__(BLK_THREADS) block_positions_kernel(const int32_t *__restrict__ ids, const int64_t *__restrict__ off, uint32_t b_lo, uint32_t n_batches,
                                                                      uint32_t per_batch, int64_t n_nodes, int32_t *__restrict__ table)
{
    uint32_t part;
    const uint32_t k = batch_of_workgroup(blockIdx.x, per_batch, &part);
    if (k >= n_batches) return;
    const int64_t u0 = off[b_lo + k], n = off[b_lo + k + 1] - u0;
    int32_t *t = table + (uint64_t)k * (uint64_t)n_nodes;
    const int64_t step = (int64_t)per_batch * BLK_THREADS;
    for (int64_t j0 = (int64_t)part * BLK_THREADS + threadIdx.x; j0 < n; j0 += BLK_IN_FLIGHT * step) {
        uint32_t v[BLK_IN_FLIGHT];
#pragma unroll
        for (int q = 0; q < BLK_IN_FLIGHT; ++q) v[q] = j0 + q * step < n ? (uint32_t)ids[u0 + j0 + q * step] : 0xFFFFFFFFu;
#pragma unroll
        for (int q = 0; q < BLK_IN_FLIGHT; ++q)
            if (v[q] < (uint64_t)n_nodes) t[v[q]] = (int32_t)(j0 + q * step);
    }
}

// src_pos[e] = table[k][samp_nbr[e]] for the samples of batch b = b_lo + k
__global__ void __launch_bounds__(BLK_THREADS) block_relabel_kernel(const int32_t *__restrict__ samp_nbr, const int64_t *__restrict__ samp_off,
                                                                    const int64_t *__restrict__ off, uint32_t b_lo, uint32_t n_batches, uint32_t per_batch, int64_t n_nodes,
                                                                    const int32_t *__restrict__ table, int32_t *__restrict__ src_pos)
{
    uint32_t part;
    const uint32_t k = batch_of_workgroup(blockIdx.x, per_batch, &part);
    if (k >= n_batches) return;
    const int64_t first = samp_off[off[b_lo + k]], end = samp_off[off[b_lo + k + 1]];
    const int32_t *t = table + (uint64_t)k * (uint64_t)n_nodes;
    const int64_t step = (int64_t)per_batch * BLK_THREADS;
    for (int64_t e0 = first + (int64_t)part * BLK_THREADS + threadIdx.x; e0 < end; e0 += BLK_IN_FLIGHT * step) {
        uint32_t u[BLK_IN_FLIGHT];
        int32_t p[BLK_IN_FLIGHT];
#pragma unroll
        for (int q = 0; q < BLK_IN_FLIGHT; ++q) u[q] = e0 + q * step < end ? (uint32_t)samp_nbr[e0 + q * step] : 0xFFFFFFFFu;
#pragma unroll
        for (int q = 0; q < BLK_IN_FLIGHT; ++q) p[q] = u[q] < (uint64_t)n_nodes ? t[u[q]] : -1;
#pragma unroll
        for (int q = 0; q < BLK_IN_FLIGHT; ++q)
            if (e0 + q * step < end) __builtin_nontemporal_store(p[q], src_pos + e0 + q * step);
    }
}

// ---------------------------------------------------------------- positions without a table
// U_L of a batch is its seeds and then, hop by hop, the hop's new IDs in ascending order.  So the position of an ID that was new at
// some hop is where that hop's begin plus its rank among them, and of a seed what a list says that is indexed by its rank among the seeds:
// a bitmap per hop, and the number of bits in front of every other word, which fit LDS where the graph is small.  A workgroup makes them
// from a batch's U_L and relabels the batch's samples of all hops, or a part of them.
//
// Bound by its scattered reads of LDS, five a sample.  (233,000 nodes, 147 batches, 29 M edges: by tables in the L2s 250 us, so 176.)
constexpr int RANK_BLOCK = 1024;
constexpr size_t RANK_LDS = 150 * 1024;
struct RankArgs {
    const int32_t *ids;                              // U_L, batches concatenated
    const int64_t *off[RG_MAX_HOPS + 1];             // the batches' ends in U_0 .. U_L
    const int32_t *samp_nbr[RG_MAX_HOPS];
    const int64_t *samp_off[RG_MAX_HOPS];
    int32_t *src_pos[RG_MAX_HOPS];
    int64_t n_nodes;
    uint32_t L, n_batches, n_words;                  // words of a bitmap, an even number
};
static size_t rank_lds_bytes(uint32_t L, uint64_t n_words, uint64_t most_seeds) { return ((uint64_t)(L + 1) * (n_words + n_words / 2) + most_seeds) * sizeof(uint32_t); }

__global__ void __launch_bounds__(RANK_BLOCK) block_ranks_kernel(RankArgs a, uint32_t parts)
{
    extern __shared__ __align__(16) uint32_t lds[];      // (read in pairs; whatever stands in front of it)
    __shared__ uint32_t ends[RG_MAX_HOPS + 1];       // where hop h's IDs end in the batch's U_L
    __shared__ uint32_t wave_sum[RANK_BLOCK / 64];
    const uint32_t n_sets = a.L + 1, n_words = a.n_words, n_pairs = n_words / 2;
    uint32_t *bits = lds, *in_front = bits + n_sets * n_words, *seed_at = in_front + n_sets * n_pairs;
    const uint32_t b = blockIdx.x % a.n_batches, part = blockIdx.x / a.n_batches;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (uint32_t w = threadIdx.x; w < n_sets * n_words; w += RANK_BLOCK) bits[w] = 0u;
    if (threadIdx.x < n_sets) ends[threadIdx.x] = (uint32_t)(a.off[threadIdx.x][b + 1] - a.off[threadIdx.x][b]);
    __syncthreads();
    const int32_t *ids = a.ids + a.off[a.L][b];
    const uint32_t n = ends[a.L];
    for (uint32_t j0 = threadIdx.x; j0 < n; j0 += BLK_IN_FLIGHT * RANK_BLOCK) {
        uint32_t v[BLK_IN_FLIGHT];
#pragma unroll
        for (int q = 0; q < BLK_IN_FLIGHT; ++q) v[q] = (uint32_t)ids[min(j0 + q * RANK_BLOCK, n - 1)];      // (past the end: the last one again, not used)
#pragma unroll
        for (int q = 0; q < BLK_IN_FLIGHT; ++q) {
            const uint32_t j = j0 + q * RANK_BLOCK;
            if (j >= n || v[q] >= (uint64_t)a.n_nodes) continue;
            uint32_t set = 0;
            for (uint32_t h = 0; h < a.L; ++h) set += j >= ends[h] ? 1u : 0u;
            atomicOr(&bits[set * n_words + (v[q] >> 5)], 1u << (v[q] & 31));
        }
    }
    __syncthreads();
    const uint32_t each = (n_pairs + RANK_BLOCK - 1) / RANK_BLOCK, p0 = min(threadIdx.x * each, n_pairs), p1 = min(p0 + each, n_pairs);
    for (uint32_t s = 0; s < n_sets; ++s) {
        const uint2 *pair = reinterpret_cast<const uint2 *>(bits + s * n_words);
        uint32_t mine = 0;
        for (uint32_t p = p0; p < p1; ++p) mine += __popc(pair[p].x) + __popc(pair[p].y);
        uint32_t incl = mine;
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t y = __shfl_up(incl, d, 64);
            if (lane >= d) incl += y;
        }
        __syncthreads();                             // the last set's sums have been read
        if (lane == 63) wave_sum[wave] = incl;
        __syncthreads();
        uint32_t run = incl - mine;
        for (int w = 0; w < wave; ++w) run += wave_sum[w];
        for (uint32_t p = p0; p < p1; ++p) {
            in_front[s * n_pairs + p] = run;
            run += __popc(pair[p].x) + __popc(pair[p].y);
        }
    }
    __syncthreads();
    // u's rank among the IDs of set s, which it is one of; word: its word of the set's bitmap
    auto rank = [&](uint32_t s, uint32_t u, uint32_t word) {
        const uint32_t w = u >> 5;
        const uint32_t left = bits[s * n_words + (w & ~1u)];                        // the pair's first word: its own, or the one in front of it
        return in_front[s * n_pairs + (w >> 1)] + __popc(word & ((1u << (u & 31)) - 1u)) + ((w & 1u) ? __popc(left) : 0);
    };
    for (uint32_t j = threadIdx.x; j < ends[0]; j += RANK_BLOCK) {
        const uint32_t v = (uint32_t)ids[j];
        if (v < (uint64_t)a.n_nodes) seed_at[rank(0, v, bits[v >> 5])] = j;
    }
    __syncthreads();
    for (uint32_t l = 0; l < a.L; ++l) {
        const int64_t first = a.samp_off[l][a.off[l][b]], m = a.samp_off[l][a.off[l][b + 1]] - first;
        const int64_t lo = first + m * part / parts, hi = first + m * (part + 1) / parts;
        for (int64_t e0 = lo + threadIdx.x; e0 < hi; e0 += BLK_IN_FLIGHT * RANK_BLOCK) {
            uint32_t u[BLK_IN_FLIGHT], word[BLK_IN_FLIGHT], set[BLK_IN_FLIGHT], at[BLK_IN_FLIGHT];
#pragma unroll
            for (int q = 0; q < BLK_IN_FLIGHT; ++q) {
                u[q] = (uint32_t)a.samp_nbr[l][min(e0 + q * RANK_BLOCK, hi - 1)];
                word[q] = 0u; set[q] = 0u; at[q] = 0u;
            }
            for (uint32_t s = 0; s < l + 2; ++s) {
                const uint32_t begin = s ? ends[s - 1] : 0u;
#pragma unroll
                for (int q = 0; q < BLK_IN_FLIGHT; ++q) {
                    const uint32_t x = u[q] < (uint64_t)a.n_nodes ? bits[s * n_words + (u[q] >> 5)] : 0u;
                    if ((x >> (u[q] & 31)) & 1u) { word[q] = x; set[q] = s; at[q] = begin; }
                }
            }
#pragma unroll
            for (int q = 0; q < BLK_IN_FLIGHT; ++q) {
                const int64_t e = e0 + q * RANK_BLOCK;
                if (e >= hi) continue;
                int32_t p = -1;                      // (of an ID that the batch does not list, which only a file may have)
                if (word[q] != 0u) {
                    const uint32_t r = rank(set[q], u[q], word[q]);
                    p = (int32_t)(set[q] == 0u ? seed_at[r] : at[q] + r);
                } else if (u[q] < (uint64_t)a.n_nodes)
                    for (uint32_t s = l + 2; s < n_sets; ++s) {      // (only a file's samples may lie in what a later hop adds)
                        const uint32_t x = bits[s * n_words + (u[q] >> 5)];
                        if ((x >> (u[q] & 31)) & 1u) p = (int32_t)(ends[s - 1] + rank(s, u[q], x));
                    }
                __builtin_nontemporal_store(p, a.src_pos[l] + e);
            }
        }
    }
}

// By ranks where they fit LDS and where that is the faster (see blocks_by_ranks).
static bool ranks_pay(const rg_schedule *s, uint64_t n_words, int n_cu, size_t *lds_bytes)
{
    uint64_t most_seeds = 0, edges = 0;
    const std::vector<int64_t> &off = s->hop[0].off_host;
    for (uint32_t b = 0; b < s->n_batches; ++b) most_seeds = std::max<uint64_t>(most_seeds, (uint64_t)(off[b + 1] - off[b]));
    for (uint32_t l = 0; l < s->L; ++l) edges += (uint64_t)s->hop[l].n_samples;
    *lds_bytes = rank_lds_bytes(s->L, n_words, most_seeds);
    if (*lds_bytes > RANK_LDS) return false;
    if (const char *force = getenv("RAPIDGNN_BLOCK_RANKS")) return force[0] == '1';      // same results either way; for tests and tuning
    return blocks_by_ranks((uint64_t)s->n_nodes, s->L, s->n_batches, edges, n_cu);
}

}  // namespace rg

using namespace rg;

extern "C" {

rg_status rg_schedule_build_blocks(rg_schedule *s, uint64_t workspace_limit_bytes, void *stream)
{
    if (!s) { set_error("rg_schedule_build_blocks: null schedule"); return RG_EINVAL; }
    if (s->blocks_built) return RG_OK;
    hipStream_t st = as_stream(stream);
    const uint64_t per_batch = (uint64_t)std::max<int64_t>(s->n_nodes, 1) * sizeof(int32_t);
    if (workspace_limit_bytes == 0) workspace_limit_bytes = (uint64_t)4 << 30;
    const uint32_t group = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(s->n_batches, workspace_limit_bytes / per_batch));
    int dev = 0, n_cu = 0;
    RG_HIP(hipGetDevice(&dev));
    RG_HIP(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
    Arena tmp(s->arena.allocator(), st);     // scratch from the allocator the schedule was built with
    int32_t *table = nullptr;
    const uint64_t n_words = ((uint64_t)s->n_nodes + 63) / 64 * 2;
    size_t lds_bytes = 0;
    const bool by_ranks = s->n_batches > 0 && s->L > 0 && s->ids_ascend && ranks_pay(s, n_words, n_cu, &lds_bytes);
    if (s->n_batches > 0 && !by_ranks) RG_TRY(tmp.dev((uint64_t)group * per_batch, (void **)&table));
    for (uint32_t l = 0; l < s->L; ++l)           // every allocation before the first launch: no early return with kernels in flight
        if (!s->hop[l].src_pos) RG_TRY(s->arena.dev_n<int32_t>((uint64_t)s->hop[l].n_samples, &s->hop[l].src_pos));
    const HopData &all = s->hop[s->L];
    if (by_ranks) {
        RankArgs a{};
        a.ids = all.ids; a.n_nodes = s->n_nodes; a.L = s->L; a.n_batches = s->n_batches; a.n_words = (uint32_t)n_words;
        for (uint32_t l = 0; l <= s->L; ++l) a.off[l] = s->hop[l].off_dev;
        for (uint32_t l = 0; l < s->L; ++l) { a.samp_nbr[l] = s->hop[l].samp_nbr; a.samp_off[l] = s->hop[l].samp_off; a.src_pos[l] = s->hop[l].src_pos; }
        const uint32_t parts = std::max<uint32_t>(1, (uint32_t)n_cu / s->n_batches);      // few batches: their samples shared out, each part with bitmaps of its own
        ScopedTimer tm(KG_BLOCKS, st);
        RG_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(block_ranks_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)RANK_LDS));
        hipLaunchKernelGGL(block_ranks_kernel, dim3(s->n_batches * parts), dim3(RANK_BLOCK), lds_bytes, st, a, parts);
    }
    for (uint32_t b_lo = 0; b_lo < s->n_batches && s->L > 0 && !by_ranks; b_lo += group) {
        const uint32_t nb = std::min(group, s->n_batches - b_lo);
        ScopedTimer tm(KG_BLOCKS, st);
        const uint32_t per_batch = workgroups_per_batch(all.off_host[s->n_batches], s->n_batches, nb, n_cu);
        hipLaunchKernelGGL(block_positions_kernel, dim3(workgroups_for(nb, per_batch)), dim3(BLK_THREADS), 0, st, all.ids, all.off_dev, b_lo, nb, per_batch, s->n_nodes, table);
        for (uint32_t l = 0; l < s->L; ++l) {
            const HopData &h = s->hop[l];
            const uint32_t per_batch = workgroups_per_batch(h.n_samples, s->n_batches, nb, n_cu);
            if (h.n_samples > 0)
                hipLaunchKernelGGL(block_relabel_kernel, dim3(workgroups_for(nb, per_batch)), dim3(BLK_THREADS), 0, st, h.samp_nbr, h.samp_off, h.off_dev, b_lo, nb, per_batch,
                                   s->n_nodes, table, h.src_pos);
        }
    }
    RG_HIP(hipGetLastError());
    RG_HIP(hipStreamSynchronize(st));            // the table is released below
    tmp.drained();
    s->blocks_built = true;
    return RG_OK;
}

rg_status rg_schedule_block(const rg_schedule *s, uint32_t hop, const int32_t **src_pos_dev)
{
    if (!s) { set_error("rg_schedule_block: null schedule"); return RG_EINVAL; }
    if (hop >= s->L) { set_error("rg_schedule_block: hop %u >= L = %u", hop, s->L); return RG_ERANGE; }
    if (!s->blocks_built) { set_error("rg_schedule_block: call rg_schedule_build_blocks first"); return RG_EINVAL; }
    if (src_pos_dev) *src_pos_dev = s->hop[hop].src_pos;
    return RG_OK;
}

}  // extern "C"
