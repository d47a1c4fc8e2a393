// Computation blocks (Sec. 4 par. (8): the sampled subgraph handed to the trainer).
//
// Block of hop l, batch b: destinations U_l of the batch, sources U_{l+1} of the batch (destination j is
// source j, since U_{l+1} starts with U_l), edges = the hop's samples.  What is computed here is the
// relabelling src_pos[k] = position of samp_nbr[k] in the batch's U_{l+1}; with samp_off it is the
// block's CSR in block-local indices, and the gathered feature block is already in source order.
//
// Method: a position table of n_nodes int32 per batch, filled by scattering j -> table[U_L[j]] and read back once per
// sampled edge.  U_{l+1} is the beginning of U_L, so the one table gives every hop's positions.  Only entries written for
// the same batch are ever read (every sampled ID is in U_L), so the table is never cleared.  Batches are processed
// in groups sized to a workspace limit: with 288 GB of HBM one group usually covers the epoch.
//
// Bound by the scattered reads of the tables.  All workgroups of a batch run on one XCD (workgroup g runs on XCD g mod
// 8), so that a batch's table is in one L2 and not read by all eight, and a thread keeps four edges in flight: 233 k nodes, 147
// batches, 29 M edges: positions and edges 616 us, 302 so.  With up to 128 workgroups per batch instead of 32, so that an XCD is at two
// batches at a time and their tables (0.9 MB each) stay in its 4 MB of L2, and four positions in flight too: 252.
#include "rg_internal.h"

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
    if (s->n_batches > 0) RG_TRY(tmp.dev((uint64_t)group * per_batch, (void **)&table));
    for (uint32_t l = 0; l < s->L; ++l)           // every allocation before the first launch: no early return with kernels in flight
        if (!s->hop[l].src_pos) RG_TRY(s->arena.dev_n<int32_t>((uint64_t)s->hop[l].n_samples, &s->hop[l].src_pos));
    const HopData &all = s->hop[s->L];
    for (uint32_t b_lo = 0; b_lo < s->n_batches && s->L > 0; b_lo += group) {
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
