// a3: per-hop fan-out sampling, SAMPLE(eta(v), f) for every frontier node of
// every batch of the epoch in one launch (Sec. 2.1 node-wise sampling; Sec. 4
// par. (2)).
//
// SAMPLE keeps the f neighbours with the smallest keys key32(S_v, u) and emits
// them in row order.  One wavefront works on one row at a time (or one tile of
// a long row), one wave per workgroup.
//
// A first, thread-per-node kernel writes one record per frontier node (row
// start, degree, batch, node state S_v, sample size, tile count), so that the
// sampling waves never chase frontier -> indptr -> row or search for a node's
// batch: a wave takes 64 consecutive frontier nodes, loads their records with
// one coalesced load each, and walks them with lane broadcasts, the next
// node's first 64 neighbour IDs already in flight while the current node is
// sampled.
//
// Fan-outs up to 64 (sample_rows_kernel):
//
//  - rows of up to 64 IDs: four at a time, sixteen lanes each (sample_short_rows).
//  - longer rows are streamed once against a cut guessed from the key distribution, what passes is listed in LDS in row
//    order, and the f smallest keys of that list are the sample.
//
// Larger fan-outs (sample_kernel), and the concatenated results of a long row's tiles (sample_merge_kernel):
//
//  - deg <= f: the row is the sample; it is copied.
//  - deg <= 256: the row sits in registers (1 or 4 IDs per lane).  A threshold
//    that exactly f keys do not exceed is found by bisection on ballots, and the
//    kept IDs are compacted straight into the output with ballot/popcount
//    ranks, which preserves row order.
//  - longer rows are streamed once in 1 KB blocks aligned to cache lines, one
//    16-byte load per lane, the next block's load already in flight.  IDs whose
//    key is not above the current cut are appended (ballot ranks again, so in
//    row order) to an LDS buffer of CAP >= f + 64 IDs; when the buffer would
//    overflow it is pruned to the f smallest keys with the same search and an
//    in-place ordered compaction, which also tightens the cut.  What is left
//    after the last block is the sample.
//
// At any fan-out:
//
//  - rows longer than BIG_ROW are cut into T near-equal tiles, each sampled by
//    its own wave into scratch (f IDs per tile, row order); a second small
//    launch samples the concatenation of a row's tile results, which is the
//    row's sample: the f smallest keys of the row are among the f smallest of
//    each tile.  This bounds the work of one wave whatever the degree skew.
//    Tiles are dealt out by workgroup index and done before the groups of
//    nodes, which the waves then take from a counter as they become free (small
//    frontiers at fan-outs up to 64: by index too).
//  - the very longest rows, where a hop holds many of them, are not read but
//    sampled from the keys' side (hub_sample_kernel).
//
// No step sorts anything.  What a batch has reached is marked in its bitmap by
// a pass over the samples (mark_pass_kernel) where they are many and dense in
// the bitmaps, else by the sampling waves as they write them.
#include "rg_internal.h"
#include "rg_device.h"
#include "rg_launch.h"

#include <algorithm>
#include <atomic>
#include <climits>
#include <cmath>
#include <cstdlib>

namespace rg {


constexpr int TINY_ROW = 8;              // rows of up to this many IDs that need no sampling are copied by one lane each
constexpr int BIG_ROW = 16384;           // rows longer than this are sampled tile by tile ...
constexpr int TILE_PIECE = 65536;        // ... in near-equal pieces of at most this many IDs.  (A row of 16,385 to 65,536 IDs is one tile: it is
                                         // sampled among the tile jobs, where the batches that share it meet in the caches.  Measured on the five
                                         // workloads: pieces of 16,384 cost 8 % more sampling time on the largest graph, pieces of 131,072 7 %;
                                         // tiling from 8,192 IDs on is 3 % slower there and 3 % faster on large_sparse.)
// Where a hop's long rows are too few to fill the chip, a piece is what its launch waits for, at one memory latency per kilobyte: pieces of
// SMALL_PIECE there, that is where pieces of TILE_PIECE are no more than FEW_TILES per compute unit.  More of them fill it as they are, and four times as
// many no longer fit into the waves that run at once.  Sampling of one hop's rows in pieces of 16,384 / of 65,536, by how many rows, each one piece of the
// larger: rows of 60,000 IDs, fan-out 10 500 30 / 50 us, 1,000 50 / 58, 1,500 90 / 96, 2,000 123 / 109, 3,000 165 / 149, 8,000 407 / 383; fan-out 60
// 1,000 54 / 60, 2,000 128 / 116; rows of 34,000, fan-out 25 1,000 35 / 38, 2,000 62 / 57; rows of 20,000, fan-out 10 1,000 26 / 28, 2,000 40 / 35.
constexpr int SMALL_PIECE = 16384;
constexpr int FEW_TILES = 6;
__device__ __host__ __forceinline__ int64_t tiles_of(int64_t deg, int64_t piece) { return deg > BIG_ROW ? (deg + piece - 1) / piece : 0; }

// Per frontier node, by position: where its row starts, its degree, its batch and its stream.
struct NodeRecs {
    int64_t *row_begin;
    int32_t *deg;
    uint32_t *batch;
    uint64_t *state;      // S_v = combine(combine(S_{e,i}, hop + 1), v)
};

// ---------------------------------------------------------------- hub rows: found by node_records_kernel
// The longest rows may be sampled without being read (see hub_sample_kernel): each distinct one gets an entry in a small
// hash table keyed by node, and the frontier positions that hold one are flagged in their count word.  Whether they become
// jobs of that kernel or tile jobs like every other long row is decided by the host once it knows how many there are.
constexpr int HUB_SLOTS = 4096;                 // distinct hub rows; a row that finds no place is sampled in tiles
constexpr int HUB_PROBES = 64;
constexpr uint32_t HUB_MAX_FANOUT = 448;
struct HubRow {
    int64_t begin;
    unsigned long long first;                   // its first bucket
    int32_t deg;
    int32_t shift;                              // bucket of ID u: u >> shift
};
struct HubJob { int64_t i; int32_t slot; int32_t pad; };
struct HubCounts { unsigned long long buckets; uint32_t n_rows, n_jobs, damaged, pad; };       // damaged: a row that is not strictly ascending inside [0, n_nodes), for which its table does not hold
// A bucket: the IDs of 2^shift consecutive ones that the row holds, as their low bits, in order; HUB_EMPTY behind them.  A
// bucket that is full may have had no room for all.
constexpr int HUB_BUCKET = 16;
constexpr uint32_t HUB_EMPTY = 0xFFFFu;
constexpr int HUB_MAX_SHIFT = 15;               // low bits stay below HUB_EMPTY
struct alignas(32) HubBucket { uint16_t id[HUB_BUCKET]; };
struct HubTable {
    int32_t min_deg;                            // rows from this length on; INT32_MAX: none
    HubCounts *counts;                          // clear on entry, as are the keys
    uint32_t *keys;                             // [HUB_SLOTS]: node + 1, 0 = free
    HubRow *rows;                               // [HUB_SLOTS]
    int32_t *list;                              // [HUB_SLOTS]: the slots in use
};
__device__ __forceinline__ uint32_t first_hub_slot(uint32_t v)
{
    static_assert(HUB_SLOTS == 1 << 12, "twelve bits of hash");
    return (v * 0x9E3779B1u) >> 20;
}
// Gives node v's row an entry, if it has none yet; false: no place left.
__device__ __forceinline__ bool add_hub_row(const HubTable &h, uint32_t v, int64_t begin, int64_t deg, int64_t n_nodes)
{
    uint32_t slot = first_hub_slot(v);
    for (int t = 0; t < HUB_PROBES; ++t) {
        uint32_t have = h.keys[slot];
        if (have == 0u) {
            have = atomicCAS(&h.keys[slot], 0u, v + 1u);
            if (have == 0u) {                   // this thread's: the row is described once
                int32_t shift = 0;
                while (shift < HUB_MAX_SHIFT && (n_nodes >> shift) > deg / 4) ++shift;         // 4 to 8 IDs per bucket on average
                const int64_t buckets = ((n_nodes - 1) >> shift) + 1;
                h.rows[slot] = HubRow{begin, atomicAdd(&h.counts->buckets, (unsigned long long)buckets), (int32_t)deg, shift};
                h.list[atomicAdd(&h.counts->n_rows, 1u)] = (int32_t)slot;
                return true;
            }
        }
        if (have == v + 1u) return true;
        slot = (slot + 1) & (HUB_SLOTS - 1);
    }
    return false;
}

// A frontier's new IDs ascend, so the like places of all batches hold about the same nodes: taken one after the other (unit u:
// round u / n_batches of batch u mod n_batches), what they read of a graph that many batches cover is still in the caches.
// Small batches would leave many units unfilled, batches of very different sizes leave many empty, and where the frontiers together
// have less than half as many entries as the graph has nodes there is little to share: those go by frontier position (n_batches = 0).
// By position / by place: 233,000 nodes, 147 batches of 80,000, fan-out 10: the sampling launches 3.06 / 2.84 ms; 2.45 M nodes, 196 of 110,000, 7.17 / 6.94, and the
// records of its nodes (random 128-byte lines of indptr) 448 / 308 us; 147 of 14,000, records 82 / 52 us; 111 M nodes, 147 of 5,800, 1.45 / 1.49 ms.
// The positions sampler alike: 233,000 nodes, 147 batches of 25,000, fan-out 10, 649 / 535 us; 2.45 M nodes, 196 of 170,000, fan-out 5, 1,956 / 1,465; 15 M nodes, 147 of
// 16,000 1,075 / 1,501; but rows that are copied whole (2.45 M nodes, 196 of 51,000, fan-out 50 of 50 IDs) 2,007 / 2,353.
struct ByPlace {
    const int64_t *batch_off;                   // dev
    uint32_t n_batches;
    int64_t longest;                            // nodes of the largest batch
};
constexpr int PLACE_NODES = 1024;               // nodes per batch, on average, from which on
static ByPlace by_place(const HopData &cur, uint32_t beta, int64_t n_nodes)
{
    ByPlace p{cur.off_dev, beta, 0};
    for (uint32_t b = 0; b < beta; ++b) p.longest = std::max(p.longest, cur.off_host[b + 1] - cur.off_host[b]);
    const int64_t n = cur.off_host[beta];
    if (n < (int64_t)beta * PLACE_NODES || 2 * n < n_nodes || p.longest * beta > 2 * n || n >= (int64_t)1 << 30) p.n_batches = 0;
    return p;
}

// Also adds up, over the frontier, what the hop will read of the adjacency: [0] the sum of the degrees (in IDs),
// [1] the part of it in rows of up to BIG_ROW IDs (the rows that are not sampled as tiles), [2] the number of rows of
// 1 .. SHORT_ROW IDs and [3] the IDs in them; of flagged hub rows, [4] how many and [5] how many tiles they make, or, where none are looked
// for, [4] how many tiles all rows make in pieces of TILE_PIECE.  The sums (the first five where no hub rows are looked for) are spread over DEG_SUM_SLOTS sets of counters, total[number of
// sums * slot + k], which the host adds up: thousands of workgroups adding to one address would queue up behind each other.
constexpr int DEG_SUM_SLOTS = 64;
constexpr int DEG_SUMS = 6;
constexpr int SHORT_ROW = 64;            // rows of up to this many IDs are sampled four at a time, sixteen lanes each

// Bound by its bytes (a random 16-byte read of indptr and 28 bytes written per node), so a workgroup takes NODE_CHUNK
// consecutive positions, whose batch and hop stream it looks up once, and a thread has four nodes' reads in flight.
// How many IDs each node will sample, how many tile jobs its row makes and whether it is a hub row go into one word,
// count[i] = samples | tiles << 12 | hub << 31, and the chunk's sums of samples and tiles into chunk_sum (tiles in the
// upper half; those of hub rows apart, into chunk_hub): two prefix sums over the nodes become one scan of the chunks and
// one pass (24.8 M nodes of an epoch's three hops, with their prefix sums: 980 us as two separate scans, 600 so).
// HUBS: rows from hubs.min_deg on are looked for (an instantiation of its own, with two sums more).
constexpr int NODE_THREADS = 256;
constexpr int NODE_PER_THREAD = 4;
constexpr int NODE_CHUNK = NODE_THREADS * NODE_PER_THREAD;
constexpr uint32_t COUNT_BITS = 12;      // samples: at most RG_MAX_FANOUT; tiles: at most 2^31 / SMALL_PIECE = 2^17
constexpr uint32_t HUB_FLAG = 1u << 31;
static_assert(RG_MAX_FANOUT < (1u << COUNT_BITS) && (((uint64_t)1 << 31) / SMALL_PIECE) < (1u << (31 - COUNT_BITS)), "");
__device__ __forceinline__ uint32_t samples_of(uint32_t count) { return count & ((1u << COUNT_BITS) - 1u); }
// The tile jobs of a node's row among those of the rows asked for.
enum { TILES_OF_ROWS = 1, TILES_OF_HUB_ROWS = 2 };
__device__ __forceinline__ uint32_t tiles_in(uint32_t count, int which)
{
    return (which & ((count & HUB_FLAG) ? TILES_OF_HUB_ROWS : TILES_OF_ROWS)) ? (count & ~HUB_FLAG) >> COUNT_BITS : 0u;
}

template <bool HUBS>
__global__ void __launch_bounds__(NODE_THREADS) node_records_kernel(const int64_t *__restrict__ indptr, const int32_t *__restrict__ frontier, int64_t n,
                                                                    const int64_t *__restrict__ batch_off, uint32_t n_batches, const uint64_t *__restrict__ batch_seed,
                                                                    uint32_t hop, uint32_t fanout, int64_t tile_piece, NodeRecs r, uint32_t *__restrict__ count,
                                                                    unsigned long long *__restrict__ chunk_sum, uint32_t *__restrict__ chunk_hub /* HUBS */, int64_t n_nodes,
                                                                    unsigned long long *__restrict__ total, HubTable hubs, int by_place)
{
    // by_place: the workgroup's chunk is one of those that begin in batch (blockIdx mod n_batches), see ByPlace
    int64_t chunk = blockIdx.x;
    if (by_place) {
        const uint32_t round = blockIdx.x / n_batches, b = blockIdx.x - round * n_batches;
        chunk = batch_off[b] / NODE_CHUNK + round;
        if (chunk >= (b + 1 < n_batches ? batch_off[b + 1] / NODE_CHUNK : (n + NODE_CHUNK - 1) / NODE_CHUNK)) return;
    }
    constexpr int SUMS = HUBS ? DEG_SUMS : DEG_SUMS - 1;
    __shared__ unsigned long long part[SUMS + 1][NODE_THREADS / 64];
    unsigned long long acc[SUMS + 1] = {};       // see above; and the chunk's sums
    const int64_t base = chunk * NODE_CHUNK;
    int32_t v[NODE_PER_THREAD];
    int64_t b0[NODE_PER_THREAD], deg[NODE_PER_THREAD];
#pragma unroll
    for (int k = 0; k < NODE_PER_THREAD; ++k) {
        const int64_t i = base + k * NODE_THREADS + threadIdx.x;
        v[k] = i < n ? frontier[i] : -1;
    }
#pragma unroll
    for (int k = 0; k < NODE_PER_THREAD; ++k) {
        const bool known = v[k] >= 0 && (int64_t)v[k] < n_nodes;      // (a seed out of range is refused by the host at the hop's readback; until then it has no row)
        b0[k] = known ? indptr[v[k]] : 0;
        deg[k] = known ? indptr[v[k] + 1] : 0;
    }
    const uint32_t b_first = batch_of(batch_off, n_batches, base);
    const int64_t first_end = batch_off[b_first + 1];
    const uint64_t first_stream = combine(batch_seed[b_first], (uint64_t)hop + 1u);
#pragma unroll
    for (int k = 0; k < NODE_PER_THREAD; ++k) {
        const int64_t i = base + k * NODE_THREADS + threadIdx.x;
        if (i >= n) continue;
        const int64_t d = deg[k] > b0[k] ? deg[k] - b0[k] : 0;
        uint32_t b = b_first;
        uint64_t stream = first_stream;
        if (i >= first_end) {
            b = batch_of(batch_off, n_batches, i);
            stream = combine(batch_seed[b], (uint64_t)hop + 1u);
        }
        r.row_begin[i] = b0[k];
        r.deg[i] = (int32_t)d;
        r.batch[i] = b;
        r.state[i] = combine(stream, (uint64_t)(uint32_t)v[k]);
        const uint32_t samples = (uint32_t)(d < (int64_t)fanout ? d : (int64_t)fanout);
        const uint32_t tiles = (uint32_t)tiles_of(d, tile_piece);
        const bool hub = HUBS && d >= hubs.min_deg && add_hub_row(hubs, (uint32_t)v[k], b0[k], d, n_nodes);
        count[i] = samples | tiles << COUNT_BITS | (hub ? HUB_FLAG : 0u);
        acc[0] += (unsigned long long)d;
        if (d <= (int64_t)BIG_ROW) acc[1] += (unsigned long long)d;
        if (d > 0 && d <= (int64_t)SHORT_ROW) { acc[2] += 1; acc[3] += (unsigned long long)d; }
        if (HUBS && hub) { acc[4] += 1; acc[5 % SUMS] += tiles; }
        if (!HUBS) acc[4] += (unsigned long long)tiles_of(d, TILE_PIECE);
        acc[SUMS] += (unsigned long long)samples | (unsigned long long)(hub ? 0u : tiles) << 32;
    }
#pragma unroll
    for (int k = 0; k <= SUMS; ++k) {
        for (int o = 32; o > 0; o >>= 1) acc[k] += __shfl_down(acc[k], o, 64);
        if ((threadIdx.x & 63) == 0) part[k][threadIdx.x >> 6] = acc[k];
    }
    __syncthreads();
    if (threadIdx.x <= SUMS) {
        const unsigned long long a = part[threadIdx.x][0] + part[threadIdx.x][1] + part[threadIdx.x][2] + part[threadIdx.x][3];
        if (HUBS && threadIdx.x == 5) chunk_hub[chunk] = (uint32_t)a;
        if (threadIdx.x == SUMS) chunk_sum[chunk] = a;
        else if (a) atomicAdd(total + SUMS * (blockIdx.x % DEG_SUM_SLOTS) + threadIdx.x, a);
    }
}

// One workgroup: chunk_sum -> exclusive prefix sums of both halves, samples and tiles in front of each chunk, with the
// totals behind the last; the total of the samples also to *samp_end.  chunk_hub (or NULL): tiles that count with the others.
constexpr int CHUNK_SCAN_THREADS = 1024;
constexpr int CHUNK_SCAN_PER_THREAD = 8;
__global__ void __launch_bounds__(CHUNK_SCAN_THREADS) scan_chunks_kernel(const unsigned long long *__restrict__ chunk_sum, const uint32_t *__restrict__ chunk_hub, int64_t n_chunks,
                                                                         int64_t *__restrict__ samp_base, int64_t *__restrict__ tile_base, int64_t *__restrict__ samp_end)
{
    __shared__ int64_t wave_sum[2][CHUNK_SCAN_THREADS / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t carry[2] = {0, 0};
    for (int64_t c0 = 0; c0 < n_chunks; c0 += CHUNK_SCAN_THREADS * CHUNK_SCAN_PER_THREAD) {
        const int64_t first = c0 + (int64_t)threadIdx.x * CHUNK_SCAN_PER_THREAD;
        unsigned long long x[CHUNK_SCAN_PER_THREAD];
        int64_t mine[2] = {0, 0};
#pragma unroll
        for (int k = 0; k < CHUNK_SCAN_PER_THREAD; ++k) x[k] = first + k < n_chunks ? chunk_sum[first + k] + (chunk_hub ? (unsigned long long)chunk_hub[first + k] << 32 : 0ull) : 0ull;
#pragma unroll
        for (int k = 0; k < CHUNK_SCAN_PER_THREAD; ++k) { mine[0] += (int64_t)(uint32_t)x[k]; mine[1] += (int64_t)(x[k] >> 32); }
        int64_t run[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            int64_t incl = mine[h];
            for (int d = 1; d < 64; d <<= 1) {
                const int64_t y = __shfl_up(incl, d, 64);
                if (lane >= d) incl += y;
            }
            if (lane == 63) wave_sum[h][wave] = incl;
            run[h] = carry[h] + incl - mine[h];
        }
        __syncthreads();
#pragma unroll
        for (int h = 0; h < 2; ++h)
            for (int w = 0; w < CHUNK_SCAN_THREADS / 64; ++w) {
                if (w < wave) run[h] += wave_sum[h][w];
                carry[h] += wave_sum[h][w];
            }
        __syncthreads();                                         // before the next round's sums
#pragma unroll
        for (int k = 0; k < CHUNK_SCAN_PER_THREAD; ++k) {
            if (first + k < n_chunks) { samp_base[first + k] = run[0]; tile_base[first + k] = run[1]; }
            run[0] += (int64_t)(uint32_t)x[k];
            run[1] += (int64_t)(x[k] >> 32);
        }
    }
    if (threadIdx.x == 0) { samp_base[n_chunks] = carry[0]; tile_base[n_chunks] = carry[1]; *samp_end = carry[0]; }
}

// A chunk's exclusive prefix sum of x, one value per thread (the sums of a chunk fit 32 bits).
__device__ __forceinline__ uint32_t chunk_exclusive_scan(uint32_t x)
{
    __shared__ uint32_t wave_sum[NODE_THREADS / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl = x;
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(incl, d, 64);
        if (lane >= d) incl += y;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    for (int w = 0; w < wave; ++w) incl += wave_sum[w];
    return incl - x;
}

__device__ __forceinline__ void load_counts(const uint32_t *__restrict__ count, int64_t first, int64_t n, uint32_t (&c)[NODE_PER_THREAD])
{
    static_assert(NODE_PER_THREAD == 4, "one 16-byte load");
    if (first + 4 <= n) {
        const uint4 x = *reinterpret_cast<const uint4 *>(count + first);
        c[0] = x.x; c[1] = x.y; c[2] = x.z; c[3] = x.w;
        return;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) c[k] = first + k < n ? count[first + k] : 0u;
}

// samp_off[i] for the nodes of a chunk; a thread takes four consecutive ones.
__global__ void __launch_bounds__(NODE_THREADS) sample_offsets_kernel(const uint32_t *__restrict__ count, int64_t n, const int64_t *__restrict__ samp_base,
                                                                      int64_t *__restrict__ samp_off)
{
    const int64_t first = (int64_t)blockIdx.x * NODE_CHUNK + (int64_t)threadIdx.x * NODE_PER_THREAD;
    uint32_t c[NODE_PER_THREAD];
    load_counts(count, first, n, c);
    const uint32_t s0 = samples_of(c[0]), s1 = s0 + samples_of(c[1]), s2 = s1 + samples_of(c[2]), s3 = s2 + samples_of(c[3]);
    const int64_t at = samp_base[blockIdx.x] + (int64_t)chunk_exclusive_scan(s3);
    if (first + 4 <= n) {
        *reinterpret_cast<longlong2 *>(samp_off + first) = make_longlong2(at, at + s0);
        *reinterpret_cast<longlong2 *>(samp_off + first + 2) = make_longlong2(at + s1, at + s2);
    } else {
        if (first < n) samp_off[first] = at;
        if (first + 1 < n) samp_off[first + 1] = at + s0;
        if (first + 2 < n) samp_off[first + 2] = at + s1;
    }
}

// Number of set bits of m below this lane's bit (m wave-uniform): the two mbcnt instructions.
__device__ __forceinline__ int lanes_below(unsigned long long m, int lane)
{
    (void)lane;
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// This lane's bit of a wave-uniform mask, as a condition the vector unit takes straight from the scalar pair.
__device__ __forceinline__ bool my_bit(unsigned long long m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// The lane mask of a predicate, taken straight from the compare.
__device__ __forceinline__ unsigned long long ballot64(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// Values that are the same in every lane of the wave, pinned to scalar registers so that the
// branches and loops they steer are scalar too.
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ uint32_t uni(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
__device__ __forceinline__ bool uni(bool x) { return __builtin_amdgcn_readfirstlane((int)x) != 0; }

__device__ __forceinline__ int64_t bcast64(int64_t x, int src_lane)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, src_lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)x >> 32), src_lane);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// The lanes 0 .. n-1 (n clamped to [0, 64]) as a mask.
__device__ __forceinline__ unsigned long long low_lanes(int n)
{
    return n >= 64 ? ~0ull : (n <= 0 ? 0ull : (1ull << n) - 1ull);
}

// Lane masks instead of per-lane booleans: a mask is one compare (ballot of a single comparison)
// and everything after it -- AND with the valid lanes, population counts, comparisons with f --
// is scalar work that the vector unit never sees.

// A threshold that exactly `keep` of the keys held in registers do not exceed.  k[e] is valid in
// the lanes of vm[e]; `total` >= keep keys are valid in all.  Search on the key value: the
// keep-th smallest key stays inside [lo, lo + 2^(bit+1)), and the search stops as soon as the
// number of keys below the bracket's upper end is exactly `keep` -- after about log2(total)
// bits for spread-out keys, 32 at most (keys are distinct).  Two bits are decided per step: the three
// inner quarter points are compared at once (independent compares and counts), which halves the
// number of dependent compare -> count -> decide chains a wave has to sit through; the outcome is
// that of two halving steps.  `upper` is a bound no valid key exceeds (the cut the keys were
// collected under, else 2^32 - 1): the search starts at its leading bit instead of bit 31.
template <int E>
__device__ __forceinline__ uint32_t kth_key_threshold(const uint32_t (&k)[E], const unsigned long long (&vm)[E], int keep, int total,
                                                      uint32_t upper = 0xFFFFFFFFu)
{
    keep = uni(keep);
    uint32_t lo = 0;
    int below_hi = uni(total);
    int bit = uni(31 - __clz((int)(upper | 1u)));
    while (below_hi != keep && bit >= 1) {
        const uint32_t q = 1u << (bit - 1);
        const uint32_t t1 = lo | q, t2 = lo | (q << 1), t3 = t2 | q;
        int c1 = 0, c2 = 0, c3 = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            c1 += __popcll(ballot64(k[e] < t1) & vm[e]);
            c2 += __popcll(ballot64(k[e] < t2) & vm[e]);
            c3 += __popcll(ballot64(k[e] < t3) & vm[e]);
        }
        if (c1 >= keep) below_hi = c1;                           // first quarter
        else if (c2 >= keep) { lo = t1; below_hi = c2; }
        else if (c3 >= keep) { lo = t2; below_hi = c3; }
        else lo = t3;                                            // last quarter: the count below its upper end is unchanged
        bit -= 2;
    }
    if (below_hi != keep && bit == 0) {                          // a single bit left
        const uint32_t trial = lo | 1u;
        int below = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) below += __popcll(ballot64(k[e] < trial) & vm[e]);
        if (below < keep) lo = trial; else below_hi = below;
        bit = -1;
    }
    return lo + (uint32_t)((((uint64_t)1) << (bit + 1)) - 1u);
}

// How many IDs of a row a guessed cut lets through on average.  Keys are uniform 32-bit words, so about lambda of the
// row's keys lie at or below lambda / len of the key range; the guess decides only how much work is done, never the
// result: if fewer than f keys turn up (a Poisson count: one row in 600 to 900 for fan-outs of 5 to 25), the exact
// procedure runs.  Every candidate is an append and widens the final cut, so the guess is as low as the misses allow:
// with f + 4 sqrt(f) + 8 a row is missed once in 10^5 but three candidates in ten are superfluous.  A missed row is streamed twice
// by its wave.  For the pieces of long rows that is the tail of the launch (they run a wave each, in one round or a few), and eight
// more candidates are nothing to 16,384 IDs: they get the safe guess.  A share of 15 M nodes, 177 batches of 163 seeds, fan-outs
// 15, 10: the schedule 669 us with the low guess for all rows, 579 so; eight batches of 32 on 32 M nodes: 401 and 318.
__device__ __forceinline__ float guessed_candidates(int f) { return (float)f + 3.0f * __fsqrt_rn((float)f) + 3.0f; }
__device__ __forceinline__ float safely_guessed_candidates(int f) { return (float)f + 4.0f * __fsqrt_rn((float)f) + 8.0f; }
// The cut itself, its lower half all ones (see key32_open); share <= 0.5.
__device__ __forceinline__ uint32_t guessed_cut_of(float share) { return (uint32_t)(share * 4294967296.0f) | 0xFFFFu; }

// The f smallest keys among cnt candidates buf[0 .. cnt) (row order; f <= cnt <= 64, one per lane), none above `upper`,
// written to out in row order and marked.  The IDs go from the candidate's lane straight to their place: the
// row's registers, or the buffer, are not passed over again.
template <int MARK>
__device__ __forceinline__ void emit_candidates(const uint32_t *buf, int cnt, int f, uint32_t lo, uint32_t hi, uint32_t upper, int lane,
                                                int32_t *__restrict__ out, const ReachedOfBatch &reached_b)
{
    cnt = uni(cnt); f = uni(f); lo = uni(lo); hi = uni(hi);
    const uint32_t u = lane < cnt ? buf[lane] : 0u;
    const uint32_t k[1] = {key32(lo, hi, u)};
    const unsigned long long vm[1] = {low_lanes(cnt)};
    const uint32_t cut = uni(kth_key_threshold<1>(k, vm, f, cnt, uni(upper)));       // (may be the end of its bracket: no candidate lies between upper and it)
    const unsigned long long m = ballot64(k[0] <= cut) & vm[0];
    if (my_bit(m)) {
        out[lanes_below(m, lane)] = (int32_t)u;
        mark_reached<MARK>(reached_b, u);
    }
}

// Row of f < len <= 64 * E IDs held in registers (u[e] of lane l is row[e * 64 + l]),
// sampled and written to out in row order.  buf: scratch of at least 64 entries (used when GUESS).  GUESS: a fan-out at which 64
// candidates may do (merged tiles of fan-outs up to 64; at larger ones the guess lets more than 64 through as a rule).
template <int E, int MARK, bool GUESS>
__device__ __forceinline__ void sample_registers(const uint32_t (&u)[E], int len, int f, uint32_t lo, uint32_t hi, int lane, uint32_t *buf,
                                                 int32_t *__restrict__ out, const ReachedOfBatch &reached_b)
{
    len = uni(len); f = uni(f); lo = uni(lo); hi = uni(hi);
    uint32_t k[E];
    unsigned long long vm[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        vm[e] = low_lanes(len - e * 64);
        k[e] = key32_open(lo, hi, u[e]);
    }
    if (GUESS && E > 1) {
        // As for long rows, a cut guessed from the key distribution first.  If between f and 64 IDs pass, they are
        // listed one per lane and the threshold is searched among those alone, from the guessed cut's leading bit down.
        const float lambda = guessed_candidates(f);
        if (uni(lambda * 2.0f <= (float)len && lambda <= 56.0f)) {
            const uint32_t guessed = uni(guessed_cut_of(lambda / (float)len));
            unsigned long long m[E];
            int total = 0;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                m[e] = ballot64(k[e] <= guessed) & vm[e];
                total += __popcll(m[e]);
            }
            if (total >= f && total <= 64) {
                int base = 0;
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    if (my_bit(m[e])) buf[base + lanes_below(m[e], lane)] = u[e];
                    base += __popcll(m[e]);
                }
                __syncthreads();
                emit_candidates<MARK>(buf, total, f, lo, hi, guessed, lane, out, reached_b);
                __syncthreads();      // the scratch is free again
                return;
            }
        }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) k[e] ^= k[e] >> 16;
    const uint32_t cut = kth_key_threshold<E>(k, vm, f, len);
    int base = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const unsigned long long m = ballot64(k[e] <= cut) & vm[e];
        if (e * 64 + lane < len && k[e] <= cut) {
            out[base + lanes_below(m, lane)] = (int32_t)u[e];
            mark_reached<MARK>(reached_b, u[e]);
        }
        base += __popcll(m);
    }
}

// Keeps the `keep` smallest-key entries of buf[0..cnt), order preserved; returns a threshold that
// exactly those entries' keys do not exceed.
// Precondition: cnt > keep >= 1, cnt <= CAP.
template <int CAP>
__device__ __forceinline__ uint32_t prune_buffer(uint32_t *buf, int cnt, int keep, uint32_t lo, uint32_t hi, int lane, uint32_t upper)
{
    constexpr int E = CAP / 64;
    cnt = uni(cnt); keep = uni(keep); lo = uni(lo); hi = uni(hi);
    uint32_t u[E], k[E];
    unsigned long long vm[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int idx = e * 64 + lane;
        vm[e] = low_lanes(cnt - e * 64);
        u[e] = idx < cnt ? buf[idx] : 0u;
        k[e] = key32(lo, hi, u[e]);
    }
    const uint32_t cut = uni(kth_key_threshold<E>(k, vm, keep, cnt, uni(upper)));
    __syncthreads();          // every lane has read its entries before any is overwritten
    int base = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const unsigned long long m = ballot64(k[e] <= cut) & vm[e];
        if (e * 64 + lane < cnt && k[e] <= cut) buf[base + lanes_below(m, lane)] = u[e];
        base += __popcll(m);
    }
    __syncthreads();
    return cut;
}

// State of the candidate buffer while a long row streams by.
struct Stream {
    int cnt;          // entries in the buffer (wave-uniform)
    bool open;        // no cut yet: every ID is a candidate
    uint32_t cut;     // candidates must have key <= cut once !open
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// A block is up to 256 consecutive IDs of the row; lane l holds IDs 4l .. 4l+3 of the block (one
// 16-byte load), so row order is lane-major and ID e of a lane is valid in the lanes of vm[e].
// Appends the block's candidates to the buffer in row order.  If they do not fit, the buffer is
// pruned first (which tightens the cut and may drop some of them); if they still do not fit, the
// block goes in four quarters of 64 consecutive IDs.
// MAYBE_OPEN = false: the caller knows a cut is in force (s.open is false), which takes the test out of the loop.
template <int CAP, bool MAYBE_OPEN = true>
__device__ __forceinline__ void append_block(const uint32_t (&u)[4], const uint32_t (&k)[4], const unsigned long long (&vm)[4], int f, uint32_t lo,
                                             uint32_t hi, int lane, uint32_t *buf, Stream &s)
{
    f = uni(f); lo = uni(lo); hi = uni(hi);
    s.cnt = uni(s.cnt); s.open = MAYBE_OPEN ? uni(s.open) : false; s.cut = uni(s.cut);
    unsigned long long m[4];
    int total = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        m[e] = (MAYBE_OPEN && s.open) ? vm[e] : (ballot64(k[e] <= s.cut) & vm[e]);
        total += __popcll(m[e]);
    }
    if (total == 0) return;
    if (s.cnt + total > CAP && s.cnt > f) {
        s.cut = prune_buffer<CAP>(buf, s.cnt, f, lo, hi, lane, ((MAYBE_OPEN && s.open) ? 0xFFFFFFFFu : s.cut));
        s.cnt = f;
        s.open = false;
        total = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            m[e] &= ballot64(k[e] <= s.cut);
            total += __popcll(m[e]);
        }
        if (total == 0) return;
    }
    if (s.cnt + total <= CAP) {
        const unsigned long long any = m[0] | m[1] | m[2] | m[3];
        if (__popcll(any) == total) {
            // The usual event: no lane holds two candidates, so lane order is row order: one rank, one store.
            if (my_bit(any)) {
                const uint32_t v = my_bit(m[0]) ? u[0] : my_bit(m[1]) ? u[1] : my_bit(m[2]) ? u[2] : u[3];
                buf[s.cnt + lanes_below(any, lane)] = v;
            }
            s.cnt += total;
            return;
        }
        int rank = s.cnt;
#pragma unroll
        for (int e = 0; e < 4; ++e) rank += lanes_below(m[e], lane);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (my_bit(m[e])) buf[rank++] = u[e];
        s.cnt += total;
        return;
    }
    for (int q = 0; q < 4; ++q) {             // lanes 16q .. 16q+15 hold 64 consecutive IDs
        if (s.cnt > CAP - 64) {
            s.cut = prune_buffer<CAP>(buf, s.cnt, f, lo, hi, lane, ((MAYBE_OPEN && s.open) ? 0xFFFFFFFFu : s.cut));
            s.cnt = f;
            s.open = false;
        }
        const unsigned long long quarter = 0xFFFFull << (16 * q);
        unsigned long long mq[4];
        int rank = s.cnt, sub = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            mq[e] = m[e] & quarter;
            if (!(MAYBE_OPEN && s.open)) mq[e] &= ballot64(k[e] <= s.cut);
            rank += lanes_below(mq[e], lane);
            sub += __popcll(mq[e]);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (my_bit(mq[e])) buf[rank++] = u[e];
        s.cnt += sub;
    }
}

// IDs p[4 * lane .. 4 * lane + 3] of a block of which `left` (> 0) IDs lie inside the row; p is 16-byte aligned.
__device__ __forceinline__ u32x4 load_block(const int32_t *__restrict__ p, int left, int lane)
{
    const int j = 4 * lane;
    if (left >= 256 || j + 3 < left) return *reinterpret_cast<const u32x4 *>(p + j);
    u32x4 r = {0u, 0u, 0u, 0u};
    if (j < left) r.x = (uint32_t)p[j];
    if (j + 1 < left) r.y = (uint32_t)p[j + 1];
    if (j + 2 < left) r.z = (uint32_t)p[j + 2];
    return r;
}

// Valid lanes of ID e of a block that holds `count` IDs: 4 * lane + e < count.
__device__ __forceinline__ unsigned long long block_lanes(int count, int e) { return low_lanes((count - e + 3) >> 2); }

// A long row is read as its head (the IDs in front of the first 128-byte boundary, fewer than 32) and aligned blocks.
__device__ __forceinline__ int row_head(const int32_t *row, int len)
{
    const int head = (32 - (int)(((uintptr_t)row >> 2) & 31)) & 31;
    return head > len ? len : head;
}
// What a row of len > 64 IDs needs besides its leading 64, fetched ahead of the row's turn: for len <= 256 the IDs
// row[64 + lane], row[128 + lane], row[192 + lane] (x, y, z; 0 past the end), for longer rows the first aligned block.
__device__ __forceinline__ u32x4 row_ahead(const int32_t *__restrict__ row, int len, int lane)
{
    len = uni(len);
    if (len <= 256) {
        u32x4 r = {0u, 0u, 0u, 0u};
        if (64 + lane < len) r.x = (uint32_t)row[64 + lane];
        if (128 + lane < len) r.y = (uint32_t)row[128 + lane];
        if (192 + lane < len) r.z = (uint32_t)row[192 + lane];
        return r;
    }
    const int head = uni(row_head(row, len));
    return load_block(row + head, len - head, lane);
}

template <int CAP, bool FULL, bool MAYBE_OPEN = true>
__device__ __forceinline__ void stream_block(const u32x4 &blk, int count, int f, uint32_t lo, uint32_t hi, int lane, uint32_t *buf, Stream &s)
{
    count = uni(count); f = uni(f); lo = uni(lo); hi = uni(hi);
    const uint32_t u[4] = {blk.x, blk.y, blk.z, blk.w};
    uint32_t k[4];
    unsigned long long vm[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        k[e] = key32(lo, hi, u[e]);
        vm[e] = FULL ? ~0ull : block_lanes(count, e);
    }
    append_block<CAP, MAYBE_OPEN>(u, k, vm, f, lo, hi, lane, buf, s);
}

// A full block while a cut whose lower half is all ones is in force, the common outcomes only: no candidate, or candidates that fit the buffer.
// Returns false, with nothing done, when they do not fit; the caller then takes the block through append_block.
template <int CAP>
__device__ __forceinline__ bool stream_full_block_fast(const u32x4 &blk, uint32_t lo, uint32_t hi, int lane, uint32_t *buf, Stream &s)
{
    const uint32_t u[4] = {blk.x, blk.y, blk.z, blk.w};
    const uint32_t cut = uni(s.cut);
    s.cnt = uni(s.cnt);
    unsigned long long m[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) m[e] = ballot64(key32_open(lo, hi, u[e]) <= cut);
    const unsigned long long any = m[0] | m[1] | m[2] | m[3];
    if (any == 0ull) return true;
    const int total = __popcll(m[0]) + __popcll(m[1]) + __popcll(m[2]) + __popcll(m[3]);
    if (s.cnt + total > CAP) return false;
    if (__popcll(any) == total) {
        if (my_bit(any)) {
            const uint32_t v = my_bit(m[0]) ? u[0] : my_bit(m[1]) ? u[1] : my_bit(m[2]) ? u[2] : u[3];
            buf[s.cnt + lanes_below(any, lane)] = v;
        }
    } else {
        int rank = s.cnt;
#pragma unroll
        for (int e = 0; e < 4; ++e) rank += lanes_below(m[e], lane);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (my_bit(m[e])) buf[rank++] = u[e];
    }
    s.cnt += total;
    return true;
}

// Row of len > 256 IDs streamed once, its sample written to out in row order and marked.  The IDs in
// front of the first 128-byte boundary go first (one per lane); from there on the row is read in
// blocks of 1 KB, one aligned 16-byte load per lane, so no two loads of a wave share a cache line,
// and the next block's load is in flight while the current block's keys are computed.
// first = row[lane] and blk0 = row_ahead(row, len, lane), loaded by the caller.
template <int CAP, int MARK>
__device__ __forceinline__ void sample_long_row(const int32_t *__restrict__ row, int len, uint32_t first, int f, uint32_t lo, uint32_t hi, int lane,
                                                uint32_t *buf, const u32x4 &blk0, int32_t *__restrict__ out, const ReachedOfBatch &reached_b)
{
    len = uni(len); f = uni(f); lo = uni(lo); hi = uni(hi);
    const int head = uni(row_head(row, len));
    const int32_t *p = row + head;
    const int rem = len - head;                                  // > 0: len > 256 and head < 32
    const int n_blocks = (rem + 255) >> 8;
    const uint32_t head_u = lane < head ? first : 0u;          // the head is part of the row's leading 64 IDs, which the caller holds
    // First attempt with a guessed cut (see guessed_candidates): streaming with it from the start collects the few IDs
    // that can be in the sample and skips the first cut and the prunes of the exact procedure.  Every ID with a key up to
    // the cut is kept, so if at least f turn up, the f smallest keys of the row are among them; if fewer do, the row is
    // streamed again with the exact procedure.
    const float lambda = len > BIG_ROW ? safely_guessed_candidates(f) : guessed_candidates(f);
    const bool can_guess = uni(lambda * 4.0f <= (float)len);
    const uint32_t guessed_cut = guessed_cut_of(fminf(lambda / (float)len, 0.5f));
    Stream s{0, true, 0u};
    const int first_attempt = uni(can_guess ? 0 : 1);
  for (int attempt = first_attempt; attempt < 2; attempt = uni(attempt + 1)) {
    const bool guess = attempt == 0;
    s = guess ? Stream{0, false, guessed_cut} : Stream{0, true, 0u};
    u32x4 cur = attempt == first_attempt ? blk0 : load_block(p, rem, lane), nxt = {0u, 0u, 0u, 0u};
    int c0 = 0;
    const int count0 = rem < 256 ? rem : 256;
    if (!guess && head + count0 > f) {
        // The usual case: the head and the first block (up to 287 IDs, all in registers) already hold more
        // than f IDs.  Their f smallest keys give the first cut directly; only those f IDs enter the buffer.
        if (rem > 256) nxt = load_block(p + 256, rem - 256, lane);
        const uint32_t u[5] = {head_u, cur.x, cur.y, cur.z, cur.w};
        uint32_t k[5];
        unsigned long long vm[5];
        vm[0] = low_lanes(head);
#pragma unroll
        for (int e = 1; e < 5; ++e) vm[e] = block_lanes(count0, e - 1);
#pragma unroll
        for (int e = 0; e < 5; ++e) k[e] = key32(lo, hi, u[e]);
        s.cut = uni(kth_key_threshold<5>(k, vm, f, head + count0));
        s.open = false;
        s.cnt = f;
            unsigned long long m[5];
        int rank = 0;
#pragma unroll
        for (int e = 0; e < 5; ++e) m[e] = ballot64(k[e] <= s.cut) & vm[e];
        if (my_bit(m[0])) buf[lanes_below(m[0], lane)] = u[0];
        rank = __popcll(m[0]);
#pragma unroll
        for (int e = 1; e < 5; ++e) rank += lanes_below(m[e], lane);
#pragma unroll
        for (int e = 1; e < 5; ++e)
            if (my_bit(m[e])) buf[rank++] = u[e];
        cur = nxt;
        c0 = 1;
    } else if (guess && head > 0) {
        // under the guessed cut the head's candidates (at most 31, into an empty buffer) need no more than a rank
        const unsigned long long m = ballot64(key32(lo, hi, head_u) <= s.cut) & low_lanes(head);
        if (my_bit(m)) buf[lanes_below(m, lane)] = head_u;
        s.cnt = __popcll(m);
    } else if (head > 0) {
        const uint32_t u[4] = {head_u, 0u, 0u, 0u};
        const uint32_t k[4] = {key32(lo, hi, u[0]), 0u, 0u, 0u};
        const unsigned long long vm[4] = {low_lanes(head), 0ull, 0ull, 0ull};
        append_block<CAP>(u, k, vm, f, lo, hi, lane, buf, s);
    }
    if (guess && rem >= 256) {
        // The full blocks under the guessed cut, two in flight behind the one whose keys are computed: block j lives in
        // register quartet j mod 3 and the loop is unrolled by three, so no block is copied from one quartet to another
        // (a copy would have to wait for a load that has only just been issued).  Leaves at the first block it does not
        // take -- the partial last one, or a full one whose candidates do not fit -- which the loop below picks up.
        const int n_full = rem >> 8;
        auto load = [&](int j) {                                                                   // block j < n_blocks
            if (j < n_full) return *reinterpret_cast<const u32x4 *>(p + j * 256 + 4 * lane);
            return load_block(p + j * 256, rem - j * 256, lane);
        };
        u32x4 r0 = cur, r1 = {0u, 0u, 0u, 0u}, r2 = {0u, 0u, 0u, 0u};
        if (1 < n_blocks) r1 = load(1);
        int c = 0;
        for (;;) {
            if (c + 2 < n_blocks) r2 = load(c + 2);
            if (!stream_full_block_fast<CAP>(r0, lo, hi, lane, buf, s)) break;
            c = uni(c + 1);
            if (c >= n_full) break;
            if (c + 2 < n_blocks) r0 = load(c + 2);
            if (!stream_full_block_fast<CAP>(r1, lo, hi, lane, buf, s)) break;
            c = uni(c + 1);
            if (c >= n_full) break;
            if (c + 2 < n_blocks) r1 = load(c + 2);
            if (!stream_full_block_fast<CAP>(r2, lo, hi, lane, buf, s)) break;
            c = uni(c + 1);
            if (c >= n_full) break;
        }
        c0 = c;
        const int which = c % 3;
        cur = which == 0 ? r0 : which == 1 ? r1 : r2;            // (unused when c == n_blocks)
    }
    for (int c = uni(c0); c < n_blocks; c = uni(c + 1)) {
        const int left = uni(rem - c * 256);                     // IDs left, this block included
        if (left > 256) nxt = load_block(p + (c + 1) * 256, left - 256, lane);
        if (left >= 256) {
            if (guess) stream_block<CAP, true, false>(cur, 256, f, lo, hi, lane, buf, s);
            else stream_block<CAP, true, true>(cur, 256, f, lo, hi, lane, buf, s);
        } else stream_block<CAP, false>(cur, left, f, lo, hi, lane, buf, s);
        cur = nxt;
    }
    __syncthreads();
    if (s.cnt >= f) break;                                       // (always, in the exact attempt: len > f)
  }
    const uint32_t upper = s.open ? 0xFFFFFFFFu : s.cut;
    if (s.cnt <= 64) {                                           // the usual case after a guessed cut: one ID per lane
        emit_candidates<MARK>(buf, s.cnt, f, lo, hi, upper, lane, out, reached_b);
    } else {
        if (s.cnt > f) (void)prune_buffer<CAP>(buf, s.cnt, f, lo, hi, lane, upper);
        for (int j = lane; j < f; j += 64) {
            const uint32_t u = buf[j];
            out[j] = (int32_t)u;
            mark_reached<MARK>(reached_b, u);
        }
    }
    __syncthreads();      // the buffer is reused by the wave's next row
}

// SAMPLE of a row of len > f IDs into out (row order), marking the sampled IDs as MARK says.
// `first` holds row[lane] for lane < len; ahead = row_ahead(row, len, lane) when len > 64 (unused otherwise).
template <int CAP, int MARK>
__device__ __forceinline__ void sample_row(const int32_t *__restrict__ row, int len, uint32_t first, const u32x4 &ahead, int f, uint32_t lo, uint32_t hi,
                                           int lane, uint32_t *buf, int32_t *__restrict__ out, const ReachedOfBatch &reached_b)
{
    if (len <= 64) {
        const uint32_t u[1] = {first};
        sample_registers<1, MARK, false>(u, len, f, lo, hi, lane, buf, out, reached_b);
    } else if (len <= 256) {
        const uint32_t u[4] = {first, ahead.x, ahead.y, ahead.z};
        sample_registers<4, MARK, CAP <= 128>(u, len, f, lo, hi, lane, buf, out, reached_b);
    } else {
        sample_long_row<CAP, MARK>(row, len, first, f, lo, hi, lane, buf, ahead, out, reached_b);
    }
}

// ---------------------------------------------------------------- rows of up to SHORT_ROW IDs, four at a time
// A wave that samples one short row at a time spends its time waiting: a row of 30 IDs is one load and a few dozen
// instructions, and the next row's load cannot start much earlier than this row's ends.  Here a wave takes 64
// consecutive frontier nodes, lists the ones with 1 .. SHORT_ROW neighbours -- shortest first, so that rows of a
// round are of a kind -- and samples four of them at once, one per row of sixteen lanes (lane l of a row holds IDs
// l, l + 16, l + 32, l + 48 of it), with the next four rows' IDs already on their way.  How the f smallest keys are found
// and put in order: emit_rows.  At fan-outs above 64 such rows are their own samples and are copied.
struct ShortRec {
    int64_t row_begin, out;
    uint64_t state;
    int32_t deg;
    uint32_t batch;
    int32_t lane;         // whose row it is
};

template <int R> __device__ __forceinline__ uint32_t rotate16(uint32_t x)      // the value R lanes away within the lane's row of sixteen
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x120 + R, 0xF, 0xF, false);
}

// cnt += the keys among a row of sixteen lanes' `theirs`, this lane's own left out, that are smaller than this lane's `mine`: each of the
// fifteen others comes by as the row is rotated, a subtraction takes it in and leaves the answer in the carry, and the carry is added.
// (Two instructions per key; the compiler's own are three.)  The waits are those that the hardware leaves to the program and the
// compiler puts into its own code, but not into this text: two states from the write of `theirs` to its rotation, two from a
// carry's write to its read.  cnt is written before the inputs are read for the last time, so it may share a register with neither.
__device__ __forceinline__ void add_smaller16(uint32_t theirs, uint32_t mine, uint32_t &cnt)
{
    uint32_t scrap;
#define RG_ROT(R) "v_sub_co_u32_dpp %0, vcc, %2, %3 row_ror:" #R " row_mask:0xf bank_mask:0xf\n\ts_nop 1\n\tv_addc_co_u32_e32 %1, vcc, 0, %1, vcc\n\t"
    asm("s_nop 1\n\t" RG_ROT(1) RG_ROT(2) RG_ROT(3) RG_ROT(4) RG_ROT(5) RG_ROT(6) RG_ROT(7) RG_ROT(8)
        RG_ROT(9) RG_ROT(10) RG_ROT(11) RG_ROT(12) RG_ROT(13) RG_ROT(14) RG_ROT(15)
        : "=&v"(scrap), "+&v"(cnt) : "v"(theirs), "v"(mine) : "vcc");
#undef RG_ROT
}

// The sum of x over the lane's row of sixteen lanes, in all of them.
__device__ __forceinline__ int sum16(int x)
{
    x += (int)rotate16<8>((uint32_t)x);
    x += (int)rotate16<4>((uint32_t)x);
    x += (int)rotate16<2>((uint32_t)x);
    x += (int)rotate16<1>((uint32_t)x);
    return x;
}
// The sum of x over the lanes of the row up to and with this one, byte by byte (no byte may overflow).
template <int N> __device__ __forceinline__ uint32_t from_left16(uint32_t x)      // the value N lanes to the left in the row of sixteen; 0 past its start
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x110 + N, 0xF, 0xF, true);
}
__device__ __forceinline__ uint32_t prefix16(uint32_t x)
{
    x += from_left16<1>(x);
    x += from_left16<2>(x);
    x += from_left16<4>(x);
    x += from_left16<8>(x);
    return x;
}
__device__ __forceinline__ uint32_t last_of16(uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x15F, 0xF, 0xF, false); }      // lane 15's value of the row of sixteen

// Four rows' IDs, one row per sixteen lanes: lane l16 of a row holds IDs l16, l16 + 16, ... in u[0 .. E), n of them in the
// row (same in its lanes).  The min(n, f) with the smallest keys go to `out` in order and are marked.  All 64 lanes call it.
// One or two IDs per lane are decided by rank; more by halving the range of key values until exactly f keys
// lie below, all four rows side by side and in vector instructions alone: counts taken from lane masks are scalar work, and that
// unit is as busy as the vector units (see sample_rows_kernel).
template <int E, int MARK>
__device__ __forceinline__ void emit_rows(const uint32_t (&u)[E], int n, int f, uint32_t lo, uint32_t hi, int l16, int32_t *__restrict__ out,
                                          const ReachedOfBatch &reached_b)
{
    bool sel[E];
#pragma unroll
    for (int e = 0; e < E; ++e) sel[e] = l16 + 16 * e < n;
    const bool search = n > f;
    if (ballot64(search) != 0ull) {
        uint32_t k[E];
#pragma unroll
        for (int e = 0; e < E; ++e) k[e] = sel[e] ? key32(lo, hi, u[e]) : 0xFFFFFFFFu;       // (a missing key's stand-in is below nothing)
        if (E <= 2) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                uint32_t smaller = 0;
#pragma unroll
                for (int q = 0; q < E; ++q) {
                    add_smaller16(k[q], k[e], smaller);
                    if (q != e) smaller += k[q] < k[e] ? 1u : 0u;
                }
                if (search) sel[e] = sel[e] && smaller < (uint32_t)f;
            }
        } else {
            uint32_t from = 0, to = 0xFFFFFFFFu, t = to >> 1;     // fewer than f keys lie below `from`, at least f at or below `to`
            for (int step = 0; step < 34; ++step) {              // (distinct keys are told apart in 32 steps; repeated IDs of a damaged row never)
                int c = 0;
#pragma unroll
                for (int e = 0; e < E; ++e) c += k[e] <= t ? 1 : 0;
                c = sum16(c);
                if (ballot64(search && c != f) == 0ull) break;
                const bool few = c < f;
                if (c <= f) from = t + (few ? 1u : 0u);
                if (!few) to = t;                                // (exactly f: this row's t stays as it is)
                t = from + ((to - from) >> 1);
            }
            if (search) {
#pragma unroll
                for (int e = 0; e < E; ++e) sel[e] = sel[e] && k[e] <= t;
            }
        }
    }
    // an ID's place is the number of selected ones in front of it: those of the lanes to the left in its own step of sixteen,
    // from a prefix sum of four steps' flags packed in a word, and all of the steps before
    const uint32_t keep = (uint32_t)(search ? f : n);
    uint32_t in_front = 0;                                       // of the words before, in every byte
#pragma unroll
    for (int w = 0; w < (E + 3) / 4; ++w) {
        uint32_t x = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (4 * w + q < E) x |= sel[4 * w + q] ? 1u << (8 * q) : 0u;
        const uint32_t incl = prefix16(x), all = last_of16(incl);
        const uint32_t place = incl - x + all * 0x01010100u + in_front;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = 4 * w + q;
            if (e >= E) break;
            const uint32_t at = (place >> (8 * q)) & 0xFFu;
            if (sel[e] && at < keep) {                           // (at < keep but for repeated IDs)
                out[at] = (int32_t)u[e];
                mark_reached<MARK>(reached_b, u[e]);
            }
        }
        if (E > 4) in_front += ((all * 0x01010101u) >> 24) * 0x01010101u;
    }
}

// The listed short rows (recs[0 .. count), shortest first; LDS) sampled four per round.  All 64 lanes call it.  COPY: none is longer
// than the fan-out.
template <int MARK, bool COPY>
__device__ __forceinline__ void sample_short_rows(const ShortRec *recs, int count, const int32_t *__restrict__ indices, int f,
                                                  int32_t *__restrict__ samp_nbr, const ReachedMaps &reached, int lane)
{
    const int l16 = lane & 15, sg = lane >> 4;
    const int n_it = (count + 3) >> 2;
    // this lane's row of the round, and its IDs (0 where the row has none)
    auto fetch = [&](int it, ShortRec &r, uint32_t (&u)[4]) {
        const int slot = it * 4 + sg;
        r = slot < count ? recs[slot] : ShortRec{};
        const int32_t *row = indices + r.row_begin;
#pragma unroll
        for (int e = 0; e < 4; ++e) u[e] = l16 + 16 * e < r.deg ? (uint32_t)row[l16 + 16 * e] : 0u;
    };
    ShortRec r, r_next;
    uint32_t u[4], u_next[4];
    fetch(0, r, u);
    for (int it = 0; it < n_it; ++it) {
        if (it + 1 < n_it) fetch(it + 1, r_next, u_next);
        const ReachedOfBatch reached_b = reached_of<MARK>(reached, r.batch);
        int32_t *out = samp_nbr + r.out;
        const uint32_t lo = (uint32_t)r.state, hi = (uint32_t)(r.state >> 32);
        const uint32_t u1[1] = {u[0]}, u2[2] = {u[0], u[1]};
        if (COPY) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (l16 + 16 * e < r.deg) { out[l16 + 16 * e] = (int32_t)u[e]; mark_reached<MARK>(reached_b, u[e]); }
        } else if (ballot64(r.deg > 32) != 0ull) emit_rows<4, MARK>(u, r.deg, f, lo, hi, l16, out, reached_b);
        else if (ballot64(r.deg > 16) != 0ull) emit_rows<2, MARK>(u2, r.deg, f, lo, hi, l16, out, reached_b);
        else emit_rows<1, MARK>(u1, r.deg, f, lo, hi, l16, out, reached_b);
        r = r_next;
#pragma unroll
        for (int e = 0; e < 4; ++e) u[e] = u_next[e];
    }
}

// Where a lane's row goes in the list of a group's rows that are sampled four at a time: shortest rows first, by the number of
// IDs per lane ((deg - 1) >> SHIFT, below 4), lane order within a kind.  mine: this lane has such a row.  All 64 lanes call it.
template <int SHIFT>
__device__ __forceinline__ int short_row_slot(bool mine, int deg, int lane)
{
    const int kind = mine ? (deg - 1) >> SHIFT : -1;
    int at = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const unsigned long long m = ballot64(kind == c);
        if (c < kind) at += __popcll(m);
        else if (c == kind) at += lanes_below(m, lane);
    }
    return at;
}

// Per tile job j: the frontier position whose row it belongs to, which of the row's tiles it is, where its piece of the
// row starts in `indices`, how long it is (near-equal pieces, each longer than 2 * RG_MAX_FANOUT) and the node's
// stream S_v: a wave finds everything about its piece in one round of loads.
struct TileRecs {
    int64_t *node;
    int32_t *t;
    int64_t *begin;
    int32_t *len;
    uint64_t *state;
};
// The tile jobs of a chunk's nodes, in frontier order; which: see tiles_in.
__global__ void __launch_bounds__(NODE_THREADS) tile_nodes_kernel(const uint32_t *__restrict__ count, int64_t n, const int64_t *__restrict__ tile_base, int which, TileRecs r)
{
    const int64_t base = tile_base[blockIdx.x];
    if (tile_base[blockIdx.x + 1] == base) return;
    const int64_t first = (int64_t)blockIdx.x * NODE_CHUNK + (int64_t)threadIdx.x * NODE_PER_THREAD;
    uint32_t c[NODE_PER_THREAD], tiles[NODE_PER_THREAD];
    load_counts(count, first, n, c);
#pragma unroll
    for (int k = 0; k < NODE_PER_THREAD; ++k) tiles[k] = tiles_in(c[k], which);
    int64_t j = base + (int64_t)chunk_exclusive_scan(tiles[0] + tiles[1] + tiles[2] + tiles[3]);
#pragma unroll
    for (int k = 0; k < NODE_PER_THREAD; ++k)
        for (uint32_t t = 0; t < tiles[k]; ++t, ++j) { r.node[j] = first + k; r.t[j] = (int32_t)t; }
}
// One thread per tile job.
__global__ void tile_records_kernel(const int64_t *__restrict__ row_begin, const int32_t *__restrict__ deg, const uint64_t *__restrict__ state, int64_t n_tiles, int64_t tile_piece, TileRecs r)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n_tiles) return;
    const int64_t i = r.node[j], t = r.t[j];
    const int64_t d = deg[i];
    const int64_t T = tiles_of(d, tile_piece);
    const int64_t first_pos = t * d / T, last_pos = (t + 1) * d / T;
    r.begin[j] = row_begin[i] + first_pos;
    r.len[j] = (int32_t)(last_pos - first_pos);
    r.state[j] = state[i];
}

// Tile jobs grouped by the piece of adjacency they read.  A hub's row is in the frontier of most batches, so the same
// piece is read once per batch; in frontier order those reads lie a whole batch apart and every one of them comes
// from HBM.  Handed out in an order in which the jobs of a piece follow each other, they run at about the same time
// and all but the first are served by the caches.  Grouping, not sorting: a job's bucket is a hash of its piece's
// start (pieces are thousands of IDs apart), jobs are counted per bucket, the counts prefix-summed, and every job
// takes the next place of its bucket (in whatever order the adds arrive: a job's result goes to the job's own
// place, so the order changes nothing but the timing).
__device__ __forceinline__ uint32_t tile_bucket(int64_t begin, int bits)
{
    return ((uint32_t)((uint64_t)begin >> 12) * 0x9E3779B1u) >> (32 - bits);
}
// rank[j] = how many jobs of j's bucket came before it (by arrival); cnt[b] ends as the bucket's size
__global__ void tile_bucket_count_kernel(const int64_t *__restrict__ begin, int64_t n_tiles, int bits, int32_t *__restrict__ cnt, int32_t *__restrict__ rank)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j < n_tiles) rank[j] = atomicAdd(&cnt[tile_bucket(begin[j], bits)], 1);
}
__global__ void tile_bucket_place_kernel(const int64_t *__restrict__ begin, int64_t n_tiles, int bits, const int64_t *__restrict__ off,
                                         const int32_t *__restrict__ rank, int32_t *__restrict__ order)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j < n_tiles) order[off[tile_bucket(begin[j], bits)] + rank[j]] = (int32_t)j;
}

struct HopArgs {
    const int32_t *indices;
    const int32_t *frontier; int64_t n_frontier;
    int64_t n_full_groups, n_units;                                    // set by launch_hop: see there ...
    int tail_shift; int64_t n_own, first_own;                          // ... as are these, for sample_rows_kernel: nodes of a unit behind the full groups (their logarithm), units that go by index, and the first one's workgroup
    ByPlace place; int64_t n_full_rounds;                              // (rounds of full groups, where units go by place)
    int64_t tile_piece;                                                // tiles_of
    int min_deg;                                                       // rows of up to this many IDs are not copied one per wave but four at a time, a group's short rows first (sample_kernel<.., true>); 0: none are
    NodeRecs rec;
    uint32_t fanout;
    const int64_t *samp_off; int32_t *samp_nbr;
    TileRecs tile; int64_t n_tiles; int32_t *tile_out;      // tile j writes tile_out[j * fanout ..)
    int merge_span;                                                    // tiles a wave of sample_merge_kernel looks at per round
    const int32_t *tile_order;                                         // the k-th tile job to hand out, or NULL: job k
    ReachedMaps reached;
    unsigned long long *next_work;                                     // work items are handed out in order through this counter
    float guess_scale;                                                 // of the candidates a row's first cut is to let through (1; for tests: sample_rows_kernel)
};

// The next unclaimed work item (lane 0 asks, every lane gets the answer).
__device__ __forceinline__ int64_t grab_work(unsigned long long *counter, int lane)
{
    unsigned long long v = 0;
    if (lane == 0) v = atomicAdd(counter, 1ull);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// The work of a hop: n_tiles tiles of long rows (done first, so the longest-running work starts first) and the groups
// of 64 consecutive frontier nodes.
// Fan-outs above 64.  SHORT_INLINE: each group's rows of up to SHORT_ROW IDs are copied four at a time before its other rows (an
// instantiation of its own: the code costs the streaming loop a few registers).
template <int CAP, int MARK, bool SHORT_INLINE>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(CAP <= 256 ? 7 : 1))) sample_kernel(HopArgs a)
{
    __shared__ uint32_t buf[CAP];
    __shared__ ShortRec short_recs[SHORT_INLINE ? 64 : 1];
    const int lane = threadIdx.x;
    const int f = (int)a.fanout;
    // Tiles first, dealt out in turn (workgroup k takes tiles k, k + grid, ...): they are all of about the same
    // length, the whole grid is resident (see launch_hop), and with the next tile known in advance its record is
    // fetched while the current one is streamed -- no wave waits for a counter or a record between tiles.
    {
        // Workgroup g runs on XCD g mod 8 (workgroups are dealt out to the XCDs in turn), and every XCD has an L2 of its
        // own: in each round XCD x takes a contiguous eighth of the round's jobs, so the jobs of a piece -- neighbours
        // in the grouped order -- meet in one L2 instead of being spread over all eight.
        int64_t k = blockIdx.x;
        if (a.tile_order && (gridDim.x & 7u) == 0) k = (int64_t)(blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
        int64_t w = 0, nb = 0; int nl = 0; uint64_t nS = 0;
        if (k < a.n_tiles) { w = a.tile_order ? a.tile_order[k] : k; nb = a.tile.begin[w]; nl = a.tile.len[w]; nS = a.tile.state[w]; }
        while (k < a.n_tiles) {
            const int32_t *row = a.indices + nb;
            const int len = nl;
            const uint64_t S = nS;
            const int64_t w_now = w;
            const uint32_t first = (uint32_t)row[lane];
            const u32x4 ahead = row_ahead(row, len, lane);
            k += gridDim.x;
            if (k < a.n_tiles) { w = a.tile_order ? a.tile_order[k] : k; nb = a.tile.begin[w]; nl = a.tile.len[w]; nS = a.tile.state[w]; }
            sample_row<CAP, MARK_NONE>(row, len, first, ahead, f, (uint32_t)S, (uint32_t)(S >> 32), lane, buf, a.tile_out + w_now * f,
                                       ReachedOfBatch{nullptr, nullptr});
        }
    }
    // Then the groups of 64 consecutive frontier nodes, taken as waves become free, so that uneven rows do not leave
    // part of the chip idle at the end -- and for the same reason the launch's last nodes come in groups of 16 (a group
    // of 64 nodes with long rows is a sizeable part of a launch's whole duration); every wave leaves once the counter
    // has passed the last group.
    for (int64_t w = grab_work(a.next_work, lane); w < a.n_units; w = grab_work(a.next_work, lane)) {
        const bool full = w < a.n_full_groups;                  // 64 nodes, or 16 of the launch's last nodes
        const int64_t i_lane = (full ? w << 6 : (a.n_full_groups << 6) + ((w - a.n_full_groups) << 4)) + lane;
        const bool in = (full || lane < 16) && i_lane < a.n_frontier;
        const int64_t rb_lane = in ? a.rec.row_begin[i_lane] : 0;
        const int deg_lane = in ? a.rec.deg[i_lane] : 0;
        const uint32_t b_lane = in ? a.rec.batch[i_lane] : 0u;
        const int64_t S_lane = in ? (int64_t)a.rec.state[i_lane] : 0;
        const int64_t out_lane = in ? a.samp_off[i_lane] : 0;
        if (SHORT_INLINE) {
            // the group's rows of up to SHORT_ROW IDs first, four at a time (their marks and scattered little reads then
            // run beside the streaming of the other waves' long rows)
            // A row of at most TINY_ROW IDs that is no longer than the fan-out is its own sample: its node's lane copies
            // and marks it, 64 rows at a time, four IDs of each in flight (on a graph whose typical row has two or three
            // IDs these are nine rows in ten, and four at a time is sixteen rounds for what is one or two here).
            const bool tiny = in && deg_lane > 0 && deg_lane <= f && deg_lane <= TINY_ROW;
            if (ballot64(tiny) != 0ull) {
                const int32_t *row = a.indices + rb_lane;
                int32_t *out = a.samp_nbr + out_lane;
                const ReachedOfBatch reached_b = reached_of<MARK>(a.reached, b_lane);
                for (int j0 = 0; ballot64(tiny && j0 < deg_lane) != 0ull; j0 += 4) {
                    int32_t u[4] = {0, 0, 0, 0};
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (tiny && j0 + k < deg_lane) u[k] = row[j0 + k];
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (tiny && j0 + k < deg_lane) { out[j0 + k] = u[k]; mark_reached<MARK>(reached_b, (uint32_t)u[k]); }
                }
            }
            const bool mine = in && !tiny && deg_lane > 0 && deg_lane <= SHORT_ROW;
            const int count = __popcll(ballot64(mine));
            if (count != 0) {
                const int at = short_row_slot<4>(mine, deg_lane, lane);
                __syncthreads();
                if (mine) short_recs[at] = ShortRec{rb_lane, out_lane, (uint64_t)S_lane, deg_lane, b_lane, lane};
                __syncthreads();
                sample_short_rows<MARK, true>(short_recs, count, a.indices, f, a.samp_nbr, a.reached, lane);
            }
        }
        unsigned long long todo = ballot64(deg_lane > a.min_deg && deg_lane <= BIG_ROW);
        if (todo == 0ull) continue;
        // the first node's leading 64 IDs; from then on the next node's are fetched while the current one is sampled
        int l = __builtin_amdgcn_readfirstlane(__ffsll((long long)todo) - 1);
        int64_t rb = bcast64(rb_lane, l);
        int deg = __builtin_amdgcn_readlane(deg_lane, l);
        uint32_t first = lane < deg ? (uint32_t)a.indices[rb + lane] : 0u;
        u32x4 ahead = {0u, 0u, 0u, 0u};
        if (deg > 64 && deg > f) ahead = row_ahead(a.indices + rb, deg, lane);
        while (todo != 0ull) {
            todo &= todo - 1ull;
            const int cl = l, cdeg = deg;
            const int64_t crb = rb;
            const uint32_t cfirst = first;
            const u32x4 cahead = ahead;
            if (todo != 0ull) {
                l = __builtin_amdgcn_readfirstlane(__ffsll((long long)todo) - 1);
                rb = bcast64(rb_lane, l);
                deg = __builtin_amdgcn_readlane(deg_lane, l);
                first = lane < deg ? (uint32_t)a.indices[rb + lane] : 0u;
                if (deg > 64 && deg > f) ahead = row_ahead(a.indices + rb, deg, lane);
            }
            const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)b_lane, cl);
            const ReachedOfBatch reached_b = reached_of<MARK>(a.reached, b);
            const int32_t *row = a.indices + crb;
            int32_t *out = a.samp_nbr + bcast64(out_lane, cl);
            if (cdeg <= f) {                  // the whole row is the sample
                if (lane < cdeg) { out[lane] = (int32_t)cfirst; mark_reached<MARK>(reached_b, cfirst); }
                for (int j = 64 + lane; j < cdeg; j += 64) {
                    const int32_t u = row[j];
                    out[j] = u;
                    mark_reached<MARK>(reached_b, (uint32_t)u);
                }
            } else {
                const uint64_t S = (uint64_t)bcast64(S_lane, cl);
                sample_row<CAP, MARK>(row, cdeg, cfirst, cahead, f, (uint32_t)S, (uint32_t)(S >> 32), lane, buf, out, reached_b);
            }
        }
    }
}

// ---------------------------------------------------------------- fan-outs up to 64
// The same work for fan-outs of at most ROWS_FANOUT.  Bound by the vector units' integer rate, and next to it by the scalar
// unit, which a compute unit's four SIMDs share and which takes one instruction per SIMD and four cycles, as the vector units do.
// sample_kernel issues as many of the one as of the other, both pipes were four fifths busy, and no more than 1.9 instructions
// per SIMD and four cycles come through, whatever their kind; so here instructions are what is saved: no tests inside a chunk's
// inner blocks, no cases at a block's load, no copies between the two chunks' registers, one compare per step of the last cut.
// Per block of 256 IDs, everything a row costs included (233,000 nodes, rows of 13 blocks, fan-outs 25, 10): 57 vector and 59 scalar
// instructions before, 49 and 36 so; the launches 3.65 -> 3.1 ms (2.45 M nodes: 15, 10, 5 9.6 -> 7.7, 50, 50 2.09 -> 1.6).
//
// A row's IDs are streamed once against a guessed cut (a key and its compare are eight vector
// instructions per ID, see key32_open_of_row), what passes, a few dozen IDs, is listed in LDS in row order, and the f smallest keys of the list are
// the sample.  If fewer than f IDs pass, or more than fit, the row is streamed again with another cut (retry_row).
//
// A row is read in blocks of 256 IDs, 16 bytes per lane.  Rows above MID_ROW IDs are read from the last 128-byte boundary in
// front of them (`skip` IDs early, which do not count), so that no two loads share a line; lanes of the last block that would read past the row
// read its last 16 bytes instead, and only the IDs that no other lane has count.  Blocks come in chunks of ROWS_CHUNK; while one is
// looked through the next one of the row, or the first one of the next row, is on its way.
constexpr int ROWS_FANOUT = 64;
constexpr int ROWS_ROOM = 128;           // candidates of one row of four
constexpr int STREAM_ROOM = 192;         // of a row that the whole wave streams: the safe guess lets 104 through at a fan-out of 64, and one tile in 100 more than 128
                                         // (2,000 tiles of 60,000 IDs, fan-out 60: 204 us with room for 128, where some are streamed twice, 105 so)
constexpr int ROWS_CHUNK = 2;
constexpr int MID_ROW = 256;

typedef u32x4 u32x4_dword_aligned __attribute__((aligned(4)));

struct StreamedRow {
    const int32_t *from;                 // where block 0 starts: `skip` IDs in front of the row
    int skip, len, n_blocks;
};

// Block j; lanes past the row's last four IDs hold those.
__device__ __forceinline__ u32x4 load_row_block(const StreamedRow &r, int j, int lane)
{
    const uint32_t at = min(1024u * (uint32_t)j + 16u * (uint32_t)lane, 4u * (uint32_t)(r.skip + r.len - 4));
    return *reinterpret_cast<const u32x4_dword_aligned *>(reinterpret_cast<const char *>(r.from) + at);
}

__device__ __forceinline__ int places(unsigned long long m, int first)      // first + the number of set bits of m below this lane's
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)first));
}

// key32_open with its addition inside the second product, (x + hi) * HA32 = x * HA32 + hi * HA32: the 64-bit multiply-add issues at the
// rate of the 32-bit product, and the step x ^= x >> 16 that the addition was fused with is one instruction by itself.  Eight
// instructions with the compare where key32_open makes nine (keys against a cut from registers alone: 3.95 -> 4.34 x 10^12 per second;
// the sampling launches of an epoch: a 111 M node share 1.95 -> 1.80 ms, 2.45 M nodes 6.92 -> 6.80, 233,000 2.83 -> 2.77).
// Only the low half of c counts, hi * HA32; its high half may be anything, so hi itself is kept there.
__device__ __forceinline__ uint64_t key_state(uint32_t hi) { return (uint64_t)hi << 32 | (hi * HA32); }
__device__ __forceinline__ uint32_t hi_of(uint64_t c) { return (uint32_t)(c >> 32); }
__device__ __forceinline__ uint32_t key32_after_mad(uint64_t y)
{
    asm("" : "+v"(y));                                           // (the whole sum is wanted, or it would be narrowed to a product and an addition again)
    uint32_t x = (uint32_t)y;
    x ^= x >> 15;
    return x * HB32;
}
// c the same in all lanes; ha32: HA32 in a register of the lanes (the instruction takes one operand from the scalar registers)
__device__ __forceinline__ uint32_t key32_open_of_row(uint32_t lo, uint64_t c, uint32_t ha32, uint32_t u)
{
    uint32_t x = (u ^ lo) * HG32;
    x ^= x >> 16;
    return key32_after_mad((uint64_t)x * ha32 + c);
}
// c a lane's own
__device__ __forceinline__ uint32_t key32_open_of_lane(uint32_t lo, uint64_t c, uint32_t u)
{
    uint32_t x = (u ^ lo) * HG32;
    x ^= x >> 16;
    return key32_after_mad((uint64_t)x * HA32 + c);
}

// Appends the IDs of a block whose key is not above `cut` to cand[cnt ..), in row order, unless they do not fit; cnt counts on
// in any case.  OPEN: the cut's lower half is all ones (see key32_open).  EDGE: the first or the last block of its row, of which
// not all IDs count; p: the position in the row that the lane's first ID should have (in front of the row: negative).
// The empty asm statements keep the branches that lanes take apart from those that the wave takes, so that cnt stays in a
// scalar register and the two ways of writing are not folded into one.
template <bool OPEN, bool EDGE>
__device__ __forceinline__ void take_block(const u32x4 &blk, int p, int last_four, uint32_t lo, uint64_t c, uint32_t ha32, uint32_t cut, uint32_t *cand, int &cnt)
{
    const uint32_t u[4] = {blk.x, blk.y, blk.z, blk.w};
    unsigned long long m[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) m[e] = ballot64((OPEN ? key32_open_of_row(lo, c, ha32, u[e]) : key32(lo, hi_of(c), u[e])) <= cut);
    if (EDGE) {
        const int first = max(p, 0) - min(p, last_four);         // from which of the lane's four IDs on they count
#pragma unroll
        for (int e = 0; e < 4; ++e) m[e] &= ballot64(first <= e);
    }
    const unsigned long long m01 = m[0] | m[1], m012 = m01 | m[2], any = m012 | m[3];
    if (any == 0ull) return;
    if (__builtin_expect(((m[0] & m[1]) | (m01 & m[2]) | (m012 & m[3])) == 0ull, 1)) {      // no lane holds two candidates: lane order is row order
        const int before = cnt;
        cnt += __popcll(any);
        if (cnt <= STREAM_ROOM) {
            uint32_t v = my_bit(m[2]) ? u[2] : u[3];
            v = my_bit(m[1]) ? u[1] : v;
            v = my_bit(m[0]) ? u[0] : v;
            const int at = places(any, before);
            if (my_bit(any)) cand[at] = v;
            asm volatile("; one each");
        }
    } else {
        const int before = cnt;
        cnt += __popcll(m[0]) + __popcll(m[1]) + __popcll(m[2]) + __popcll(m[3]);
        if (cnt <= STREAM_ROOM) {
            int at = places(m[3], places(m[2], places(m[1], places(m[0], before))));
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (my_bit(m[e])) cand[at++] = u[e];
            asm volatile("; several");
        }
    }
}

// The row again, with finished keys, until between f and STREAM_ROOM IDs pass: the cut is moved by what the count says is missing
// or too much, inside what the tries so far leave.  Returns how many, and the cut.  (Only a row that repeats IDs can have no
// such cut; its first f IDs stand for it then.)
__device__ __forceinline__ int retry_row(const StreamedRow &r, int f, uint32_t lo, uint64_t c, int cnt, uint32_t *cut_io, int lane, uint32_t *cand)
{
    uint32_t cut = *cut_io;
    uint64_t low = 0, high = (uint64_t)1 << 32;                  // cuts below `low` let too few through, from `high` on too many
    const float spare = 2.0f * __fsqrt_rn((float)f) + 4.0f;
    for (int t = 0; t < 48 && (cnt < f || cnt > STREAM_ROOM); ++t) {
        uint64_t next;
        if (cnt < f) {
            low = (uint64_t)cut + 1;
            next = (uint64_t)cut + 1 + (uint64_t)(((float)(f - cnt) + spare) / (float)r.len * 4294967296.0f);
        } else {
            high = cut;
            next = (uint64_t)((float)cut * (((float)f + spare) / (float)cnt));
        }
        if (t >= 4 || next < low || next >= high) next = low + (high - low) / 2;
        if (low >= high) break;
        cut = uni((uint32_t)next);
        cnt = 0;
        for (int j = 0; j < r.n_blocks; ++j) take_block<false, true>(load_row_block(r, j, lane), 256 * j + 4 * lane - r.skip, r.len - 4, lo, c, 0u, cut, cand, cnt);
        cnt = uni(cnt);
    }
    if (cnt < f || cnt > STREAM_ROOM) {
        if (lane < f) cand[lane] = (uint32_t)r.from[r.skip + lane];
        cnt = f;
    }
    *cut_io = cut;
    return cnt;
}

// The f smallest keys of cand[0 .. cnt), 64 * (E - 1) < cnt <= 64 * E, none above `cut`, written to `out` in row order and marked.
// Their bound is found bit by bit from the cut's leading bit down, one compare per step and the rest on the scalar
// unit, until exactly f keys lie below it: 4 to 6 steps.  (Four rows at once, a row per sixteen lanes, took twice the vector
// instructions of this: the steps are those of the slowest row, and counts over sixteen lanes are four additions each.)
template <int E, int MARK>
__device__ __forceinline__ void emit_row(const uint32_t *cand, int cnt, int f, uint32_t lo, uint32_t hi, uint32_t cut, int lane, int32_t *__restrict__ out, bool mark,
                                         const ReachedOfBatch &reached_b)
{
    uint32_t u[E], k[E];
    unsigned long long vm[E], m[E];
#pragma unroll
    for (int e = 0; e < E; ++e) u[e] = cand[64 * e + lane];      // (past cnt: what an earlier row left)
#pragma unroll
    for (int e = 0; e < E; ++e) {
        vm[e] = m[e] = low_lanes(cnt - 64 * e);
        k[e] = key32(lo, hi, u[e]);
    }
    if (cnt > f) {
        uint32_t from = 0, bit = 1u << (31 - __clz((int)(cut | 1u)));      // the f-th smallest key lies in [from, from + 2 * bit)
        int c;
        do {
            const uint32_t t = from | bit;
            c = 0;
#pragma unroll
            for (int e = 0; e < E; ++e) { m[e] = ballot64(k[e] < t) & vm[e]; c += __popcll(m[e]); }
            if (c < f) from = t;
            bit >>= 1;
        } while (c != f && bit != 0u);
        if (c != f) {
#pragma unroll
            for (int e = 0; e < E; ++e) m[e] = ballot64(k[e] <= from) & vm[e];
        }
    }
    int first = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int at = places(m[e], first);
        if (my_bit(m[e]) && at < f) {                            // (at < f but for repeated IDs)
            out[at] = (int32_t)u[e];
            if (MARK != MARK_NONE && mark) mark_reached<MARK>(reached_b, u[e]);
        }
        first += __popcll(m[e]);
    }
}

// Four rows of 65 .. MID_ROW IDs, sixteen lanes each (they are listed shortest first, so those of a round are of a kind).  A lane
// takes four consecutive IDs of every 64; what passes the guessed cut goes to the row's list (`mine`), in order, from where
// emit_rows takes it.  Returns the lanes (of the group) whose rows let too few or too many through: they are streamed like longer rows.
// NQ: how many times 64 IDs the round's longest row has.
// A row on its own spends more on its set-up and its cut, on the scalar unit above all, than on its keys: 2.45 M nodes, 5.8 M such rows,
// fan-outs 15, 10, 5, some 230 instructions a row against 110 so, the launches 7.7 -> 7.3 ms; 50, 50 1.60 -> 1.45.
constexpr int MID_STRIDE = ROWS_ROOM + 16;       // (sixteen banks further on for the next row)
template <int NQ, int MARK>
__device__ __forceinline__ unsigned long long sample_mid_round(const ShortRec &r, bool active, const int32_t *__restrict__ indices, int f, float lambda,
                                                               int32_t *__restrict__ samp_nbr, const ReachedMaps &reached, int l16, uint32_t *mine)
{
    const uint32_t lo = (uint32_t)r.state, hi = (uint32_t)(r.state >> 32);
    const char *row = reinterpret_cast<const char *>(indices + r.row_begin);
    u32x4 u[NQ];
    int first[NQ];                                               // from which of a lane's four IDs on they count
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int p = 64 * q + 4 * l16, at = min(p, r.deg - 4);
        first[q] = active ? p - at : 4;
        u[q] = *reinterpret_cast<const u32x4_dword_aligned *>(row + 4u * (uint32_t)at);
    }
    const uint32_t cut = guessed_cut_of(fminf(lambda / (float)r.deg, 0.99f));
    const uint64_t key = key_state(hi);
    bool sel[NQ][4];
    uint32_t x = 0;                                              // how many of each four, in a byte each
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const uint32_t id[4] = {u[q].x, u[q].y, u[q].z, u[q].w};
        uint32_t c = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            sel[q][e] = key32_open_of_lane(lo, key, id[e]) <= cut && first[q] <= e;
            c += sel[q][e] ? 1u : 0u;
        }
        x |= c << (8 * q);
    }
    const uint32_t incl = prefix16(x), all = last_of16(incl), place = incl - x + all * 0x01010100u;
    const int n = (int)((all * 0x01010101u) >> 24);
    const bool fits = n >= f && n <= ROWS_ROOM;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const uint32_t id[4] = {u[q].x, u[q].y, u[q].z, u[q].w};
        uint32_t *to = mine + ((place >> (8 * q)) & 0xFFu);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (sel[q][e] && fits) *to++ = id[e];
    }
    wave_lds_order();
    const int take = fits && active ? n : 0;
    const ReachedOfBatch reached_b = reached_of<MARK>(reached, r.batch);
    int32_t *out = samp_nbr + r.out;
#define RG_EMIT(E)                                                                                                    \
    do {                                                                                                              \
        uint32_t v[E];                                                                                                \
        _Pragma("unroll") for (int e = 0; e < E; ++e) v[e] = mine[l16 + 16 * e];                                      \
        emit_rows<E, MARK>(v, take, f, lo, hi, l16, out, reached_b);                                                  \
    } while (0)
    if (ballot64(take > 64) != 0ull) RG_EMIT(8);
    else if (ballot64(take > 32) != 0ull) RG_EMIT(4);
    else if (ballot64(take > 16) != 0ull) RG_EMIT(2);
    else RG_EMIT(1);
#undef RG_EMIT
    wave_lds_order();
    unsigned long long again = 0ull, failed = ballot64(active && !fits && l16 == 0);
    while (failed != 0ull) {
        const int l = __builtin_amdgcn_readfirstlane(__ffsll((long long)failed) - 1);
        failed &= failed - 1ull;
        again |= 1ull << __builtin_amdgcn_readlane(r.lane, l);
    }
    return again;
}

// Six waves per SIMD, 80 registers: eleven or twelve of them spill, to 40 or 52 bytes of scratch per lane, reloaded once per row or round of rows.  At
// seven waves (72 registers, up to 20 spilled) what a row costs besides its keys is slower, at five nothing spills but fewer waves wait together:
// sampling launches and mark pass at seven / six / five waves, 233,000 nodes 2,807 / 2,786 / 2,781 us, 2.45 M nodes, 15, 10, 5 7,077 / 7,039 / 7,036, 50, 50
// 1,745 / 1,720 / 1,778, 111 M nodes 1,885 / 1,884 / 1,915; one hop of 200,000 rows of 100 IDs, fan-out 60 123 / 115; 16,000 rows of 20,000 IDs, fan-out 10 272 / 255.
template <int MARK>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(6))) sample_rows_kernel(HopArgs a)
{
    __shared__ uint32_t cand[4 * MID_STRIDE];                    // one streamed row's candidates, or those of four rows
    static_assert(STREAM_ROOM <= 4 * MID_STRIDE && STREAM_ROOM % 64 == 0, "");
    __shared__ ShortRec short_recs[64];
    const int lane = threadIdx.x;
    const int f = (int)a.fanout;
    uint32_t ha32 = HA32;
    asm volatile("" : "+v"(ha32));                               // (not a constant to the compiler, which would put it back)
    // Tiles first, dealt out in turn; in each round XCD x takes a contiguous eighth of the round's jobs (see sample_kernel).
    int64_t k = blockIdx.x;
    if (a.tile_order && (gridDim.x & 7u) == 0) k = (int64_t)(blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    int64_t own_unit = k - a.first_own + (k < a.first_own ? gridDim.x : 0);
    if (own_unit >= a.n_own) own_unit = -1;
    int64_t w = 0, tile_begin = 0; int tile_len = 0; uint64_t tile_state = 0;
    if (k < a.n_tiles) { w = a.tile_order ? a.tile_order[k] : k; tile_begin = a.tile.begin[w]; tile_len = a.tile.len[w]; tile_state = a.tile.state[w]; }
    for (;;) {
        // a tile (one row, the first lane's), or the next group of nodes, a lane each
        const bool is_tile = k < a.n_tiles;
        int64_t rb_lane = 0;
        int deg_lane = 0;
        uint32_t b_lane = 0;
        uint64_t S_lane = 0;
        int64_t out_lane = 0;
        int32_t *const out_base = is_tile ? a.tile_out : a.samp_nbr;
        if (is_tile) {
            rb_lane = tile_begin; deg_lane = lane == 0 ? tile_len : 0; S_lane = tile_state; out_lane = w * f;
            k += gridDim.x;
            if (k < a.n_tiles) { w = a.tile_order ? a.tile_order[k] : k; tile_begin = a.tile.begin[w]; tile_len = a.tile.len[w]; tile_state = a.tile.state[w]; }
        } else {
            // Workgroups without a tile have their first unit of nodes by index, and where a frontier is small all units go by index, a wave every
            // grid's one; the others come through the counter.  It answers one wave every 4 to 8 ns: thousands that ask at once wait 25 us for their turns,
            // which is a small launch's whole time, more where they all come from a tile (6,000 rows of 20,000 IDs, fan-out 10, by the counter / by index
            // 167 / 106 us), and more where the units are small (13 batches of 7,500 nodes, 450 IDs each, in units of four: 384 / 160 us for two hops).
            int64_t g = own_unit;
            own_unit = g >= 0 && g + gridDim.x < a.n_own ? g + gridDim.x : -1;
            if (g < 0) {
                if (a.n_own >= a.n_units) break;
                g = a.n_own + grab_work(a.next_work, lane);
            }
            if (g >= a.n_units) break;
            const bool full = g < a.n_full_groups;               // 64 nodes, or fewer of the launch's last nodes
            // its nodes: in frontier order, or the like places of all batches one after the other
            int64_t i0 = full ? g << 6 : (a.n_full_groups << 6) + ((g - a.n_full_groups) << a.tail_shift), i_end = a.n_frontier;
            if (a.place.n_batches) {
                const uint32_t at = (uint32_t)(full ? g : g - a.n_full_groups), round = at / a.place.n_batches, b = at - round * a.place.n_batches;
                i0 = a.place.batch_off[b] + (full ? (int64_t)round << 6 : (a.n_full_rounds << 6) + ((int64_t)round << a.tail_shift));
                i_end = a.place.batch_off[b + 1];
            }
            const int64_t i_lane = i0 + lane;
            const bool in = (full || lane < 1 << a.tail_shift) && i_lane < i_end;
            if (in) {
                rb_lane = a.rec.row_begin[i_lane];
                deg_lane = a.rec.deg[i_lane];
                b_lane = a.rec.batch[i_lane];
                S_lane = a.rec.state[i_lane];
                out_lane = a.samp_off[i_lane];
            }
            // A row of at most TINY_ROW IDs that is no longer than the fan-out is its own sample: its node's lane copies
            // and marks it, 64 rows at a time, four IDs of each in flight.
            const bool tiny = deg_lane > 0 && deg_lane <= f && deg_lane <= TINY_ROW;
            if (ballot64(tiny) != 0ull) {
                const int32_t *row = a.indices + rb_lane;
                int32_t *out = a.samp_nbr + out_lane;
                const ReachedOfBatch reached_b = reached_of<MARK>(a.reached, b_lane);
                for (int j0 = 0; ballot64(tiny && j0 < deg_lane) != 0ull; j0 += 4) {
                    int32_t u[4] = {0, 0, 0, 0};
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (tiny && j0 + q < deg_lane) u[q] = row[j0 + q];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (tiny && j0 + q < deg_lane) { out[j0 + q] = u[q]; mark_reached<MARK>(reached_b, (uint32_t)u[q]); }
                }
            }
            const bool mine = !tiny && deg_lane > 0 && deg_lane <= SHORT_ROW;
            const int count = __popcll(ballot64(mine));
            if (count != 0) {
                const int at = short_row_slot<4>(mine, deg_lane, lane);
                wave_lds_order();
                if (mine) short_recs[at] = ShortRec{rb_lane, out_lane, S_lane, deg_lane, b_lane, lane};
                wave_lds_order();
                sample_short_rows<MARK, false>(short_recs, count, a.indices, f, a.samp_nbr, a.reached, lane);
            }
        }
        unsigned long long todo = ballot64(deg_lane > MID_ROW && (is_tile || deg_lane <= BIG_ROW));      // rows that the whole wave streams
        const bool mid = deg_lane > SHORT_ROW && deg_lane <= MID_ROW;
        if (const int count = __popcll(ballot64(mid))) {
            const int at = short_row_slot<6>(mid, deg_lane, lane);
            wave_lds_order();
            if (mid) short_recs[at] = ShortRec{rb_lane, out_lane, S_lane, deg_lane, b_lane, lane};
            wave_lds_order();
            const float lambda = guessed_candidates(f) * a.guess_scale;
            const int l16 = lane & 15, sg = lane >> 4;
            for (int k0 = 0; k0 < count; k0 += 4) {
                const ShortRec r = short_recs[min(k0 + sg, count - 1)];
                const bool active = k0 + sg < count;
                uint32_t *mine = cand + sg * MID_STRIDE;
                if (ballot64(r.deg > 192) != 0ull) todo |= sample_mid_round<4, MARK>(r, active, a.indices, f, lambda, a.samp_nbr, a.reached, l16, mine);
                else if (ballot64(r.deg > 128) != 0ull) todo |= sample_mid_round<3, MARK>(r, active, a.indices, f, lambda, a.samp_nbr, a.reached, l16, mine);
                else todo |= sample_mid_round<2, MARK>(r, active, a.indices, f, lambda, a.samp_nbr, a.reached, l16, mine);
            }
        }
        if (todo == 0ull) continue;
        // the guessed cut of this lane's row; a row that fits the candidates' room and would lose little is taken whole
        uint32_t cut_lane = 0xFFFFFFFFu;
        {
            const float lambda = (is_tile ? safely_guessed_candidates(f) : guessed_candidates(f)) * a.guess_scale;
            if (deg_lane > STREAM_ROOM || lambda * 2.0f <= (float)deg_lane) cut_lane = guessed_cut_of(fminf(lambda / (float)deg_lane, 0.99f));
        }
        // where the wave is: chunk j of the row of lane l
        struct Cursor { StreamedRow r; int l, j; uint32_t lo, cut; uint64_t key; };
        auto first_chunk_of = [&](int l) {
            const int64_t rb = bcast64(rb_lane, l);
            Cursor c;
            c.l = l;
            c.j = 0;
            c.r.len = __builtin_amdgcn_readlane(deg_lane, l);
            c.r.from = a.indices + rb;
            c.r.skip = c.r.len > MID_ROW && (rb >> 5) != 0 ? (int)(((uintptr_t)c.r.from >> 2) & 31u) : 0;      // (no fewer than 32 IDs in front of the row)
            c.r.from -= c.r.skip;
            c.r.n_blocks = (c.r.skip + c.r.len + 255) >> 8;
            c.lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)S_lane, l);
            c.key = key_state((uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(S_lane >> 32), l));
            c.cut = (uint32_t)__builtin_amdgcn_readlane((int)cut_lane, l);
            return c;
        };
        auto next_lane = [&]() {
            const int l = __builtin_amdgcn_readfirstlane(__ffsll((long long)todo) - 1);
            todo &= todo - 1ull;
            return l;
        };
        auto load_chunk = [&](const Cursor &c, u32x4 (&to)[ROWS_CHUNK]) {
#pragma unroll
            for (int e = 0; e < ROWS_CHUNK; ++e) to[e] = load_row_block(c.r, c.j + e, lane);
        };
        Cursor at = first_chunk_of(next_lane()), ahead = at;     // the chunk that is looked through, and the one that is loaded
        int cnt = 0;
        // One chunk, held in `now`, while the next one is loaded into `then`; false: it was the last.
        auto step = [&](u32x4 (&now)[ROWS_CHUNK], u32x4 (&then)[ROWS_CHUNK]) {
            const bool last = at.j + ROWS_CHUNK >= at.r.n_blocks;      // of its row
            bool more = true;
            ahead.j += ROWS_CHUNK;
            if (last) {
                more = todo != 0ull;
                if (more) ahead = first_chunk_of(next_lane());
            }
            __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0): this chunk is here, and only then the next is asked for (behind the last one, the end of its row again)
            load_chunk(ahead, then);
            if (at.j > 0 && !last) {
#pragma unroll
                for (int q = 0; q < ROWS_CHUNK; ++q) take_block<true, false>(now[q], 0, 0, at.lo, at.key, ha32, at.cut, cand, cnt);
            } else {
#pragma unroll
                for (int q = 0; q < ROWS_CHUNK; ++q)
                    if (q == 0 || at.j + q < at.r.n_blocks)
                        take_block<true, true>(now[q], 256 * (at.j + q) + 4 * lane - at.r.skip, at.r.len - 4, at.lo, at.key, ha32, at.cut, cand, cnt);
            }
            at.j += ROWS_CHUNK;
            if (last) {
                uint32_t cut = at.cut;
                int n = cnt;
                wave_lds_order();
                if (n < f || n > STREAM_ROOM) {
                    n = uni(retry_row(at.r, f, at.lo, at.key, n, &cut, lane, cand));
                    cut = uni(cut);
                    wave_lds_order();
                }
                n = uni(n);
                int32_t *out = out_base + bcast64(out_lane, at.l);
                const ReachedOfBatch reached_b = reached_of<MARK>(a.reached, MARK == MARK_NONE ? 0u : (uint32_t)__builtin_amdgcn_readlane((int)b_lane, at.l));
                const uint32_t lo = at.lo, hi = hi_of(at.key);
                at = ahead;
                cnt = 0;
                if (n <= 64) emit_row<1, MARK>(cand, n, f, lo, hi, cut, lane, out, !is_tile, reached_b);
                else if (n <= 128) emit_row<2, MARK>(cand, n, f, lo, hi, cut, lane, out, !is_tile, reached_b);
                else emit_row<3, MARK>(cand, n, f, lo, hi, cut, lane, out, !is_tile, reached_b);
                wave_lds_order();
            }
            return more;
        };
        u32x4 x[ROWS_CHUNK], y[ROWS_CHUNK];
        load_chunk(at, x);
        while (step(x, y) && step(y, x)) {}
    }
}

// A long row's concatenated tile results (T * f IDs, row order, all distinct) are sampled into the final output by
// the wave that finds the row's first tile.  A wave looks at 64 tiles at once, a lane each (hub rows have hundreds of
// tiles, so first tiles are few: walking the tiles one per wave-iteration cost two dependent loads per tile), and
// then takes the rows whose first tiles it found one after the other.  a.merge_span <= 64 tiles per look: fewer
// where the launch has too few tiles to give every wave 64 of them (rows of two or three tiles would queue up).
template <int CAP, int MARK>
__global__ void __launch_bounds__(64) sample_merge_kernel(HopArgs a)
{
    __shared__ uint32_t buf[CAP];
    const int lane = threadIdx.x;
    const int f = (int)a.fanout;
    const int span = a.merge_span;
    for (int64_t base = (int64_t)blockIdx.x * span; base < a.n_tiles; base += (int64_t)gridDim.x * span) {
        int64_t i_lane = -1;
        if (lane < span && base + lane < a.n_tiles) {
            if (a.tile.t[base + lane] == 0) i_lane = a.tile.node[base + lane];
        }
        unsigned long long firsts = ballot64(i_lane >= 0);
        while (firsts != 0ull) {
            const int l = __builtin_amdgcn_readfirstlane(__ffsll((long long)firsts) - 1);
            firsts &= firsts - 1ull;
            const int64_t i = bcast64(i_lane, l);
            const int64_t w = base + l;
            const int64_t T = tiles_of(a.rec.deg[i], a.tile_piece);
            const uint32_t b = a.rec.batch[i];
            const uint64_t S = a.rec.state[i];
            const int32_t *row = a.tile_out + w * f;
            const int len = (int)(T * f);
            u32x4 ahead = {0u, 0u, 0u, 0u};
            if (len > 64) ahead = row_ahead(row, len, lane);
            sample_row<CAP, MARK>(row, len, lane < len ? (uint32_t)row[lane] : 0u, ahead, f, (uint32_t)S, (uint32_t)(S >> 32), lane, buf,
                                  a.samp_nbr + a.samp_off[i], reached_of<MARK>(a.reached, b));
        }
    }
}


// ---------------------------------------------------------------- hub rows: sampled from the keys' side
// A row of d IDs holds about lambda keys up to the cut lambda / d * 2^32.  Reading the row finds them with d keys; but
// key32 is a bijection, so they are found as well by taking the key values 0, 1, 2, ... up to the cut, undoing each
// (key32_inverse) and asking whether the row holds the ID that comes out.  That is lambda / d * 2^32 values, of which only
// the share n_nodes / 2^32 are IDs at all and have to be looked up: the longer the row the fewer, and fewer than d from
// d = sqrt(lambda * 2^32) on.  A row of 6.7 M IDs takes 14,000 values instead of 6.7 M keys. 
// On 111 M nodes and 405 M edges in 147 batches, fan-out 10 behind 15, the sampling launches took 4.5 ms, nine tenths of
// it vector instructions; with the rows from 450,000 IDs on taken out (half the length the rule takes): 1.66 ms, and 0.26 for the key values, 0.17 for the
// tables, 0.05 to clear them.  (A directory of positions into the row in place of the tables cost 0.09 to build but three
// dependent reads per lookup: 0.38 ms for the key values.)
// Results are those of reading the row: all IDs with a key in the range come out, the f smallest keys are taken.
//
// Lookup: a table per distinct row, a bucket of sixteen 16-bit entries for every 2^shift consecutive IDs, so that one
// 32-byte read settles nearly every ID (a search of the whole row where a full bucket does not hold it); built by one
// pass over the row.  Rows are shared by most batches, so the pass is paid once for many jobs.  The IDs to look up are
// collected per wave and looked up 64 at a time: only one value in 40 (of 10^8 nodes) needs it.
__global__ void __launch_bounds__(256) hub_table_kernel(const int32_t *__restrict__ indices, int64_t n_nodes, HubTable h, HubBucket *__restrict__ buckets)
{
    const int32_t slot = h.list[blockIdx.y];
    const HubRow r = h.rows[slot];
    const int32_t *row = indices + r.begin;
    HubBucket *mine = buckets + r.first;
    const uint32_t n = (uint32_t)n_nodes;
    bool damaged = false;
    const int lane = threadIdx.x & 63;
    // A wave takes 64 consecutive IDs; an ID's place in its bucket is its distance from the lane its bucket starts in, and
    // for the bucket the wave starts in the middle of, also from the up to sixteen IDs in front of the wave.
    for (int64_t base = (int64_t)blockIdx.x * 256 + (threadIdx.x & ~63u); base < r.deg; base += (int64_t)gridDim.x * 256) {
        const int64_t i = base + lane;
        const bool in = i < r.deg;
        const uint32_t u = in ? (uint32_t)row[i] : 0xFFFFFFFFu, before = in && i > 0 ? (uint32_t)row[i - 1] : 0u;
        const int64_t behind = base - 1 - lane;                  // lanes 0 .. 15: the IDs in front of the wave, nearest first
        const uint32_t back = lane < HUB_BUCKET && behind >= 0 ? (uint32_t)row[behind] : 0xFFFFFFFFu;
        const uint32_t b = u >> r.shift, b0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)b);
        const unsigned long long not_mine = ~__ballot(lane < HUB_BUCKET && behind >= 0 && back >> r.shift == b0);
        const int carried = __ffsll((long long)not_mine) - 1;    // how many of them, without a gap, are in the first lane's bucket
        const unsigned long long starts = __ballot(in && (i == 0 || before >> r.shift != b)) & (lane == 63 ? ~0ull : (2ull << lane) - 1ull);
        const int rank = starts ? lane - (63 - __clzll((long long)starts)) : lane + carried;
        if (!in) continue;
        if (u >= n || (i > 0 && before >= u)) damaged = true;
        else if (rank < HUB_BUCKET) mine[b].id[rank] = (uint16_t)(u & ((1u << r.shift) - 1u));
    }
    if (damaged) h.counts->damaged = 1u;
}

// A job for every frontier position that holds a hub row, in whatever order they arrive (a job's samples go to the
// position's own place).
__global__ void __launch_bounds__(NODE_THREADS) hub_jobs_kernel(const uint32_t *__restrict__ count, const int32_t *__restrict__ frontier, int64_t n,
                                                                const uint32_t *__restrict__ chunk_hub, HubTable h, HubJob *__restrict__ jobs)
{
    if (chunk_hub[blockIdx.x] == 0u) return;
    const int64_t first = (int64_t)blockIdx.x * NODE_CHUNK + (int64_t)threadIdx.x * NODE_PER_THREAD;
    uint32_t c[NODE_PER_THREAD];
    load_counts(count, first, n, c);
#pragma unroll
    for (int k = 0; k < NODE_PER_THREAD; ++k) {
        if (!(c[k] & HUB_FLAG)) continue;
        const uint32_t v = (uint32_t)frontier[first + k];
        uint32_t slot = first_hub_slot(v);
        for (int t = 0; t < HUB_PROBES && h.keys[slot] != v + 1u; ++t) slot = (slot + 1) & (HUB_SLOTS - 1);
        jobs[atomicAdd(&h.counts->n_jobs, 1u)] = HubJob{first + k, (int32_t)slot, 0};
    }
}

// Whether the row (ascending) holds u < n_nodes.
__device__ __forceinline__ bool hub_holds(const HubBucket *__restrict__ mine, const HubRow &r, const int32_t *__restrict__ row, uint32_t u)
{
    const uint4 *p = reinterpret_cast<const uint4 *>(mine + (u >> r.shift));
    const uint4 x = p[0], y = p[1];
    const uint32_t want = (u & ((1u << r.shift) - 1u)) * 0x00010001u;
    const uint32_t w[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
    uint32_t any = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t d = w[k] ^ want;                          // a 16-bit half that is zero: found
        any |= (d - 0x00010001u) & ~d & 0x80008000u;
    }
    if (any) return true;
    if (y.w >> 16 == HUB_EMPTY) return false;
    int32_t lo = 0, hi = r.deg;
    while (lo < hi) {                                            // the first position whose ID is not below u
        const int32_t m = lo + ((hi - lo) >> 1);
        if ((uint32_t)row[m] < u) lo = m + 1; else hi = m;
    }
    return lo < r.deg && (uint32_t)row[lo] == u;
}

struct HubArgs {
    const int32_t *indices;
    int64_t n_nodes;
    const HubRow *rows;
    const HubBucket *buckets;
    const HubJob *jobs;
    uint32_t n_jobs;
    float first_range;                          // of the guessed range of key values, how much is looked through first (1; for tests)
    NodeRecs rec;
    uint32_t fanout;
    const int64_t *samp_off; int32_t *samp_nbr;
    ReachedMaps reached;
};

constexpr int HUB_THREADS = 256;
constexpr int HUB_WAVES = HUB_THREADS / 64;
constexpr int HUB_HITS = 1024;                  // the guess lets 515 through at the largest fan-out; 15 KB of LDS, so that eight workgroups of a compute unit wait for their lookups together
constexpr int HUB_QUEUE = 64 + 4 * 64;          // a wave's IDs waiting to be looked up: fewer than 64 left over, and a step's four per lane

template <int MARK>
__global__ void __launch_bounds__(HUB_THREADS) hub_sample_kernel(HubArgs a)
{
    __shared__ uint32_t hit_key[HUB_HITS], hit_id[HUB_HITS];
    __shared__ uint8_t hit_taken[HUB_HITS];
    __shared__ uint32_t queue[HUB_WAVES][HUB_QUEUE];                                // keys of IDs below n_nodes
    __shared__ uint32_t n_hits;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int f = (int)a.fanout;
    const uint32_t n = (uint32_t)a.n_nodes;
    for (uint32_t j = blockIdx.x; j < a.n_jobs; j += gridDim.x) {
        const HubJob job = a.jobs[j];
        const HubRow r = a.rows[job.slot];
        const int32_t *row = a.indices + r.begin;
        const HubBucket *mine = a.buckets + r.first;
        const uint64_t S = a.rec.state[job.i];
        const uint32_t lo = uni((uint32_t)S), hi = uni((uint32_t)(S >> 32));
        uint64_t from = 0, to = (uint64_t)fminf(guessed_candidates(f) / (float)r.deg * a.first_range * 4294967296.0f, 4294967296.0f) + 1;     // key values [from, to)
        uint32_t kept = 0;                                       // hits with keys below `from` (fewer than f)
        for (;;) {
            if (to > ((uint64_t)1 << 32)) to = (uint64_t)1 << 32;
            __syncthreads();                                     // the hits of the job before, or of the round before, have been read
            if (threadIdx.x == 0) n_hits = kept;
            __syncthreads();
            int waiting = 0;                                     // in this wave's queue (the same in all its lanes)
            auto look_up = [&](int count) {                      // the queue's last `count` <= 64 entries
                if (lane < count) {
                    const uint32_t key = queue[wave][waiting - count + lane], u = key32_inverse(lo, hi, key);
                    if (hub_holds(mine, r, row, u)) {
                        const uint32_t k = atomicAdd(&n_hits, 1u);
                        if (k < HUB_HITS) { hit_key[k] = key; hit_id[k] = u; }
                    }
                }
                waiting -= count;
            };
            for (uint64_t base = from + (uint64_t)wave * 256; base < to; base += HUB_THREADS * 4) {
                const uint32_t left = (uint32_t)(to - base < 256 ? to - base : 256);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t at = (uint32_t)(64 * e + lane), key = (uint32_t)base + at;
                    const unsigned long long m = ballot64(key32_inverse(lo, hi, key) < n && at < left);
                    if (my_bit(m)) queue[wave][waiting + lanes_below(m, lane)] = key;
                    waiting += __popcll(m);
                }
                waiting = uni(waiting);
                wave_lds_order();
                while (waiting >= 64) look_up(64);
                wave_lds_order();
            }
            if (waiting > 0) look_up(waiting);
            __syncthreads();
            const uint32_t found = n_hits;
            if (found > HUB_HITS) { to = from + (to - from) / 2; continue; }        // too many for the list: a smaller range (the hits kept so far stay; a single key value is one hit at most)
            if (found >= (uint32_t)f || to == ((uint64_t)1 << 32)) break;
            kept = found;
            const uint64_t step = 2 * (to - from);               // too few: the next key values, twice as many
            from = to;
            to += step;
        }
        // the f smallest keys, in row order: the row ascends, so in the order of the IDs
        const int c = (int)n_hits;
        for (int k = threadIdx.x; k < c; k += HUB_THREADS) {
            const uint32_t key = hit_key[k];
            int smaller = 0;
            for (int q = 0; q < c; ++q) smaller += hit_key[q] < key ? 1 : 0;
            hit_taken[k] = smaller < f ? 1 : 0;
        }
        __syncthreads();
        int32_t *out = a.samp_nbr + a.samp_off[job.i];
        const ReachedOfBatch reached_b = reached_of<MARK>(a.reached, a.rec.batch[job.i]);
        for (int k = threadIdx.x; k < c; k += HUB_THREADS) {
            if (!hit_taken[k]) continue;
            const uint32_t id = hit_id[k];
            int in_front = 0;
            for (int q = 0; q < c; ++q) in_front += hit_taken[q] && hit_id[q] < id ? 1 : 0;
            out[in_front] = (int32_t)id;
            mark_reached<MARK>(reached_b, id);
        }
    }
}

// From which length on a row is sampled from the keys' side: twice the length at which its key values cost what its IDs
// would.  A value costs about 1.6 times what an ID does (twice the arithmetic, no read), and the share of values that are
// IDs one more scattered read each.  Near the even length nothing is won and a few jobs do not fill the chip.  Schedules by where the line
// lies, in even lengths, 0.75 / 1 / 1.4 / 2 / 2.8 / no hub rows: 111 M nodes, 147 batches 3,171 / 2,749 / 2,775 / 2,828 / 2,919 / 3,516 us, 60 M
// 2,316 / 2,199 / 2,178 / 2,196 / 2,248 / 2,359, 30 M 1,933 / 1,854 / 1,865 / 1,839 / 1,859 / 1,831, 15 M, 177 batches 1,340 / 1,119 / 1,114 / 971 / 974 / 945.
static double hub_line(int64_t n_nodes, uint32_t fanout)
{
    const double f = (double)fanout, lambda = f + 3.0 * std::sqrt(f) + 3.0;
    const double per_value = 1.6 + 20.0 * (double)n_nodes / 4294967296.0;
    return 2.0 * std::sqrt(per_value * lambda * 4294967296.0);
}

// How many tile jobs the hub rows must make, per compute unit, to be worth their tables: clearing and building those and a
// wait for the rows' order cost 70 to 130 us (2 to 28 M distinct IDs), a tile job 17 ns.  Schedules with hub jobs / with tile jobs / by
// this line: 111 M nodes, 147 batches 2,828 / 3,516 / 2,812 us, 20 batches of 512 585 / 626 / 580, 40 of 1,024 1,022 / 993 / 1,000; 60 M, 147 2,196 / 2,359 / 2,176,
// 30 of 2,048 865 / 856 / 860; 30 M 1,839 / 1,831 / 1,831; 15 M, 176 of 163 614 / 598 / 604.
constexpr int HUB_TILES_PER_CU = 24;
// Epochs of fewer batches seldom hold so many (the 100 M nodes, 15 batches of 2,048 seeds: 6,525), and looking for them costs
// some 10 us a hop.
constexpr uint32_t HUB_BATCHES = 16;

// Nodes per compute unit from which on a frontier gives every resident wave a group of 64.
constexpr int SMALL_FRONTIER = 24 * 64;

// Every workgroup of the sampling launch must be resident from the start (tiles are dealt out by workgroup index), so
// the grid is what the chip holds of this kernel, or the amount of work if that is less.
typedef void (*HopKernel)(HopArgs);
template <bool ROWS, HopKernel SAMPLE, HopKernel MERGE>
static rg_status launch_hop(const HopArgs &args, int n_cu, unsigned merge_grid, bool fine_tail, bool fine_if_few, hipStream_t st)
{
    HopArgs a = args;
    static std::atomic<int> asked{0};                   // the same answer every time; asked once (schedules may be built from several threads)
    int per_cu = asked.load(std::memory_order_relaxed);
    if (per_cu == 0) {
        int v = 0;
        RG_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&v, SAMPLE, 64, 0));
        per_cu = v > 0 ? v : 1;
        asked.store(per_cu, std::memory_order_relaxed);
    }
    // Groups of 64 nodes, except that with fine_tail the last 128 nodes per resident wave (and always what is left of
    // the frontier after the last whole group) are handed out 16 at a time.
    const int64_t resident = (int64_t)n_cu * per_cu;
    const bool few = a.n_frontier < resident * 64;               // fewer groups of 64 than waves
    int64_t tail_nodes = fine_tail ? std::min<int64_t>(a.n_frontier, resident * 128) : 0;
    a.tail_shift = 4;
    if (ROWS) {
        // A frontier that leaves waves without a group of 64 is split so that all waves that it can occupy have one unit, of as few nodes as that
        // takes (four at least: rows up to MID_ROW IDs are sampled four at a time), or four times as fine where rows are long work.
        if (few) {
            int shift = 2;
            while (shift < 6 && (a.n_frontier >> shift) > resident) shift += 2;
            if (fine_if_few && shift > 2) shift -= 2;
            if (shift < 6) { a.tail_shift = shift; tail_nodes = a.n_frontier; }
        }
    } else if (fine_if_few && few) tail_nodes = a.n_frontier;    // sixteens throughout
    if (ROWS && a.place.n_batches) {
        const int64_t n_batches = a.place.n_batches, longest = a.place.longest;
        a.n_full_rounds = std::max<int64_t>(0, longest - (tail_nodes + n_batches - 1) / n_batches) / 64;
        a.n_full_groups = a.n_full_rounds * n_batches;
        a.n_units = a.n_full_groups + (((longest - a.n_full_rounds * 64 - 1) >> a.tail_shift) + 1) * n_batches;
    } else {
        a.n_full_groups = (a.n_frontier - tail_nodes) / 64;
        a.n_units = a.n_full_groups + (((a.n_frontier - a.n_full_groups * 64 - 1) >> a.tail_shift) + 1);
    }
    const int64_t n_work = a.n_tiles + a.n_units;
    const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>(n_work, resident));
    a.n_own = few ? a.n_units : std::max<int64_t>(0, (int64_t)grid - a.n_tiles);
    a.first_own = a.n_tiles % grid;                              // (waves without a tile, or without one more, come first)
    hipLaunchKernelGGL(SAMPLE, dim3(grid), dim3(64), 0, st, a);
    if (a.n_tiles > 0) hipLaunchKernelGGL(MERGE, dim3(merge_grid), dim3(64), 0, st, a);
    return RG_OK;
}

// The O(f) sampler.  A node with deg <= f copies its row; otherwise draw t reads the row at its drawn position (rg_device.h) and
// nothing else of the row.
//
// Bound by the walks of the drawn positions, some 110 vector instructions a step, and by the lines of the rows' IDs.  A walk takes 1.4 steps on
// average, but the longest of 64 takes four to six, which is what a lane per draw waits for.  So a wave takes a unit of nodes, up to
// POS_DRAWS draws, lists the draws that walk and deals them out to its lanes as they come free; positions are kept in LDS, and
// the rows read at all of them afterwards (233,000 nodes, 147 batches, fan-outs 25, 10, 29 M draws: a lane per draw / so 452 / 343 us).
// BY_PLACE (see ByPlace): an instantiation of its own (one kernel that looks whether units go by place, units by position: sampling 10 M nodes, fan-out 50, rows of 50,
// 2,007 / 2,019 us; 3.7 M, fan-out 10, 649 / 651).
constexpr int POS_IN_FLIGHT = 4;
struct PosNode {
    uint64_t state;
    int64_t row_begin, out;
    uint32_t deg, batch;
};
template <int MARK, bool BY_PLACE>
__global__ void __launch_bounds__(POS_THREADS) sample_positions_kernel(const int32_t *__restrict__ indices, NodeRecs rec, int64_t n_cur, uint32_t f, uint32_t unit_nodes,
                                                                       const int64_t *__restrict__ samp_off, int32_t *__restrict__ samp_nbr,
                                                                       ReachedMaps reached, ByPlace place, int64_t n_units)
{
    __shared__ PosNode all_nodes[POS_WAVES][64];
    __shared__ uint32_t all_pos[POS_WAVES][POS_DRAWS];
    __shared__ uint16_t all_walks[POS_WAVES][POS_DRAWS];
    constexpr uint32_t NO_DRAW = 0xFFFFFFFFu;                                  // (no position: rows are shorter than 2^31)
    const int lane = threadIdx.x & 63;
    const int wave = uni((int)threadIdx.x >> 6);
    PosNode *nodes = all_nodes[wave];
    uint32_t *pos = all_pos[wave];
    uint16_t *walks = all_walks[wave];
    const float per_node = 1.0f / (float)f;
    // draw d of the unit: node d / f, and its draw number (exact: where a unit has several nodes, d + 1/2 below 2^8 is 1/256 of a node or more away from any edge)
    auto node_of = [&](uint32_t d) { return unit_nodes == 1 ? 0u : (uint32_t)(((float)d + 0.5f) * per_node); };
    for (int64_t at = (int64_t)blockIdx.x * POS_WAVES + wave; at < n_units; at += (int64_t)gridDim.x * POS_WAVES) {
        int64_t i0 = at * unit_nodes, i_end = n_cur;
        if (BY_PLACE) {
            const uint32_t round = (uint32_t)at / place.n_batches, b = (uint32_t)at - round * place.n_batches;
            i0 = place.batch_off[b] + (int64_t)round * unit_nodes;
            i_end = place.batch_off[b + 1];
        }
        if (i0 >= i_end) continue;
        const uint32_t n_nodes = (uint32_t)min((int64_t)unit_nodes, i_end - i0);
        wave_lds_order();                                                      // the last unit's have been read
        uint32_t my_deg = 0;
        if ((uint32_t)lane < n_nodes) {
            const int64_t i = i0 + lane;
            my_deg = (uint32_t)rec.deg[i];
            nodes[lane] = PosNode{rec.state[i], rec.row_begin[i], samp_off[i], my_deg, rec.batch[i]};
        }
        const bool selects = my_deg > f && my_deg <= DRAW_SELECT;
        wave_lds_order();
        // (A node that is a unit by itself has rounds for what it draws, not for all of f: 100,000 rows of five IDs, fan-out 1,984, a schedule 344 us
        // with rounds for f, so 186, with a lane per draw 197.)
        const uint32_t n_draws = unit_nodes == 1 ? uni(min(f, nodes[0].deg)) : n_nodes * f;
        for (uint32_t d0 = 0; d0 < n_draws; d0 += POS_DRAWS) {
            const uint32_t n = uni(min((uint32_t)POS_DRAWS, n_draws - d0));
            uint32_t n_walks = 0;
            for (uint32_t q0 = 0; q0 < n; q0 += 64) {
                const uint32_t j = q0 + lane;
                bool walk = false;
                if (j < n) {
                    const uint32_t k = node_of(d0 + j), t = d0 + j - k * f, deg = nodes[k].deg;
                    walk = deg > f && deg > DRAW_SELECT;
                    pos[j] = walk ? NO_DRAW : deg > f ? draw32(nodes[k].state, t) : t < deg ? t : NO_DRAW;      // (a walk's until it has ended: nothing is read where a loop failed to end one)
                }
                const unsigned long long m = ballot64(walk);
                if (walk) walks[n_walks + lanes_below(m, lane)] = (uint16_t)j;
                n_walks = uni(n_walks + (uint32_t)__popcll(m));
            }
            wave_lds_order();
            // Rows selected from: the draws of a node follow from one another, so a node's lane goes through them, the random words at hand (a lane
            // per draw that repeated all draws before its own / so, schedules of 2.45 M nodes, fan-outs 15, 10, 5 3,440 / 2,478 us, 50, 50 4,352 / 3,099).
            if (selects) {
                uint64_t free_slots = low_lanes((int)my_deg);
                for (uint32_t t = 0; t < f; ++t) {                             // (a unit of such rows is one round: f < DRAW_SELECT)
                    const uint32_t p = nth_set_bit(free_slots, __umulhi(pos[lane * f + t], my_deg - t));
                    free_slots &= ~(1ull << p);
                    pos[lane * f + t] = p;
                }
            }
            // One step of every lane's walk; lanes whose walk has ended take the next ones of the list.  All lanes go round together until the last
            // walk has ended: the counts are the wave's, in scalar registers, and the barrier at the loop's end is its one way back (with a way back
            // for lanes that walk on, the compiler made a loop of its own of it, in which they went round without the others).
            uint32_t next = 64, left = n_walks, j = 0, deg = 0, n_bits = 0, x = 0;
            uint64_t S = 0;
            auto take = [&](uint32_t w) {
                j = walks[w];
                const uint32_t k = node_of(d0 + j);
                x = d0 + j - k * f;
                deg = nodes[k].deg;
                S = nodes[k].state;
                n_bits = 32u - (uint32_t)__clz((int)(deg - 1u));
            };
            bool on = (uint32_t)lane < n_walks;
            if (on) take((uint32_t)lane);
            while (left != 0u) {
                bool ended = false;
                if (on) {
                    x = feistel(x, n_bits, S);
                    ended = x < deg;
                    if (ended) pos[j] = x;
                }
                const unsigned long long m = ballot64(ended);
                const uint32_t w = next + (uint32_t)lanes_below(m, lane);
                const uint32_t n_ended = (uint32_t)__popcll(m);
                next = uni(next + n_ended);
                left = uni(left - n_ended);
                if (ended) {
                    on = w < n_walks;
                    if (on) take(w);
                }
                __builtin_amdgcn_wave_barrier();
            }
            wave_lds_order();
            for (uint32_t q0 = 0; q0 < n; q0 += 64 * POS_IN_FLIGHT) {
                int32_t u[POS_IN_FLIGHT];
                uint32_t k[POS_IN_FLIGHT], p[POS_IN_FLIGHT];
#pragma unroll
                for (int q = 0; q < POS_IN_FLIGHT; ++q) {
                    const uint32_t jq = q0 + 64 * q + lane;
                    p[q] = jq < n ? pos[jq] : NO_DRAW;
                    k[q] = jq < n ? node_of(d0 + jq) : 0u;
                    if (p[q] != NO_DRAW) u[q] = indices[nodes[k[q]].row_begin + p[q]];
                }
#pragma unroll
                for (int q = 0; q < POS_IN_FLIGHT; ++q)
                    if (p[q] != NO_DRAW) {
                        const uint32_t d = d0 + q0 + 64 * q + lane;
                        samp_nbr[nodes[k[q]].out + (d - k[q] * f)] = u[q];
                        mark_reached<MARK>(reached_of<MARK>(reached, nodes[k[q]].batch), (uint32_t)u[q]);
                    }
            }
            wave_lds_order();                                                  // the positions have been read
        }
    }
}

// ---------------------------------------------------------------- the samples marked in the reached bitmaps
// Bound by reading the samples once per piece of the bitmap.  A workgroup puts MARK_WORDS words of one batch's bitmap
// together in LDS from all of the batch's samples, or a part of them, and writes them and the flags of the groups that
// hold bits: nothing scattered leaves the compute unit.  Marked one by one from the sampling kernels, the memory system takes 25 G
// atomic ORs or 88 G byte stores a second and the kernels carry the address arithmetic.  233 k nodes, 29 M samples: 0.04 ms; 2.45 M nodes, 167 M samples:
// 0.30, and the launches that marked bytes themselves 3.9 -> 2.2 ms; 146 M samples in three hops: 0.20, launches that marked
// bits 10.6 -> 9.6.  A lane reads four IDs at a time: one at a time, twice as many loads of a quarter the size in flight, 424 us instead of 327 and 328 instead of 293.
// The pieces of a batch run on one XCD (workgroup g runs on XCD g mod 8) at about the same time and share the reads; the
// batches left over from whole eights are dealt out over all XCDs, or one batch would have an eighth of the chip.
constexpr int MARK_THREADS = 1024;
constexpr int MARK_WORDS = 38400;                        // a piece's words at most: 150 KB of LDS, 1,228,800 IDs
constexpr int MARK_XCDS = 8;
constexpr int MARK_IN_FLIGHT = 4;                        // loads of four IDs
constexpr uint64_t MARK_SPARSE = 512, MARK_MANY = 1 << 21, MARK_CROWD = 64;      // see marks_want_a_pass
constexpr uint64_t MARK_PASS = 320 << 10, MARK_ROUND = 240 << 10, MARK_FULL = 32768;
constexpr int64_t MARK_PART = 1 << 18;                   // samples per part, at least, where there are too few pieces to fill the chip

__global__ void __launch_bounds__(MARK_THREADS) mark_pass_kernel(const int32_t *__restrict__ samp_nbr, const int64_t *__restrict__ samp_off, const int64_t *__restrict__ batch_off,
                                                                 uint32_t n_batches, uint32_t pieces, uint32_t parts, uint32_t piece_words, ReachedMaps m)
{
    extern __shared__ __align__(16) uint32_t bits[];     // [piece_words], read in fours
    const uint32_t per_batch = pieces * parts, whole = n_batches / MARK_XCDS * MARK_XCDS, rest = n_batches - whole;
    uint32_t b, at;                                      // the batch, and which of its workgroups
    if (blockIdx.x < whole * per_batch) {
        const uint32_t r = blockIdx.x / MARK_XCDS;
        b = r / per_batch * MARK_XCDS + blockIdx.x % MARK_XCDS;
        at = r % per_batch;
    } else {
        const uint32_t r = blockIdx.x - whole * per_batch;
        b = whole + r % rest;
        at = r / rest;
    }
    const uint32_t piece = at % pieces, part = at / pieces;
    for (uint32_t w = threadIdx.x; w < piece_words; w += MARK_THREADS) bits[w] = 0u;
    __syncthreads();
    const int64_t first = samp_off[batch_off[b]], n = samp_off[batch_off[b + 1]] - first;
    const int64_t lo = first + n * part / parts, hi = first + n * (part + 1) / parts;
    const uint32_t id0 = piece * piece_words * 32u, n_ids = piece_words * 32u;
    auto mark = [&](uint32_t id) {
        const uint32_t u = id - id0;
        if (u < n_ids) atomicOr(&bits[u >> 5], 1u << (u & 31));
    };
    const int64_t whole_end = lo + (hi - lo) / 4 * 4;            // (vectors need no more than the alignment of an ID)
    // (Each round's loads are under way while the bits of the round before are set: a read of four IDs and its marks by turns 321 us, so 300, on the 167 M samples.)
    auto load = [&](int64_t j0, u32x4 (&to)[MARK_IN_FLIGHT]) {
#pragma unroll
        for (int q = 0; q < MARK_IN_FLIGHT; ++q) to[q] = *reinterpret_cast<const u32x4_dword_aligned *>(samp_nbr + min(j0 + q * 4 * MARK_THREADS, whole_end - 4));      // (past the end: the last ones again)
    };
    auto mark_all = [&](int64_t j0, const u32x4 (&u)[MARK_IN_FLIGHT]) {
#pragma unroll
        for (int q = 0; q < MARK_IN_FLIGHT; ++q)
            if (j0 + q * 4 * MARK_THREADS < whole_end) { mark(u[q].x); mark(u[q].y); mark(u[q].z); mark(u[q].w); }      // (thousands of threads' marks on the last ones' words would queue up: 98 batches of 41,000 samples 14.5 us, so 8.3)
    };
    constexpr int64_t ROUND = 4 * MARK_IN_FLIGHT * MARK_THREADS;
    if (whole_end > lo) {
        u32x4 x[MARK_IN_FLIGHT], y[MARK_IN_FLIGHT];
        int64_t j0 = lo + 4 * threadIdx.x;
        load(j0, x);
        while (j0 < whole_end) {
            load(j0 + ROUND, y);
            mark_all(j0, x);
            j0 += ROUND;
            if (j0 >= whole_end) break;
            load(j0 + ROUND, x);
            mark_all(j0, y);
            j0 += ROUND;
        }
    }
    if (whole_end + threadIdx.x < hi) mark((uint32_t)samp_nbr[whole_end + threadIdx.x]);
    __syncthreads();
    // a thread per group of eight words: written where it holds bits (the map is clear otherwise), its flag set
    const uint64_t word0 = (uint64_t)piece * piece_words;
    uint32_t *map = m.words + (uint64_t)b * m.words_per_batch + word0;
    uint8_t *flags = m.flags + (((uint64_t)b * m.words_per_batch + word0) >> 3);
    const uint32_t n_groups = (uint32_t)(min((uint64_t)piece_words, m.words_per_batch - word0) >> 3);
    for (uint32_t g = threadIdx.x; g < n_groups; g += MARK_THREADS) {
        const uint4 x = *reinterpret_cast<const uint4 *>(bits + 8 * g), y = *reinterpret_cast<const uint4 *>(bits + 8 * g + 4);
        if ((x.x | x.y | x.z | x.w | y.x | y.y | y.z | y.w) == 0u) continue;
        if (parts == 1) {
            *reinterpret_cast<uint4 *>(map + 8 * g) = x;
            *reinterpret_cast<uint4 *>(map + 8 * g + 4) = y;
        } else {
            const uint32_t w[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (w[k]) (void)__hip_atomic_fetch_or(map + 8 * g + k, w[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        flags[g] = 1;
    }
}

// Every piece reads all samples of its batch, so the pieces are as few as LDS allows, of equal size; one more where that
// costs no further round of workgroups, since a workgroup then has fewer bits to set (2.45 M nodes in two pieces / three: 147 batches of
// 1.1 M samples in 294 or 441 workgroups on 256 compute units 345 / 327 us, 196 batches of 0.7 M in 392 or 588 233 / 293).  So are those of a bitmap of
// more than MARK_FULL words that would fit one piece (1.1 M nodes, 75 batches of 0.6 M samples in one piece, two parts / in two pieces 160 / 72 us).
static uint32_t mark_pieces(const ReachedMaps &m, uint32_t beta, int n_cu)
{
    const uint64_t least = (m.words_per_batch + MARK_WORDS - 1) / MARK_WORDS, cus = (uint64_t)n_cu;
    const auto rounds = [&](uint64_t pieces) { return (pieces * beta + cus - 1) / cus; };
    return (uint32_t)(m.words_per_batch > MARK_FULL && rounds(least + 1) == rounds(least) ? least + 1 : least);
}
static uint32_t mark_piece_words(const ReachedMaps &m, uint32_t pieces) { return (uint32_t)(((m.words_per_batch + pieces - 1) / pieces + 7) / 8 * 8); }

// By a pass or by the sampling kernels themselves.  The pass clears and looks through the words of every batch's bitmap, some
// 6 us per 128 KB of LDS and compute unit, and 8 us for itself, more where a few workgroups have all the samples; an atomic OR
// costs 25 to 40 ps where little hides it, next to nothing while rows are read, and more where many meet on a word.  So the pass
// (schedules, marked by the kernels / by the pass)
//  - from one sample per MARK_SPARSE IDs of bitmap on: 2.45 M nodes, one hop, 1.6 M samples, keys sampler one per 2,816 685 / 758 us, 1,432
//    616 / 604, 710 449 / 426, 355 347 / 319; the positions sampler, whose launch is shorter, is faster by the pass at one per 1,531 already (524 / 503, 766 389 / 371,
//    383 311 / 277), and with fewer samples than MARK_MANY (1.6 M in 16 batches 236 / 203): the lines are the keys sampler's;
//  - there, from MARK_MANY samples on, or MARK_CROWD per word (one batch, fan-outs 50, 50, 2.45 M nodes, 0.5 M samples in the second hop
//    289 / 310, 1.0 M 321 / 317, 1.8 M 387 / 348, 3.3 M 508 / 393, 9.8 M 1,067 / 531; 30,000 nodes, one batch, 237 per word 329 / 263; ten batches on
//    40,000 nodes, 15 per word 243 / 247, 26 267 / 268, 46 300 / 297, 77 328 / 317);
//  - and where its workgroups are a quarter of the compute units and more, from as many samples on as cost what it does: MARK_PASS
//    and MARK_ROUND per round of full workgroups (113 batches on 76,000 nodes, 0.5 M samples 324 / 324, 1.0 M 372 / 369, 1.8 M 422 / 418, 3.3 M 495 / 479).
static bool marks_want_a_pass(const ReachedMaps &m, uint32_t beta, uint64_t n_marks, int n_cu)
{
    const uint64_t words = m.words_per_batch * (uint64_t)beta;
    if (n_marks * MARK_SPARSE < words * 32) return false;
    if (n_marks >= MARK_MANY || n_marks >= words * MARK_CROWD) return true;
    const uint32_t pieces = mark_pieces(m, beta, n_cu);
    const uint64_t units = (uint64_t)pieces * beta, cus = (uint64_t)n_cu;
    return units * 4 >= cus && n_marks >= MARK_PASS + MARK_ROUND * ((units + cus - 1) / cus) * mark_piece_words(m, pieces) / MARK_FULL;
}

static rg_status launch_mark_pass(const HopData &cur, uint32_t beta, const ReachedMaps &m, int n_cu, hipStream_t st)
{
    if (cur.n_samples == 0) return RG_OK;
    const uint32_t pieces = mark_pieces(m, beta, n_cu), piece_words = mark_piece_words(m, pieces);
    // a few batches of many samples are read in parts, whose bits are ORed into the map
    const uint64_t units = (uint64_t)pieces * beta;
    const uint32_t parts = (uint32_t)std::max<int64_t>(1, std::min<int64_t>(cur.n_samples / beta / MARK_PART, n_cu / (int64_t)units));
    const uint64_t grid = (uint64_t)beta * pieces * parts;
    if (grid > 0x7FFFFFFFull) { set_error("rg_build_schedule: %llu pieces of bitmaps in one hop", (unsigned long long)grid); return RG_ERANGE; }
    RG_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(mark_pass_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, MARK_WORDS * (int)sizeof(uint32_t)));
    hipLaunchKernelGGL(mark_pass_kernel, dim3((unsigned)grid), dim3(MARK_THREADS), piece_words * sizeof(uint32_t), st, cur.samp_nbr, cur.samp_off, cur.off_dev, beta, pieces,
                       parts, piece_words, m);
    RG_HIP(hipGetLastError());
    return RG_OK;
}

// Samples hop `hop` of every batch: fills cur.samp_off / samp_nbr / n_samples and marks the reached-ID bitmaps.
// tmp: scratch of this hop alone.  hubs_allowed: hub rows may be looked for, *looked_for_hubs: they were, which takes
// memory that the hop can do without.
// also_read_dev (or NULL): one more device value copied to *also_read_host behind the hop's own readback; if it
// comes back non-zero the hop stops there (the caller is about to refuse its input).
rg_status sample_hop(const rg_graph *g, HopData &cur, uint32_t beta, const uint64_t *batch_seed, uint32_t hop, uint32_t fanout,
                     uint32_t sampler, const ReachedMaps &reached, Arena &keep, Arena &tmp, int n_cu,
                     hipStream_t st, bool hubs_allowed, bool *looked_for_hubs, const unsigned long long *also_read_dev, unsigned long long *also_read_host)
{
    const int64_t n_cur = cur.off_host[beta];
    const int64_t n_chunks = (n_cur + NODE_CHUNK - 1) / NODE_CHUNK;
    const ByPlace place = by_place(cur, beta, g->n_nodes);
    // Hub rows (see hub_sample_kernel): where the table of a row is shared by the batches of an epoch -- behind the seeds,
    // which hold a node once.
    HubTable hubs{INT32_MAX, nullptr, nullptr, nullptr, nullptr};
    const char *forced_line = getenv("RAPIDGNN_HUB_ROWS");                            // same results either way; for tests and tuning
    if (hubs_allowed) {
        double line = hop > 0 && beta >= HUB_BATCHES ? hub_line(g->n_nodes, fanout) : 2147483647.0;
        if (forced_line) line = std::max(atof(forced_line), 4.0 * RG_MAX_FANOUT);
        if (sampler == RG_SAMPLER_KEYS && fanout > 0 && fanout <= HUB_MAX_FANOUT && line <= (double)g->n_nodes)
            hubs.min_deg = std::max((int32_t)std::min(line, 2147483647.0), BIG_ROW + 1);
    }
    const bool look_for_hubs = *looked_for_hubs = hubs.min_deg != INT32_MAX;
    int64_t tile_piece = fanout <= (uint32_t)ROWS_FANOUT && (hop == 0 || beta < HUB_BATCHES) && !look_for_hubs && n_cur < (int64_t)n_cu * SMALL_FRONTIER ? SMALL_PIECE : TILE_PIECE;
    uint32_t *count = nullptr, *chunk_hub = nullptr;
    unsigned long long *chunk_sum = nullptr;
    int64_t *samp_base = nullptr, *tile_base = nullptr;
    NodeRecs rec{nullptr, nullptr, nullptr, nullptr};
    RG_TRY(tmp.dev_n<uint32_t>((uint64_t)n_cur, &count));
    RG_TRY(tmp.dev_n<unsigned long long>((uint64_t)n_chunks, &chunk_sum));
    RG_TRY(tmp.dev_n<int64_t>((uint64_t)n_chunks + 1, &samp_base));
    RG_TRY(tmp.dev_n<int64_t>((uint64_t)n_chunks + 1, &tile_base));
    RG_TRY(tmp.dev_n<int64_t>((uint64_t)n_cur, &rec.row_begin));
    RG_TRY(tmp.dev_n<int32_t>((uint64_t)n_cur, &rec.deg));
    RG_TRY(tmp.dev_n<uint32_t>((uint64_t)n_cur, &rec.batch));
    RG_TRY(tmp.dev_n<uint64_t>((uint64_t)n_cur, &rec.state));
    RG_TRY(keep.dev_n<int64_t>((uint64_t)n_cur + 1, &cur.samp_off));
    unsigned long long sums[DEG_SUMS] = {}, *sum_deg_dev = nullptr;       // see node_records_kernel
    unsigned long long sum_parts[DEG_SUMS * DEG_SUM_SLOTS];
    const int n_sums = look_for_hubs ? DEG_SUMS : DEG_SUMS - 1;
    const size_t sum_bytes = (size_t)n_sums * DEG_SUM_SLOTS * sizeof(unsigned long long);
    const size_t hub_cleared = look_for_hubs ? sizeof(HubCounts) + HUB_SLOTS * sizeof(uint32_t) : 0;      // behind the sums, cleared with them
    unsigned long long *next_work = nullptr;                              // the sampling launch's work counter, cleared with them too (sixteen bytes in front)
    RG_TRY(tmp.dev(2 * sizeof(unsigned long long) + sum_bytes + hub_cleared, (void **)&next_work));
    RG_HIP(hipMemsetAsync(next_work, 0, 2 * sizeof(unsigned long long) + sum_bytes + hub_cleared, st));
    sum_deg_dev = next_work + 2;
    if (look_for_hubs) {
        hubs.counts = reinterpret_cast<HubCounts *>(sum_deg_dev + DEG_SUMS * DEG_SUM_SLOTS);
        hubs.keys = reinterpret_cast<uint32_t *>(hubs.counts + 1);
        RG_TRY(tmp.dev(HUB_SLOTS * (sizeof(HubRow) + sizeof(int32_t)), (void **)&hubs.rows));
        hubs.list = reinterpret_cast<int32_t *>(hubs.rows + HUB_SLOTS);
        RG_TRY(tmp.dev_n<uint32_t>((uint64_t)n_chunks, &chunk_hub));
    }
    const dim3 grid((unsigned)n_chunks), block(NODE_THREADS);
    auto launch_records = [&] {
        // (the chunks that begin in a batch, at most one more than fit it)
        const dim3 record_grid(place.n_batches ? (unsigned)((place.longest / NODE_CHUNK + 2) * beta) : (unsigned)n_chunks);
        if (look_for_hubs)
            hipLaunchKernelGGL(node_records_kernel<true>, record_grid, block, 0, st, g->indptr, cur.ids, n_cur, cur.off_dev, beta, batch_seed, hop, fanout, tile_piece, rec, count, chunk_sum,
                               chunk_hub, (int64_t)g->n_nodes, sum_deg_dev, hubs, place.n_batches ? 1 : 0);
        else
            hipLaunchKernelGGL(node_records_kernel<false>, record_grid, block, 0, st, g->indptr, cur.ids, n_cur, cur.off_dev, beta, batch_seed, hop, fanout, tile_piece, rec, count, chunk_sum,
                               chunk_hub, (int64_t)g->n_nodes, sum_deg_dev, hubs, place.n_batches ? 1 : 0);
        hipLaunchKernelGGL(scan_chunks_kernel, dim3(1), dim3(CHUNK_SCAN_THREADS), 0, st, chunk_sum, (const uint32_t *)nullptr, n_chunks, samp_base, tile_base, cur.samp_off + n_cur);
    };
    {
        ScopedTimer tm(KG_OFFSETS, st);
        launch_records();
        hipLaunchKernelGGL(sample_offsets_kernel, grid, block, 0, st, count, n_cur, samp_base, cur.samp_off);
        RG_HIP(hipGetLastError());
    }
    int64_t n_tiles = 0;                          // of the rows that are no hub rows, at first
    HubCounts hub_counts{};
    {
        Readback rb(st);
        RG_TRY(rb.add(sum_parts, sum_deg_dev, sum_bytes));
        RG_TRY(rb.add(&cur.n_samples, cur.samp_off + n_cur, sizeof(int64_t)));
        RG_TRY(rb.add(&n_tiles, tile_base + n_chunks, sizeof(int64_t)));
        if (look_for_hubs) RG_TRY(rb.add(&hub_counts, hubs.counts, sizeof(hub_counts)));
        if (also_read_dev) RG_TRY(rb.add(also_read_host, also_read_dev, sizeof(unsigned long long)));     // a value the caller wants behind the same wait
        RG_TRY(rb.wait());
        for (int k = 0; k < DEG_SUM_SLOTS; ++k)
            for (int q = 0; q < n_sums; ++q) sums[q] += sum_parts[n_sums * k + q];
        if (also_read_dev && *also_read_host != 0) return RG_OK;        // the caller refuses the build: nothing more to launch
    }
    bool inline_marks = reached.paired || !marks_want_a_pass(reached, beta, (uint64_t)cur.n_samples, n_cu);
    if (const char *force = getenv("RAPIDGNN_MARK_PASS"); force && !reached.paired) inline_marks = force[0] == '0';       // same results either way; for tests and tuning
    RG_TRY(keep.dev_n<int32_t>((uint64_t)cur.n_samples, &cur.samp_nbr));
    if (sampler == RG_SAMPLER_POSITIONS) {
        if (fanout > 0 && n_cur > 0) {
            ScopedTimer tm(KG_SAMPLER, st);
            const PositionUnits units = position_units(n_cur, cur.n_samples, fanout, place.n_batches != 0, place.longest, beta, n_cu, reached.paired);
#define RG_POSITIONS(M, P) hipLaunchKernelGGL((sample_positions_kernel<M, P>), dim3(units.grid), dim3(POS_THREADS), 0, st, g->indices, rec, n_cur, fanout, units.nodes, cur.samp_off, cur.samp_nbr, reached, place, units.n)
            if (inline_marks && place.n_batches) RG_POSITIONS(MARK_BITS, true);
            else if (inline_marks) RG_POSITIONS(MARK_BITS, false);
            else if (place.n_batches) RG_POSITIONS(MARK_NONE, true);
            else RG_POSITIONS(MARK_NONE, false);
#undef RG_POSITIONS
            RG_HIP(hipGetLastError());
            if (!inline_marks) RG_TRY(launch_mark_pass(cur, beta, reached, n_cu, st));
        }
        return RG_OK;
    }
    if (tile_piece == SMALL_PIECE && sums[4] > (uint64_t)FEW_TILES * n_cu) {      // not so few after all: the same records, the rows in larger pieces
        tile_piece = TILE_PIECE;
        n_tiles = (int64_t)sums[4];
        ScopedTimer tm(KG_OFFSETS, st);
        launch_records();
    }
    // The hub rows: as jobs of hub_sample_kernel where that saves more than it costs, the tables and jobs find memory and the
    // rows turn out to be in order; else as tile jobs like the other long rows.
    const uint64_t n_hub_jobs = look_for_hubs ? sums[4] : 0, n_hub_tiles = sums[5];
    HubBucket *buckets = nullptr;
    HubJob *jobs = nullptr;
    bool hub_jobs = n_hub_jobs > 0 && n_hub_jobs <= 0x7FFFFFFFull && (forced_line || n_hub_tiles >= (uint64_t)HUB_TILES_PER_CU * n_cu) &&
                    tmp.dev_spare(hub_counts.buckets * sizeof(HubBucket), (void **)&buckets) && tmp.dev_spare(n_hub_jobs * sizeof(HubJob), (void **)&jobs);
    if (hub_jobs) {
        {
            ScopedTimer tm(KG_SAMPLER, st);
            RG_HIP(hipMemsetAsync(buckets, 0xFF, hub_counts.buckets * sizeof(HubBucket), st));
            const uint32_t per_row = std::max<uint32_t>(64, std::min<uint32_t>(1024, 64u * (uint32_t)n_cu / hub_counts.n_rows));       // few rows, long ones: the workgroups of the chip shared out among them
            hipLaunchKernelGGL(hub_table_kernel, dim3(per_row, hub_counts.n_rows), dim3(256), 0, st, g->indices, g->n_nodes, hubs, buckets);
            hipLaunchKernelGGL(hub_jobs_kernel, dim3((unsigned)n_chunks), dim3(NODE_THREADS), 0, st, count, cur.ids, n_cur, chunk_hub, hubs, jobs);
            RG_HIP(hipGetLastError());
        }
        Readback rb(st);
        RG_TRY(rb.add(&hub_counts, hubs.counts, sizeof(hub_counts)));
        RG_TRY(rb.wait());
        hub_jobs = hub_counts.damaged == 0;
    }
    if (!hub_jobs && n_hub_jobs > 0) {        // the tiles in front of each chunk once more, with those of the hub rows
        tmp.free_one(buckets);                // (the host has waited for what read them)
        tmp.free_one(jobs);
        n_tiles += (int64_t)n_hub_tiles;
        ScopedTimer tm(KG_OFFSETS, st);
        hipLaunchKernelGGL(scan_chunks_kernel, dim3(1), dim3(CHUNK_SCAN_THREADS), 0, st, chunk_sum, chunk_hub, n_chunks, samp_base, tile_base, cur.samp_off + n_cur);
    }
    if (fanout == 0) n_tiles = 0;             // nothing is drawn; every sample is empty
    int32_t *tile_out = nullptr;
    TileRecs tile{nullptr, nullptr, nullptr, nullptr, nullptr};
    RG_TRY(tmp.dev_n<int32_t>((uint64_t)n_tiles * fanout, &tile_out));
    RG_TRY(tmp.dev_n<int64_t>((uint64_t)n_tiles, &tile.node));
    RG_TRY(tmp.dev_n<int32_t>((uint64_t)n_tiles, &tile.t));
    RG_TRY(tmp.dev_n<int64_t>((uint64_t)n_tiles, &tile.begin));
    RG_TRY(tmp.dev_n<int32_t>((uint64_t)n_tiles, &tile.len));
    RG_TRY(tmp.dev_n<uint64_t>((uint64_t)n_tiles, &tile.state));
    if (n_tiles > 0) {
        ScopedTimer tm(KG_OFFSETS, st);
        hipLaunchKernelGGL(tile_nodes_kernel, dim3((unsigned)n_chunks), dim3(NODE_THREADS), 0, st, count, n_cur, tile_base, hub_jobs ? TILES_OF_ROWS : TILES_OF_ROWS | TILES_OF_HUB_ROWS, tile);
        hipLaunchKernelGGL(tile_records_kernel, dim3((unsigned)((n_tiles + 255) / 256)), dim3(256), 0, st, rec.row_begin, rec.deg, rec.state, n_tiles, tile_piece, tile);
    }
    int32_t *tile_order = nullptr;
    bool group_tiles = n_tiles >= (int64_t)n_cu * 64 && n_tiles <= 0x7FFFFFFF;     // fewer jobs than two rounds of the resident waves: nothing to bring together
    if (const char *force = getenv("RAPIDGNN_GROUP_TILES")) group_tiles = force[0] == '1' && n_tiles > 0 && n_tiles <= 0x7FFFFFFF;     // same results either way; for tests and tuning
    if (group_tiles) {
        int bits = 12;                                    // about 32 jobs to a bucket: buckets that share pieces only widen the set in flight
        while (bits < 20 && ((int64_t)32 << bits) < n_tiles) ++bits;
        const uint64_t n_buckets = (uint64_t)1 << bits;
        int32_t *cnt = nullptr, *rank = nullptr;
        int64_t *off = nullptr;
        RG_TRY(tmp.dev_n<int32_t>(n_buckets, &cnt));
        RG_TRY(tmp.dev_n<int32_t>((uint64_t)n_tiles, &rank));
        RG_TRY(tmp.dev_n<int64_t>(n_buckets + 1, &off));
        RG_TRY(tmp.dev_n<int32_t>((uint64_t)n_tiles, &tile_order));
        ScopedTimer tm(KG_OFFSETS, st);
        RG_HIP(hipMemsetAsync(cnt, 0, n_buckets * sizeof(int32_t), st));
        const dim3 grid((unsigned)((n_tiles + 255) / 256));
        hipLaunchKernelGGL(tile_bucket_count_kernel, grid, dim3(256), 0, st, tile.begin, n_tiles, bits, cnt, rank);
        RG_TRY(scan_i32_to_i64(cnt, off, (int64_t)n_buckets, tmp, st));
        hipLaunchKernelGGL(tile_bucket_place_kernel, grid, dim3(256), 0, st, tile.begin, n_tiles, bits, off, rank, tile_order);
        RG_HIP(hipGetLastError());
    }

    if (fanout > 0 && n_cur > 0) {
        // Rows of up to SHORT_ROW IDs are taken four at a time wherever a frontier has any.  Same samples either way; at fan-outs above 64
        // RAPIDGNN_SHORT_ROWS = 0 forces one row per wave.
        bool short_rows = sums[2] != 0;
        if (const char *force = getenv("RAPIDGNN_SHORT_ROWS")) short_rows = force[0] != '0';
        const uint32_t need = fanout + 64;
        int merge_span = 64;                              // tiles per look of a merging wave: 64 if that still occupies the chip's waves
        while (merge_span > 1 && n_tiles / merge_span < (int64_t)n_cu * 32) merge_span >>= 1;
        const unsigned merge_grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((n_tiles + merge_span - 1) / merge_span, (int64_t)n_cu * 64));
        HopArgs a{};
        a.indices = g->indices;
        a.frontier = cur.ids; a.n_frontier = n_cur;
        a.min_deg = short_rows ? SHORT_ROW : 0;
        a.rec = rec;
        a.fanout = fanout;
        a.samp_off = cur.samp_off; a.samp_nbr = cur.samp_nbr;
        a.tile = tile; a.n_tiles = n_tiles; a.tile_out = tile_out; a.tile_piece = tile_piece;
        a.merge_span = merge_span;
        a.tile_order = tile_order;
        a.reached = reached;
        a.next_work = next_work;
        a.guess_scale = 1.0f;
        a.place = place;
        if (const char *scale = getenv("RAPIDGNN_GUESS_SCALE")) a.guess_scale = std::min(std::max((float)atof(scale), 1e-3f), 1e3f);      // same results either way; for tests
        ScopedTimer tm(KG_SAMPLER, st);
        if (hub_jobs) {
            const char *range = getenv("RAPIDGNN_HUB_RANGE");                         // same results either way; for tests
            const HubArgs ha{g->indices, g->n_nodes, hubs.rows, buckets, jobs, (uint32_t)n_hub_jobs, range ? std::max((float)atof(range), 0.0f) : 1.0f, rec, fanout, cur.samp_off, cur.samp_nbr, reached};
            const dim3 grid(std::min<uint32_t>((uint32_t)n_hub_jobs, (uint32_t)n_cu * 64)), block(HUB_THREADS);
            if (inline_marks) hipLaunchKernelGGL(hub_sample_kernel<MARK_BITS>, grid, block, 0, st, ha);
            else hipLaunchKernelGGL(hub_sample_kernel<MARK_NONE>, grid, block, 0, st, ha);
            RG_HIP(hipGetLastError());
        }
        // worth it where a group is long work: rows of a thousand IDs on average, tiles aside (short rows finish a
        // group of 64 in no time, and four times the requests to the work counter then cost more than the tail does;
        // measured: Medium, 2,500 IDs per row, 4 % faster; large_sparse and partition_share, a few hundred, 1-8 % slower)
        const unsigned long long ids_here = sums[1] - (short_rows ? sums[3] : 0), rows_here = (unsigned long long)n_cur - (short_rows ? sums[2] : 0);
        const bool fine_tail = ids_here >= 1024ull * rows_here;
        // a frontier that does not give every resident wave a group of 64 (the seed hop) is split finer from rows of 256 IDs on
        const bool fine_if_few = ids_here >= 256ull * rows_here;
#define RG_LAUNCH(...) RG_TRY((launch_hop<__VA_ARGS__>(a, n_cu, merge_grid, fine_tail, fine_if_few, st)))
#define RG_HOP(CAP)                                                                                                   \
    do {                                                                                                              \
        if (inline_marks && short_rows) RG_LAUNCH(false, sample_kernel<CAP, MARK_BITS, true>, sample_merge_kernel<CAP, MARK_BITS>);  \
        else if (inline_marks) RG_LAUNCH(false, sample_kernel<CAP, MARK_BITS, false>, sample_merge_kernel<CAP, MARK_BITS>);   \
        else if (short_rows) RG_LAUNCH(false, sample_kernel<CAP, MARK_NONE, true>, sample_merge_kernel<CAP, MARK_NONE>);      \
        else RG_LAUNCH(false, sample_kernel<CAP, MARK_NONE, false>, sample_merge_kernel<CAP, MARK_NONE>);                     \
    } while (0)
        if (fanout <= (uint32_t)ROWS_FANOUT) {
            if (inline_marks) RG_LAUNCH(true, sample_rows_kernel<MARK_BITS>, sample_merge_kernel<128, MARK_BITS>);
            else RG_LAUNCH(true, sample_rows_kernel<MARK_NONE>, sample_merge_kernel<128, MARK_NONE>);
        } else if (need <= 256) RG_HOP(256);
        else if (need <= 512) RG_HOP(512);
        else if (need <= 1024) RG_HOP(1024);
        else RG_HOP(2048);
#undef RG_HOP
#undef RG_LAUNCH
        RG_HIP(hipGetLastError());
        if (!inline_marks) RG_TRY(launch_mark_pass(cur, beta, reached, n_cu, st));
    }
    return RG_OK;
}

}  // namespace rg

