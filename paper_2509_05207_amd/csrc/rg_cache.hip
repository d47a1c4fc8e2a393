// rg_build_cache: access-frequency tally, TopHot selection, VectorPull into the
// device table, and the per-batch routing plans (Alg. 1 steps 2-4).
#include "rg_internal.h"
#include "rg_device.h"

#include <algorithm>
#include <type_traits>

namespace rg {

thread_local std::atomic<uint64_t> *tls_table_bytes_sink = nullptr;

// ---------------------------------------------------------------- a6: freq(v)
// Every batch's input set is duplicate free, so each listed ID adds one.
// The counters are uint32_t, or -- when no frequency can exceed 255 (at most 255 batches over the epochs given) --
// uint8_t, four to a word: an add of 1 << 8 * (id & 3) to the word can then never carry into the next counter.  A
// tally of 10^8 nodes is a quarter of the bytes to clear and to read in every later pass, and small enough for
// its scattered adds to stay in the last-level cache.
template <typename F>
__global__ void tally_kernel(const int32_t *__restrict__ ids, int64_t n, F *__restrict__ freq)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint32_t v = (uint32_t)ids[i];
        if (sizeof(F) == 1) atomicAdd(reinterpret_cast<uint32_t *>(freq) + (v >> 2), 1u << (8 * (v & 3)));
        else atomicAdd(reinterpret_cast<uint32_t *>(freq) + v, 1u);
    }
}

// freq += the frequencies an epoch's schedule already holds (computed from its bitmaps when it was built); FIRST: freq holds nothing yet
template <typename F, bool FIRST>
__global__ void add_epoch_freq_kernel(const uint32_t *__restrict__ epoch_freq, int64_t n, F *__restrict__ freq)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) freq[i] = (F)((FIRST ? 0u : (uint32_t)freq[i]) + epoch_freq[i]);
}

// The uint8_t tally as the uint32_t array the cache's view hands out (made when first asked for).
__global__ void widen_freq_kernel(const uint8_t *__restrict__ freq8, int64_t n, uint32_t *__restrict__ freq)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) freq[i] = freq8[i];
}

// ---------------------------------------------------------------- a7: TopHot
// Candidates: remote IDs with freq > 0.  The K-th largest frequency t is found
// by a most-significant-digit-first radix select over the candidates' freq
// values (8-bit digits, as many passes as max_freq needs; LDS-privatised digit
// histograms merged with atomics).  Selected: freq > t, plus the first r
// candidates with freq == t in ascending ID order (the tie-break), found by one
// prefix sum over the nodes that also yields the slots: cache_ids ascending.
struct SelectState {
    uint32_t prefix;        // digits of t decided so far (high bits), already shifted into place
    uint32_t prefix_mask;   // which bits of prefix are decided
    uint64_t want;          // how many still to take among candidates matching the prefix
    uint64_t n_candidates;  // set by the first pass
    uint32_t take_all;      // 1: K >= #candidates, every candidate is selected
    uint32_t t;             // final threshold
    uint64_t r;             // how many of the freq == t candidates to take
    uint64_t k_eff;
};

constexpr int TOPK_THREADS = 256;
constexpr int DIGIT_BITS = 8;
constexpr int DIGIT_BINS = 1 << DIGIT_BITS;
constexpr int SEL_PER_THREAD = 8;         // runs of eight consecutive nodes: a quarter of a slot-map record per thread (sixteen measured 8 % slower over the byte tally)
constexpr int SEL_TILE = TOPK_THREADS * SEL_PER_THREAD;
constexpr int BIN_COPIES = 64;            // the digit histogram is kept in this many copies, summed when a digit is chosen

// QUADS: a lane takes four consecutive nodes per round (one 16-byte and one 4-byte load; is_local must be 4-byte
// aligned), the few nodes after the last whole quad one by one.
template <bool QUADS>
__global__ void __launch_bounds__(TOPK_THREADS) digit_histogram_kernel(const uint32_t *__restrict__ freq, const uint8_t *__restrict__ is_local, int64_t n,
                                                                       const SelectState *__restrict__ stp, int shift,
                                                                       unsigned long long *__restrict__ bins)
{
    __shared__ unsigned int h[DIGIT_BINS];
    for (int k = threadIdx.x; k < DIGIT_BINS; k += TOPK_THREADS) h[k] = 0;
    __syncthreads();
    const uint32_t prefix = stp->prefix, pmask = stp->prefix_mask;
    if (stp->take_all) return;
    auto count = [&](uint32_t fv, uint32_t local) {
        if (fv != 0 && !local && (fv & pmask) == prefix) atomicAdd(&h[(fv >> shift) & (DIGIT_BINS - 1)], 1u);
    };
    int64_t done = 0;
    if (QUADS) {
        auto count4 = [&](const uint4 fv, uint32_t loc) {
            if ((fv.x | fv.y | fv.z | fv.w) == 0u) return;                     // most nodes are never listed
            count(fv.x, loc & 0xFFu); count(fv.y, (loc >> 8) & 0xFFu); count(fv.z, (loc >> 16) & 0xFFu); count(fv.w, loc >> 24);
        };
        // a workgroup reads one contiguous span of quads, four independent loads of each kind in flight per lane
        const int64_t n_quads = n >> 2;
        const int64_t span = (n_quads + gridDim.x - 1) / gridDim.x;
        const int64_t q_end = min(n_quads, (int64_t)(blockIdx.x + 1) * span);
        int64_t q = (int64_t)blockIdx.x * span + threadIdx.x;
        for (; q + 3 * TOPK_THREADS < q_end; q += 4 * TOPK_THREADS) {
            uint4 fv[4]; uint32_t loc[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) fv[u] = reinterpret_cast<const uint4 *>(freq)[q + u * TOPK_THREADS];
#pragma unroll
            for (int u = 0; u < 4; ++u) loc[u] = reinterpret_cast<const uint32_t *>(is_local)[q + u * TOPK_THREADS];
#pragma unroll
            for (int u = 0; u < 4; ++u) count4(fv[u], loc[u]);
        }
        for (; q < q_end; q += TOPK_THREADS) count4(reinterpret_cast<const uint4 *>(freq)[q], reinterpret_cast<const uint32_t *>(is_local)[q]);
        done = n_quads << 2;
    }
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t v = done + t0; v < n; v += stride) count(freq[v], is_local[v]);
    __syncthreads();
    // workgroups spread their adds over BIN_COPIES copies of the bins: few digits are in use, and thousands of adds
    // to the same few addresses would queue up behind each other
    unsigned long long *mine = bins + (size_t)(blockIdx.x % BIN_COPIES) * DIGIT_BINS;
    for (int k = threadIdx.x; k < DIGIT_BINS; k += TOPK_THREADS)
        if (h[k]) atomicAdd(&mine[k], (unsigned long long)h[k]);
}

// The same for the uint8_t tally: one digit, so no prefix to match.  WIDE (is_local 16-byte aligned; the tally always
// is): a lane takes sixteen consecutive nodes per round, one 16-byte load of each array, and visits only the
// bytes that are candidates (non-zero count, not local).
__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t w) { return (w | ((w & 0x7F7F7F7Fu) + 0x7F7F7F7Fu)) & 0x80808080u; }   // bit 7 of every non-zero byte

// The candidates among four and among sixteen consecutive nodes into the histogram h (LDS); how many they are.
__device__ __forceinline__ int count_word(unsigned int *h, uint32_t fw, uint32_t lw)
{
    uint32_t cand = nonzero_bytes(fw) & ~nonzero_bytes(lw);
    const int n_here = __popc(cand);
    while (cand) {
        const int top = __ffs((int)cand) - 1;                  // bit 7 of the candidate's byte
        cand &= cand - 1;
        atomicAdd(&h[(fw >> (top - 7)) & 0xFFu], 1u);
    }
    return n_here;
}
__device__ __forceinline__ int count16(unsigned int *h, const uint4 fv, const uint4 lv)
{
    if ((fv.x | fv.y | fv.z | fv.w) == 0u) return 0;          // most nodes are never listed
    return count_word(h, fv.x, lv.x) + count_word(h, fv.y, lv.y) + count_word(h, fv.z, lv.z) + count_word(h, fv.w, lv.w);
}

// A wave takes SEL_TILE consecutive nodes at a time and also leaves their number of candidates, which is the select passes' total of those nodes wherever all
// candidates are taken (111 M nodes: a pass of 58 us that need not be).  In the last tile a lane has sixteen nodes to a load as far as they go, then
// one (one after the other from its start: 10 M nodes, the selection 46 us -> 52).
template <bool WIDE>
__global__ void __launch_bounds__(TOPK_THREADS) digit_histogram8_kernel(const uint8_t *__restrict__ freq, const uint8_t *__restrict__ is_local, int64_t n,
                                                                        unsigned long long *__restrict__ bins, uint64_t *__restrict__ block_tot)
{
    __shared__ unsigned int h[DIGIT_BINS];
    for (int k = threadIdx.x; k < DIGIT_BINS; k += TOPK_THREADS) h[k] = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    constexpr int LOADS = SEL_TILE / (64 * 16), IN_FLIGHT = 8;
    static_assert(SEL_TILE == LOADS * 64 * 16, "a wave's loads are a tile");
    auto count_tile = [&](int64_t t, auto is_whole) {
        constexpr bool WHOLE = decltype(is_whole)::value;
        const int64_t first = t * SEL_TILE, left = n - first;
        int here = 0;
        if constexpr (WIDE) {
            const uint4 *fq = reinterpret_cast<const uint4 *>(freq + first), *lq = reinterpret_cast<const uint4 *>(is_local + first);
            uint4 f[LOADS], l[LOADS];
#pragma unroll
            for (int k = 0; k < LOADS; ++k) {
                if (!WHOLE) f[k] = l[k] = make_uint4(0u, 0u, 0u, 0u);
                if (WHOLE || (k * 64 + lane + 1) * 16 <= left) { f[k] = fq[k * 64 + lane]; l[k] = lq[k * 64 + lane]; }
            }
#pragma unroll
            for (int k = 0; k < LOADS; ++k) here += count16(h, f[k], l[k]);
            if (!WHOLE && lane < (left & 15)) {
                const int64_t v = n - (left & 15) + lane;
                if (freq[v] != 0 && !is_local[v]) { atomicAdd(&h[freq[v]], 1u); ++here; }
            }
        } else {
            for (int64_t j = lane; j < (WHOLE ? SEL_TILE : left); j += 64 * IN_FLIGHT) {
                uint8_t f[IN_FLIGHT], l[IN_FLIGHT];
#pragma unroll
                for (int k = 0; k < IN_FLIGHT; ++k) f[k] = WHOLE || j + 64 * k < left ? freq[first + j + 64 * k] : 0;
#pragma unroll
                for (int k = 0; k < IN_FLIGHT; ++k) l[k] = f[k] != 0 ? is_local[first + j + 64 * k] : 1;
#pragma unroll
                for (int k = 0; k < IN_FLIGHT; ++k)
                    if (!l[k]) { atomicAdd(&h[f[k]], 1u); ++here; }
            }
        }
        for (int o = 32; o > 0; o >>= 1) here += __shfl_down(here, o, 64);
        if (lane == 0) block_tot[t] = (uint64_t)here << 32;
    };
    // a wave's tiles are consecutive; the last one of all may be a part
    const int64_t n_whole = n / SEL_TILE, n_tiles = (n + SEL_TILE - 1) / SEL_TILE, n_waves = (int64_t)gridDim.x * (TOPK_THREADS / 64);
    const int64_t per_wave = (n_tiles + n_waves - 1) / n_waves, wave = (int64_t)blockIdx.x * (TOPK_THREADS / 64) + (threadIdx.x >> 6);
    const int64_t t_end = min(n_whole, (wave + 1) * per_wave);
    for (int64_t t = wave * per_wave; t < t_end; ++t) count_tile(t, std::true_type{});
    if (n_whole < n_tiles && wave == n_whole / per_wave) count_tile(n_whole, std::false_type{});
    __syncthreads();
    unsigned long long *mine = bins + (size_t)(blockIdx.x % BIN_COPIES) * DIGIT_BINS;
    for (int k = threadIdx.x; k < DIGIT_BINS; k += TOPK_THREADS)
        if (h[k]) atomicAdd(&mine[k], (unsigned long long)h[k]);
}

// One workgroup of DIGIT_BINS threads: sum the copies of each bin (and clear them for the next pass), then find the bin
// from the top in which `want` is covered.  Bound by the latency of its loads and of whatever runs in one thread: the
// copies are read eight at a time and the bins above each bin added up by a scan (bins walked by one thread, copies
// read one after the other: 15-20 us; so: under 5).
__global__ void __launch_bounds__(DIGIT_BINS) choose_digit_kernel(SelectState *__restrict__ stp, unsigned long long *__restrict__ bins_copies, int shift,
                                                                  int first_pass, uint64_t K)
{
    __shared__ unsigned long long wave_sum[DIGIT_BINS / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int bin = DIGIT_BINS - 1 - (int)threadIdx.x;                 // thread 0 has the top bin
    unsigned long long mine = 0;
    for (int c0 = 0; c0 < BIN_COPIES; c0 += 8) {
        unsigned long long x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = bins_copies[(size_t)(c0 + u) * DIGIT_BINS + bin];
#pragma unroll
        for (int u = 0; u < 8; ++u) { mine += x[u]; bins_copies[(size_t)(c0 + u) * DIGIT_BINS + bin] = 0; }
    }
    unsigned long long incl = mine;                                    // of this bin and the bins above it
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long y = __shfl_up(incl, d, 64);
        if (lane >= d) incl += y;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    unsigned long long total = 0;
    for (int w = 0; w < DIGIT_BINS / 64; ++w) {
        if (w < wave) incl += wave_sum[w];
        total += wave_sum[w];
    }
    const SelectState was = *stp;
    __syncthreads();                                                   // everyone has read the state before one thread writes it
    const uint64_t want = first_pass ? K : was.want;
    const bool all = first_pass ? K >= total : was.take_all != 0;
    if (all) {
        if (first_pass && threadIdx.x == 0) {
            SelectState st = was;
            st.n_candidates = total; st.want = K; st.take_all = 1; st.t = 0; st.r = 0; st.k_eff = total;
            *stp = st;
        }
        return;
    }
    // the bin in which the count from the top first reaches `want`; the last one if none does
    const unsigned long long above = incl - mine;
    const bool chosen = bin > 0 ? above + mine >= want && (threadIdx.x == 0 || above < want) : above < want || threadIdx.x == 0;
    if (!chosen) return;
    SelectState st = was;
    if (first_pass) { st.n_candidates = total; st.k_eff = K; }
    st.want = want - above;                                            // still to take inside this digit
    st.prefix |= (uint32_t)bin << shift;
    st.prefix_mask |= (uint32_t)(DIGIT_BINS - 1) << shift;
    if (shift == 0) { st.t = st.prefix; st.r = st.want; }
    *stp = st;
}

// Packed counters per node: high 32 bits = selected outright (freq > t), low 32 bits = tied (freq == t).
__device__ __forceinline__ uint64_t classify_node(uint32_t fv, uint8_t local, const SelectState &st)
{
    if (fv == 0 || local) return 0;
    if (st.take_all || fv > st.t) return (uint64_t)1 << 32;
    return fv == st.t ? 1ull : 0ull;
}


// The eight consecutive nodes of a thread, classified.  ALIGNED8 (is_local 8-byte aligned; freq always is, and a
// thread's first node is a multiple of eight): two 16-byte loads and one 8-byte load when all eight exist.
template <bool ALIGNED8>
__device__ __forceinline__ void classify_eight(const uint32_t *__restrict__ freq, const uint8_t *__restrict__ is_local, int64_t first, int64_t n,
                                               const SelectState &st, uint64_t *c /* [8] */)
{
    if (ALIGNED8 && first + 8 <= n) {
        const uint4 a = *reinterpret_cast<const uint4 *>(freq + first), b = *reinterpret_cast<const uint4 *>(freq + first + 4);
        const uint64_t loc = *reinterpret_cast<const uint64_t *>(is_local + first);
        const uint32_t fv[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int k = 0; k < 8; ++k) c[k] = classify_node(fv[k], (uint8_t)(loc >> (8 * k)), st);
        return;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int64_t v = first + k;
        c[k] = v < n ? classify_node(freq[v], is_local[v], st) : 0;
    }
}
// The same over the uint8_t tally: one 8-byte load of each array.
template <bool ALIGNED8>
__device__ __forceinline__ void classify_eight(const uint8_t *__restrict__ freq, const uint8_t *__restrict__ is_local, int64_t first, int64_t n,
                                               const SelectState &st, uint64_t *c /* [8] */)
{
    if (ALIGNED8 && first + 8 <= n) {
        const uint64_t fw = *reinterpret_cast<const uint64_t *>(freq + first);
        if (fw == 0ull) {
#pragma unroll
            for (int k = 0; k < 8; ++k) c[k] = 0;
            return;
        }
        const uint64_t loc = *reinterpret_cast<const uint64_t *>(is_local + first);
#pragma unroll
        for (int k = 0; k < 8; ++k) c[k] = classify_node((uint32_t)(fw >> (8 * k)) & 0xFFu, (uint8_t)(loc >> (8 * k)), st);
        return;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int64_t v = first + k;
        c[k] = v < n ? classify_node(freq[v], is_local[v], st) : 0;
    }
}
// The SEL_PER_THREAD consecutive nodes of a thread.
template <bool ALIGNED8, typename F>
__device__ __forceinline__ void classify_mine(const F *__restrict__ freq, const uint8_t *__restrict__ is_local, int64_t first, int64_t n,
                                              const SelectState &st, uint64_t (&c)[SEL_PER_THREAD])
{
#pragma unroll
    for (int h = 0; h < SEL_PER_THREAD / 8; ++h) classify_eight<ALIGNED8>(freq, is_local, first + 8 * h, n, st, c + 8 * h);
}

__device__ __forceinline__ uint64_t block_exclusive_scan_u64(uint64_t x, uint64_t *total, uint64_t *lds)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint64_t incl = x;
    for (int d = 1; d < 64; d <<= 1) {
        uint64_t y = __shfl_up(incl, d, 64);
        if (lane >= d) incl += y;
    }
    if (lane == 63) lds[wave] = incl;
    __syncthreads();
    uint64_t base = 0, tot = 0;
    for (int w = 0; w < TOPK_THREADS / 64; ++w) {
        const uint64_t s = lds[w];
        if (w < wave) base += s;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return base + incl - x;
}

template <bool ALIGNED8, typename F>
__global__ void __launch_bounds__(TOPK_THREADS) select_block_totals(const F *__restrict__ freq, const uint8_t *__restrict__ is_local, int64_t n,
                                                                    const SelectState *__restrict__ stp, uint64_t *__restrict__ block_tot)
{
    __shared__ uint64_t lds[TOPK_THREADS / 64];
    const SelectState st = *stp;
    if (sizeof(F) == 1 && st.take_all) return;                 // (digit_histogram8_kernel has left the totals)
    const int64_t n_blocks = (n + SEL_TILE - 1) / SEL_TILE;
    for (int64_t block = blockIdx.x; block < n_blocks; block += gridDim.x) {
        const int64_t first = block * SEL_TILE + (int64_t)threadIdx.x * SEL_PER_THREAD;
        uint64_t c[SEL_PER_THREAD];
        classify_mine<ALIGNED8, F>(freq, is_local, first, n, st, c);
        uint64_t s = 0;
#pragma unroll
        for (int k = 0; k < SEL_PER_THREAD; ++k) s += c[k];
        uint64_t tot;
        (void)block_exclusive_scan_u64(s, &tot, lds);
        if (threadIdx.x == 0) block_tot[block] = tot;
    }
}

// The exclusive scan of the per-workgroup totals, in two levels: every workgroup scans its own SCAN_TILE totals in
// place and leaves their sum in tile_tot; one workgroup then scans tile_tot (select_scan_totals); the emit pass adds
// the two.  (10^8 nodes are 54,000 totals: one workgroup alone spends longer walking them than a pass over the nodes' flags takes.)
constexpr int SCAN_TILE = TOPK_THREADS * 8;
__global__ void __launch_bounds__(TOPK_THREADS) select_scan_tiles(uint64_t *__restrict__ block_tot, int64_t n_blocks, uint64_t *__restrict__ tile_tot)
{
    __shared__ uint64_t lds[TOPK_THREADS / 64];
    const int64_t i0 = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * 8;
    uint64_t x[8], sum = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) { x[k] = i0 + k < n_blocks ? block_tot[i0 + k] : 0; sum += x[k]; }
    uint64_t tot;
    uint64_t run = block_exclusive_scan_u64(sum, &tot, lds);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        if (i0 + k < n_blocks) block_tot[i0 + k] = run;
        run += x[k];
    }
    if (threadIdx.x == 0) tile_tot[blockIdx.x] = gridDim.x > 1 ? tot : 0;      // (a single tile has nothing in front: no second level)
}

// One workgroup; a thread takes eight consecutive totals per round.
__global__ void __launch_bounds__(TOPK_THREADS) select_scan_totals(uint64_t *__restrict__ block_tot, int64_t n_blocks)
{
    __shared__ uint64_t lds[TOPK_THREADS / 64];
    uint64_t carry = 0;
    for (int64_t base = 0; base < n_blocks; base += (int64_t)TOPK_THREADS * 8) {
        const int64_t i0 = base + (int64_t)threadIdx.x * 8;
        uint64_t x[8], sum = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) { x[k] = i0 + k < n_blocks ? block_tot[i0 + k] : 0; sum += x[k]; }
        uint64_t tot;
        uint64_t run = carry + block_exclusive_scan_u64(sum, &tot, lds);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            if (i0 + k < n_blocks) block_tot[i0 + k] = run;
            run += x[k];
        }
        carry += tot;
    }
}

template <bool ALIGNED8, typename F>
__global__ void __launch_bounds__(TOPK_THREADS) select_emit_kernel(const F *__restrict__ freq, const uint8_t *__restrict__ is_local, int64_t n,
                                                                   const SelectState *__restrict__ stp, const uint64_t *__restrict__ block_base,
                                                                   const uint64_t *__restrict__ tile_base, int32_t *__restrict__ cache_ids, SlotRec *__restrict__ slot_pairs,
                                                                   const int32_t *__restrict__ row_of, uint32_t *__restrict__ fill_codes)
{
    // fill_codes[slot]: where VectorPull finds the row of the node in that slot (a8), written here while the node is at hand
    __shared__ uint64_t lds[TOPK_THREADS / 64];
    __shared__ uint16_t lists[TOPK_THREADS / 64][64 * SEL_PER_THREAD];
    const SelectState st = *stp;
    const int64_t first = (int64_t)blockIdx.x * SEL_TILE + (int64_t)threadIdx.x * SEL_PER_THREAD;
    uint32_t local8 = 0;                                    // which of this thread's eight nodes are local
    if (ALIGNED8 && first + SEL_PER_THREAD <= n) {
        const uint64_t loc = *reinterpret_cast<const uint64_t *>(is_local + first);
#pragma unroll
        for (int k = 0; k < SEL_PER_THREAD; ++k)
            if ((loc >> (8 * k)) & 0xFFull) local8 |= 1u << k;
    } else {
#pragma unroll
        for (int k = 0; k < SEL_PER_THREAD; ++k)
            if (first + k < n && is_local[first + k]) local8 |= 1u << k;
    }
    uint64_t c[SEL_PER_THREAD];
    classify_mine<ALIGNED8, F>(freq, is_local, first, n, st, c);
    uint64_t s = 0;
#pragma unroll
    for (int k = 0; k < SEL_PER_THREAD; ++k) s += c[k];
    uint64_t tot;
    uint64_t run = block_base[blockIdx.x] + tile_base[blockIdx.x / SCAN_TILE] + block_exclusive_scan_u64(s, &tot, lds);
    static_assert(SEL_PER_THREAD == 8, "four consecutive lanes make up one pair of the slot map");
    const uint64_t gt_start = run >> 32, eq_start = run & 0xFFFFFFFFull;
    const int64_t slot0 = (int64_t)(gt_start + (eq_start < st.r ? eq_start : st.r));      // of the first selected node of this thread
    uint32_t mine = 0;                                      // which of this thread's eight nodes are selected
#pragma unroll
    for (int k = 0; k < SEL_PER_THREAD; ++k) {
        const bool sel = first + k < n && ((c[k] >> 32) != 0 || (c[k] == 1 && (run & 0xFFFFFFFFull) < st.r));
        if (sel) mine |= 1u << k;
        run += c[k];
    }
    // The wave's selected nodes are listed first and then taken one per lane: rows are asked for and IDs and entries stored 64 at a time,
    // not by the one or two lanes that have a node selected at the same place of their eight (111 M nodes, 3.9 M of them selected, 198 us so, 146 with the list).
    const int lane = threadIdx.x & 63;
    uint16_t *list = lists[threadIdx.x >> 6];
    const int64_t wave_slot0 = __shfl(slot0, 0, 64), wave_first = first - lane * SEL_PER_THREAD;
    int at = (int)(slot0 - wave_slot0);
#pragma unroll
    for (int k = 0; k < SEL_PER_THREAD; ++k)
        if ((mine >> k) & 1u) list[at++] = (uint16_t)(lane * SEL_PER_THREAD + k);
    const int n_listed = __shfl(at, 63, 64);
    wave_lds_order();
    for (int j = lane; j < n_listed; j += 64) {
        const int64_t v = wave_first + list[j];
        cache_ids[wave_slot0 + j] = (int32_t)v;
        fill_codes[wave_slot0 + j] = make_code(false, false, (uint32_t)row_of[v]);
    }
    // the slot map's record for 32 node IDs (see slot_lookup): bits from four lanes, the rank from the first of them
    uint32_t word = mine << (8 * (lane & 3)), lword = local8 << (8 * (lane & 3));
    word |= __shfl_xor(word, 1, 64); lword |= __shfl_xor(lword, 1, 64);
    word |= __shfl_xor(word, 2, 64); lword |= __shfl_xor(lword, 2, 64);
    if ((lane & 3) == 0) {
        slot_pairs[first >> 5] = make_uint4(word, (uint32_t)slot0, lword, 0u);
    }
}

// The slot map as the int32_t[n_nodes] array the cache's view hands out (made when first asked for).
__global__ void widen_slots_kernel(const SlotRec *__restrict__ pairs, int64_t n, int32_t *__restrict__ slot_of)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) slot_of[v] = slot_lookup(pairs, (uint32_t)v);
}

// ---------------------------------------------------------------- a5/a9: routing plan
// Where a request for v's feature row is served from.  One record of the slot map says whether v
// is local and whether (and where) it is cached; row_of is read for the others only, and not even for those where the
// tables hold the nodes' rows in the order of their IDs: row_of is then a rank, which the record gives too.
struct RouteSources {
    const int32_t *row_of;
    const SlotRec *slot_pairs;       // see slot_lookup
    const uint32_t *not_ranks;       // dev: 0 = row_of[v] is the number of local (of remote) IDs in front of v, for every v; NULL: not known
};

// Reading row_of is two thirds of what a plan over many input nodes moves (a batch's IDs touch nearly every line of it), so it
// is first checked, in one pass, for being the ranks that the slot map knows anyway.  The pass reads row_of once and is a few
// launches: 8 to 16 us where there is little to save, so it wants RANK_INPUTS_PER_NODE input nodes per node, and RANK_INPUTS
// (plans that read row_of / that know the ranks: 0.6 M inputs on 30,000 nodes 120 / 131 us, 8.5 M on 1 M 161 / 171, 17 M on
// 1 M 266 / 243, 42 M on 1 M 475 / 376, 28 M on 233,000 281 / 281, 84 M on 233,000 876 / 793).
constexpr int64_t RANK_INPUTS_PER_NODE = 8;
constexpr int64_t RANK_INPUTS = 1 << 24;
// local_cnt[r] = local IDs among record r's 32
__global__ void local_counts_kernel(const SlotRec *__restrict__ recs, int64_t n_recs, int32_t *__restrict__ local_cnt)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r < n_recs) local_cnt[r] = __popc(recs[r].z);
}
// The records' w, and whether row_of is what they make of it: *not_ranks = 1 if any node's differs.
__global__ void row_ranks_kernel(SlotRec *recs, int64_t n, const int64_t *__restrict__ local_off, const int32_t *__restrict__ row_of, uint32_t *__restrict__ not_ranks)
{
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool differs = false;
    if (v < n) {
        const uint32_t z = recs[v >> 5].z, bit = 1u << (v & 31);
        const int64_t in_front = local_off[v >> 5], local = in_front + __popc(z & (bit - 1));
        differs = row_of[v] != ((z & bit) ? local : v - local);
        if ((v & 31) == 0) recs[v >> 5].w = (uint32_t)in_front;
    }
    if (__ballot(differs) != 0ull && (threadIdx.x & 63) == 0) *not_ranks = 1u;
}

// route[j] = where ids[j] is served from, for every listed input node, and how many local rows and misses each PLAN_GROUP of
// them holds (misses in the upper half of the word).  Nothing is added up per batch here: the tiles of a batch run at the
// same time, and two adds per tile to the batch's counters queued up behind each other (an epoch of 80 M input nodes in
// 196 batches: 712 us with the adds, 494 without them).  The kernel waits for its dependent reads (ID, slot-map record, row), so
// each kind is asked for by all of a thread's positions before the first answer is used; a thread's positions come in fours, which
// are one load of IDs and one store of codes.
// A route is a code or, where codes have met a row they cannot hold (*no_codes = 1; see make_code), an entry.
constexpr int PLAN_THREADS = 256;
constexpr int PLAN_QUADS = 2;
constexpr int PLAN_PER_THREAD = 4 * PLAN_QUADS;
constexpr int PLAN_TILE = PLAN_THREADS * PLAN_PER_THREAD;
constexpr int PLAN_GROUP = 2 * PLAN_THREADS;             // positions to a word of counts: a quad of two waves
constexpr int PLAN_TILE_GROUPS = PLAN_TILE / PLAN_GROUP;

template <typename ROUTE>
__global__ void __launch_bounds__(PLAN_THREADS) plan_kernel(const int32_t *__restrict__ ids, int64_t n, RouteSources rs, uint32_t last_remote, ROUTE *__restrict__ route,
                                                            uint32_t *__restrict__ no_codes, uint32_t *__restrict__ group_counts /* [tiles * PLAN_TILE_GROUPS] */)
{
    static_assert(PLAN_GROUP == 4 * 64 * 2 && PLAN_THREADS == 4 * 64, "two waves' quads are a group");
    typedef uint32_t id4 __attribute__((ext_vector_type(4), aligned(4)));              // (an allocator of the caller's may align less than sixteen bytes)
    typedef ROUTE route4 __attribute__((ext_vector_type(4), aligned(sizeof(ROUTE))));
    __shared__ uint32_t red[PLAN_QUADS][PLAN_THREADS / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool ranks = rs.not_ranks && *rs.not_ranks == 0u;
    const int64_t j0 = (int64_t)blockIdx.x * PLAN_TILE + 4 * (int64_t)threadIdx.x;      // of the first quad; the next one 4 * PLAN_THREADS on
    uint32_t v[PLAN_PER_THREAD];
    SlotRec rec[PLAN_PER_THREAD];
    int32_t row[PLAN_PER_THREAD];
#pragma unroll
    for (int q = 0; q < PLAN_QUADS; ++q) {
        const int64_t j = j0 + q * 4 * PLAN_THREADS;
        if (j + 4 <= n) {
            const id4 x = *reinterpret_cast<const id4 *>(ids + j);
            v[4 * q] = x.x; v[4 * q + 1] = x.y; v[4 * q + 2] = x.z; v[4 * q + 3] = x.w;
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) v[4 * q + k] = (uint32_t)ids[min(j + k, n - 1)];      // (past the end: the last ID again, not used)
        }
    }
#pragma unroll
    for (int k = 0; k < PLAN_PER_THREAD; ++k) rec[k] = rs.slot_pairs[v[k] >> 5];
#pragma unroll
    for (int k = 0; k < PLAN_PER_THREAD; ++k) {
        const uint32_t bit = 1u << (v[k] & 31);
        // a cached row is at its rank among the cached IDs, the others at row_of
        if (rec[k].x & ~rec[k].z & bit) row[k] = (int32_t)(rec[k].y + __popc(rec[k].x & (bit - 1)));
        else if (ranks) {
            const uint32_t local = rec[k].w + __popc(rec[k].z & (bit - 1));
            row[k] = (int32_t)((rec[k].z & bit) ? local : v[k] - local);
        } else row[k] = rs.row_of[v[k]];
    }
    bool no_code = false;
#pragma unroll
    for (int q = 0; q < PLAN_QUADS; ++q) {
        const int64_t j = j0 + q * 4 * PLAN_THREADS;
        route4 r;
        uint32_t counts = 0;                               // of the wave's quad
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const SlotRec &here = rec[4 * q + k];
            const uint32_t bit = 1u << (v[4 * q + k] & 31), at = (uint32_t)row[4 * q + k];
            const bool local = (here.z & bit) != 0, cached = !local && (here.x & bit) != 0;
            if constexpr (sizeof(ROUTE) == 4) {
                no_code |= !fits_code(local, cached, at, last_remote);      // (past the end: the last ID's answer again)
                r[k] = make_code(local, cached, at);
            } else r[k] = make_entry(local ? TAG_LOCAL : cached ? TAG_CACHE : TAG_REMOTE, row[4 * q + k]);
            counts += (uint32_t)__popcll(__ballot(j + k < n && local)) + ((uint32_t)__popcll(__ballot(j + k < n && !local && !cached)) << 16);
        }
        if (j + 4 <= n) __builtin_nontemporal_store(r, reinterpret_cast<route4 *>(route + j));
        else {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (j + k < n) route[j + k] = r[k];
        }
        if (lane == 0) red[q][wave] = counts;
    }
    if (__ballot(no_code) != 0ull && lane == 0) *no_codes = 1u;
    __syncthreads();
    if (threadIdx.x < PLAN_TILE_GROUPS) {
        const int q = threadIdx.x / 2, w = threadIdx.x % 2 * 2;
        group_counts[(uint64_t)blockIdx.x * PLAN_TILE_GROUPS + threadIdx.x] = red[q][w] + red[q][w + 1];
    }
}

// What a route adds to a word of counts.
__device__ __forceinline__ uint32_t counts_of_route(int64_t e, uint32_t) { return entry_tag(e) == TAG_LOCAL ? 1u : entry_tag(e) == TAG_REMOTE ? 1u << 16 : 0u; }
__device__ __forceinline__ uint32_t counts_of_route(uint32_t c, uint32_t last_remote) { return c < CODE_NOT_LOCAL ? 1u : c <= last_remote ? 1u << 16 : 0u; }

// One workgroup per batch: its local rows and misses, those of the whole groups between its ends and of the routes in front of
// and behind them.  Bound by its dependent reads, of which there are two: the batch's ends, then everything else at once (a
// plan of 500,000 input nodes in 145 batches 5 us; with whole tiles counted and the entries of the end tiles read, 10.0).
constexpr int COUNT_THREADS = 256;
constexpr int COUNT_IN_FLIGHT = PLAN_GROUP / COUNT_THREADS;
template <typename ROUTE>
__global__ void __launch_bounds__(COUNT_THREADS) batch_counts_kernel(const ROUTE *__restrict__ route, uint32_t last_remote, const uint32_t *__restrict__ group_counts,
                                                                     const int64_t *__restrict__ batch_off, uint32_t n_batches, int64_t *__restrict__ counts /* [2 * batches]: local rows, then misses */)
{
    __shared__ int64_t part[2][COUNT_THREADS / 64];
    const uint32_t b = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t lo = batch_off[b], hi = batch_off[b + 1];
    const int64_t g_lo = (lo + PLAN_GROUP - 1) / PLAN_GROUP, g_hi = hi / PLAN_GROUP;      // whole groups [g_lo, g_hi), if any
    const int64_t front_end = g_lo <= g_hi ? g_lo * PLAN_GROUP : hi, back = g_lo <= g_hi ? g_hi * PLAN_GROUP : hi;
    uint32_t ends = 0;
#pragma unroll
    for (int k = 0; k < COUNT_IN_FLIGHT; ++k) {
        const int64_t j = lo + k * COUNT_THREADS + threadIdx.x, i = back + k * COUNT_THREADS + threadIdx.x;
        if (j < front_end) ends += counts_of_route(route[j], last_remote);
        if (i < hi) ends += counts_of_route(route[i], last_remote);
    }
    int64_t local = ends & 0xFFFFu, miss = ends >> 16;
    for (int64_t g = g_lo + threadIdx.x; g < g_hi; g += COUNT_THREADS) {
        const uint32_t c = group_counts[g];
        local += c & 0xFFFFu;
        miss += c >> 16;
    }
    for (int o = 32; o > 0; o >>= 1) { local += __shfl_down(local, o, 64); miss += __shfl_down(miss, o, 64); }
    if (lane == 0) { part[0][wave] = local; part[1][wave] = miss; }
    __syncthreads();
    if (threadIdx.x < 2) {
        int64_t c = 0;
        for (int w = 0; w < COUNT_THREADS / 64; ++w) c += part[threadIdx.x][w];
        counts[(uint64_t)threadIdx.x * n_batches + b] = c;
    }
}

// Whether row_of is ranks (see RouteSources): asked once, in the codes of the first plan that has room for it before they are
// written, so that it takes no memory of its own.
struct RankCheck {
    SlotRec *recs;
    int64_t n_nodes;
    uint32_t *not_ranks;             // dev
    bool pending;
};
static rg_status check_row_ranks(const RankCheck &c, const int32_t *row_of, void *room, Arena &tmp, hipStream_t st)
{
    const int64_t n_recs = (c.n_nodes + 31) / 32;
    int64_t *local_off = static_cast<int64_t *>(room);
    int32_t *local_cnt = reinterpret_cast<int32_t *>(local_off + n_recs + 1);
    RG_HIP(hipMemsetAsync(c.not_ranks, 0, sizeof(uint32_t), st));
    hipLaunchKernelGGL(local_counts_kernel, dim3((unsigned)((n_recs + 255) / 256)), dim3(256), 0, st, c.recs, n_recs, local_cnt);
    RG_TRY(scan_i32_to_i64(local_cnt, local_off, n_recs, tmp, st));
    hipLaunchKernelGGL(row_ranks_kernel, dim3((unsigned)((c.n_nodes + 255) / 256)), dim3(256), 0, st, c.recs, c.n_nodes, local_off, row_of, c.not_ranks);
    RG_HIP(hipGetLastError());
    return RG_OK;
}

// The plans of all epochs: routes, and counts per batch, which the host waits for once, behind the last epoch's.  What a plan
// keeps lives in `keep`; scratch in `tmp`.  no_codes: dev, 0; *codes: whether routes are codes, false on return if
// a row turned out to be out of their reach.
static rg_status launch_plans(const rg_schedule *const *epochs, RouteSources &rs, RankCheck &check, uint64_t k_eff, uint32_t *no_codes, bool *codes, Arena &keep, Arena &tmp,
                              hipStream_t st, std::vector<Plan> &plans)
{
    const uint32_t last_remote = last_remote_code(k_eff);
    std::vector<std::vector<int64_t>> counts(plans.size());
    std::vector<int64_t *> counts_of(plans.size(), nullptr);      // dev
    uint32_t no_codes_host = 0;
    for (size_t e = 0; e < plans.size(); ++e) {
        const rg_schedule *s = epochs[e];
        Plan &plan = plans[e];
        const uint32_t beta = s->n_batches;
        const HopData &h = s->hop[s->L];
        const int64_t n = beta ? h.off_host[beta] : 0, n_tiles = (n + PLAN_TILE - 1) / PLAN_TILE;
        if (*codes) RG_TRY(keep.dev_n<uint32_t>((uint64_t)n, &plan.code));
        else RG_TRY(keep.dev_n<int64_t>((uint64_t)n, &plan.entry));
        counts[e].assign(2 * (size_t)beta, 0);
        if (n == 0) continue;
        uint32_t *group_counts = nullptr;
        RG_TRY(tmp.dev_n<uint32_t>((uint64_t)n_tiles * PLAN_TILE_GROUPS, &group_counts));
        RG_TRY(tmp.dev_n<int64_t>(2 * (uint64_t)beta, &counts_of[e]));
        ScopedTimer tm(KG_PLAN, st);
        if (check.pending && *codes && (uint64_t)n * sizeof(uint32_t) >= (uint64_t)((check.n_nodes + 31) / 32 + 1) * (sizeof(int64_t) + sizeof(int32_t))) {
            RG_TRY(check_row_ranks(check, rs.row_of, plan.code, tmp, st));
            rs.not_ranks = check.not_ranks;
            check.pending = false;
        }
        auto launch = [&](auto *route) {
            using ROUTE = std::remove_pointer_t<decltype(route)>;
            hipLaunchKernelGGL(plan_kernel<ROUTE>, dim3((unsigned)n_tiles), dim3(PLAN_THREADS), 0, st, h.ids, n, rs, last_remote, route, no_codes, group_counts);
            hipLaunchKernelGGL(batch_counts_kernel<ROUTE>, dim3(beta), dim3(COUNT_THREADS), 0, st, route, last_remote, group_counts, h.off_dev, beta, counts_of[e]);
        };
        if (*codes) launch(plan.code);
        else launch(plan.entry);
        RG_HIP(hipGetLastError());
    }
    Readback rb(st);                                              // (from here on nothing leaves between a copy asked for and the wait)
    for (size_t e = 0; e < plans.size(); ++e)
        if (counts_of[e]) RG_TRY(rb.add(counts[e].data(), counts_of[e], counts[e].size() * sizeof(int64_t)));
    RG_TRY(rb.add(&no_codes_host, no_codes, sizeof(no_codes_host)));
    RG_TRY(rb.wait());
    if (no_codes_host != 0) *codes = false;
    for (size_t e = 0; e < plans.size(); ++e) {
        const rg_schedule *s = epochs[e];
        Plan &plan = plans[e];
        const HopData &h = s->hop[s->L];
        const uint32_t beta = s->n_batches;
        plan.schedule_uid = s->uid;
        plan.miss_off.assign((size_t)beta + 1, 0);
        plan.stats.assign(beta, rg_gather_stats{0, 0, 0, 0});
        for (uint32_t b = 0; b < beta; ++b) {
            rg_gather_stats &g = plan.stats[b];
            g.n_rows = (uint64_t)(h.off_host[b + 1] - h.off_host[b]);
            g.n_local = (uint64_t)counts[e][b];
            g.n_miss = (uint64_t)counts[e][(size_t)beta + b];
            g.n_hit = g.n_rows - g.n_local - g.n_miss;
            plan.miss_off[b + 1] = plan.miss_off[b] + (int64_t)g.n_miss;
        }
    }
    return RG_OK;                 // (the caller waits for the stream before `tmp` goes back)
}

static rg_status build_plans(const rg_schedule *const *epochs, RouteSources &rs, RankCheck &check, uint64_t k_eff, uint32_t *no_codes, Arena &keep, Arena &tmp,
                             hipStream_t st, std::vector<Plan> &plans)
{
    bool codes = true;
    if (const char *force = getenv("RAPIDGNN_PLAN_CODES")) codes = force[0] != '0';      // same results either way; for tests
    const bool tried = codes;
    RG_TRY(launch_plans(epochs, rs, check, k_eff, no_codes, &codes, keep, tmp, st, plans));
    if (codes || !tried) return RG_OK;
    for (Plan &p : plans) { keep.free_one(p.code); p.code = nullptr; }          // (the host has waited for what wrote them)
    return launch_plans(epochs, rs, check, k_eff, no_codes, &codes, keep, tmp, st, plans);
}

// The tally as uint32_t[n_nodes] for rg_cache_view: the array itself, or -- where the build counted in bytes -- a
// widened copy made at the first request (device memory from the cache's allocator; the call waits for the copy).
rg_status cache_freq_view(const rg_cache *cc, const uint32_t **out)
{
    rg_cache *c = const_cast<rg_cache *>(cc);
    std::lock_guard<std::mutex> lk(c->view_mu);
    if (!c->freq && c->freq8 && c->n_nodes > 0) {
        hipStream_t side = nullptr;
        RG_TRY(helper_stream(&side));
        uint32_t *wide = nullptr;
        RG_TRY(c->arena.dev_n<uint32_t>((uint64_t)c->n_nodes, &wide));
        const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((c->n_nodes + 255) / 256, 1 << 16));
        hipLaunchKernelGGL(widen_freq_kernel, dim3(grid), dim3(256), 0, side, c->freq8, c->n_nodes, wide);
        RG_HIP(hipGetLastError());
        RG_HIP(hipStreamSynchronize(side));
        c->freq = wide;
    }
    *out = c->freq;
    return RG_OK;
}

// slot_of as int32_t[n_nodes] for rg_cache_view, made from the slot map at the first request in the same way.
rg_status cache_slot_view(const rg_cache *cc, const int32_t **out)
{
    rg_cache *c = const_cast<rg_cache *>(cc);
    std::lock_guard<std::mutex> lk(c->view_mu);
    if (!c->slot_of && c->slot_pairs && c->n_nodes > 0) {
        hipStream_t side = nullptr;
        RG_TRY(helper_stream(&side));
        int32_t *wide = nullptr;
        RG_TRY(c->arena.dev_n<int32_t>((uint64_t)c->n_nodes, &wide));
        const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((c->n_nodes + 255) / 256, 1 << 16));
        hipLaunchKernelGGL(widen_slots_kernel, dim3(grid), dim3(256), 0, side, c->slot_pairs, c->n_nodes, wide);
        RG_HIP(hipGetLastError());
        RG_HIP(hipStreamSynchronize(side));
        c->slot_of = wide;
    }
    *out = c->slot_of;
    return RG_OK;
}

static rg_status build_cache_impl(const rg_schedule *const *epochs, uint32_t n_epochs, const rg_features *f, uint64_t K,
                                  const rg_allocator *a, hipStream_t st, rg_cache *c)
{
    const int64_t n = epochs[0]->n_nodes;
    c->n_nodes = n;
    c->row_bytes = f->row_bytes;
    c->stride = ((uint64_t)f->row_bytes + 15) / 16 * 16;
    c->remote_rows_seen = f->remote_rows;
    c->remote_is_device = is_device_memory(f->remote_rows);
    Arena tmp(a, st);
    RG_HIP(hipEventCreateWithFlags(&c->ev_fork, hipEventDisableTiming));
    RG_HIP(hipEventCreateWithFlags(&c->ev_join, hipEventDisableTiming));

    int dev = 0, n_cu = 256;
    RG_HIP(hipGetDevice(&dev));
    RG_HIP(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));

    // ---- a6: tally
    uint64_t max_freq = 0;
    bool from_bitmaps = false;
    for (uint32_t e = 0; e < n_epochs; ++e) { max_freq += epochs[e]->n_batches; from_bitmaps = from_bitmaps || epochs[e]->epoch_freq; }
    bool narrow = max_freq <= 255;                       // byte counters suffice
    if (const char *force = getenv("RAPIDGNN_NARROW_TALLY"); force && force[0] == '0') narrow = false;      // same results either way; for tests and tuning
    const uint64_t tally_bytes = narrow ? ((uint64_t)n + 15) / 16 * 16 : (uint64_t)n * sizeof(uint32_t);
    void *tally = nullptr;
    RG_TRY(c->arena.dev(tally_bytes ? tally_bytes : 16, &tally));
    if (narrow) c->freq8 = (uint8_t *)tally; else c->freq = (uint32_t *)tally;
    bool counted = false;                                // the tally holds counts (or zeros)
    for (uint32_t e = 0; e < n_epochs; ++e) {
        const rg_schedule *s = epochs[e];
        if (s->n_batches == 0) continue;
        const HopData &h = s->hop[s->L];
        const int64_t m = h.off_host[s->n_batches];
        if (m == 0) continue;
        ScopedTimer tm(KG_HIST, st);
        if (s->epoch_freq) {
            const dim3 grid((unsigned)((n + 255) / 256));
            if (narrow && counted) hipLaunchKernelGGL((add_epoch_freq_kernel<uint8_t, false>), grid, dim3(256), 0, st, s->epoch_freq, n, c->freq8);
            else if (narrow) hipLaunchKernelGGL((add_epoch_freq_kernel<uint8_t, true>), grid, dim3(256), 0, st, s->epoch_freq, n, c->freq8);
            else if (counted) hipLaunchKernelGGL((add_epoch_freq_kernel<uint32_t, false>), grid, dim3(256), 0, st, s->epoch_freq, n, c->freq);
            else hipLaunchKernelGGL((add_epoch_freq_kernel<uint32_t, true>), grid, dim3(256), 0, st, s->epoch_freq, n, c->freq);
            counted = true;
            continue;
        }
        if (!counted) RG_HIP(hipMemsetAsync(tally, 0, tally_bytes, st));
        counted = true;
        const unsigned grid = (unsigned)std::min<int64_t>((m + 255) / 256, (int64_t)n_cu * 32);
        if (narrow) hipLaunchKernelGGL(tally_kernel<uint8_t>, dim3(grid), dim3(256), 0, st, h.ids, m, c->freq8);
        else hipLaunchKernelGGL(tally_kernel<uint32_t>, dim3(grid), dim3(256), 0, st, h.ids, m, c->freq);
    }
    if (!counted) RG_HIP(hipMemsetAsync(tally, 0, tally_bytes, st));
    RG_HIP(hipGetLastError());

    // ---- a7: TopHot
    SelectState *stp = nullptr;
    unsigned long long *bins = nullptr;
    // cleared together: the state of the selection, what the plans report of their codes, the digit's bins
    struct SelectScratch { SelectState state; uint32_t no_codes, pad; unsigned long long bins[BIN_COPIES * DIGIT_BINS]; };
    SelectScratch *sel = nullptr;
    RG_TRY(tmp.dev_n<SelectScratch>(1, &sel));
    RG_HIP(hipMemsetAsync(sel, 0, sizeof(SelectScratch), st));
    stp = &sel->state;
    bins = sel->bins;
    int bits = 1;
    while (bits < 32 && (max_freq >> bits) != 0) ++bits;
    const int passes = (bits + DIGIT_BITS - 1) / DIGIT_BITS;
    const bool local4 = ((uintptr_t)f->is_local & 3) == 0, local8 = ((uintptr_t)f->is_local & 7) == 0,      // the caller's array: wide loads only if it allows them
               local16 = ((uintptr_t)f->is_local & 15) == 0;
    const int64_t sel_blocks = (n + SEL_TILE - 1) / SEL_TILE;
    uint64_t *block_tot = nullptr;
    RG_TRY(tmp.dev_n<uint64_t>((uint64_t)(sel_blocks ? sel_blocks : 1), &block_tot));
    const int64_t sel_tiles = (sel_blocks + SCAN_TILE - 1) / SCAN_TILE;
    uint64_t *tile_tot = nullptr;
    RG_TRY(tmp.dev_n<uint64_t>((uint64_t)(sel_tiles ? sel_tiles : 1), &tile_tot));
    {
        ScopedTimer tm(KG_TOPK, st);
        const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + TOPK_THREADS - 1) / TOPK_THREADS, (int64_t)n_cu * 16));
        for (int p = 0; p < passes; ++p) {
            const int shift = (passes - 1 - p) * DIGIT_BITS;
            if (narrow) {
                if (local16) hipLaunchKernelGGL(digit_histogram8_kernel<true>, dim3(grid), dim3(TOPK_THREADS), 0, st, c->freq8, f->is_local, n, bins, block_tot);
                else hipLaunchKernelGGL(digit_histogram8_kernel<false>, dim3(grid), dim3(TOPK_THREADS), 0, st, c->freq8, f->is_local, n, bins, block_tot);
            } else if (local4) hipLaunchKernelGGL(digit_histogram_kernel<true>, dim3(grid), dim3(TOPK_THREADS), 0, st, c->freq, f->is_local, n, stp, shift, bins);
            else hipLaunchKernelGGL(digit_histogram_kernel<false>, dim3(grid), dim3(TOPK_THREADS), 0, st, c->freq, f->is_local, n, stp, shift, bins);
            hipLaunchKernelGGL(choose_digit_kernel, dim3(1), dim3(DIGIT_BINS), 0, st, stp, bins, shift, p == 0 ? 1 : 0, K);
        }
        if (sel_blocks > 0) {
            const dim3 tg((unsigned)std::min<int64_t>(sel_blocks, (int64_t)n_cu * 32)), sb(TOPK_THREADS);
            if (narrow && local8) hipLaunchKernelGGL((select_block_totals<true, uint8_t>), tg, sb, 0, st, c->freq8, f->is_local, n, stp, block_tot);
            else if (narrow) hipLaunchKernelGGL((select_block_totals<false, uint8_t>), tg, sb, 0, st, c->freq8, f->is_local, n, stp, block_tot);
            else if (local8) hipLaunchKernelGGL((select_block_totals<true, uint32_t>), tg, sb, 0, st, c->freq, f->is_local, n, stp, block_tot);
            else hipLaunchKernelGGL((select_block_totals<false, uint32_t>), tg, sb, 0, st, c->freq, f->is_local, n, stp, block_tot);
            hipLaunchKernelGGL(select_scan_tiles, dim3((unsigned)sel_tiles), dim3(TOPK_THREADS), 0, st, block_tot, sel_blocks, tile_tot);
            if (sel_tiles > 1) hipLaunchKernelGGL(select_scan_totals, dim3(1), dim3(TOPK_THREADS), 0, st, tile_tot, sel_tiles);
        }
    }
    SelectState hs;
    {
        Readback rb(st);
        RG_TRY(rb.add(&hs, stp, sizeof(SelectState)));
        RG_TRY(rb.wait());
    }
    c->K_eff = hs.k_eff;
    RG_TRY(c->arena.dev_n<int32_t>(c->K_eff, &c->cache_ids));
    uint32_t *fill_codes = nullptr;
    RG_TRY(tmp.dev_n<uint32_t>(c->K_eff ? c->K_eff : 1, &fill_codes));
    RG_TRY(c->arena.dev_n<SlotRec>((uint64_t)std::max<int64_t>(sel_blocks, 1) * (SEL_TILE / 32), &c->slot_pairs));      // whole tiles: every thread of the select pass writes its share
    if (sel_blocks > 0) {
        ScopedTimer tm(KG_TOPK, st);
        const dim3 sg((unsigned)sel_blocks), sb(TOPK_THREADS);
        if (narrow && local8)
            hipLaunchKernelGGL((select_emit_kernel<true, uint8_t>), sg, sb, 0, st, c->freq8, f->is_local, n, stp, block_tot, tile_tot, c->cache_ids, c->slot_pairs, f->row_of, fill_codes);
        else if (narrow)
            hipLaunchKernelGGL((select_emit_kernel<false, uint8_t>), sg, sb, 0, st, c->freq8, f->is_local, n, stp, block_tot, tile_tot, c->cache_ids, c->slot_pairs, f->row_of, fill_codes);
        else if (local8)
            hipLaunchKernelGGL((select_emit_kernel<true, uint32_t>), sg, sb, 0, st, c->freq, f->is_local, n, stp, block_tot, tile_tot, c->cache_ids, c->slot_pairs, f->row_of, fill_codes);
        else
            hipLaunchKernelGGL((select_emit_kernel<false, uint32_t>), sg, sb, 0, st, c->freq, f->is_local, n, stp, block_tot, tile_tot, c->cache_ids, c->slot_pairs, f->row_of, fill_codes);
    }
    RG_HIP(hipGetLastError());

    // ---- a8: VectorPull -- one bulk gather of the selected rows out of the remote table.  It streams rows while the
    // plans below are bound by dependent lookups, and neither reads what the other writes: the fill goes to the
    // library's helper stream and runs beside them.
    RG_TRY(c->arena.dev(c->K_eff * c->stride, &c->rows));
    if (tls_table_bytes_sink) tls_table_bytes_sink->store(c->K_eff * c->stride, std::memory_order_release);
    struct Forked {                                       // declared after `tmp`: on every exit the fill has ended before tmp's blocks go back
        hipStream_t side = nullptr;
        ~Forked() { if (side) (void)hipStreamSynchronize(side); }
    } forked;
    if (c->K_eff > 0) {
        hipStream_t side = nullptr;
        RG_TRY(helper_stream(&side));
        RG_HIP(hipEventRecord(c->ev_fork, st));
        RG_HIP(hipStreamWaitEvent(side, c->ev_fork, 0));
        forked.side = side;
        RowSources src{(const uint8_t *)f->local_rows, f->local_stride, (const uint8_t *)c->rows, c->stride,
                       (const uint8_t *)f->remote_rows, f->remote_stride};
        RG_TRY(launch_gather(Routes{nullptr, fill_codes, last_remote_code(0)}, (int64_t)c->K_eff, ROWS_ALL, src, f->row_bytes, (uint8_t *)c->rows, c->stride, side, KG_FILL));
        RG_HIP(hipEventRecord(c->ev_join, side));
    }

    // ---- a5/a9: plans and counts for every batch of every epoch
    c->plans.resize(n_epochs);
    RouteSources rs{f->row_of, c->slot_pairs, nullptr};
    int64_t n_inputs = 0;
    for (uint32_t e = 0; e < n_epochs; ++e) n_inputs += epochs[e]->n_batches ? epochs[e]->hop[epochs[e]->L].off_host[epochs[e]->n_batches] : 0;
    bool look_for_ranks = n_inputs >= RANK_INPUTS_PER_NODE * n && n_inputs >= RANK_INPUTS;
    if (const char *force = getenv("RAPIDGNN_ROW_RANKS")) look_for_ranks = force[0] == '1';      // same results either way; for tests and tuning
    RankCheck check{c->slot_pairs, n, reinterpret_cast<uint32_t *>(bins), look_for_ranks && n > 0};       // (the digits have been chosen)
    RG_TRY(build_plans(epochs, rs, check, c->K_eff, &sel->no_codes, c->arena, tmp, st, c->plans));
    if (forked.side) RG_HIP(hipStreamWaitEvent(st, c->ev_join, 0));
    RG_HIP(hipStreamSynchronize(st));
    if (forked.side) { RG_HIP(hipStreamSynchronize(forked.side)); forked.side = nullptr; }
    tmp.drained();
    return RG_OK;
}

}  // namespace rg

using namespace rg;

extern "C" rg_status rg_build_cache(const rg_schedule *const *epochs, uint32_t n_epochs, const rg_features *f, uint64_t K,
                                    const rg_allocator *a, void *stream, rg_cache **out)
{
    if (!epochs || n_epochs == 0 || !f || !out) { set_error("rg_build_cache: null argument or no epoch"); return RG_EINVAL; }
    for (uint32_t e = 0; e < n_epochs; ++e) {
        if (!epochs[e]) { set_error("rg_build_cache: epochs[%u] is null", e); return RG_EINVAL; }
        if (epochs[e]->n_nodes != epochs[0]->n_nodes) { set_error("rg_build_cache: epochs disagree on n_nodes"); return RG_EINVAL; }
    }
    if (epochs[0]->n_nodes > 0 && (!f->is_local || !f->row_of)) { set_error("rg_build_cache: null is_local / row_of"); return RG_EINVAL; }
    if (f->row_bytes == 0) { set_error("rg_build_cache: row_bytes must be > 0"); return RG_EINVAL; }
    if (f->local_stride < f->row_bytes || f->remote_stride < f->row_bytes) { set_error("rg_build_cache: a stride is smaller than row_bytes"); return RG_EINVAL; }

    rg_cache *c = new (std::nothrow) rg_cache(a);
    if (!c) { set_error("rg_build_cache: out of host memory"); return RG_ENOMEM; }
    rg_status rc = build_cache_impl(epochs, n_epochs, f, K, a, as_stream(stream), c);
    if (rc != RG_OK) {
        (void)hipStreamSynchronize(as_stream(stream));
        rg_cache_destroy(c);
        return rc;
    }
    *out = c;
    return RG_OK;
}
