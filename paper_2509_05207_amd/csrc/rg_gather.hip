// rg_gather_batch: the feature block of one batch (Alg. 1 inner loop).
//
// A batch's block is n_rows byte rows; the kernel works on the flat space of
// (row, vector) pairs so that consecutive lanes copy consecutive vectors of a
// row and run on into the next row: no lane idles whatever the row width.
// Each thread keeps CHUNKS_IN_FLIGHT independent loads outstanding before it
// stores (stores are non-temporal: the block is consumed by a later kernel,
// not by this one).  The source of a row comes from its routing entry or code:
// local table, cache table or remote table.
//
// When the remote table is pinned host memory (mapped into the device's address
// space) the miss set is copied by a launch of its own, on the side stream: a
// wave finds the misses among a run of rows and copies those, and its loads
// cross the host link -- SyncPull without host-side packing or staging, and
// without a list of the misses.  When the remote table is device memory, one
// launch on the main stream copies every row.
#include "rg_internal.h"
#include "rg_device.h"
#include "rg_launch.h"

#include <algorithm>
#include <mutex>

namespace rg {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

template <int W> struct VecT;
template <> struct VecT<16> { using type = u32x4; };
template <> struct VecT<8> { using type = u32x2; };
template <> struct VecT<4> { using type = uint32_t; };
template <> struct VecT<2> { using type = uint16_t; };
template <> struct VecT<1> { using type = uint8_t; };

// A piece of W bytes at an address that is only known to be a multiple of A bytes.  Global memory takes
// vector accesses at any dword-aligned address, so rows whose base and stride are multiples of 4 (any
// fp32 width, even bf16/fp16 widths) are copied with 16-byte vectors whatever their 16-byte phase.
template <int W, int A> struct PieceT { typedef typename VecT<W>::type type __attribute__((aligned(A < W ? A : W))); };

template <int W, int A>
__device__ __forceinline__ void copy_piece(const uint8_t *src, uint8_t *dst)
{
    using P = typename PieceT<W, A>::type;
    *reinterpret_cast<P *>(dst) = *reinterpret_cast<const P *>(src);
}

template <int VEC, int A>
__device__ __forceinline__ void copy_tail(const uint8_t *src, uint8_t *dst, uint32_t tail)
{
    // tail < VEC, at an offset that is a multiple of VEC; pieces of decreasing power-of-two width
    if constexpr (VEC > 8) { if (tail & 8u) { copy_piece<8, A>(src, dst); src += 8; dst += 8; } }
    if constexpr (VEC > 4) { if (tail & 4u) { copy_piece<4, A>(src, dst); src += 4; dst += 4; } }
    if constexpr (VEC > 2) { if (tail & 2u) { copy_piece<2, A>(src, dst); src += 2; dst += 2; } }
    if constexpr (VEC > 1) { if (tail & 1u) { copy_piece<1, A>(src, dst); } }
}

constexpr int GATHER_THREADS = 256;

// Where a row comes from, out of a routing entry or a routing code.
__device__ __forceinline__ void decode_route(int64_t e, uint32_t, int64_t &tag, uint64_t &row) { tag = entry_tag(e); row = (uint64_t)entry_row(e); }
__device__ __forceinline__ void decode_route(uint32_t c, uint32_t last_remote, int64_t &tag, uint64_t &row)
{
    tag = c < CODE_NOT_LOCAL ? TAG_LOCAL : c > last_remote ? TAG_CACHE : TAG_REMOTE;
    row = c > last_remote ? ~c : c & ~CODE_NOT_LOCAL;
}

// TAILPIECE = false: every piece is a full vector.  Either row_bytes is a multiple of VEC, or the last piece of a
// row is the vector that ENDS at the row's end and overlaps its predecessor (both write the same bytes there), so
// that no lane leaves the vector path.  TAILPIECE = true (row widths that are no multiple of 4, or below VEC): the
// last piece is copied in 8/4/2/1-byte parts.
template <int VEC, int A, bool TAILPIECE, typename ROUTE>
__global__ void __launch_bounds__(GATHER_THREADS) gather_rows_kernel(const ROUTE *__restrict__ routes, uint32_t last_remote, int64_t n_rows, int skip_remote,
                                                                     RowSources src, uint32_t row_bytes,
                                                                     uint8_t *__restrict__ out, uint64_t out_stride, int chunks)
{
    using T = typename VecT<VEC>::type;
    using P = typename PieceT<VEC, A>::type;
    const uint32_t cpr = row_bytes / VEC, tail = row_bytes % VEC;
    const uint32_t cpt = cpr + (tail ? 1u : 0u);                  // pieces per row: full vectors, then the last piece
    const uint32_t last_off = TAILPIECE ? cpr * VEC : row_bytes - VEC;     // where the piece after the full vectors starts
    const uint64_t total = (uint64_t)n_rows * cpt;
    // A workgroup takes GATHER_THREADS * chunks consecutive pieces per round (chunks <= CHUNKS_IN_FLIGHT, fewer for
    // a block of rows too small to fill the chip otherwise): one contiguous span of the output, 32 KB with 16-byte
    // pieces.  Within a round the flat index -> (row, piece) pair is advanced by GATHER_THREADS without
    // dividing again.
    const uint32_t ROUND = GATHER_THREADS * (uint32_t)chunks;
    const uint32_t dq = GATHER_THREADS / cpt;
    const uint32_t dr = GATHER_THREADS - dq * cpt;

    for (uint64_t base = (uint64_t)blockIdx.x * ROUND + threadIdx.x; base < total; base += (uint64_t)gridDim.x * ROUND) {
        uint64_t idx = base;
        uint64_t w = idx / cpt;
        uint32_t c = (uint32_t)(idx - w * cpt);
        T v[CHUNKS_IN_FLIGHT];
        const uint8_t *sp[CHUNKS_IN_FLIGHT];
        uint8_t *dp[CHUNKS_IN_FLIGHT];
        int kind[CHUNKS_IN_FLIGHT];                                // 0 nothing, 1 full vector, 2 last piece in parts
#pragma unroll
        for (int k = 0; k < CHUNKS_IN_FLIGHT; ++k) {
            kind[k] = 0;
            sp[k] = nullptr; dp[k] = nullptr;
            if (k < chunks && idx < total) {
                int64_t tag;
                uint64_t row;
                decode_route(routes[(int64_t)w], last_remote, tag, row);
                if (!(skip_remote && tag == TAG_REMOTE)) {
                    const uint8_t *base = tag == TAG_LOCAL ? src.local_rows + row * src.local_stride
                                        : tag == TAG_CACHE ? src.cache_rows + row * src.cache_stride
                                                           : src.remote_rows + row * src.remote_stride;
                    const uint32_t o = c < cpr ? c * VEC : last_off;
                    sp[k] = base + o;
                    dp[k] = out + w * out_stride + o;
                    kind[k] = (!TAILPIECE || c < cpr) ? 1 : 2;
                    if (kind[k] == 1) v[k] = *reinterpret_cast<const P *>(sp[k]);
                }
            }
            idx += GATHER_THREADS;
            w += dq;
            c += dr;
            if (c >= cpt) { c -= cpt; ++w; }
        }
#pragma unroll
        for (int k = 0; k < CHUNKS_IN_FLIGHT; ++k) {
            if (kind[k] == 1) __builtin_nontemporal_store(v[k], reinterpret_cast<P *>(dp[k]));
            else if (TAILPIECE && kind[k] == 2) copy_tail<VEC, A>(sp[k], dp[k], tail);
        }
    }
}

// The remote rows alone.  A wave takes per_wave consecutive rows (a power of two up to 64) per round, one route a lane, lists the
// remote ones in LDS and copies those as the kernel above copies all: flat pieces, one per lane, CHUNKS_IN_FLIGHT under way.  Bound by
// the host link.  (A list of the misses made with every plan took 79 us per 80 M input nodes, and a wait for its length.)
// parts > 1 (then per_wave is 1): a row's pieces are shared out among that many waves.
template <int VEC, int A, bool TAILPIECE, typename ROUTE>
__global__ void __launch_bounds__(GATHER_THREADS) gather_remote_kernel(const ROUTE *__restrict__ routes, uint32_t last_remote, int64_t n_rows, int per_wave, uint32_t parts,
                                                                       RowSources src, uint32_t row_bytes, uint8_t *__restrict__ out, uint64_t out_stride)
{
    using T = typename VecT<VEC>::type;
    using P = typename PieceT<VEC, A>::type;
    struct Miss { uint64_t src_row, out_row; };
    __shared__ Miss lists[GATHER_THREADS / 64][64];
    const uint32_t cpr = row_bytes / VEC, tail = row_bytes % VEC;
    const uint32_t cpt = cpr + (tail ? 1u : 0u);
    const uint32_t last_off = TAILPIECE ? cpr * VEC : row_bytes - VEC;
    const uint32_t dq = 64 / cpt, dr = 64 - dq * cpt;
    const int lane = threadIdx.x & 63;
    const int wave_here = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);        // (a scalar: the rounds are the wave's)
    Miss *mine = lists[wave_here];
    const int64_t n_waves = (int64_t)gridDim.x * (GATHER_THREADS / 64), wave = (int64_t)blockIdx.x * (GATHER_THREADS / 64) + wave_here;
    for (int64_t unit = wave; unit * per_wave < n_rows * parts; unit += n_waves) {
        const int64_t first = parts == 1 ? unit * per_wave : unit / parts;
        const uint32_t part = parts == 1 ? 0u : (uint32_t)(unit - first * parts);
        int64_t tag = TAG_LOCAL;
        uint64_t row = 0;
        if (lane < per_wave && first + lane < n_rows) decode_route(routes[first + lane], last_remote, tag, row);
        const bool miss = tag == TAG_REMOTE;
        const unsigned long long all = __ballot(miss);
        wave_lds_order();                                          // the last round's list has been read
        if (miss) mine[__popcll(all & ((1ull << lane) - 1ull))] = Miss{row, (uint64_t)(first + lane)};
        wave_lds_order();
        const uint64_t pieces = (uint64_t)__popcll(all) * cpt;     // (64 rows of up to 2^32 bytes)
        const uint64_t begin = parts == 1 ? 0u : pieces * part / parts, total = parts == 1 ? pieces : pieces * (part + 1) / parts;
        uint32_t m = (uint32_t)lane / cpt, c = (uint32_t)lane - m * cpt;
        if (parts != 1) { m = 0; c = (uint32_t)begin + lane; }
        for (uint64_t idx = begin + lane; idx < total;) {
            T v[CHUNKS_IN_FLIGHT];
            const uint8_t *sp[CHUNKS_IN_FLIGHT];
            uint8_t *dp[CHUNKS_IN_FLIGHT];
            int kind[CHUNKS_IN_FLIGHT];                            // 0 nothing, 1 full vector, 2 last piece in parts
#pragma unroll
            for (int k = 0; k < CHUNKS_IN_FLIGHT; ++k) {
                kind[k] = 0;
                sp[k] = nullptr; dp[k] = nullptr;
                if (idx < total) {
                    const uint32_t o = c < cpr ? c * VEC : last_off;
                    sp[k] = src.remote_rows + mine[m].src_row * src.remote_stride + o;
                    dp[k] = out + mine[m].out_row * out_stride + o;
                    kind[k] = (!TAILPIECE || c < cpr) ? 1 : 2;
                    if (kind[k] == 1) v[k] = *reinterpret_cast<const P *>(sp[k]);
                }
                idx += 64;
                m += dq;
                c += dr;
                if (c >= cpt) { c -= cpt; ++m; }
            }
#pragma unroll
            for (int k = 0; k < CHUNKS_IN_FLIGHT; ++k) {
                if (kind[k] == 1) __builtin_nontemporal_store(v[k], reinterpret_cast<P *>(dp[k]));
                else if (TAILPIECE && kind[k] == 2) copy_tail<VEC, A>(sp[k], dp[k], tail);
            }
        }
    }
}

// The routes of a plan's input nodes from position `at` on.
static Routes plan_routes(const Plan &p, const rg_cache *c, int64_t at)
{
    return p.code ? Routes{nullptr, p.code + at, last_remote_code(c->K_eff)} : Routes{p.entry + at, nullptr, 0};
}

static int common_alignment(const RowSources &s, const uint8_t *out, uint64_t out_stride)
{
    uint64_t bits = (uint64_t)(uintptr_t)s.local_rows | s.local_stride | (uint64_t)(uintptr_t)s.cache_rows | s.cache_stride |
                    (uint64_t)(uintptr_t)s.remote_rows | s.remote_stride | (uint64_t)(uintptr_t)out | out_stride;
    if ((bits & 15) == 0) return 16;
    if ((bits & 7) == 0) return 8;
    if ((bits & 3) == 0) return 4;
    return 1;
}

rg_status launch_gather(const Routes &routes, int64_t n_rows, RowsWanted wanted, const RowSources &src, uint32_t row_bytes, uint8_t *out, uint64_t out_stride,
                        hipStream_t st, int group, int64_t n_remote)
{
    if (n_rows <= 0) return RG_OK;
    int align = common_alignment(src, out, out_stride);
    const int vec = align >= 4 ? 16 : 1;                        // dword-aligned rows take 16-byte vectors, anything else goes byte by byte
    const uint32_t tail = row_bytes % (uint32_t)vec;
    // A row that ends between vectors: if its width is a multiple of 4 and at least one vector, the last piece is the
    // vector ending at the row's end, at the alignment the width leaves; otherwise the last piece goes in parts.
    const bool overlap_last = vec == 16 && tail != 0 && row_bytes >= 16 && row_bytes % 4 == 0;
    const bool tailpiece = tail != 0 && !overlap_last;
    if (overlap_last) align = std::min(align, (row_bytes % 8 == 0) ? 8 : 4);
    const uint64_t cpt = row_bytes / (uint32_t)vec + (tail ? 1 : 0);
    int n_cu = 256;
    RG_TRY(compute_units(&n_cu));
    // pieces per thread and round: as many as stay in flight, fewer when that would leave compute units without a workgroup
    const uint64_t total = (uint64_t)n_rows * cpt;
    const uint64_t want_blocks = (uint64_t)n_cu * 8;
    int chunks = CHUNKS_IN_FLIGHT;
    while (chunks > 1 && (total + (uint64_t)GATHER_THREADS * chunks - 1) / ((uint64_t)GATHER_THREADS * chunks) < want_blocks) --chunks;
    const uint64_t per_block = (uint64_t)GATHER_THREADS * chunks;
    const uint64_t blocks = std::max<uint64_t>(1, std::min<uint64_t>((total + per_block - 1) / per_block, (uint64_t)n_cu * 32));
    const int skip_remote = wanted == ROWS_NOT_REMOTE ? 1 : 0;
    const RemoteShape remote = remote_shape(n_rows, n_remote, cpt, vec, n_cu);
    const unsigned remote_blocks = (unsigned)((remote.waves + GATHER_THREADS / 64 - 1) / (GATHER_THREADS / 64));
    ScopedTimer tm(group, st);
#define RG_GATHER_ROWS(V, AL, TAIL, ROUTE, FROM)                                                                                              \
    do {                                                                                                                                      \
        if (wanted == ROWS_REMOTE)                                                                                                            \
            hipLaunchKernelGGL((gather_remote_kernel<V, AL, TAIL, ROUTE>), dim3(remote_blocks), dim3(GATHER_THREADS), 0, st, FROM,            \
                               routes.last_remote, n_rows, remote.per_wave, (uint32_t)remote.parts, src, row_bytes, out, out_stride);         \
        else                                                                                                                                  \
            hipLaunchKernelGGL((gather_rows_kernel<V, AL, TAIL, ROUTE>), dim3((unsigned)blocks), dim3(GATHER_THREADS), 0, st, FROM,           \
                               routes.last_remote, n_rows, skip_remote, src, row_bytes, out, out_stride, chunks);                             \
    } while (0)
#define RG_GATHER_LAUNCH(V, AL)                                                                                                               \
    do {                                                                                                                                      \
        if (tailpiece && routes.entry) RG_GATHER_ROWS(V, AL, true, int64_t, routes.entry);                                                    \
        else if (tailpiece) RG_GATHER_ROWS(V, AL, true, uint32_t, routes.code);                                                               \
        else if (routes.entry) RG_GATHER_ROWS(V, AL, false, int64_t, routes.entry);                                                           \
        else RG_GATHER_ROWS(V, AL, false, uint32_t, routes.code);                                                                             \
    } while (0)
    switch (align) {
    case 16: RG_GATHER_LAUNCH(16, 16); break;
    case 8:  RG_GATHER_LAUNCH(16, 8); break;
    case 4:  RG_GATHER_LAUNCH(16, 4); break;
    default: RG_GATHER_LAUNCH(1, 1); break;
    }
#undef RG_GATHER_LAUNCH
#undef RG_GATHER_ROWS
    RG_HIP(hipGetLastError());
    return RG_OK;
}

// True when p is device memory (then "remote" rows are plain HBM reads and need no side stream).
bool is_device_memory(const void *p)
{
    if (!p) return false;
    hipPointerAttribute_t attr;
    if (hipPointerGetAttributes(&attr, p) != hipSuccess) { (void)hipGetLastError(); return false; }
    return attr.type == hipMemoryTypeDevice;
}

// Routing of a single batch computed on the spot (no cache, or a schedule the cache has no plan for).
//
// Bound by its scattered reads (is_local, row_of and a slot-map record per listed ID), so a thread takes ROUTE_PER_THREAD
// IDs and has the reads of all of them in flight at once.  The counts go through LDS to two adds per workgroup, spread
// over ROUTE_COUNT_SLOTS pairs of counters which the host adds up: three adds per wave to the same three addresses queued
// up behind each other at 11 ns apiece and were nine tenths of the kernel (a batch of 1.2 M rows of 512 bytes: routing
// 615 us, now under 20; the whole call 852 -> 243 us, its gather 227).  Misses are not counted: they are the rows that are
// neither local nor cached.
constexpr int ROUTE_THREADS = 256;
constexpr int ROUTE_PER_THREAD = 4;
constexpr int ROUTE_TILE = ROUTE_THREADS * ROUTE_PER_THREAD;
constexpr int ROUTE_COUNT_SLOTS = 16;
constexpr size_t ROUTE_COUNT_BYTES = 2 * ROUTE_COUNT_SLOTS * sizeof(unsigned long long);      // local, hit per slot

// entry == NULL: the counts alone.  counts == NULL: the entries alone.
__global__ void __launch_bounds__(ROUTE_THREADS) route_batch_kernel(const int32_t *__restrict__ ids, int64_t n, const uint8_t *__restrict__ is_local,
                                                                    const int32_t *__restrict__ row_of,
                                                                    const SlotRec *__restrict__ slot_pairs /* see slot_lookup; NULL: no cache */,
                                                                    int64_t *__restrict__ entry, unsigned long long *__restrict__ counts)
{
    __shared__ unsigned int red[2][ROUTE_THREADS / 64];
    const int64_t j0 = (int64_t)blockIdx.x * ROUTE_TILE + threadIdx.x;
    int32_t v[ROUTE_PER_THREAD], row[ROUTE_PER_THREAD], slot[ROUTE_PER_THREAD];
    uint8_t local[ROUTE_PER_THREAD];
#pragma unroll
    for (int k = 0; k < ROUTE_PER_THREAD; ++k) v[k] = ids[min(j0 + k * ROUTE_THREADS, n - 1)];        // (past the end: the last ID again, not used)
#pragma unroll
    for (int k = 0; k < ROUTE_PER_THREAD; ++k) local[k] = is_local[v[k]];
#pragma unroll
    for (int k = 0; k < ROUTE_PER_THREAD; ++k) slot[k] = slot_pairs ? slot_lookup(slot_pairs, (uint32_t)v[k]) : -1;
    if (entry)
#pragma unroll
        for (int k = 0; k < ROUTE_PER_THREAD; ++k) row[k] = row_of[v[k]];
    unsigned int n_local = 0, n_hit = 0;                       // of the wave
#pragma unroll
    for (int k = 0; k < ROUTE_PER_THREAD; ++k) {
        const int64_t j = j0 + k * ROUTE_THREADS;
        const bool is_loc = local[k] != 0, is_hit = !is_loc && slot[k] >= 0;
        if (entry && j < n) entry[j] = make_entry(is_loc ? TAG_LOCAL : is_hit ? TAG_CACHE : TAG_REMOTE, is_hit ? slot[k] : row[k]);
        n_local += (unsigned int)__popcll(__ballot(is_loc && j < n));
        n_hit += (unsigned int)__popcll(__ballot(is_hit && j < n));
    }
    if (!counts) return;
    if ((threadIdx.x & 63) == 0) { red[0][threadIdx.x >> 6] = n_local; red[1][threadIdx.x >> 6] = n_hit; }
    __syncthreads();
    if (threadIdx.x < 2) {
        unsigned int c = 0;
        for (int w = 0; w < ROUTE_THREADS / 64; ++w) c += red[threadIdx.x][w];
        if (c) atomicAdd(&counts[2 * (blockIdx.x % ROUTE_COUNT_SLOTS) + threadIdx.x], (unsigned long long)c);
    }
}

static void launch_route(const int32_t *ids, int64_t n, const rg_features *f, const SlotRec *slot_pairs, int64_t *entry, unsigned long long *counts, hipStream_t st)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(route_batch_kernel, dim3((unsigned)((n + ROUTE_TILE - 1) / ROUTE_TILE)), dim3(ROUTE_THREADS), 0, st, ids, n, f->is_local, f->row_of,
                       slot_pairs, entry, counts);
}

static void sum_route_counts(const unsigned long long *counts /* host, [2 * ROUTE_COUNT_SLOTS] */, int64_t n_rows, rg_gather_stats *stats)
{
    uint64_t local = 0, hit = 0;
    for (int s = 0; s < ROUTE_COUNT_SLOTS; ++s) { local += counts[2 * s]; hit += counts[2 * s + 1]; }
    stats->n_rows = (uint64_t)n_rows; stats->n_local = local; stats->n_hit = hit; stats->n_miss = (uint64_t)n_rows - local - hit;
}

// ---------------------------------------------------------------- the entry point that allocates nothing
// Its scratch -- the counters and one routing entry per row of the batch -- lives in the library's image: one
// copy per GPU, at an address of that GPU's own, which the host asks for once per device.  The array's name is only a
// stand-in on the host; kernels and copies get the pointer kept here.
constexpr uint64_t NOALLOC_HEAD_BYTES = 256;                       // the counters, in front of the entries
static_assert(ROUTE_COUNT_BYTES <= NOALLOC_HEAD_BYTES, "the counters fit in front of the entries");
static __device__ __align__(256) unsigned char scratch[NOALLOC_HEAD_BYTES + RG_NOALLOC_MAX_ROWS * sizeof(int64_t)];

constexpr int MAX_DEVICES = 64;
static std::mutex g_scratch_mu;
static void *g_scratch_ptr[MAX_DEVICES];                           // per device; NULL until asked for

// The current device's copy of `scratch`.
static rg_status scratch_of_current_device(unsigned char **out)
{
    int dev = 0;
    RG_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) { set_error("rg_gather_batch_noalloc: device %d beyond the %d this build keeps scratch for", dev, MAX_DEVICES); return RG_ERANGE; }
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        RG_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) { set_error("rg_gather_batch_noalloc: no address for the scratch array on device %d", dev); return RG_EHIP; }
        g_scratch_ptr[dev] = p;
    }
    *out = static_cast<unsigned char *>(g_scratch_ptr[dev]);
    return RG_OK;
}

// (a fill kernel, not hipMemsetAsync: the call may be recorded into a graph)
__global__ void clear_counts_kernel(unsigned long long *__restrict__ counts)
{
    if (threadIdx.x < 2 * ROUTE_COUNT_SLOTS) counts[threadIdx.x] = 0ull;
}

}  // namespace rg

using namespace rg;

extern "C" rg_status rg_gather_batch_noalloc(const rg_schedule *s, const rg_cache *c, const rg_features *f, uint32_t batch, void *out,
                                             uint64_t out_stride, uint64_t out_capacity_rows, void *stream, rg_gather_stats *stats)
{
    if (!s || !f) { set_error("rg_gather_batch_noalloc: null schedule or features"); return RG_EINVAL; }
    if (batch >= s->n_batches) { set_error("rg_gather_batch_noalloc: batch %u >= n_batches = %u", batch, s->n_batches); return RG_ERANGE; }
    if (f->row_bytes == 0 || out_stride < f->row_bytes || f->local_stride < f->row_bytes || f->remote_stride < f->row_bytes) {
        set_error("rg_gather_batch_noalloc: row_bytes = %u with strides out %llu local %llu remote %llu", f->row_bytes,
                  (unsigned long long)out_stride, (unsigned long long)f->local_stride, (unsigned long long)f->remote_stride);
        return RG_EINVAL;
    }
    if (c && (c->n_nodes != s->n_nodes || c->row_bytes != f->row_bytes)) { set_error("rg_gather_batch_noalloc: cache does not match schedule / features"); return RG_EINVAL; }
    const HopData &h = s->hop[s->L];
    const int64_t off = h.off_host[batch];
    const int64_t m = h.off_host[batch + 1] - off;
    if ((uint64_t)m > RG_NOALLOC_MAX_ROWS) {
        set_error("rg_gather_batch_noalloc: batch %u has %lld rows, the built-in scratch holds RG_NOALLOC_MAX_ROWS = %llu", batch, (long long)m,
                  (unsigned long long)RG_NOALLOC_MAX_ROWS);
        return RG_ERANGE;
    }
    if ((uint64_t)m > out_capacity_rows) {
        set_error("rg_gather_batch_noalloc: batch %u has %lld rows, output holds %llu", batch, (long long)m, (unsigned long long)out_capacity_rows);
        return RG_ERANGE;
    }
    if (m > 0 && !out) { set_error("rg_gather_batch_noalloc: null output"); return RG_EINVAL; }
    unsigned char *base = nullptr;
    RG_TRY(scratch_of_current_device(&base));
    unsigned long long *counts = reinterpret_cast<unsigned long long *>(base);
    int64_t *entry = reinterpret_cast<int64_t *>(base + NOALLOC_HEAD_BYTES);
    hipStream_t st = as_stream(stream);
    RowSources src{(const uint8_t *)f->local_rows, f->local_stride, c ? (const uint8_t *)c->rows : (const uint8_t *)f->local_rows,
                   c ? c->stride : f->local_stride, (const uint8_t *)f->remote_rows, f->remote_stride};
    if (stats) hipLaunchKernelGGL(clear_counts_kernel, dim3(1), dim3(64), 0, st, counts);
    if (m > 0) {
        launch_route(h.ids + off, m, f, c ? c->slot_pairs : nullptr, entry, stats ? counts : nullptr, st);
        RG_HIP(hipGetLastError());
        RG_TRY(launch_gather(Routes{entry, nullptr, 0}, m, ROWS_ALL, src, f->row_bytes, (uint8_t *)out, out_stride, st, -1));      // (group -1: no event timers, they are created on demand)
    }
    RG_HIP(hipGetLastError());
    if (stats) {
        unsigned long long hc[2 * ROUTE_COUNT_SLOTS];
        RG_HIP(hipMemcpyAsync(hc, counts, sizeof(hc), hipMemcpyDeviceToHost, st));
        RG_HIP(hipStreamSynchronize(st));
        sum_route_counts(hc, m, stats);
    }
    return RG_OK;
}

extern "C" rg_status rg_gather_batch(const rg_schedule *s, const rg_cache *c, const rg_features *f, uint32_t batch, void *out,
                                     uint64_t out_stride, uint64_t out_capacity_rows, void *stream, void *side_stream,
                                     rg_gather_stats *stats)
{
    if (!s || !f) { set_error("rg_gather_batch: null schedule or features"); return RG_EINVAL; }
    if (batch >= s->n_batches) { set_error("rg_gather_batch: batch %u >= n_batches = %u", batch, s->n_batches); return RG_ERANGE; }
    if (f->row_bytes == 0 || out_stride < f->row_bytes || f->local_stride < f->row_bytes || f->remote_stride < f->row_bytes) {
        set_error("rg_gather_batch: row_bytes = %u with strides out %llu local %llu remote %llu", f->row_bytes,
                  (unsigned long long)out_stride, (unsigned long long)f->local_stride, (unsigned long long)f->remote_stride);
        return RG_EINVAL;
    }
    if (c && (c->n_nodes != s->n_nodes || c->row_bytes != f->row_bytes)) { set_error("rg_gather_batch: cache does not match schedule / features"); return RG_EINVAL; }
    const HopData &h = s->hop[s->L];
    const int64_t off = h.off_host[batch];
    const int64_t m = h.off_host[batch + 1] - off;
    if ((uint64_t)m > out_capacity_rows) {
        set_error("rg_gather_batch: batch %u has %lld rows, output holds %llu", batch, (long long)m, (unsigned long long)out_capacity_rows);
        return RG_ERANGE;
    }
    if (m > 0 && !out) { set_error("rg_gather_batch: null output"); return RG_EINVAL; }
    hipStream_t st = as_stream(stream);
    hipStream_t side = side_stream ? as_stream(side_stream) : st;
    RowSources src{(const uint8_t *)f->local_rows, f->local_stride, c ? (const uint8_t *)c->rows : (const uint8_t *)f->local_rows,
                   c ? c->stride : f->local_stride, (const uint8_t *)f->remote_rows, f->remote_stride};

    const Plan *plan = nullptr;
    if (c)
        for (const Plan &p : c->plans)
            if (p.schedule_uid == s->uid) { plan = &p; break; }

    if (plan) {
        const int64_t n_miss = plan->miss_off[batch + 1] - plan->miss_off[batch];
        const Routes routes = plan_routes(*plan, c, off);
        const bool remote_in_hbm = n_miss > 0 && (f->remote_rows == c->remote_rows_seen ? c->remote_is_device : is_device_memory(f->remote_rows));
        if (n_miss == 0 || remote_in_hbm) {
            // every source is HBM: one launch copies the whole block
            RG_TRY(launch_gather(routes, m, ROWS_ALL, src, f->row_bytes, (uint8_t *)out, out_stride, st, KG_GATHER));
        } else if (side != st) {
            RG_HIP(hipEventRecord(c->ev_fork, st));            // earlier work on `stream` may still use `out`
            RG_HIP(hipStreamWaitEvent(side, c->ev_fork, 0));
            RG_TRY(launch_gather(routes, m, ROWS_REMOTE, src, f->row_bytes, (uint8_t *)out, out_stride, side, KG_MISS, n_miss));
            RG_HIP(hipEventRecord(c->ev_join, side));
            RG_TRY(launch_gather(routes, m, ROWS_NOT_REMOTE, src, f->row_bytes, (uint8_t *)out, out_stride, st, KG_GATHER));
            RG_HIP(hipStreamWaitEvent(st, c->ev_join, 0));
        } else {
            RG_TRY(launch_gather(routes, m, ROWS_NOT_REMOTE, src, f->row_bytes, (uint8_t *)out, out_stride, st, KG_GATHER));
            RG_TRY(launch_gather(routes, m, ROWS_REMOTE, src, f->row_bytes, (uint8_t *)out, out_stride, st, KG_MISS, n_miss));
        }
        UseLog::note(s->uses, c->uses, st);                    // the launches above read the schedule's and the cache's arrays after this call returns
        if (stats) *stats = plan->stats[batch];
        return RG_OK;
    }

    // No prepared plan: classify this batch now, copy every row on `stream`, wait for both.
    Arena tmp(s->arena.allocator(), st);     // scratch from the allocator the schedule was built with
    int64_t *entry = nullptr;
    unsigned long long *counts = nullptr, hc[2 * ROUTE_COUNT_SLOTS] = {};
    RG_TRY(tmp.dev_n<int64_t>((uint64_t)m, &entry));
    if (stats) {
        RG_TRY(tmp.dev(ROUTE_COUNT_BYTES, (void **)&counts));
        RG_HIP(hipMemsetAsync(counts, 0, ROUTE_COUNT_BYTES, st));
    }
    if (m > 0) {
        {
            ScopedTimer tm(KG_PLAN, st);
            launch_route(h.ids + off, m, f, c ? c->slot_pairs : nullptr, entry, counts, st);
        }
        RG_HIP(hipGetLastError());
        RG_TRY(launch_gather(Routes{entry, nullptr, 0}, m, ROWS_ALL, src, f->row_bytes, (uint8_t *)out, out_stride, st, KG_GATHER));
    }
    if (stats) RG_HIP(hipMemcpyAsync(hc, counts, sizeof(hc), hipMemcpyDeviceToHost, st));
    RG_HIP(hipStreamSynchronize(st));
    tmp.drained();
    if (stats) sum_route_counts(hc, m, stats);
    return RG_OK;
}

// Blocks of consecutive batches, back to back in one output buffer.  A schedule keeps the frontiers of its batches
// concatenated, and so does a plan its routing entries: a range of batches is a range of rows, and one launch
// copies it (fewer, larger launches: the ramp and tail of a launch are paid once per range, not once per batch).
extern "C" rg_status rg_gather_batches(const rg_schedule *s, const rg_cache *c, const rg_features *f, uint32_t first_batch,
                                       uint32_t n_batches, void *out, uint64_t out_stride, uint64_t out_capacity_rows, void *stream,
                                       void *side_stream, rg_gather_stats *stats)
{
    if (!s || !f) { set_error("rg_gather_batches: null schedule or features"); return RG_EINVAL; }
    if ((uint64_t)first_batch + n_batches > s->n_batches) {
        set_error("rg_gather_batches: batches [%u, %u + %u) beyond n_batches = %u", first_batch, first_batch, n_batches, s->n_batches);
        return RG_ERANGE;
    }
    if (n_batches == 0) return RG_OK;
    const HopData &h = s->hop[s->L];
    const int64_t off0 = h.off_host[first_batch];
    const int64_t m = h.off_host[first_batch + n_batches] - off0;
    if ((uint64_t)m > out_capacity_rows) {
        set_error("rg_gather_batches: %u batches from %u have %lld rows, output holds %llu", n_batches, first_batch, (long long)m,
                  (unsigned long long)out_capacity_rows);
        return RG_ERANGE;
    }
    const Plan *plan = nullptr;
    if (c)
        for (const Plan &p : c->plans)
            if (p.schedule_uid == s->uid) { plan = &p; break; }
    if (!plan || n_batches == 1) {
        // no prepared routing for this schedule: batch by batch (each call classifies on the fly and waits for its counts)
        for (uint32_t k = 0; k < n_batches; ++k) {
            const uint32_t b = first_batch + k;
            const int64_t at = h.off_host[b] - off0;
            RG_TRY(rg_gather_batch(s, c, f, b, (uint8_t *)out + (uint64_t)at * out_stride, out_stride, out_capacity_rows - (uint64_t)at, stream,
                                   side_stream, stats ? stats + k : nullptr));
        }
        return RG_OK;
    }
    if (f->row_bytes == 0 || out_stride < f->row_bytes || f->local_stride < f->row_bytes || f->remote_stride < f->row_bytes) {
        set_error("rg_gather_batches: row_bytes = %u with strides out %llu local %llu remote %llu", f->row_bytes,
                  (unsigned long long)out_stride, (unsigned long long)f->local_stride, (unsigned long long)f->remote_stride);
        return RG_EINVAL;
    }
    if (c->n_nodes != s->n_nodes || c->row_bytes != f->row_bytes) { set_error("rg_gather_batches: cache does not match schedule / features"); return RG_EINVAL; }
    if (m > 0 && !out) { set_error("rg_gather_batches: null output"); return RG_EINVAL; }
    hipStream_t st = as_stream(stream);
    hipStream_t side = side_stream ? as_stream(side_stream) : st;
    RowSources src{(const uint8_t *)f->local_rows, f->local_stride, (const uint8_t *)c->rows, c->stride, (const uint8_t *)f->remote_rows, f->remote_stride};
    const int64_t n_miss = plan->miss_off[first_batch + n_batches] - plan->miss_off[first_batch];
    const Routes routes = plan_routes(*plan, c, off0);
    const bool remote_in_hbm = n_miss > 0 && (f->remote_rows == c->remote_rows_seen ? c->remote_is_device : is_device_memory(f->remote_rows));
    if (n_miss == 0 || remote_in_hbm) {
        RG_TRY(launch_gather(routes, m, ROWS_ALL, src, f->row_bytes, (uint8_t *)out, out_stride, st, KG_GATHER));
    } else {
        // rows with HBM sources in one launch, the misses in another
        if (side != st) {
            RG_HIP(hipEventRecord(c->ev_fork, st));
            RG_HIP(hipStreamWaitEvent(side, c->ev_fork, 0));
        }
        RG_TRY(launch_gather(routes, m, ROWS_NOT_REMOTE, src, f->row_bytes, (uint8_t *)out, out_stride, st, KG_GATHER));
        RG_TRY(launch_gather(routes, m, ROWS_REMOTE, src, f->row_bytes, (uint8_t *)out, out_stride, side, KG_MISS, n_miss));
        if (side != st) {
            RG_HIP(hipEventRecord(c->ev_join, side));
            RG_HIP(hipStreamWaitEvent(st, c->ev_join, 0));
        }
    }
    UseLog::note(s->uses, c->uses, st);
    if (stats)
        for (uint32_t k = 0; k < n_batches; ++k) stats[k] = plan->stats[first_batch + k];
    return RG_OK;
}

// The batch's counts alone: a9 without the copy (Alg. 1 inner loop, rpc_e += |M_i^e|).
extern "C" rg_status rg_classify_batch(const rg_schedule *s, const rg_cache *c, const rg_features *f, uint32_t batch, void *stream,
                                       rg_gather_stats *stats)
{
    if (!s || !f || !stats) { set_error("rg_classify_batch: null argument"); return RG_EINVAL; }
    if (batch >= s->n_batches) { set_error("rg_classify_batch: batch %u >= n_batches = %u", batch, s->n_batches); return RG_ERANGE; }
    if (c && c->n_nodes != s->n_nodes) { set_error("rg_classify_batch: cache does not match the schedule"); return RG_EINVAL; }
    if (c)
        for (const Plan &p : c->plans)
            if (p.schedule_uid == s->uid) { *stats = p.stats[batch]; return RG_OK; }
    const HopData &h = s->hop[s->L];
    const int64_t off = h.off_host[batch], m = h.off_host[batch + 1] - off;
    hipStream_t st = as_stream(stream);
    Arena tmp(s->arena.allocator(), st);     // scratch from the allocator the schedule was built with
    unsigned long long *counts = nullptr;
    RG_TRY(tmp.dev(ROUTE_COUNT_BYTES, (void **)&counts));
    RG_HIP(hipMemsetAsync(counts, 0, ROUTE_COUNT_BYTES, st));
    if (m > 0) {
        ScopedTimer tm(KG_PLAN, st);
        launch_route(h.ids + off, m, f, c ? c->slot_pairs : nullptr, nullptr, counts, st);
    }
    unsigned long long hc[2 * ROUTE_COUNT_SLOTS] = {};
    hipError_t e1 = hipGetLastError();
    hipError_t e2 = hipMemcpyAsync(hc, counts, sizeof(hc), hipMemcpyDeviceToHost, st);
    hipError_t e3 = hipStreamSynchronize(st);                    // also before `tmp` is released
    if (e3 == hipSuccess) tmp.drained();
    if (e1 != hipSuccess || e2 != hipSuccess || e3 != hipSuccess) { set_error("rg_classify_batch: HIP call failed"); return RG_EHIP; }
    sum_route_counts(hc, m, stats);
    return RG_OK;
}
