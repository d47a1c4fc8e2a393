// Error reporting, memory arena, kernel-group timers, the device prefix sum,
// graph validation and the handle accessors.
#include "rg_internal.h"

#include <cstring>

#include <algorithm>
#include <atomic>
#include <cstdarg>
#include <cstdio>
#include <map>
#include <mutex>

namespace rg {

// ---------------------------------------------------------------- errors
static thread_local char g_err[512] = "";

void set_error(const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
}

// ---------------------------------------------------------------- device block cache
// hipMalloc / hipFree cost tens of microseconds to milliseconds each and hipFree synchronises the
// device.  An epoch's build allocates a few dozen buffers whose sizes repeat from epoch to epoch, so
// released blocks are kept (per device) and handed out again to requests of nearly the same size.
// Blocks only come back here after the work that used them has completed: a call's scratch arena drains
// the call's stream before it lets go (on every way out of the call), and a handle is released only once
// the gathers that read it have finished (UseLog).  rg_trim_memory() returns everything to the driver.
namespace {
struct BlockCache {
    std::mutex mu;
    std::multimap<std::pair<int, uint64_t>, void *> free_blocks;      // (device, bytes) -> block
    std::multimap<std::pair<int, uint64_t>, void *> zero_blocks;      // the same, blocks whose every byte is known to be zero
    std::map<void *, std::pair<int, uint64_t>> live;                  // blocks handed out
    uint64_t cached_bytes = 0;

    static uint64_t round_up(uint64_t bytes)
    {
        if (bytes <= 4096) return 4096;
        if (bytes < (1ull << 20)) { uint64_t r = 4096; while (r < bytes) r <<= 1; return r; }
        return (bytes + (1ull << 20) - 1) >> 20 << 20;
    }

    // zeroed: prefer a block that is known to hold nothing but zero bytes (*was_zero says whether one was found;
    // otherwise the caller clears what it got).  A request that finds no ordinary block takes a zeroed one.
    // spare: the caller can do without; nothing is given back to the driver for it.
    void *take(uint64_t bytes, hipError_t *err, bool zeroed = false, bool *was_zero = nullptr, bool spare = false)
    {
        int dev = 0;
        (void)hipGetDevice(&dev);
        const uint64_t want = round_up(bytes);
        if (was_zero) *was_zero = false;
        {
            std::lock_guard<std::mutex> lk(mu);
            auto fits = [&](std::multimap<std::pair<int, uint64_t>, void *> &pool) -> void * {
                auto it = pool.lower_bound({dev, want});
                if (it == pool.end() || it->first.first != dev || it->first.second > want + want / 8 + (1ull << 20)) return nullptr;
                void *p = it->second;
                live[p] = it->first;
                cached_bytes -= it->first.second;
                pool.erase(it);
                return p;
            };
            if (zeroed) {
                if (void *p = fits(zero_blocks)) { if (was_zero) *was_zero = true; return p; }
                if (void *p = fits(free_blocks)) return p;
            } else {
                if (void *p = fits(free_blocks)) return p;
                if (void *p = fits(zero_blocks)) return p;
            }
        }
        void *p = nullptr;
        hipError_t e = hipMalloc(&p, want);
        if (e != hipSuccess && !spare) {             // release what waits for its readers, give the cache back to the driver, try once more
            (void)hipGetLastError();
            reap_retired(true);
            trim();
            e = hipMalloc(&p, want);
        }
        if (e != hipSuccess) { (void)hipGetLastError(); *err = e; return nullptr; }
        std::lock_guard<std::mutex> lk(mu);
        live[p] = {dev, want};
        return p;
    }

    uint64_t size_of(void *p)
    {
        std::lock_guard<std::mutex> lk(mu);
        auto it = live.find(p);
        return it == live.end() ? 0 : it->second.second;
    }

    // all_zero: the caller vouches that every byte of the block is zero and that nothing will write it any more
    void give(void *p, bool all_zero = false)
    {
        std::lock_guard<std::mutex> lk(mu);
        auto it = live.find(p);
        if (it == live.end()) { (void)hipFree(p); return; }
        (all_zero ? zero_blocks : free_blocks).insert({it->second, p});
        cached_bytes += it->second.second;
        live.erase(it);
    }

    void trim()
    {
        std::lock_guard<std::mutex> lk(mu);
        for (auto &kv : free_blocks) (void)hipFree(kv.second);
        for (auto &kv : zero_blocks) (void)hipFree(kv.second);
        free_blocks.clear();
        zero_blocks.clear();
        cached_bytes = 0;
    }
};
BlockCache g_blocks;
}  // namespace

// ---------------------------------------------------------------- small readbacks
namespace {
constexpr size_t STAGE_BYTES = 8192;
struct StagePool {
    std::mutex mu;
    std::vector<uint8_t *> free_blocks;
    uint8_t *take()
    {
        {
            std::lock_guard<std::mutex> lk(mu);
            if (!free_blocks.empty()) { uint8_t *p = free_blocks.back(); free_blocks.pop_back(); return p; }
        }
        void *p = nullptr;
        if (hipHostMalloc(&p, STAGE_BYTES, hipHostMallocDefault) != hipSuccess) { (void)hipGetLastError(); return nullptr; }
        return static_cast<uint8_t *>(p);
    }
    void give(uint8_t *p) { std::lock_guard<std::mutex> lk(mu); free_blocks.push_back(p); }
};
StagePool g_stages;
}  // namespace

// Several small pieces are fetched by one kernel that writes them straight into the pinned block (host memory the
// device can address), not by a copy each: a copy is a launch of its own, and they run one after the other.
constexpr int PACK_PARTS = 8;
struct PackArgs {
    const uint8_t *src[PACK_PARTS];
    uint32_t at[PACK_PARTS], bytes[PACK_PARTS];
    int n;
};
__global__ void __launch_bounds__(256) pack_pieces_kernel(PackArgs a, uint8_t *__restrict__ stage)
{
    for (int p = 0; p < a.n; ++p) {
        const uint8_t *src = a.src[p];
        uint8_t *dst = stage + a.at[p];
        const uint32_t bytes = a.bytes[p];
        if ((((uintptr_t)src | bytes) & 3u) == 0) {                     // (the block's offsets are multiples of 16)
            for (uint32_t i = threadIdx.x; i < bytes / 4; i += blockDim.x) reinterpret_cast<uint32_t *>(dst)[i] = reinterpret_cast<const uint32_t *>(src)[i];
        } else {
            for (uint32_t i = threadIdx.x; i < bytes; i += blockDim.x) dst[i] = src[i];
        }
    }
}

Readback::Readback(hipStream_t st) : st_(st) {}
Readback::~Readback()
{
    if (!stage_) return;
    if (in_flight_) (void)hipStreamSynchronize(st_);      // left in the middle of wait() (an error path): writes into the block may still be in flight
    g_stages.give(stage_);
}

rg_status Readback::add(void *host_dst, const void *dev_src, size_t bytes)
{
    if (bytes == 0) return RG_OK;
    if (!stage_) stage_ = g_stages.take();
    const size_t at = (used_ + 15) & ~(size_t)15;
    if (!stage_ || at + bytes > STAGE_BYTES) {           // too large for the block (or no pinned memory to be had): straight to the destination
        RG_HIP(hipMemcpyAsync(host_dst, dev_src, bytes, hipMemcpyDeviceToHost, st_));
        return RG_OK;
    }
    parts_.push_back({host_dst, dev_src, at, bytes});
    used_ = at + bytes;
    return RG_OK;
}

rg_status Readback::wait()
{
    in_flight_ = true;
    if (parts_.size() == 1) {
        RG_HIP(hipMemcpyAsync(stage_ + parts_[0].at, parts_[0].src, parts_[0].bytes, hipMemcpyDeviceToHost, st_));
    } else {
        for (size_t first = 0; first < parts_.size(); first += PACK_PARTS) {
            PackArgs a{};
            a.n = (int)std::min<size_t>(PACK_PARTS, parts_.size() - first);
            for (int p = 0; p < a.n; ++p) {
                const Part &part = parts_[first + p];
                a.src[p] = static_cast<const uint8_t *>(part.src);
                a.at[p] = (uint32_t)part.at;
                a.bytes[p] = (uint32_t)part.bytes;
            }
            hipLaunchKernelGGL(pack_pieces_kernel, dim3(1), dim3(256), 0, st_, a, stage_);
            RG_HIP(hipGetLastError());
        }
    }
    RG_HIP(hipStreamSynchronize(st_));
    in_flight_ = false;
    for (const Part &p : parts_) memcpy(p.dst, stage_ + p.at, p.bytes);
    parts_.clear();
    used_ = 0;
    return RG_OK;
}

// ---------------------------------------------------------------- arena
Arena::Arena(const rg_allocator *a)
{
    custom_ = (a != nullptr && a->alloc != nullptr && a->free != nullptr);
    if (custom_) a_ = *a; else a_ = rg_allocator{nullptr, nullptr, nullptr};
}

Arena::Arena(const rg_allocator *a, hipStream_t st) : Arena(a)
{
    drain_ = true;
    drain_stream_ = st;
}

Arena::~Arena() { release_all(); }

rg_status Arena::dev(uint64_t bytes, void **out)
{
    uint64_t want = bytes ? bytes : 256;
    void *p = nullptr;
    if (custom_) {
        p = a_.alloc(want, 1, a_.ctx);
        if (!p) { set_error("allocator callback returned NULL for %llu device bytes", (unsigned long long)want); return RG_ENOMEM; }
    } else {
        hipError_t e = hipSuccess;
        p = g_blocks.take(want, &e);
        if (!p) {
            set_error("hipMalloc(%llu) failed: %s", (unsigned long long)want, hipGetErrorString(e));
            return RG_ENOMEM;
        }
    }
    items_.push_back({p, 1, want});
    in_use_ += want;
    *out = p;
    return RG_OK;
}

bool Arena::dev_spare(uint64_t bytes, void **out)
{
    const uint64_t want = bytes ? bytes : 256;
    hipError_t e = hipSuccess;
    void *p = custom_ ? a_.alloc(want, 1, a_.ctx) : g_blocks.take(want, &e, false, nullptr, true);
    if (!p) return false;
    items_.push_back({p, 1, want});
    in_use_ += want;
    *out = p;
    return true;
}

rg_status Arena::dev_zeroed(uint64_t bytes, void **out, hipStream_t st)
{
    if (custom_) {
        RG_TRY(dev(bytes, out));
        RG_HIP(hipMemsetAsync(*out, 0, bytes ? bytes : 256, st));
        return RG_OK;
    }
    const uint64_t want = bytes ? bytes : 256;
    hipError_t e = hipSuccess;
    bool was_zero = false;
    void *p = g_blocks.take(want, &e, true, &was_zero);
    if (!p) {
        set_error("hipMalloc(%llu) failed: %s", (unsigned long long)want, hipGetErrorString(e));
        return RG_ENOMEM;
    }
    items_.push_back({p, 1, want});
    in_use_ += want;
    *out = p;
    if (!was_zero) RG_HIP(hipMemsetAsync(p, 0, g_blocks.size_of(p), st));      // the whole block: it may come back as all-zero for a larger request
    return RG_OK;
}

void Arena::free_zeroed(void *p)
{
    if (!p) return;
    for (size_t i = 0; i < items_.size(); ++i) {
        if (items_[i].p == p) {
            if (custom_) a_.free(p, items_[i].kind, a_.ctx);
            else g_blocks.give(p, true);
            in_use_ -= items_[i].bytes;
            items_[i] = items_.back();
            items_.pop_back();
            return;
        }
    }
}

rg_status Arena::pinned(uint64_t bytes, void **out)
{
    uint64_t want = bytes ? bytes : 256;
    void *p = nullptr;
    if (custom_) {
        p = a_.alloc(want, 0, a_.ctx);
        if (!p) { set_error("allocator callback returned NULL for %llu pinned bytes", (unsigned long long)want); return RG_ENOMEM; }
    } else {
        hipError_t e = hipHostMalloc(&p, want, hipHostMallocDefault);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            set_error("hipHostMalloc(%llu) failed: %s", (unsigned long long)want, hipGetErrorString(e));
            return RG_ENOMEM;
        }
    }
    items_.push_back({p, 0, want});
    in_use_ += want;
    *out = p;
    return RG_OK;
}

void Arena::free_one(void *p)
{
    if (!p) return;
    for (size_t i = 0; i < items_.size(); ++i) {
        if (items_[i].p == p) {
            if (custom_) a_.free(p, items_[i].kind, a_.ctx);
            else if (items_[i].kind == 1) g_blocks.give(p);
            else (void)hipHostFree(p);
            in_use_ -= items_[i].bytes;
            items_[i] = items_.back();
            items_.pop_back();
            return;
        }
    }
}

void Arena::release_all()
{
    if (drain_ && !items_.empty()) (void)hipStreamSynchronize(drain_stream_);     // kernels of the call that owns this scratch may still run
    drain_ = false;
    for (auto &it : items_) {
        if (custom_) a_.free(it.p, it.kind, a_.ctx);
        else if (it.kind == 1) g_blocks.give(it.p);
        else (void)hipHostFree(it.p);
    }
    items_.clear();
    in_use_ = 0;
}

// ---------------------------------------------------------------- last uses, retired handles
static std::atomic<uint64_t> g_next_log_id{1};
UseLog::UseLog() : id_(g_next_log_id.fetch_add(1)) {}
UseLog::Event::~Event()
{
    if (ev) (void)hipEventDestroy(ev);
}

void UseLog::note(UseLog &a, UseLog &b, hipStream_t st)
{
    std::scoped_lock lk(a.mu_, b.mu_);
    for (Use &u : a.uses_)
        if (u.st == st && u.partner == b.id_) {
            if (hipEventRecord(u.at->ev, st) != hipSuccess) { (void)hipGetLastError(); a.lost_ = b.lost_ = true; }
            return;
        }
    // The pair's first use on this stream.  An event whose other holder has let go of it is recorded again, here behind what it stood for, so that a
    // schedule served from cache after cache does not collect events.  (Not found by asking which have completed: hipEventQuery ends a global
    // capture that is under way on any other stream.)
    std::shared_ptr<Event> at;
    a.take_unshared(st, &at);
    b.take_unshared(st, &at);
    if (!at) at = std::make_shared<Event>();
    if (!at->ev && hipEventCreateWithFlags(&at->ev, hipEventDisableTiming) != hipSuccess) { (void)hipGetLastError(); at->ev = nullptr; a.lost_ = b.lost_ = true; return; }
    if (hipEventRecord(at->ev, st) != hipSuccess) { (void)hipGetLastError(); a.lost_ = b.lost_ = true; return; }
    a.uses_.push_back({st, b.id_, at});
    b.uses_.push_back({st, a.id_, at});
}

void UseLog::take_unshared(hipStream_t st, std::shared_ptr<Event> *first)
{
    size_t kept = 0;
    for (Use &u : uses_) {
        if (u.st == st && u.at.use_count() == 1) {
            if (!*first) *first = std::move(u.at);
        } else {
            if (&uses_[kept] != &u) uses_[kept] = std::move(u);
            ++kept;
        }
    }
    uses_.resize(kept);
}

bool UseLog::idle()
{
    std::lock_guard<std::mutex> lk(mu_);
    if (lost_) return false;
    for (Use &u : uses_) {
        const hipError_t e = hipEventQuery(u.at->ev);
        if (e == hipErrorNotReady) return false;
        if (e != hipSuccess) { (void)hipGetLastError(); return false; }
    }
    return true;
}

void UseLog::wait()
{
    std::lock_guard<std::mutex> lk(mu_);
    if (lost_) { (void)hipDeviceSynchronize(); lost_ = false; return; }
    for (Use &u : uses_)
        if (hipEventSynchronize(u.at->ev) != hipSuccess) { (void)hipGetLastError(); (void)hipDeviceSynchronize(); return; }
}

rg_status compute_units(int *n_cu)
{
    static std::atomic<int> known[64];                   // per device; 0: not asked yet
    int dev = 0;
    RG_HIP(hipGetDevice(&dev));
    int n = dev >= 0 && dev < 64 ? known[dev].load(std::memory_order_relaxed) : 0;
    if (n == 0) {
        RG_HIP(hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev));
        if (dev >= 0 && dev < 64) known[dev].store(n, std::memory_order_relaxed);
    }
    *n_cu = n;
    return RG_OK;
}

namespace {
struct Retired {
    std::mutex mu;
    std::vector<rg_schedule *> schedules;
    std::vector<rg_cache *> caches;
};
Retired &retired() { static Retired *r = new Retired(); return *r; }     // (never destructed: no HIP calls at process exit)

template <typename H> void reap_list(std::vector<H *> &list, bool wait)
{
    size_t kept = 0;
    for (H *h : list) {
        if (wait) h->uses.wait();
        if (wait || h->uses.idle()) delete h;
        else list[kept++] = h;
    }
    list.resize(kept);
}

// A handle leaves: at once when nothing reads it any more; with a caller's allocator after a wait for its own
// readers (the allocator may not outlive the call); otherwise it is parked until a later call finds it idle.
template <typename H> void retire(H *h, std::vector<H *> Retired::*list)
{
    reap_retired(false);
    if (h->arena.allocator()) h->uses.wait();
    if (h->arena.allocator() || h->uses.idle()) { delete h; return; }
    Retired &r = retired();
    std::lock_guard<std::mutex> lk(r.mu);
    (r.*list).push_back(h);
}
}  // namespace

rg_status helper_stream(hipStream_t *out)
{
    static std::mutex mu;
    static hipStream_t streams[64] = {};
    int dev = 0;
    RG_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) { set_error("helper_stream: device %d out of range", dev); return RG_EINVAL; }
    std::lock_guard<std::mutex> lk(mu);
    if (!streams[dev]) RG_HIP(hipStreamCreateWithFlags(&streams[dev], hipStreamNonBlocking));
    *out = streams[dev];
    return RG_OK;
}

void reap_retired(bool wait)
{
    Retired &r = retired();
    std::lock_guard<std::mutex> lk(r.mu);
    reap_list(r.schedules, wait);
    reap_list(r.caches, wait);
}

// ---------------------------------------------------------------- profiling
static std::atomic<int> g_prof_on{0};
static std::mutex g_prof_mu;
struct Pending { int group; hipEvent_t e0, e1; };
static std::vector<Pending> g_pending;
static std::vector<hipEvent_t> g_free_events;
static double g_ms[RG_N_KERNEL_GROUPS];
static uint64_t g_launches[RG_N_KERNEL_GROUPS];

bool profiling_on() { return g_prof_on.load(std::memory_order_relaxed) != 0; }

ScopedTimer::ScopedTimer(int g, hipStream_t s) : group(g), st(s)
{
    if (g < 0 || !profiling_on()) return;       // group -1: a launch that is never timed
    {
        std::lock_guard<std::mutex> lk(g_prof_mu);
        if (g_free_events.size() >= 2) {
            e0 = g_free_events.back(); g_free_events.pop_back();
            e1 = g_free_events.back(); g_free_events.pop_back();
        }
    }
    if (!e0 && (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)) { e0 = e1 = nullptr; return; }
    (void)hipEventRecord(e0, st);
}

ScopedTimer::~ScopedTimer()
{
    if (!e0) return;
    (void)hipEventRecord(e1, st);
    std::lock_guard<std::mutex> lk(g_prof_mu);
    g_pending.push_back({group, e0, e1});
}

static void drain_pending_locked()
{
    for (auto &p : g_pending) {
        float ms = 0.f;
        if (hipEventSynchronize(p.e1) == hipSuccess && hipEventElapsedTime(&ms, p.e0, p.e1) == hipSuccess) {
            g_ms[p.group] += ms;
            g_launches[p.group] += 1;
        }
        g_free_events.push_back(p.e0);
        g_free_events.push_back(p.e1);
    }
    g_pending.clear();
}

// ---------------------------------------------------------------- prefix sum
// Per-block totals, then per-block local scans plus the sum of the totals in front: one launch for a single block,
// two while a block can add up its predecessors' totals itself, three (with a scan of the totals between) beyond.
// Each block covers SCAN_TILE consecutive elements.
constexpr int SCAN_THREADS = 256;
constexpr int SCAN_PER_THREAD = 16;
constexpr int SCAN_TILE = SCAN_THREADS * SCAN_PER_THREAD;

__device__ __forceinline__ int64_t block_exclusive_scan_i64(int64_t x, int64_t *total, int64_t *lds /* [SCAN_THREADS/64 + 1] */)
{
    // wave-level inclusive scan by shuffles, then across the block's waves through LDS
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t incl = x;
    for (int d = 1; d < 64; d <<= 1) {
        int64_t y = __shfl_up(incl, d, 64);
        if (lane >= d) incl += y;
    }
    if (lane == 63) lds[wave] = incl;
    __syncthreads();
    int64_t base = 0, tot = 0;
    const int nw = blockDim.x >> 6;
    for (int w = 0; w < nw; ++w) {
        int64_t s = lds[w];
        if (w < wave) base += s;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return base + incl - x;
}

__global__ void __launch_bounds__(SCAN_THREADS) scan_block_totals(const int32_t *__restrict__ in, int64_t n, int64_t *__restrict__ block_tot)
{
    __shared__ int64_t lds[SCAN_THREADS / 64 + 1];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
    int64_t s = 0;
    for (int k = 0; k < SCAN_PER_THREAD; ++k) {
        int64_t i = base + (int64_t)k * SCAN_THREADS + threadIdx.x;
        if (i < n) s += in[i];
    }
    int64_t tot;
    (void)block_exclusive_scan_i64(s, &tot, lds);
    if (threadIdx.x == 0) block_tot[blockIdx.x] = tot;
}

__global__ void __launch_bounds__(SCAN_THREADS) scan_of_totals(int64_t *__restrict__ block_tot, int64_t n_blocks, int64_t *__restrict__ grand_total)
{
    __shared__ int64_t lds[SCAN_THREADS / 64 + 1];
    int64_t carry = 0;
    for (int64_t base = 0; base < n_blocks; base += SCAN_THREADS) {
        int64_t i = base + threadIdx.x;
        int64_t x = i < n_blocks ? block_tot[i] : 0;
        int64_t tot;
        int64_t ex = block_exclusive_scan_i64(x, &tot, lds);
        if (i < n_blocks) block_tot[i] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) *grand_total = carry;
}

// FUSED: block_base is the raw per-block totals; the block adds up the totals in front of its own (a few thousand
// at most, see scan_i32_to_i64) instead of reading a scanned table, and the last block writes the grand total.
template <bool FUSED>
__global__ void __launch_bounds__(SCAN_THREADS) scan_apply(const int32_t *__restrict__ in, int64_t n, const int64_t *__restrict__ block_base,
                                                           int64_t *__restrict__ out)
{
    __shared__ int64_t lds[SCAN_THREADS / 64 + 1];
    int64_t base;
    if (FUSED) {
        int64_t part = 0;
        for (int64_t j = threadIdx.x; j < (int64_t)blockIdx.x; j += SCAN_THREADS) part += block_base[j];
        (void)block_exclusive_scan_i64(part, &base, lds);
    } else base = block_base[blockIdx.x];
    // thread t owns SCAN_PER_THREAD consecutive elements so one block scan suffices
    const int64_t first = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_PER_THREAD;
    int32_t v[SCAN_PER_THREAD];
    int64_t s = 0;
    for (int k = 0; k < SCAN_PER_THREAD; ++k) {
        int64_t i = first + k;
        v[k] = i < n ? in[i] : 0;
        s += v[k];
    }
    int64_t tot;
    int64_t run = base + block_exclusive_scan_i64(s, &tot, lds);
    for (int k = 0; k < SCAN_PER_THREAD; ++k) {
        int64_t i = first + k;
        if (i < n) out[i] = run;
        run += v[k];
    }
    if (FUSED && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[n] = base + tot;
}

constexpr int64_t SCAN_FUSED_BLOCKS = 4096;      // up to here a block adds up its predecessors' totals itself (16 M elements)

rg_status scan_i32_to_i64(const int32_t *in, int64_t *out, int64_t n, Arena &tmp, hipStream_t st)
{
    const int64_t n_blocks = (n + SCAN_TILE - 1) / SCAN_TILE;
    if (n_blocks <= 1) {
        // one block: nothing in front of it, its own total is the grand total (n = 0 writes out[0] = 0)
        hipLaunchKernelGGL(scan_apply<true>, dim3(1), dim3(SCAN_THREADS), 0, st, in, n, (const int64_t *)nullptr, out);
        RG_HIP(hipGetLastError());
        return RG_OK;
    }
    int64_t *block_tot = nullptr;
    RG_TRY(tmp.dev_n<int64_t>((uint64_t)n_blocks, &block_tot));
    hipLaunchKernelGGL(scan_block_totals, dim3((unsigned)n_blocks), dim3(SCAN_THREADS), 0, st, in, n, block_tot);
    if (n_blocks <= SCAN_FUSED_BLOCKS) {
        hipLaunchKernelGGL(scan_apply<true>, dim3((unsigned)n_blocks), dim3(SCAN_THREADS), 0, st, in, n, block_tot, out);
    } else {
        hipLaunchKernelGGL(scan_of_totals, dim3(1), dim3(SCAN_THREADS), 0, st, block_tot, n_blocks, out + n);
        hipLaunchKernelGGL(scan_apply<false>, dim3((unsigned)n_blocks), dim3(SCAN_THREADS), 0, st, in, n, block_tot, out);
    }
    RG_HIP(hipGetLastError());
    return RG_OK;
}

// ---------------------------------------------------------------- graph validation
// Bound by reading indptr and indices once.  Where indptr ascends from 0 -- every graph but a damaged one -- the rows
// lie back to back, and the violations are counted over the flat array: every ID out of range and every ID not above the one
// in front of it, less the latter at the starts of rows.  A wave per row, which is what finds the violations of any indptr (validate_rows, now run only where
// the rows are out of order), spends its time on 2.45 M rows' dependent loads: a graph of 122 M edges 4.4 ms, the two
// streaming passes together 0.1 (0.5 GB).
// The starts of the rows are scattered reads of lines that the flat pass reads too, so a wave of that pass looks at those among
// the IDs it has just read (found in indptr, which is known to ascend by then), while they are in a cache: 2.45 M rows,
// 122 M edges, starts with the pass over indptr 43 + 90 us, so 9 + 107.  (Per 64 KB and workgroup, behind a barrier: 6 + 129.)
// Many rows to few IDs take the wave many turns, and small graphs feel its search for its first row: there the starts stay with
// the pass over indptr (starts there / behind the IDs: 50 M nodes, 2 IDs each 238 / 292 us, 7 in one of 100 134 / 534; 8,000 nodes, 8 each 32.8 / 34.6).
// So do, in any graph, those of 64 consecutive rows (from a multiple of 64 on) with few IDs together: however the rows are spread, a wave has
// no more than three blocks of 64 to look at for every 1,024 IDs it reads, and few steps between two of them.  Where the line lies (all starts with the
// pass over indptr / behind the IDs / blocks from 256, 384, 512, 1,024 IDs on behind the IDs): a few rows with most IDs and the others with some 5 to 20, 2.4 M nodes,
// 45 M IDs 83 / 79 / 78, 80, 88, 96 us, 70 M 104 / 98 / 97, 98, 98, 112; 2.45 M rows sorted by length 157 / 156 / 168, 160, 156, 152; 7 M nodes, 100
// rows of 1.2 M IDs, then one ID in each 148 / 302 / 156 at any, in every 64th 143 / 10,070 / 146 at any.
constexpr int VAL_THREADS = 256;
constexpr int VAL_SLOTS = 16;                  // each count is kept in this many copies, summed by the host (adds to one address queue up)
constexpr int64_t VAL_ROW_IDS = 16;            // IDs per row, on average, from which on a wave looks at the starts among its IDs ...
constexpr int64_t VAL_MANY_IDS = 1 << 24;      // ... where there are so many,
constexpr int64_t VAL_BLOCK_IDS = 384;         // in blocks of 64 rows that hold so many
__device__ __forceinline__ bool starts_with_the_ids(int64_t n_nodes, int64_t n) { return n >= VAL_ROW_IDS * n_nodes && n >= VAL_MANY_IDS; }
__device__ __forceinline__ int64_t from_lane(int64_t x, int lane)      // (lane the same in the whole wave)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, lane), hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)x >> 32), lane);
    return (int64_t)((uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ bool long_block(int64_t start, int64_t end) { return end - start >= VAL_BLOCK_IDS; }
enum { VAL_ROWS = 0, VAL_FLAT = 1, VAL_STARTS = 2, VAL_GENERAL = 3, VAL_COUNTS = 4 };

__device__ __forceinline__ void add_block_count(unsigned long long x, unsigned long long *counts, int which)
{
    __shared__ unsigned long long part[VAL_THREADS / 64];
    for (int o = 32; o > 0; o >>= 1) x += __shfl_down(x, o, 64);
    __syncthreads();                            // (a second call in the same kernel: the first one's sums have been read)
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = x;
    __syncthreads();
    if (threadIdx.x != 0) return;
    x = 0;
    for (int w = 0; w < VAL_THREADS / 64; ++w) x += part[w];
    if (x) atomicAdd(&counts[which * VAL_SLOTS + blockIdx.x % VAL_SLOTS], x);
}

// Rows that decrease (and an indptr that does not start at 0), and the non-empty rows whose first ID is in range but not
// above the ID in front of it in the flat array, where the flat pass does not look at those.  A wave has 64 consecutive rows at a time.
__global__ void __launch_bounds__(VAL_THREADS) validate_indptr(int64_t n_nodes, const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                                               unsigned long long *__restrict__ counts)
{
    const int64_t n = indptr[n_nodes];
    const bool flat_looks = starts_with_the_ids(n_nodes, n);
    unsigned long long bad = 0, starts = 0;
    const int lane = threadIdx.x & 63;
    const int64_t step = (int64_t)gridDim.x * VAL_THREADS;
    for (int64_t v0 = (int64_t)blockIdx.x * VAL_THREADS + threadIdx.x; v0 - lane < n_nodes; v0 += 4 * step) {
        int64_t b[4], e[4];
        int32_t here[4], front[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t v = v0 + k * step;
            b[k] = v < n_nodes ? indptr[v] : n;
            e[k] = v < n_nodes ? indptr[v + 1] : n;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bool mine = !flat_looks || !long_block(from_lane(b[k], 0), from_lane(e[k], 63));
            const bool look = mine && b[k] > 0 && b[k] < e[k];
            here[k] = look ? indices[b[k]] : -1;
            front[k] = look ? indices[b[k] - 1] : -1;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (e[k] < b[k] || (v0 + k * step == 0 && b[k] != 0)) ++bad;
            if (here[k] >= 0 && here[k] < n_nodes && front[k] >= here[k]) ++starts;
        }
    }
    add_block_count(bad, counts, VAL_ROWS);
    add_block_count(starts, counts, VAL_STARTS);
}

__device__ __forceinline__ bool any_row_bad(const unsigned long long *counts)
{
    unsigned long long x = 0;
    for (int k = 0; k < VAL_SLOTS; ++k) x |= counts[VAL_ROWS * VAL_SLOTS + k];
    return x != 0;
}

// The first v with indptr[v] >= x, by a wave that looks at 64 places at a time (x the same in all lanes, 0 <= x <=
// indptr[n_nodes]; indptr ascends from 0).
__device__ __forceinline__ int64_t first_row_from(const int64_t *__restrict__ indptr, int64_t n_nodes, int64_t x, int lane)
{
    int64_t lo = 0, hi = n_nodes;                // the answer lies in [lo, hi]
    while (lo < hi) {
        const int64_t step = (hi - lo + 63) / 64, at = lo + lane * step;
        const int k = __popcll(__ballot(at < hi && indptr[min(at, hi)] < x));      // the first k places lie in front of it
        if (k == 0) return lo;
        hi = min(lo + k * step, hi);
        lo += (k - 1) * step + 1;
    }
    return lo;
}

// The first long block of 64 rows from block k on, or no block of those that start in front of id_stop; *start: where it starts (INT64_MAX: there is
// none).  By a wave, 64 blocks at a time; where those hold few IDs together, 64 groups of 64 blocks at a time, and so on (a group that holds
// few IDs has no long block; the first that may have one is looked into).
__device__ __forceinline__ int64_t next_long_block(const int64_t *__restrict__ indptr, int64_t n_nodes, int64_t k, int64_t id_stop, int lane, int64_t *start)
{
    int64_t group = 1;                           // blocks per lane
    while (64 * k < n_nodes) {
        const int64_t s = indptr[min(64 * (k + lane * group), n_nodes)], e = indptr[min(64 * (k + (lane + 1) * group), n_nodes)];
        const int64_t first = from_lane(s, 0);
        if (first >= id_stop) break;
        const unsigned long long m = __ballot(long_block(s, e));
        if (m != 0ull) {
            const int l = __builtin_amdgcn_readfirstlane(__ffsll((long long)m) - 1);
            k += l * group;
            *start = from_lane(s, l);
            if (group == 1) return k;
            group /= 64;
        } else {
            k += 64 * group;
            if (!long_block(first, from_lane(e, 63)) && 64 * k < n_nodes) group *= 64;      // (at most three times: the rows are fewer than 2^31)
        }
    }
    *start = INT64_MAX;
    return k;
}

// The flat array, 4 KB at a time per wave: 16-byte loads from the first aligned ID on, four in flight per lane; the IDs
// in front of the first whole vector and after the last by the first workgroup.  Where rows are looked at too, a wave has a contiguous
// part, and behind each 4 KB come the rows of the long blocks that start in them: the non-empty ones whose first ID is in range but not above
// the ID in front of it.  Elsewhere the waves read side by side (50 M nodes, 2 IDs each, parts / side by side 236 / 231 us).
constexpr int64_t VAL_ROUND = 4 * 64;            // vectors that a wave reads at once
__global__ void __launch_bounds__(VAL_THREADS) validate_flat(int64_t n_nodes, const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                                             unsigned long long *__restrict__ counts)
{
    if (any_row_bad(counts)) return;
    const int64_t n = indptr[n_nodes];
    const uint32_t limit = (uint32_t)n_nodes;
    auto wrong = [&](int32_t front, int32_t u) { return ((uint32_t)u >= limit || front >= u) ? 1u : 0u; };
    unsigned long long bad = 0, starts = 0;
    int64_t head = (int64_t)((16 - ((uintptr_t)indices & 15)) & 15) / 4;
    if (head > n) head = n;
    const int64_t n_vec = (n - head) >> 2;
    const int4 *vec = reinterpret_cast<const int4 *>(indices + head);
    const int lane = threadIdx.x & 63;
    const int64_t n_waves = (int64_t)gridDim.x * (VAL_THREADS / 64), wave = (int64_t)blockIdx.x * (VAL_THREADS / 64) + (threadIdx.x >> 6);
    const bool look_at_starts = starts_with_the_ids(n_nodes, n);
    const int64_t part = look_at_starts ? ((n_vec + n_waves - 1) / n_waves + VAL_ROUND - 1) / VAL_ROUND * VAL_ROUND : VAL_ROUND;      // (a division in 64 bits is a microsecond of a small check)
    const int64_t i_first = wave * part, i_step = look_at_starts ? VAL_ROUND : n_waves * VAL_ROUND;
    const int64_t i_end = look_at_starts ? min((wave + 1) * part, n_vec) : n_vec;
    const int64_t part_end = (wave + 1) * part >= n_vec ? n : head + 4 * (wave + 1) * part;
    int64_t block = 0, start = 0;                // the next block of 64 rows, and where it starts
    if (look_at_starts && wave > 0 && wave * part < n_vec) {
        block = (first_row_from(indptr, n_nodes, head + 4 * wave * part, lane) + 63) / 64;
        start = 64 * block < n_nodes ? indptr[64 * block] : INT64_MAX;
    }
    for (int64_t i_lo = i_first; i_lo < i_end; i_lo += i_step) {
        int4 x[4];
        int32_t front[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t i = i_lo + k * 64 + lane;
            x[k] = i < i_end ? vec[i] : make_int4(0, 0, 0, 0);
            front[k] = lane == 0 && i < i_end && head + 4 * i > 0 ? indices[head + 4 * i - 1] : -1;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int32_t left = __shfl_up(x[k].w, 1, 64);
            const int32_t f = lane == 0 ? front[k] : left;
            if (i_lo + k * 64 + lane < i_end) bad += wrong(f, x[k].x) + wrong(x[k].x, x[k].y) + wrong(x[k].y, x[k].z) + wrong(x[k].z, x[k].w);
        }
        if (!look_at_starts) continue;
        const int64_t id_end = i_lo + VAL_ROUND >= n_vec ? n : head + 4 * (i_lo + VAL_ROUND);       // (a part that is not the last is whole rounds)
        while (start < id_end) {
            const int64_t v = 64 * block + lane, b = indptr[min(v, n_nodes)], e = indptr[min(v + 1, n_nodes)], end = from_lane(e, 63);
            ++block;
            if (long_block(start, end)) {
                const bool look = b > 0 && b < e;
                const int32_t here = look ? indices[b] : -1, before = look ? indices[b - 1] : -1;
                if (here >= 0 && here < n_nodes && before >= here) ++starts;
                start = 64 * block < n_nodes ? end : INT64_MAX;
            } else block = next_long_block(indptr, n_nodes, block, part_end, lane, &start);
        }
    }
    if (blockIdx.x == 0 && threadIdx.x < 8) {
        const int64_t j = threadIdx.x < 4 ? (int64_t)threadIdx.x : head + 4 * n_vec + threadIdx.x - 4;
        if (threadIdx.x < 4 ? j < head : j < n) bad += wrong(j > 0 ? indices[j - 1] : -1, indices[j]);
    }
    add_block_count(bad, counts, VAL_FLAT);
    if (look_at_starts) add_block_count(starts, counts, VAL_STARTS);
}

// Any indptr: one wave per row, grid-stride; nothing to do where validate_indptr found no row that decreases.  With more
// workgroups than the chip holds, because the longest rows are the tail and waves that come free must find other rows (20 M
// nodes, 40 M edges, one row that decreases: 3.3 ms with a grid of what the chip holds, 2.2 so).  That many are launched only
// once the host knows that they are needed; a few at once, which costs less than a second wait.
__global__ void __launch_bounds__(VAL_THREADS) validate_rows(int64_t n_nodes, const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                                             unsigned long long *__restrict__ counts)
{
    if (!any_row_bad(counts)) return;
    const int lane = threadIdx.x & 63;
    const int64_t wave0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t n_waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    unsigned long long bad = 0;
    for (int64_t v = wave0; v < n_nodes; v += n_waves) {
        const int64_t b = indptr[v], e = indptr[v + 1];
        if (e < b || (v == 0 && b != 0)) { if (lane == 0) ++bad; continue; }
        for (int64_t j = b + lane; j < e; j += 64) {
            const int32_t u = indices[j];
            if (u < 0 || u >= n_nodes) ++bad;
            else if (j > b && indices[j - 1] >= u) ++bad;
        }
    }
    add_block_count(bad, counts, VAL_GENERAL);
}

}  // namespace rg

rg_cache::~rg_cache()
{
    if (ev_fork) (void)hipEventDestroy(ev_fork);
    if (ev_join) (void)hipEventDestroy(ev_join);
}

using namespace rg;

extern "C" {

const char *rg_last_error(void) { return g_err; }

void rg_profile_enable(int on) { g_prof_on.store(on ? 1 : 0); }

void rg_profile_reset(void)
{
    std::lock_guard<std::mutex> lk(g_prof_mu);
    drain_pending_locked();
    for (int i = 0; i < RG_N_KERNEL_GROUPS; ++i) { g_ms[i] = 0.0; g_launches[i] = 0; }
}

rg_status rg_profile_read(double *ms, uint64_t *launches)
{
    if (!ms || !launches) { set_error("rg_profile_read: null output"); return RG_EINVAL; }
    std::lock_guard<std::mutex> lk(g_prof_mu);
    drain_pending_locked();
    for (int i = 0; i < RG_N_KERNEL_GROUPS; ++i) { ms[i] = g_ms[i]; launches[i] = g_launches[i]; }
    return RG_OK;
}

rg_status rg_graph_validate(const rg_graph *g, void *stream, uint64_t *n_bad)
{
    if (!g || !n_bad || !g->indptr) { set_error("rg_graph_validate: null argument"); return RG_EINVAL; }
    if (g->n_nodes < 0 || g->n_nodes >= ((int64_t)1 << 31)) { set_error("rg_graph_validate: n_nodes out of range"); return RG_ERANGE; }
    hipStream_t st = as_stream(stream);
    if (g->n_nodes == 0) { *n_bad = 0; return RG_OK; }
    Arena tmp(nullptr, st);
    unsigned long long *counts = nullptr, host[VAL_COUNTS * VAL_SLOTS];
    RG_TRY(tmp.dev(sizeof(host), (void **)&counts));
    RG_HIP(hipMemsetAsync(counts, 0, sizeof(host), st));
    int dev = 0, n_cu = 256;
    RG_HIP(hipGetDevice(&dev));
    RG_HIP(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
    const unsigned row_grid = (unsigned)std::min<int64_t>((g->n_nodes + 4 * VAL_THREADS - 1) / (4 * VAL_THREADS), (int64_t)n_cu * 8);
    hipLaunchKernelGGL(validate_indptr, dim3(row_grid), dim3(VAL_THREADS), 0, st, g->n_nodes, g->indptr, g->indices, counts);
    hipLaunchKernelGGL(validate_flat, dim3((unsigned)n_cu * 8), dim3(VAL_THREADS), 0, st, g->n_nodes, g->indptr, g->indices, counts);
    const int64_t general_grid = std::min<int64_t>((g->n_nodes + 3) / 4, 65536);
    auto general = [&] { hipLaunchKernelGGL(validate_rows, dim3((unsigned)general_grid), dim3(VAL_THREADS), 0, st, g->n_nodes, g->indptr, g->indices, counts); };
    const bool at_once = general_grid <= (int64_t)n_cu * 16;
    if (at_once) general();
    RG_HIP(hipGetLastError());
    uint64_t sum[VAL_COUNTS] = {};
    auto fetch = [&]() -> rg_status {
        Readback rb(st);
        RG_TRY(rb.add(host, counts, sizeof(host)));
        RG_TRY(rb.wait());
        for (uint64_t &x : sum) x = 0;
        for (int k = 0; k < VAL_COUNTS * VAL_SLOTS; ++k) sum[k / VAL_SLOTS] += host[k];
        return RG_OK;
    };
    RG_TRY(fetch());
    if (sum[VAL_ROWS] != 0 && !at_once) {
        general();
        RG_HIP(hipGetLastError());
        RG_TRY(fetch());
    }
    tmp.drained();
    *n_bad = sum[VAL_ROWS] ? sum[VAL_GENERAL] : sum[VAL_FLAT] - sum[VAL_STARTS];
    return RG_OK;
}

rg_status rg_schedule_info(const rg_schedule *s, uint32_t *n_batches, uint32_t *L, int64_t *n_nodes)
{
    if (!s) { set_error("rg_schedule_info: null schedule"); return RG_EINVAL; }
    if (n_batches) *n_batches = s->n_batches;
    if (L) *L = s->L;
    if (n_nodes) *n_nodes = s->n_nodes;
    return RG_OK;
}

rg_status rg_schedule_frontier(const rg_schedule *s, uint32_t hop, const int32_t **ids_dev,
                               const int64_t **batch_off_dev, const int64_t **batch_off_host)
{
    if (!s) { set_error("rg_schedule_frontier: null schedule"); return RG_EINVAL; }
    if (hop > s->L) { set_error("rg_schedule_frontier: hop %u > L = %u", hop, s->L); return RG_ERANGE; }
    const HopData &h = s->hop[hop];
    if (ids_dev) *ids_dev = h.ids;
    if (batch_off_dev) *batch_off_dev = h.off_dev;
    if (batch_off_host) *batch_off_host = h.off_host.data();
    return RG_OK;
}

rg_status rg_schedule_seeds(const rg_schedule *s, const int32_t **seeds_dev, const int64_t **batch_off_dev)
{
    if (!s) { set_error("rg_schedule_seeds: null schedule"); return RG_EINVAL; }
    return rg_schedule_frontier(s, 0, seeds_dev, batch_off_dev, nullptr);
}

rg_status rg_schedule_samples(const rg_schedule *s, uint32_t hop, const int64_t **samp_off_dev,
                              const int32_t **samp_nbr_dev, int64_t *n_samples)
{
    if (!s) { set_error("rg_schedule_samples: null schedule"); return RG_EINVAL; }
    if (hop >= s->L) { set_error("rg_schedule_samples: hop %u >= L = %u", hop, s->L); return RG_ERANGE; }
    const HopData &h = s->hop[hop];
    if (samp_off_dev) *samp_off_dev = h.samp_off;
    if (samp_nbr_dev) *samp_nbr_dev = h.samp_nbr;
    if (n_samples) *n_samples = h.n_samples;
    return RG_OK;
}

rg_status rg_cache_view(const rg_cache *c, uint64_t *K_eff, const int32_t **cache_ids_dev, const uint32_t **freq_dev,
                        const int32_t **slot_of_dev, const void **rows_dev, uint64_t *stride)
{
    if (!c) { set_error("rg_cache_view: null cache"); return RG_EINVAL; }
    if (K_eff) *K_eff = c->K_eff;
    if (cache_ids_dev) *cache_ids_dev = c->cache_ids;
    if (freq_dev) RG_TRY(cache_freq_view(c, freq_dev));
    if (slot_of_dev) RG_TRY(cache_slot_view(c, slot_of_dev));
    if (rows_dev) *rows_dev = c->rows;
    if (stride) *stride = c->stride;
    return RG_OK;
}

void rg_schedule_destroy(rg_schedule *s)
{
    if (s) retire(s, &Retired::schedules);
}

void rg_trim_memory(void)
{
    reap_retired(true);
    g_blocks.trim();
}

void rg_cache_destroy(rg_cache *c)
{
    if (c) retire(c, &Retired::caches);
}

}  // extern "C"
