// Device-side helpers shared by the schedule kernels: the hash family, the
// batch lookup and the per-batch reached-ID bitmaps.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rg {

// ---------------------------------------------------------------- hash family
// H of Sec. 3 "Seeding and reproducibility": a 64-bit multiply / xor-shift
// mixer.  Constants: floor(2^64/phi), frac(sqrt 2) * 2^64 made odd,
// frac(sqrt 3) * 2^64; the 32-bit ones are the top words of the same numbers.
constexpr uint64_t HG64 = 0x9E3779B97F4A7C15ull;
constexpr uint64_t HA64 = 0x6A09E667F3BCC909ull;
constexpr uint64_t HB64 = 0xBB67AE8584CAA73Bull;
constexpr uint32_t HG32 = 0x9E3779B9u;
constexpr uint32_t HA32 = 0x6A09E667u;
constexpr uint32_t HB32 = 0xBB67AE85u;

__host__ __device__ __forceinline__ uint64_t mix64(uint64_t x)
{
    x ^= x >> 32; x *= HA64; x ^= x >> 29; x *= HB64; x ^= x >> 32;
    return x;
}
__host__ __device__ __forceinline__ uint64_t combine(uint64_t h, uint64_t x) { return mix64(h ^ mix64(x + HG64)); }

// Key of neighbour u under a node's state (lo, hi).  For fixed state this is a
// bijection of 32-bit words, so the keys of one row never tie.
//
// key32_open is the key without its last step, x ^= x >> 16, which leaves the upper half of the word alone: where the
// lower half of a cut is all ones, key <= cut exactly when open key <= cut.  A row is streamed against such a cut with
// two operations less per ID.
__device__ __forceinline__ uint32_t key32_open(uint32_t lo, uint32_t hi, uint32_t u)
{
    uint32_t x = u ^ lo;
    x *= HG32; x ^= x >> 16;
    x += hi;
    x *= HA32; x ^= x >> 15;
    x *= HB32;
    return x;
}
__device__ __forceinline__ uint32_t key32(uint32_t lo, uint32_t hi, uint32_t u)
{
    const uint32_t x = key32_open(lo, hi, u);
    return x ^ (x >> 16);
}

// The neighbour ID whose key is x: key32 undone step by step (an odd multiplier's inverse modulo 2^32 by Newton's
// iteration, which doubles the right low bits each time).
constexpr uint32_t inverse32(uint32_t a)
{
    uint32_t y = a;                                // right in the low 3 bits: a * a = 1 modulo 8
    for (int k = 0; k < 4; ++k) y *= 2u - a * y;
    return y;
}
static_assert(inverse32(HG32) * HG32 == 1u && inverse32(HA32) * HA32 == 1u && inverse32(HB32) * HB32 == 1u, "");
__device__ __forceinline__ uint32_t key32_inverse(uint32_t lo, uint32_t hi, uint32_t x)
{
    x ^= x >> 16; x *= inverse32(HB32);
    x ^= (x >> 15) ^ (x >> 30); x *= inverse32(HA32);
    x -= hi;
    x ^= x >> 16; x *= inverse32(HG32);
    return x ^ lo;
}

// ---------------------------------------------------------------- drawn positions (the O(f) sampler)
// Position p_t of draw t among the deg > f slots of a row, for a node state s; p_0, p_1, ... are distinct.
//   deg <= 64: selection without replacement.  Draw k takes r_k = floor(u_k * (deg - k)), u_k the top 32 bits of
//              mix64(s + (k + 1) G) read as a fraction, and picks the r_k-th slot not picked by draws 0 .. k-1.
//   deg > 64:  p_t = pi_s(t), pi_s a permutation of [0, deg): an alternating Feistel network on
//              n = bitlen(deg - 1) bits (left part n - n/2 bits, right part n/2 bits, six rounds, round value =
//              top 32 bits of mix64((s ^ other part) + (r + 1) G)), walked along its cycle until the value is
//              below deg.  The walk ends: the cycle through t comes back to t < deg.
constexpr uint32_t DRAW_SELECT = 64;
__device__ __forceinline__ uint32_t draw32(uint64_t s, uint32_t k) { return (uint32_t)(mix64(s + (uint64_t)(k + 1u) * HG64) >> 32); }

__device__ __forceinline__ uint32_t feistel(uint32_t x, uint32_t n_bits, uint64_t s)
{
    const uint32_t hb = n_bits >> 1, ha = n_bits - hb;
    const uint32_t mask_a = (1u << ha) - 1u, mask_b = (1u << hb) - 1u;        // n_bits <= 31: both parts below 32 bits
    uint32_t a = x >> hb, b = x & mask_b;
#pragma unroll
    for (uint32_t r = 0; r < 6; ++r) {
        if ((r & 1u) == 0) a ^= (uint32_t)(mix64((s ^ (uint64_t)b) + (uint64_t)(r + 1u) * HG64) >> 32) & mask_a;
        else               b ^= (uint32_t)(mix64((s ^ (uint64_t)a) + (uint64_t)(r + 1u) * HG64) >> 32) & mask_b;
    }
    return (a << hb) | b;
}

// The r-th (from 0) set bit of m; m has more than r set bits.
__device__ __forceinline__ uint32_t nth_set_bit(uint64_t m, uint32_t r)
{
    const uint32_t low = (uint32_t)__popc((uint32_t)m);
    const bool upper = r >= low;
    uint32_t x = upper ? (uint32_t)(m >> 32) : (uint32_t)m, p = upper ? 32u : 0u;
    if (upper) r -= low;
#pragma unroll
    for (uint32_t w = 16; w >= 1; w >>= 1) {
        const uint32_t c = (uint32_t)__popc(x & ((1u << w) - 1u));
        if (r >= c) { r -= c; p += w; x >>= w; }
    }
    return p;
}

// ---------------------------------------------------------------- batch lookup
// Batch of flat frontier position i: the b with off[b] <= i < off[b+1].
__device__ __forceinline__ uint32_t batch_of(const int64_t *__restrict__ off, uint32_t n_batches, int64_t i)
{
    uint32_t lo = 0, hi = n_batches;          // invariant: off[lo] <= i < off[hi]
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (off[mid] <= i) lo = mid; else hi = mid;
    }
    return lo;
}

// What a wave's lanes have written to LDS before is what they read behind it, and what they have read before is not yet
// overwritten: for memory that one wave has to itself, where no barrier of the workgroup stands between.  The hardware takes a
// wave's LDS operations in order; the fence keeps the compiler to it and costs no instruction.
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------- reached-ID maps
// Every sampled ID is marked in the batch's `reached` bitmap; which of the reached IDs are new to the batch is decided
// afterwards, group by group, against the batch's `seen` bitmap.  Beside the map there is one flag byte per 256 IDs: the
// frontier passes read the flags and touch only the flagged groups, which on a graph of 10^8 nodes is a few per cent of
// the map.  Where a hop's samples are many and dense in the bitmaps, a pass over them puts the bitmaps together in LDS piece
// by piece (mark_pass_kernel) and the sampling kernels mark nothing; elsewhere they mark each ID as they write it, by an
// atomic OR without return value which the wave does not wait for.
constexpr int MARK_NONE = 0, MARK_BITS = 1;      // what a kernel does with a sampled ID (a template argument)
// On graphs of 10^8 nodes a batch touches a few per cent of its groups, so the frontier passes read a group's words
// of `reached` and of `seen` from two unrelated places each time.  Paired, both lie in one 64-byte record: word w of
// a map that would hold both arrays apart is word paired_word(w) of the records (`seen`: eight words further on).
// Where maps are paired the sampling kernels always mark.
struct ReachedMaps {
    uint32_t *words;              // [n_batches * words_per_batch]; paired: 64-byte records, the group's words of `reached` in front
    uint8_t *flags;               // [n_batches * words_per_batch / 8]
    uint64_t words_per_batch;     // a multiple of 8
    bool paired;
};
struct ReachedOfBatch {
    uint32_t *words;
    uint8_t *flags;
    uint32_t paired;
};
__host__ __device__ __forceinline__ uint64_t paired_word(uint64_t w) { return ((w >> 3) << 4) | (w & 7); }
template <int MARK>
__device__ __forceinline__ ReachedOfBatch reached_of(const ReachedMaps &m, uint32_t batch)
{
    if (MARK == MARK_NONE) return ReachedOfBatch{nullptr, nullptr, 0};
    const uint32_t paired = m.paired ? 1u : 0u;
    return ReachedOfBatch{m.words + (uint64_t)batch * (m.words_per_batch << paired), m.flags + (uint64_t)batch * (m.words_per_batch >> 3), paired};
}
template <int MARK>
__device__ __forceinline__ void mark_reached(const ReachedOfBatch &r, uint32_t u)
{
    if (MARK == MARK_NONE) return;
    const uint32_t w = u >> 5;
    (void)__hip_atomic_fetch_or(r.words + (r.paired ? (((w >> 3) << 4) | (w & 7)) : w), 1u << (u & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    r.flags[u >> 8] = 1;
}

}  // namespace rg
