// Wavefront- and workgroup-level building blocks for gfx950 (64-wide wavefronts).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace mqg {

__device__ __forceinline__ int lane_id() { return static_cast<int>(threadIdx.x) & 63; }

__device__ __forceinline__ uint64_t lanes_below(int lane) { return (uint64_t(1) << lane) - 1; }

__device__ __forceinline__ uint64_t ballot64(bool p) { return __ballot(p); }

__device__ __forceinline__ int popc64(uint64_t m) { return __popcll(m); }

// base and how many lanes of m come before this one
__device__ __forceinline__ int rank_below(uint64_t m, int base = 0) {
    return static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                                      __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), static_cast<uint32_t>(base))));
}

// Value of v in lane `l`; l must be the same in every lane.
__device__ __forceinline__ uint32_t readlane32(uint32_t v, int l) {
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), l));
}
__device__ __forceinline__ uint64_t readlane64(uint64_t v, int l) {
    uint32_t lo = readlane32(static_cast<uint32_t>(v), l);
    uint32_t hi = readlane32(static_cast<uint32_t>(v >> 32), l);
    return (uint64_t(hi) << 32) | lo;
}

// Orders LDS traffic of one wavefront: writes before, reads after.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A bound that exactly k of the wavefront's words lie below, 0 if there is none to be found.  The words are uniform
// 31-bit values, `gap` apart on average, or kNoWord, which never lies below.  The first bound is where k words are
// expected, the next ones are moved by as many gaps as words were too many or too few, the gap a quarter smaller each
// time: four bounds on average, of one comparison per chunk each, where a radix select took eight bits and twice the scalar
// work per bit.  One search in twenty has not ended after ten; it goes on by halves.
constexpr uint32_t kNoWord = 0x7FFFFFFFu;
template <int NCH>
__device__ __forceinline__ uint32_t word_bound(const uint32_t (&w)[NCH], int k, uint32_t gap) {
    auto below = [&](uint32_t t) {
        int n = 0;
#pragma unroll
        for (int c = 0; c < NCH; ++c) n += popc64(ballot64(w[c] < t));
        return n;
    };
    uint32_t t = gap / 2 + static_cast<uint32_t>(k) * gap;
    for (int tries = 0; tries < 10; ++tries) {
        const int more = k - below(t);
        if (more == 0) return t <= kNoWord ? t : below(kNoWord) == k ? kNoWord : 0;       // (past the end all lanes lie below)
        t += static_cast<uint32_t>(more) * gap;
        gap -= gap >> 2;
    }
    uint32_t lo = 0, hi = kNoWord;                         // fewer than k lie below lo
    if (below(hi) < k) return 0;
    while (hi - lo > 0) {
        t = lo + (hi - lo) / 2;
        const int n = below(t);
        if (n == k) return t;
        if (n < k) lo = t + 1;
        else hi = t;
    }
    return below(hi) == k ? hi : 0;
}

// Inclusive prefix sum over the 64 lanes of a wavefront.
__device__ __forceinline__ int wave_incl_scan(int v) {
    const int lane = lane_id();
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        int t = __shfl_up(v, off, 64);
        if (lane >= off) v += t;
    }
    return v;
}

__device__ __forceinline__ int wave_sum(int v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Exclusive prefix sum over a workgroup of NWAVES*64 threads; *total gets the workgroup sum.
// `lds` needs NWAVES ints.  Every thread of the workgroup must call it.
template <int NWAVES>
__device__ __forceinline__ int block_excl_scan(int v, int *total, int *lds) {
    const int lane = lane_id();
    const int wave = static_cast<int>(threadIdx.x) >> 6;
    int incl = wave_incl_scan(v);
    __syncthreads();                       // lds may still be read from a previous call
    if (lane == 63) lds[wave] = incl;
    __syncthreads();
    int base = 0, sum = 0;
#pragma unroll
    for (int w = 0; w < NWAVES; ++w) {
        int t = lds[w];
        if (w < wave) base += t;
        sum += t;
    }
    *total = sum;
    return base + incl - v;
}

// Sum of tile_sums[0 .. tile): what a tile's own workgroup adds up instead of a separate scan
// launch when the tiles are few (kSelfPrefixTiles at most, i.e. at most 32 loads per thread).
// Every thread of the workgroup (256 threads) must call it; `lds` needs 4 ints.
constexpr int kSelfPrefixTiles = 8192;
constexpr int kSelfPrefixBlock = 256, kSelfPrefixWaves = kSelfPrefixBlock / 64;
__device__ __forceinline__ int tiles_before(const int32_t *__restrict__ tile_sums, int *lds, int tile) {
    int part = 0;
    for (int t = threadIdx.x; t < tile; t += kSelfPrefixBlock) part += tile_sums[t];
    part = wave_sum(part);
    __syncthreads();                                       // lds may still be read from an earlier use
    if (lane_id() == 0) lds[threadIdx.x >> 6] = part;
    __syncthreads();
    int sum = 0;
#pragma unroll
    for (int k = 0; k < kSelfPrefixWaves; ++k) sum += lds[k];
    return sum;
}
__device__ __forceinline__ int tiles_before(const int32_t *__restrict__ tile_sums, int *lds) {
    return tiles_before(tile_sums, lds, static_cast<int>(blockIdx.x));
}

// Number of the entries of the ascending list v[0..n) that are below x (STRICT) or not above it, found by a
// whole wavefront: 64 probes per step instead of one, so that a million entries take four dependent loads.
template <bool STRICT, typename V>
__device__ __forceinline__ int64_t wave_count_below(const V *__restrict__ v, int64_t n, int64_t x) {
    int64_t lo = 0, hi = n;                                // the answer lies in [lo, hi]
    while (lo < hi) {
        const int64_t step = (hi - lo + kWave - 1) / kWave;
        const int64_t i = lo + (lane_id() + 1) * step - 1;
        const bool below = i < hi && (STRICT ? static_cast<int64_t>(v[i]) < x : static_cast<int64_t>(v[i]) <= x);
        const int64_t c = popc64(ballot64(below));         // v ascends: the first c probes
        const int64_t next = lo + (c + 1) * step - 1;      // the first probe that is not
        lo += c * step;
        hi = next < hi ? next : hi;
    }
    return lo;
}

// SplitMix64 finaliser (Steele, Lea, Flood 2014): the mixing function of the sampling keys.
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z ^= z >> 30;
    z *= 0xBF58476D1CE4E5B9ULL;
    z ^= z >> 27;
    z *= 0x94D049BB133111EBULL;
    z ^= z >> 31;
    return z;
}

// key(j) = mix64(hv ^ j) for the slots j of one row, with everything that depends only on the row
// hoisted out: j < 2^31 touches only the low word of hv ^ j, so the high word after the first
// xor-shift and its share of the first multiply are per-row constants.  Written on 32-bit halves
// (funnel shifts are one v_alignbit each): 5 multiplies per key instead of 6.
struct RowKeys {
    static constexpr uint32_t kC1Lo = 0x1CE4E5B9u, kC1Hi = 0xBF58476Du;
    static constexpr uint32_t kC2Lo = 0x133111EBu, kC2Hi = 0x94D049BBu;
    uint32_t lo, hi_shl2, a_hi, c1_term;
    __device__ __forceinline__ explicit RowKeys(uint64_t hv) {
        const uint32_t hi = static_cast<uint32_t>(hv >> 32);
        lo = static_cast<uint32_t>(hv);
        hi_shl2 = hi << 2;
        a_hi = hi ^ (hi >> 30);
        c1_term = a_hi * kC1Lo;
    }
    __device__ __forceinline__ uint64_t operator()(int j) const {
        const uint32_t lo0 = lo ^ static_cast<uint32_t>(j);
        const uint32_t a_lo = lo0 ^ (hi_shl2 | (lo0 >> 30));                       // z ^= z >> 30
        const uint64_t p = static_cast<uint64_t>(a_lo) * kC1Lo;                      // z *= C1
        const uint32_t b_lo = static_cast<uint32_t>(p);
        const uint32_t b_hi = static_cast<uint32_t>(p >> 32) + a_lo * kC1Hi + c1_term;
        const uint32_t c_lo = b_lo ^ __builtin_amdgcn_alignbit(b_hi, b_lo, 27);      // z ^= z >> 27
        const uint32_t c_hi = b_hi ^ (b_hi >> 27);
        const uint64_t q = static_cast<uint64_t>(c_lo) * kC2Lo;                      // z *= C2
        const uint32_t d_lo = static_cast<uint32_t>(q);
        const uint32_t d_hi = static_cast<uint32_t>(q >> 32) + c_lo * kC2Hi + c_hi * kC2Lo;
        const uint32_t e_lo = d_lo ^ __builtin_amdgcn_alignbit(d_hi, d_lo, 31);      // z ^= z >> 31
        const uint32_t e_hi = d_hi ^ (d_hi >> 31);
        return (static_cast<uint64_t>(e_hi) << 32) | e_lo;
    }
};

// The same keys for a wavefront that walks a row 64 slots at a time, slot = base + lane with base a
// multiple of 64.  Up to the first multiplication a lane's word differs from the wavefront's only in its
// six low bits, so the product splits into a part that depends on the row and base alone (scalar unit) and
// a part that depends on the row and the lane alone (once per row): what is left of the first half of the
// mixer per key is one 64-bit addition, and three multiplications per key remain of five.  One object
// serves the slots of one range of 2^30 (the slot's two top bits reach the low bits).  Where a wavefront takes
// CHUNKS times 64 slots from a multiple of that on, those share the row's part.
constexpr uint64_t kC1 = (uint64_t(RowKeys::kC1Hi) << 32) | RowKeys::kC1Lo;
__device__ __forceinline__ uint32_t key_low(uint64_t hv, uint32_t range = 0) {           // low word after the first xor-shift, for slot 0 of the range
    const uint32_t lo = static_cast<uint32_t>(hv);
    return lo ^ static_cast<uint32_t>(((hv >> 32 << 32) | (lo ^ range)) >> 30);
}
__device__ __forceinline__ uint32_t key_hi_term(uint64_t hv) {                            // the high word's share of the first product
    const uint32_t hi = static_cast<uint32_t>(hv >> 32);
    return (hi ^ (hi >> 30)) * RowKeys::kC1Lo;
}
// The key's upper word, from the first product, before the final xor-shift, which would change its bit 0 only
__device__ __forceinline__ uint32_t key_upper(uint64_t b) {
    const uint32_t b_lo = static_cast<uint32_t>(b), b_hi = static_cast<uint32_t>(b >> 32);
    const uint32_t c_lo = b_lo ^ __builtin_amdgcn_alignbit(b_hi, b_lo, 27);
    const uint32_t c_hi = b_hi ^ (b_hi >> 27);
    return __umulhi(c_lo, RowKeys::kC2Lo) + c_lo * RowKeys::kC2Hi + c_hi * RowKeys::kC2Lo;
}
// The key itself.
__device__ __forceinline__ uint64_t key_whole(uint64_t b) {
    const uint32_t b_lo = static_cast<uint32_t>(b), b_hi = static_cast<uint32_t>(b >> 32);
    const uint32_t c_lo = b_lo ^ __builtin_amdgcn_alignbit(b_hi, b_lo, 27);
    const uint32_t c_hi = b_hi ^ (b_hi >> 27);
    const uint64_t q = static_cast<uint64_t>(c_lo) * RowKeys::kC2Lo + (static_cast<uint64_t>(c_lo * RowKeys::kC2Hi + c_hi * RowKeys::kC2Lo) << 32);
    return q ^ (q >> 31);
}
template <int CHUNKS>
struct WaveKeys {
    static constexpr uint32_t kMask = CHUNKS * kWave - 1;
    uint32_t low, hi_term;        // the same in all lanes
    uint64_t lane_prod[CHUNKS];   // (its low bits, with the slot's) * C1
    __device__ __forceinline__ WaveKeys(uint32_t low_word, uint32_t hi_share) : low(low_word), hi_term(hi_share) {
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) lane_prod[c] = static_cast<uint64_t>((low ^ static_cast<uint32_t>(c * kWave + lane_id())) & kMask) * kC1;
    }
    // the row's part for the CHUNKS * 64 slots from base on
    __device__ __forceinline__ uint64_t row_part(uint32_t base) const {
        const uint32_t rest = (low ^ base) & ~kMask;
        uint64_t p = uint64_t(rest) * RowKeys::kC1Lo + (uint64_t(rest * RowKeys::kC1Hi + hi_term) << 32);
        // (this keeps it in scalar registers: the compiler would fold the product into the addition as a vector multiply-add)
        asm("" : "+s"(p));
        return p;
    }
    __device__ __forceinline__ uint32_t upper(uint64_t part, int c = 0) const { return key_upper(part + lane_prod[c]); }
    __device__ __forceinline__ uint64_t whole(uint64_t part, int c = 0) const { return key_whole(part + lane_prod[c]); }
};

// The smallest of the wavefront's words, the same in all lanes: six steps of one instruction on the lanes' own registers (an exchange
// through LDS takes three and its latency).
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
    auto step = [&](auto ctrl, auto rows) {
        const uint32_t o = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(-1, static_cast<int>(v), decltype(ctrl)::value, decltype(rows)::value, 0xF, false));
        v = o < v ? o : v;
    };
    using std::integral_constant;
    step(integral_constant<int, 0x111>(), integral_constant<int, 0xF>());      // from the lane 1, 2, 4, 8 below in a row of 16
    step(integral_constant<int, 0x112>(), integral_constant<int, 0xF>());
    step(integral_constant<int, 0x114>(), integral_constant<int, 0xF>());
    step(integral_constant<int, 0x118>(), integral_constant<int, 0xF>());
    step(integral_constant<int, 0x142>(), integral_constant<int, 0xA>());      // from the last lane of the row before
    step(integral_constant<int, 0x143>(), integral_constant<int, 0xC>());      // from lane 31
    return readlane32(v, kWave - 1);
}

// An exponential variate from 64 random bits in integer arithmetic: -log2(r / 2^64) with 32
// fractional bits (r = 0 counts as 1).  With m = r << lz in [2^63, 2^64) the integer part is
// lz + 1; the fraction of log2(m / 2^63) comes bit by bit from repeated squaring (a square that
// reaches 2 emits a one and is halved), squares truncated to 64 bits.  The step is written without
// a data-dependent branch (selects) so that the loop compiles to straight
// vector code: with a branch the compiler wraps the low product in an exec-mask save/restore, and
// one build of a kernel around that form returned wrong tickets, different from run to run, in
// every workgroup but the first of a compute unit.
// The square of m = hi 2^32 + lo takes three multiplications: with t = hi lo + floor(lo^2 / 2^33) its upper word is
// hi^2 + floor(t / 2^31), and bit 63 of its lower one is bit 30 of t.
__device__ __forceinline__ uint64_t exp_ticket64(uint64_t r) {
    if (r == 0) r = 1;
    const int lz = __clzll(static_cast<long long>(r));
    const uint64_t m = r << lz;
    uint32_t hi = static_cast<uint32_t>(m >> 32), lo = static_cast<uint32_t>(m), frac = 0;
#pragma unroll 8
    for (int b = 0; b < 32; ++b) {
        const uint64_t t = static_cast<uint64_t>(hi) * lo + (__umulhi(lo, lo) >> 1);
        const uint64_t top = static_cast<uint64_t>(hi) * hi + (t >> 31);
        const uint32_t th = static_cast<uint32_t>(top >> 32), tl = static_cast<uint32_t>(top);
        const uint32_t below = static_cast<uint32_t>(t) >> 30 & 1u;
        const bool one = static_cast<int32_t>(th) < 0;     // the square reached 2
        frac = frac << 1 | (one ? 1u : 0u);
        hi = one ? th : __builtin_amdgcn_alignbit(th, tl, 31);        // not yet at 2: renormalise by one bit
        lo = one ? tl : tl << 1 | below;
    }
    return (static_cast<uint64_t>(lz + 1) << 32) - frac;
}

}  // namespace mqg
