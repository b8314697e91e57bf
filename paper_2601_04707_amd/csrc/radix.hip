// Stable least-significant-digit radix sort of (32-bit key, 32-bit payload) pairs and the exclusive
// scan it needs.  Used to rank nodes by degree for the cache, to transpose an adjacency and to order a
// block's edges by source node for the backward aggregation.  The element count may live on the
// device (n_dev): grids are sized by the host-side bound n_cap and every kernel clamps.  Keys of b
// significant bits take ceil(b / 11) passes (ceil(b / 9) for more than 2 M keys) with digits of
// ceil(b / passes) bits (8 at least): the 18-bit source positions of a 230 k-node block sort in two
// 9-bit passes.
//   k_radix_hist     per-workgroup digit histogram, laid out [digit][workgroup]
//   k_radix_scan     exclusive scan of every digit's counts over the workgroups, and their totals
//   k_radix_scatter  stable scatter: ballot match and running counts per wavefront, the tile sorted by
//                    digit in LDS, written from there run by run (each workgroup scans the digits'
//                    totals itself)
// Sorts of up to 32 tiles (65,536 keys: the inner blocks of a mini-batch) need no scan launch:
// the histogram table is laid out [tile][digit] and every workgroup of the scatter adds up, per
// digit, the counts of all tiles (for the digit's base) and of the tiles before its own.  (With 138
// tiles the adding-up made the scatter 25 us instead of 8: more than the two scan launches it
// saved.)  Small inputs are cut into tiles of fewer rounds, so that about 32 workgroups share them.
#include <algorithm>

#include "common.h"
#include "device_utils.h"
#include "radix.h"

namespace mqg {

namespace {

// tile_major: the table is [tile][digit] (for the scatter that adds the counts up itself), otherwise
// [digit][tile] (so that a scan of every row gives every tile its places among the keys of the digit).
// DB = bits per digit.
template <int DB>
__global__ void __launch_bounds__(kBlock)
k_radix_hist(const uint32_t *__restrict__ keys, int64_t n, const int64_t *__restrict__ n_dev, int shift,
             int32_t *__restrict__ hist, int nblocks, int items, int tile_major) {
    constexpr int D = 1 << DB, PER = D / kBlock;
    __shared__ int h[D];
    if (n_dev && *n_dev < n) n = *n_dev;
    const int me = tile_major ? static_cast<int>(blockIdx.x) : xcd_tile(n_dev ? live_tiles(n, kBlock * items) : nblocks);
    if (me >= nblocks) return;
#pragma unroll
    for (int q = 0; q < PER; ++q) h[q * kBlock + threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = int64_t(me) * kBlock * items;
    for (int r0 = 0; r0 < items; r0 += 8) {                  // eight keys on their way before the first is counted
        uint32_t key[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int64_t i = base + (r0 + r) * kBlock + threadIdx.x;
            key[r] = r0 + r < items && i < n ? keys[i] : 0;
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int64_t i = base + (r0 + r) * kBlock + threadIdx.x;
            if (r0 + r < items && i < n) atomicAdd(&h[(key[r] >> shift) & (D - 1)], 1);
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int d = q * kBlock + threadIdx.x;
        if (tile_major) hist[int64_t(me) * D + d] = h[d];
        else hist[int64_t(d) * nblocks + me] = h[d];
    }
}

// Exclusive scan, in place, of the counts of one digit (a workgroup's row of the [digit][tile] table), and
// the digit's total.  A launch of 256 or more short workgroups: what it costs is the launch and one trip to
// memory, the next counts being on their way while these are added up.  (A scan of the whole table took two
// launches, three on large ones: 4.3 M keys by 8 bits 12.9 -> 7.6 us, 100 M 63 -> 48, 1 M 13.3 -> 7.5.)
constexpr int kScanRounds = 8;
__global__ void __launch_bounds__(kBlock)
k_radix_scan(int32_t *__restrict__ hist, int stride, int32_t *__restrict__ totals, int64_t n, const int64_t *__restrict__ n_dev, int tile) {
    if (n_dev && *n_dev < n) n = *n_dev;
    const int nblocks = n_dev ? live_tiles(n, tile) : stride;
    __shared__ int lds[2][kWavesPerBlock];
    int32_t *row = hist + int64_t(blockIdx.x) * stride;
    const int mine = (static_cast<int>(threadIdx.x) >> 6) * (kWave * kScanRounds) + lane_id();
    const int wave = threadIdx.x >> 6;
    int next[kScanRounds];
    auto load = [&](int c) {
#pragma unroll
        for (int r = 0; r < kScanRounds; ++r) next[r] = c + mine + r * kWave < nblocks ? row[c + mine + r * kWave] : 0;
    };
    load(0);
    int carry = 0, side = 0;
    for (int c = 0; c < nblocks; c += kBlock * kScanRounds, side ^= 1) {
        int ex[kScanRounds], sum = 0;
        int v[kScanRounds];
#pragma unroll
        for (int r = 0; r < kScanRounds; ++r) v[r] = next[r];
        load(c + kBlock * kScanRounds);
#pragma unroll
        for (int r = 0; r < kScanRounds; ++r) {
            const int incl = wave_incl_scan(v[r]);
            ex[r] = sum + incl - v[r];
            sum += __shfl(incl, kWave - 1);
        }
        if (lane_id() == 0) lds[side][wave] = sum;
        __syncthreads();                             // the other half of lds is written next: one barrier will do
        int before = carry;
#pragma unroll
        for (int w = 0; w < kWavesPerBlock; ++w) {
            const int t = lds[side][w];
            before += w < wave ? t : 0;
            carry += t;
        }
#pragma unroll
        for (int r = 0; r < kScanRounds; ++r)
            if (c + mine + r * kWave < nblocks) row[c + mine + r * kWave] = before + ex[r];
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

__global__ void __launch_bounds__(kBlock)
k_scan_reduce(const int32_t *__restrict__ in, int64_t n, int32_t *__restrict__ tile_sums) {
    __shared__ int lds[kWavesPerBlock];
    const int64_t base = int64_t(blockIdx.x) * kScanTile + threadIdx.x * 4;
    int c = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (base + q < n) c += in[base + q];
    int s = wave_sum(c);
    if (lane_id() == 0) lds[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) tile_sums[blockIdx.x] = lds[0] + lds[1] + lds[2] + lds[3];
}

// scanned: tile_vals holds the exclusive scan of the tile sums; otherwise the sums themselves, and
// every workgroup adds up the ones before its own
__global__ void __launch_bounds__(kBlock)
k_scan_apply(int32_t *__restrict__ data, int64_t n, const int32_t *__restrict__ tile_vals, int scanned) {
    __shared__ int lds[kWavesPerBlock];
    const int tile_base = scanned ? tile_vals[blockIdx.x] : tiles_before(tile_vals, lds);
    const int64_t base = int64_t(blockIdx.x) * kScanTile + threadIdx.x * 4;
    int v[4];
    int c = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        v[q] = base + q < n ? data[base + q] : 0;
        c += v[q];
    }
    int total;
    int ex = block_excl_scan<kWavesPerBlock>(c, &total, lds) + tile_base;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (base + q < n) data[base + q] = ex;
        ex += v[q];
    }
}

// What a key carries along: vals_in[i], or (vals_in == nullptr, first pass only) its own position i.
struct RadixPayload {
    const int32_t *vals_in;
    __device__ __forceinline__ int32_t get(int64_t i) const { return vals_in ? vals_in[i] : static_cast<int32_t>(i); }
};

// SELF: `offsets` is the [tile][digit] table of counts and the bases are added up here; otherwise it
// is the [digit][tile] table, scanned row by row, and `totals` the number of keys of every digit.
// A wavefront owns `items` consecutive groups of 64 keys of the tile.  All keys and payloads are loaded
// first; a key's rank among the wavefront's keys of its digit comes from ballots and a running count in
// LDS that only this wavefront touches; three barriers later the tile lies sorted by digit in LDS and is
// written from there, every digit's run to consecutive addresses.  (Before: three barriers per 256 keys, a
// load in front of each, single words written; 4.3 M pairs by 8 bits 75 -> 33 us, 2.4 M 45 -> 16 us.  Tiles
// of 4,096 instead of 2,048 keys: the same at 4.3 M, 10.6 instead of 8.5 us at 250 k, too few workgroups.)
template <bool SELF, int DB, int ITEMS>
__global__ void __launch_bounds__(kBlock)
k_radix_scatter(const uint32_t *__restrict__ keys_in, RadixPayload payload, int64_t n,
                const int64_t *__restrict__ n_dev, int shift,
                const int32_t *__restrict__ offsets, const int32_t *__restrict__ totals, int nblocks, int items, uint32_t *__restrict__ keys_out,
                int32_t *__restrict__ vals_out) {
    constexpr int D = 1 << DB, PER = D / kBlock;
    __shared__ int wcnt[kWavesPerBlock][D];          // keys of this digit so far, then those of the wavefronts before
    __shared__ int first[D];                         // first place of the digit in the sorted tile ...
    __shared__ int gbase[D];                         // ... and in the output, less that
    __shared__ uint32_t skeys[kBlock * ITEMS];
    __shared__ int32_t svals[kBlock * ITEMS];
    __shared__ int scan_lds[kWavesPerBlock];
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int wave = tid >> 6;
    if (n_dev && *n_dev < n) n = *n_dev;
    const int me = SELF ? static_cast<int>(blockIdx.x) : xcd_tile(n_dev ? live_tiles(n, kBlock * items) : nblocks);
    if (me >= nblocks) return;
    const int64_t base = int64_t(me) * kBlock * items;
    if (base >= n) return;
    const int tile_n = n - base < kBlock * items ? static_cast<int>(n - base) : kBlock * items;
    const int wave_first = wave * kWave * items;
    uint32_t key[ITEMS];
    int32_t val[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int i = wave_first + r * kWave + lane;
        const bool in = r < items && i < tile_n;
        key[r] = in ? keys_in[base + i] : 0;
        val[r] = in ? payload.get(base + i) : 0;
    }
    int out0[PER];                                   // first output place of the digits tid * PER ... for this tile
    if (!SELF) {
        int all[PER], mine = 0, total;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            out0[q] = offsets[int64_t(tid * PER + q) * nblocks + me];
            all[q] = totals[tid * PER + q];
            mine += all[q];
        }
        int ex = block_excl_scan<kWavesPerBlock>(mine, &total, scan_lds);
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            out0[q] += ex;
            ex += all[q];
        }
    } else {
        // keys with a smaller digit in any tile, plus keys with the same digit in earlier tiles
        int all[PER], before[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) all[q] = before[q] = 0;
#pragma unroll 4
        for (int w = 0; w < nblocks; ++w) {
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const int c = offsets[int64_t(w) * D + tid * PER + q];
                all[q] += c;
                before[q] += w < me ? c : 0;
            }
        }
        int mine = 0;
#pragma unroll
        for (int q = 0; q < PER; ++q) mine += all[q];
        int total;
        int ex = block_excl_scan<kWavesPerBlock>(mine, &total, scan_lds);
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            out0[q] = ex + before[q];
            ex += all[q];
        }
    }
#pragma unroll
    for (int q = 0; q < D / kWave; ++q) wcnt[wave][q * kWave + lane] = 0;
    wave_lds_sync();
    int rank[ITEMS];                                 // among the keys of its digit in this wavefront
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        if (r < items) {                             // uniform
            const bool in = wave_first + r * kWave + lane < tile_n;
            const int digit = (key[r] >> shift) & (D - 1);
            uint64_t peers = ballot64(in);           // lanes that hold the same digit
#pragma unroll
            for (int bit = 0; bit < DB; ++bit) {
                const uint64_t m = ballot64((digit >> bit) & 1);
                peers &= ((digit >> bit) & 1) ? m : ~m;
            }
            const int in_group = popc64(peers & lanes_below(lane));
            const int so_far = wcnt[wave][digit];
            rank[r] = so_far + in_group;
            wave_lds_sync();
            if (in && in_group == 0) wcnt[wave][digit] = so_far + popc64(peers);
            wave_lds_sync();
        }
    }
    __syncthreads();
    int cnt[PER], mine = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        cnt[q] = 0;
#pragma unroll
        for (int w = 0; w < kWavesPerBlock; ++w) {
            const int c = wcnt[w][tid * PER + q];
            wcnt[w][tid * PER + q] = cnt[q];
            cnt[q] += c;
        }
        mine += cnt[q];
    }
    if constexpr (SELF) {
        // small sorts: each key straight to its place, without the second scan and the sorted tile
#pragma unroll
        for (int q = 0; q < PER; ++q) gbase[tid * PER + q] = out0[q];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            if (r < items && wave_first + r * kWave + lane < tile_n) {
                const int digit = (key[r] >> shift) & (D - 1);
                const int o = gbase[digit] + wcnt[wave][digit] + rank[r];
                keys_out[o] = key[r];
                vals_out[o] = val[r];
            }
        }
        return;
    }
    int total;
    int ex = block_excl_scan<kWavesPerBlock>(mine, &total, scan_lds);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        first[tid * PER + q] = ex;
        gbase[tid * PER + q] = out0[q] - ex;
        ex += cnt[q];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        if (r < items && wave_first + r * kWave + lane < tile_n) {
            const int digit = (key[r] >> shift) & (D - 1);
            const int p = first[digit] + wcnt[wave][digit] + rank[r];
            skeys[p] = key[r];
            svals[p] = val[r];
        }
    }
    __syncthreads();
    for (int p = tid; p < tile_n; p += kBlock) {
        const uint32_t k = skeys[p];
        const int64_t o = int64_t(gbase[(k >> shift) & (D - 1)]) + p;
        keys_out[o] = k;
        vals_out[o] = svals[p];
    }
}

}  // namespace

// Digits: as few passes as the widest digit allows, then the digit just wide enough for them (8 bits
// at least).  The widest digit is 11 bits for inputs of up to kRadixWideKeys keys, where a pass is
// mostly its launches, and 9 bits above, where it is mostly its scatter: a tile of 2,048 keys has about
// one of each of 2,048 digits, so its runs are single words.  All launches of a sort, keys spread evenly:
// 11 bits in one pass or in two of 8, 300 k keys 30 and 44 us, 1 M 40 and 50, 2 M 55 and 56, 4.3 M 104 and 79;
// 20 bits in two passes of 10 or in three of 8, 300 k 49 and 67, 2 M 84 and 87, 4.3 M 136 and 118; 22 bits in two
// of 11 or in three of 8, 300 k 59 and 67, 1 M 81 and 75, 2 M 112 and 87, 4.3 M 207 and 118.
static int max_digit_bits(int64_t n_cap) { return n_cap <= kRadixWideKeys ? kRadixMaxDigitBits : 9; }
int radix_passes(int bits, int64_t n_cap) { return bits <= 0 ? 0 : (bits + max_digit_bits(n_cap) - 1) / max_digit_bits(n_cap); }
int radix_digit_bits(int bits, int64_t n_cap) {
    const int p = radix_passes(bits, n_cap);
    return p == 0 ? 8 : std::max(8, (bits + p - 1) / p);
}
int radix_key_bits(uint64_t max_key) {
    int bits = 0;
    while (bits < 32 && (max_key >> bits) != 0) ++bits;
    return bits;
}
int64_t radix_blocks(int64_t n_cap) { return std::max<int64_t>(1, ceil_div(n_cap, kRadixTile)); }
// (small inputs have up to kRadixSelfBlocks tiles whatever their size)
int64_t radix_hist_len(int64_t n_cap, int bits) {
    return (int64_t(1) << radix_digit_bits(bits, n_cap)) * std::max<int64_t>(radix_blocks(n_cap), kRadixSelfBlocks);
}
// The largest table any sort of at most n_cap keys of at most 32 bits needs: the widest digit on the
// largest input that still takes it, or the 9-bit digit on all of n_cap.
int64_t radix_hist_len_max(int64_t n_cap) {
    const int64_t wide = (int64_t(1) << kRadixMaxDigitBits) * std::max<int64_t>(radix_blocks(std::min(n_cap, kRadixWideKeys)), kRadixSelfBlocks);
    const int64_t narrow = (int64_t(1) << 9) * radix_blocks(n_cap);
    return std::max(wide, narrow);
}

// exclusive scan of data[0..n) in place
int device_scan(mqg_ctx *ctx, int32_t *data, int64_t n, int32_t *tile_sums, hipStream_t s) {
    const int tiles = static_cast<int>(std::max<int64_t>(1, ceil_div(n, kScanTile)));
    const int scanned = tiles > kSelfPrefixTiles ? 1 : 0;     // few tiles: k_scan_apply adds the sums up itself
    if (tiles > 1) MQG_LAUNCH(ctx, "k_scan_reduce", s, (k_scan_reduce<<<tiles, kBlock, 0, s>>>(data, n, tile_sums)));
    if (scanned) {
        int rc = launch_scan_tiles(ctx, tile_sums, tiles, nullptr, nullptr, nullptr, s, "k_scan_tiles(radix)");
        if (rc != MQG_OK) return rc;
    }
    MQG_LAUNCH(ctx, "k_scan_apply", s, (k_scan_apply<<<tiles, kBlock, 0, s>>>(data, n, tile_sums, scanned)));
    return MQG_OK;
}

// rounds per tile: 8, fewer for small inputs (a round is a serial step of a workgroup; 32 tiles of
// one round sort 8 k keys faster than 4 tiles of eight)
int radix_items(int64_t n_cap) {
    return static_cast<int>(std::min<int64_t>(kRadixItems, std::max<int64_t>(1, ceil_div(n_cap, int64_t(kBlock) * kRadixSelfBlocks))));
}

int launch_radix_scan(mqg_ctx *ctx, int32_t *hist, int nblocks, int digits, int32_t *totals, int64_t n_cap, const int64_t *n_dev, int tile, hipStream_t s) {
    MQG_LAUNCH(ctx, "k_radix_scan", s, (k_radix_scan<<<digits, kBlock, 0, s>>>(hist, nblocks, totals, n_cap, n_dev, tile)));
    return MQG_OK;
}

template <int DB>
static int radix_sort_pairs_t(mqg_ctx *ctx, const uint32_t *keys_in, RadixPayload first, const RadixBufs &b, int64_t n_cap,
                              const int64_t *n_dev, int bits, hipStream_t s, int *result) {
    constexpr int D = 1 << DB;
    const int items = radix_items(n_cap);
    const int nblocks = static_cast<int>(std::max<int64_t>(1, ceil_div(n_cap, int64_t(kBlock) * items)));
    const bool self = nblocks <= kRadixSelfBlocks;
    const uint32_t *kin = keys_in;
    RadixPayload pay = first;
    int out = 0;
    *result = -1;
    const int passes = radix_passes(bits, n_cap);
    for (int p = 0; p < passes; ++p) {
        const int shift = p * DB;
        MQG_LAUNCH(ctx, "k_radix_hist", s, (k_radix_hist<DB><<<self ? nblocks : xcd_grid(nblocks), kBlock, 0, s>>>(kin, n_cap, n_dev, shift, b.hist, nblocks, items, self ? 1 : 0)));
        if (self) {
            MQG_LAUNCH(ctx, "k_radix_scatter", s,
                       (k_radix_scatter<true, DB, kRadixItems><<<nblocks, kBlock, 0, s>>>(kin, pay, n_cap, n_dev, shift, b.hist, b.totals, nblocks, items, b.keys[out], b.vals[out])));
        } else {
            int rc = launch_radix_scan(ctx, b.hist, nblocks, D, b.totals, n_cap, n_dev, kBlock * items, s);
            if (rc != MQG_OK) return rc;
            MQG_LAUNCH(ctx, "k_radix_scatter", s,
                       (k_radix_scatter<false, DB, kRadixItems><<<xcd_grid(nblocks), kBlock, 0, s>>>(kin, pay, n_cap, n_dev, shift, b.hist, b.totals, nblocks, items, b.keys[out], b.vals[out])));
        }
        kin = b.keys[out];
        pay = RadixPayload{b.vals[out]};
        *result = out;
        out ^= 1;
    }
    return MQG_OK;
}

int radix_sort_pairs(mqg_ctx *ctx, const uint32_t *keys_in, const int32_t *vals_in, const RadixBufs &b,
                     int64_t n_cap, const int64_t *n_dev, int bits, hipStream_t s, int *result) {
    const RadixPayload first{vals_in};
    switch (radix_digit_bits(bits, n_cap)) {
        case 8: return radix_sort_pairs_t<8>(ctx, keys_in, first, b, n_cap, n_dev, bits, s, result);
        case 9: return radix_sort_pairs_t<9>(ctx, keys_in, first, b, n_cap, n_dev, bits, s, result);
        case 10: return radix_sort_pairs_t<10>(ctx, keys_in, first, b, n_cap, n_dev, bits, s, result);
        default: return radix_sort_pairs_t<11>(ctx, keys_in, first, b, n_cap, n_dev, bits, s, result);
    }
}

}  // namespace mqg
