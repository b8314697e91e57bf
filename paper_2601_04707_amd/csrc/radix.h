// Radix sort of (key, payload) pairs and the device-wide exclusive scan (internal).
#pragma once

#include "common.h"

namespace mqg {

// Tiles that hold any of n keys.
__device__ __forceinline__ int live_tiles(int64_t n, int tile) { return static_cast<int>((n + tile - 1) / tile); }

// An XCD's workgroups (every eighth) take neighbouring tiles: their runs of one digit, and their counts of it,
// share cache lines, and the scatter finds in its L2 the keys that the histogram read (histograms of the seven
// passes of a 4.3 M-edge backward 77 -> 71 us, of a degree sort of 1 M nodes 23 -> 19).  The live tiles are dealt, not the
// capacity's: with half of it in use four of the XCDs went without work (a pass of 4.3 M keys in room for 8.1 M, scatter 52 -> 36 us).
// (Where the host knows the count, all tiles are live, and no workgroup divides for them.)  A result of kNoTile: no tile for this workgroup.  The grid is the number of tiles rounded up to a multiple of eight.
constexpr int kNoTile = 0x7FFFFFFF;
__device__ __forceinline__ int xcd_tile(int live) {
    const int share = (live + 7) >> 3, k = static_cast<int>(blockIdx.x >> 3);
    const int me = static_cast<int>(blockIdx.x & 7) * share + k;
    return k < share && me < live ? me : kNoTile;
}
__host__ inline int xcd_grid(int nblocks) { return (nblocks + 7) & ~7; }

constexpr int kRadixItems = 8;                      // rounds per tile
constexpr int kRadixTile = kBlock * kRadixItems;     // keys per workgroup
constexpr int kScanTile = 1024;                      // elements per workgroup in the generic scan
constexpr int kRadixSelfBlocks = 32;                 // up to this many tiles the scatter adds the tile counts up itself
constexpr int kRadixMaxDigitBits = 11;
constexpr int kRadixTotals = 1 << kRadixMaxDigitBits;  // entries of RadixBufs::totals

constexpr int64_t kRadixWideKeys = int64_t(2) << 20;  // inputs above this many keys use digits of at most 9 bits
// n_cap keys of `bits` significant bits are sorted in radix_passes passes of radix_digit_bits bits.
int radix_passes(int bits, int64_t n_cap);
int radix_digit_bits(int bits, int64_t n_cap);
int radix_key_bits(uint64_t max_key);                // significant bits of the largest key (at most 32)
int64_t radix_blocks(int64_t n_cap);
int64_t radix_hist_len(int64_t n_cap, int bits);     // table of one sort of exactly this shape
int64_t radix_hist_len_max(int64_t n_cap);            // enough for every sort of at most n_cap keys, any key width

int radix_items(int64_t n_cap);                       // rounds per tile
// exclusive scan of every row of the [digits][nblocks] table, in place, up to the last tile of min(n_cap, *n_dev) keys, and the
// rows' totals
int launch_radix_scan(mqg_ctx *ctx, int32_t *hist, int nblocks, int digits, int32_t *totals, int64_t n_cap, const int64_t *n_dev, int tile,
                      hipStream_t s);

// exclusive scan of data[0..n) in place; tile_sums needs ceil(n / kScanTile) + 1 ints
int device_scan(mqg_ctx *ctx, int32_t *data, int64_t n, int32_t *tile_sums, hipStream_t s);

// Sorts the first min(n_cap, *n_dev) pairs by the low `bits` bits of the key, stably.  The input
// arrays are only read; *result tells which of b.keys/b.vals holds the output (-1: bits == 0,
// nothing was moved and the input is the output).  b.hist needs radix_hist_len(n_cap, bits) entries,
// b.totals kRadixTotals.
// vals_in == nullptr: the payload of key i is i itself, made in the first pass (bits > 0 then).
int radix_sort_pairs(mqg_ctx *ctx, const uint32_t *keys_in, const int32_t *vals_in, const RadixBufs &b,
                     int64_t n_cap, const int64_t *n_dev, int bits, hipStream_t s, int *result);

}  // namespace mqg
