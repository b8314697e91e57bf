// The edges of a block ordered by source, stably, for the backward aggregation: the transposed operator's row offsets
// (col_ptr), and per edge its destination row and, weighted, its weight.
//
//   k_order_hist     digit histogram of every tile of edges, digit = the leading bits of the source position
//   (k_radix_scan    exclusive scan of every digit's counts over the tiles, and their totals; up to kRadixSelfBlocks
//                    tiles the scatter adds the counts up itself)
//   k_order_scatter  stable partition by that digit; an edge's destination row is found here, by its wavefront, among
//                    the offsets of 64 consecutive rows
//   k_order_buckets  a workgroup per range of up to 2,048 sources: counts its edges per source, which gives col_ptr,
//                    and writes them to their places in order; crowded buckets by several workgroups, the most crowded
//                    ones in a second launch
//
// One partition and one pass over each bucket in place of two or three passes of a radix sort (a histogram, a scan and a
// scatter each), a launch for the destination rows, a bisection for col_ptr and, weighted, a gather of the
// weights.  All launches: 4.0 M edges of 279 k rows into 1.27 M sources 194 -> 107 us; 434 k edges into
// 279 k 50 -> 38; 253 k weighted ones into 108 k 47 -> 36.
// How many leading bits there are depends on the number of sources, which only the device knows.
#include <algorithm>

#include "common.h"
#include "device_utils.h"
#include "radix.h"

namespace mqg {

namespace {

constexpr int kOrderBits = 9;                        // of the partition's digit
constexpr int kOrderDigits = 1 << kOrderBits;
// Workgroups of 512 cut more than kLargeOrder edges into tiles of 4,096: half the counts to scan and runs twice as long.  Fewer
// edges take tiles of 2,048, more workgroups (histogram, scan and partition of 245 k edges 22.0 and 23.7 us, of 4.3 M 75 and 72).
constexpr int kOrderThreads = 512;
constexpr int64_t kLargeOrder = int64_t(1) << 20;
constexpr int kSubBits = 11;                         // of a source within its workgroup's range
constexpr int kSub = 1 << kSubBits;
constexpr int kBucketThreads = 512;
constexpr int kBucketWaves = kBucketThreads / kWave;
constexpr int kSmallChunk = 4096;                    // edges of a bucket placed by one workgroup, see order_chunk
constexpr int kRecountMost = 1 << 17;                // edges of a bucket up to which a chunk's workgroup counts the other chunks too
constexpr int kMostRanges = 4;                       // of a bucket
constexpr int kStageWords = 8192;                    // of a range's edges, for a coalesced store
constexpr int kBucketGrid = 1024;

// bits of a source position below the partition's digit
__host__ __device__ inline int order_shift(int64_t num_src) {
    int bits = 0;
    while (bits < 32 && ((num_src > 0 ? num_src - 1 : 0) >> bits) != 0) ++bits;
    return bits > kOrderBits ? bits - kOrderBits : 0;
}
// words of two counts in a chunk's row of the table; at least two, which a thread reads at a time
__host__ __device__ inline int order_table_stride(int shift) { return shift > 2 ? 1 << (shift - 1) : 2; }
// Edges of a chunk (fit 16 bits, multiples of 64): few edges take small ones, so that a crowded bucket gets several workgroups (60 k edges
// of which half are in one bucket 51 us in chunks of 16,384, 22 so), at least as many as a bucket has sources, so that the table has
// room.  Many fill the chip with whole buckets (16 M evenly spread edges 287 us in chunks of 16,384, 250 so).
inline int order_chunk(int64_t nnz_cap, int shift) {
    if (nnz_cap <= kLargeOrder) return shift < 12 ? kSmallChunk : 1 << shift;
    return nnz_cap <= 8 * kLargeOrder ? 16384 : 32768;
}

template <int THREADS>
__global__ void __launch_bounds__(THREADS)
k_order_hist(const int32_t *__restrict__ indices, const int64_t *__restrict__ sizes, int64_t cap, int32_t *__restrict__ hist, int nblocks, int items,
             int tile_major, int32_t *__restrict__ totals) {
    __shared__ int h[kOrderDigits];
    const int64_t n = sizes[2] < cap ? sizes[2] : cap;
    const int me = tile_major ? static_cast<int>(blockIdx.x) : xcd_tile(live_tiles(n, THREADS * items));
    if (blockIdx.x == 0 && threadIdx.x == 0) totals[kOrderDigits] = 0;     // no bucket is counted yet, see k_order_buckets
    if (me >= nblocks) return;
    const int shift = order_shift(sizes[1]);
#pragma unroll
    for (int q = 0; q < kOrderDigits / THREADS; ++q) h[q * THREADS + threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = int64_t(me) * THREADS * items;
    uint32_t key[kRadixItems];
#pragma unroll
    for (int r = 0; r < kRadixItems; ++r) {
        const int64_t i = base + r * THREADS + threadIdx.x;
        key[r] = r < items && i < n ? static_cast<uint32_t>(indices[i]) : 0;
    }
#pragma unroll
    for (int r = 0; r < kRadixItems; ++r) {
        const int64_t i = base + r * THREADS + threadIdx.x;
        if (r < items && i < n) atomicAdd(&h[(key[r] >> shift) & (kOrderDigits - 1)], 1);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kOrderDigits / THREADS; ++q) {
        const int d = q * THREADS + threadIdx.x;
        if (tile_major) hist[int64_t(me) * kOrderDigits + d] = h[d];
        else hist[int64_t(d) * nblocks + me] = h[d];
    }
}

// The destination rows of consecutive edges, 64 at a time, for one wavefront: the last row that begins at or before an
// edge.  The lanes hold the offsets of 64 consecutive rows; the window only moves forward and ends at the last row,
// which takes every edge past the last offset.
struct RowWindow {
    const int32_t *indptr;
    int64_t num_dst, r0;
    int off, end;
    __device__ __forceinline__ int offset(int64_t r) const { return indptr[r < num_dst ? r : num_dst]; }
    __device__ __forceinline__ int64_t row_of(int64_t e) const {
        const int64_t r = wave_count_below<false>(indptr, num_dst, e) - 1;
        return r > 0 ? r : 0;
    }
    __device__ __forceinline__ RowWindow(const int32_t *p, int64_t n, int64_t first) : indptr(p), num_dst(n) {
        r0 = row_of(first);
        off = offset(r0 + lane_id());
        end = offset(r0 + kWave);
    }
    // edge e of every lane (ascending over the lanes and from call to call); only `open` ones count
    __device__ __forceinline__ int32_t rows(int64_t e, bool open) {
        int32_t row = 0;
        const int64_t e0 = e - lane_id();
        for (;;) {
            int k = 0;
#pragma unroll
            for (int h = 32; h > 0; h >>= 1)
                if (__shfl(off, k + h, 64) <= e) k += h;
            if (open && (e < end || r0 + kWave >= num_dst)) {
                const int64_t r = r0 + k < num_dst ? r0 + k : num_dst - 1;
                row = static_cast<int32_t>(r > 0 ? r : 0);
                open = false;
            }
            const uint64_t left = ballot64(open);
            if (!left) return row;
            r0 += kWave;
            const int64_t first = e0 + __ffsll(static_cast<long long>(left)) - 1;
            if (offset(r0 + kWave) <= first) {             // past a stretch of empty rows
                const int64_t r = row_of(first);
                r0 = r > r0 ? r : r0;
            }
            off = offset(r0 + lane_id());
            end = offset(r0 + kWave);
        }
    }
};

// SELF: hist is the [tile][digit] table of counts, added up here (and the totals stored); otherwise it is the
// [digit][tile] table, scanned row by row, and `totals` the edges of every digit.  The tile lies sorted by digit in LDS
// before it is written, every digit's run to consecutive addresses; see k_radix_scatter.
template <bool SELF, bool WEIGHTED, int THREADS>
__global__ void __launch_bounds__(THREADS)
k_order_scatter(const int32_t *__restrict__ indices, const int32_t *__restrict__ indptr, const float *__restrict__ edge_w,
                const int64_t *__restrict__ sizes, int64_t cap, const int32_t *__restrict__ hist, int32_t *__restrict__ totals, int nblocks, int items,
                uint16_t *__restrict__ key_out, int32_t *__restrict__ row_out, float *__restrict__ w_out) {
    constexpr int ITEMS = kRadixItems, WAVES = THREADS / kWave, PER = kOrderDigits / THREADS;
    __shared__ uint16_t wcnt[WAVES][kOrderDigits];     // edges of this digit so far, then those of the wavefronts before
    __shared__ int first[kOrderDigits];                    // first place of the digit in the sorted tile ...
    __shared__ int gbase[kOrderDigits];                    // ... and in the output, less that
    __shared__ uint32_t skeys[THREADS * ITEMS];
    __shared__ int32_t srows[THREADS * ITEMS];
    __shared__ float sw[WEIGHTED ? THREADS * ITEMS : 1];
    __shared__ int scan_lds[WAVES];
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int wave = tid >> 6;
    const int64_t n = sizes[2] < cap ? sizes[2] : cap;
    const int shift = order_shift(sizes[1]);
    const uint32_t low = (1u << shift) - 1;
    const int me = SELF ? static_cast<int>(blockIdx.x) : xcd_tile(live_tiles(n, THREADS * items));
    if (me >= nblocks) return;
    const int64_t base = int64_t(me) * THREADS * items;
    if (base >= n && !(SELF && me == 0)) return;
    const int tile_n = n - base < THREADS * items ? static_cast<int>(n > base ? n - base : 0) : THREADS * items;
    const int wave_first = wave * kWave * items;
    uint32_t key[ITEMS];
    float w[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int i = wave_first + r * kWave + lane;
        const bool in = r < items && i < tile_n;
        key[r] = in ? static_cast<uint32_t>(indices[base + i]) : 0;
        w[r] = WEIGHTED && in ? edge_w[base + i] : 0.f;
    }
    int out0[PER], all[PER], sum = 0, total;   // first output places of digits tid * PER ... for this tile
    if (!SELF) {
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            out0[q] = hist[int64_t(tid * PER + q) * nblocks + me];
            all[q] = totals[tid * PER + q];
            sum += all[q];
        }
    } else {
#pragma unroll
        for (int q = 0; q < PER; ++q) all[q] = out0[q] = 0;
#pragma unroll 4
        for (int t = 0; t < nblocks; ++t) {
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const int c = hist[int64_t(t) * kOrderDigits + tid * PER + q];
                all[q] += c;
                out0[q] += t < me ? c : 0;
            }
        }
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            if (me == 0) totals[tid * PER + q] = all[q];
            sum += all[q];
        }
    }
    int ex = block_excl_scan<WAVES>(sum, &total, scan_lds);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        out0[q] += ex;
        ex += all[q];
    }
#pragma unroll
    for (int q = 0; q < kOrderDigits / kWave; ++q) wcnt[wave][q * kWave + lane] = 0;
    wave_lds_sync();
    int rank[ITEMS];                                       // among the edges of its digit in this wavefront
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        if (r < items) {                                   // uniform
            const bool in = wave_first + r * kWave + lane < tile_n;
            const int digit = (key[r] >> shift) & (kOrderDigits - 1);
            uint64_t peers = ballot64(in);                 // lanes that hold the same digit
#pragma unroll
            for (int bit = 0; bit < kOrderBits; ++bit) {
                const int b = __builtin_amdgcn_sbfe(digit, bit, 1);              // all ones or zero
                peers &= ~(ballot64(b != 0) ^ static_cast<uint64_t>(int64_t(b)));
            }
            const int in_group = popc64(peers & lanes_below(lane));
            const int so_far = wcnt[wave][digit];
            rank[r] = so_far + in_group;
            wave_lds_sync();
            if (in && in_group == 0) wcnt[wave][digit] = static_cast<uint16_t>(so_far + popc64(peers));
            wave_lds_sync();
        }
    }
    int32_t row[ITEMS];
    if (wave_first < tile_n) {
        RowWindow window(indptr, sizes[0], base + wave_first);
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            const int i = wave_first + r * kWave + lane;
            row[r] = r < items && wave_first + r * kWave < tile_n ? window.rows(base + i, i < tile_n) : 0;
        }
    }
    __syncthreads();
    int cnt[PER];
    sum = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        cnt[q] = 0;
#pragma unroll
        for (int v = 0; v < WAVES; ++v) {
            const int c = wcnt[v][tid * PER + q];
            wcnt[v][tid * PER + q] = static_cast<uint16_t>(cnt[q]);
            cnt[q] += c;
        }
        sum += cnt[q];
    }
    if constexpr (SELF) {                                  // few edges: each straight to its place
#pragma unroll
        for (int q = 0; q < PER; ++q) gbase[tid * PER + q] = out0[q];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            if (r < items && wave_first + r * kWave + lane < tile_n) {
                const int digit = (key[r] >> shift) & (kOrderDigits - 1);
                const int o = gbase[digit] + wcnt[wave][digit] + rank[r];
                key_out[o] = static_cast<uint16_t>(key[r] & low);
                row_out[o] = row[r];
                if (WEIGHTED) w_out[o] = w[r];
            }
        }
        return;
    }
    ex = block_excl_scan<WAVES>(sum, &total, scan_lds);
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
            const int digit = (key[r] >> shift) & (kOrderDigits - 1);
            const int p = first[digit] + wcnt[wave][digit] + rank[r];
            skeys[p] = key[r];
            srows[p] = row[r];
            if (WEIGHTED) sw[p] = w[r];
        }
    }
    __syncthreads();
    for (int p = tid; p < tile_n; p += THREADS) {
        const uint32_t k = skeys[p];
        const int o = gbase[(k >> shift) & (kOrderDigits - 1)] + p;
        key_out[o] = static_cast<uint16_t>(k & low);
        row_out[o] = srows[p];
        if (WEIGHTED) w_out[o] = sw[p];
    }
}

// Lanes that add to one word of LDS are served one after the other (1.8 cycles each).  Where kHotLanes or more lanes hold an edge of the
// same source as the first lane with one, a wavefront counts, and places, these together; it looks once per batch of loads.
constexpr int kHotLanes = 8;
__device__ __forceinline__ uint64_t lanes_like_first(int d, uint64_t live) {           // live: not none
    const int first = __ffsll(static_cast<long long>(live)) - 1;
    return ballot64(d == static_cast<int>(readlane32(static_cast<uint32_t>(d), first))) & live;
}
__device__ __forceinline__ bool many_alike(int d, bool in) {
    const uint64_t live = ballot64(in);
    return live && popc64(lanes_like_first(d, live)) >= kHotLanes;
}
// add(1) for every lane with `in`, or, hot, once for all of those
template <typename Add>
__device__ __forceinline__ void add_each(bool hot, int d, bool in, Add add) {
    int n = 1;
    if (hot) {
        const uint64_t live = ballot64(in), same = live ? lanes_like_first(d, live) : 0;
        if ((same >> lane_id()) & 1) {
            n = popc64(same);
            in = (same & lanes_below(lane_id())) == 0;
        }
    }
    if (in) add(n);
}

// f(i, keys[i], hot) for the places [first, last), f(i, -1, hot) for a few around them, in no order: eight keys to a 16-byte load.
// t of `threads` threads; all lanes of a wavefront call f together.
template <typename F>
__device__ __forceinline__ void for_keys(const uint16_t *__restrict__ keys, int first, int last, int t, int threads, F f) {
    const int before = t & ~(kWave - 1);
    const uint4 *groups = reinterpret_cast<const uint4 *>(keys);
    const int end = (last + 7) >> 3;
    for (int g0 = first >> 3; g0 + before < end; g0 += 2 * threads) {
        uint4 v[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int g = g0 + u * threads + t;
            v[u] = groups[g < end ? g : end - 1];
        }
        const bool hot = many_alike(static_cast<int>(v[0].y & 0xFFFF), true);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (g0 + u * threads + before >= end) break;
            const uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int i = (g0 + u * threads + t) * 8 + e;
                f(i, i >= first && i < last ? static_cast<int>(w[e >> 1] >> ((e & 1) << 4) & 0xFFFF) : -1, hot);
            }
        }
    }
}

// A bucket's sources are cut into ranges of up to kSub.  A bucket of more than chunk_edges edges is cut into chunks of that many:
// a workgroup takes one (bucket, range, chunk) after the other, `grid` apart.  It counts the chunk's edges of its range per source and
// wavefront, which gives the places, and places them: the chunk's edges in order are cut among the wavefronts, so that counts per
// wavefront and running places keep the order.  A range in one chunk is put together in LDS and stored coalesced.
// The other chunks' counts: in a bucket of up to kRecountMost edges every chunk's workgroup reads and counts the bucket for itself.
// For larger ones, which only blocks of more edges can hold, the first launch counts each chunk once, into a table of 16-bit counts per chunk
// and source, and a second one places their edges, adding up the table's columns.  (Counting all of a bucket for every chunk is
// quadratic in its edges: the order of 4 M edges of one source took 6.7 ms, 2.1 with 30 % of them; now 0.12 and 0.11, evenly
// spread ones 0.09.)  The line: the crowded buckets of earlier frontiers hold 100 k edges, 52 us counted here and 30 + 37 in two launches; a
// second launch without work takes 2 us.
// Bound by what a wavefront does per 64 keys, of which the other ranges' are done for nothing: ballots over all bits of every key in place
// of the places taken and corrected 79 us for 4.3 M edges, 52 so; digits of 8 and 10 bits in the partition, with 4 ranges and 1,
// 14 and 7 us more in all.
constexpr int kPartAll = 0, kPartFirst = 1, kPartCounted = 2;       // one launch for all buckets (none is counted), the first of two, the second
template <bool WEIGHTED, int PART>
__global__ void __launch_bounds__(kBucketThreads)
k_order_buckets(const uint16_t *__restrict__ keys, const int32_t *__restrict__ rows, const float *__restrict__ w, const int64_t *__restrict__ sizes,
                int64_t cap, int32_t *__restrict__ totals, int chunk_edges, int grid, uint32_t *__restrict__ table, int32_t *__restrict__ range_first,
                int32_t *__restrict__ col_ptr, int32_t *__restrict__ row_out, float *__restrict__ w_out) {
    __shared__ uint32_t pairs[kBucketWaves][kSub / 2];     // two 16-bit counts a word: edges per wavefront and source
    __shared__ int base_of[kSub];                          // of the chunks after; then the first place of the source's edges
    __shared__ int32_t stage[kStageWords];                 // edges of the range; or, in several chunks, counts of the chunks before
    __shared__ int start_of[kOrderDigits + 1], item_of[kOrderDigits + 1];   // first edge and item of every bucket,
    __shared__ int row_of[PART == kPartCounted ? kOrderDigits : 1];     // and first row in the table
    __shared__ int lds[kBucketWaves];
    __shared__ int below_of[kBucketWaves];
    constexpr bool COUNTED = PART == kPartCounted;
    static_assert(kOrderDigits == kBucketThreads, "a bucket per thread");
    static_assert(kSub == 4 * kBucketThreads, "four sources per thread");
    constexpr int kStage = WEIGHTED ? kStageWords / 2 : kStageWords;
    const int tid = threadIdx.x, lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (COUNTED && totals[kOrderDigits] == 0) return;      // no bucket of that size
    const int64_t num_src = sizes[1];
    const int shift = order_shift(num_src);
    const int range_bits = shift > kSubBits ? shift - kSubBits : 0;
    const int sub_bits = shift < kSubBits ? shift : kSubBits;
    const int subs = 1 << sub_bits;                        // sources of a range
    const int stride = order_table_stride(shift);          // words of a table row
    const int used = num_src > 0 ? static_cast<int>((num_src - 1) >> shift) + 1 : 0;      // buckets
    if (!COUNTED && blockIdx.x == 0 && tid == 0) col_ptr[num_src] = static_cast<int32_t>(sizes[2] < cap ? sizes[2] : cap);
    int items, rows_mine;                                  // rows_mine: of bucket tid in the table
    {
        const int mine = totals[tid];
        int total;
        start_of[tid] = block_excl_scan<kBucketWaves>(mine, &total, lds);
        if (tid == 0) start_of[kOrderDigits] = total;
        const int chunks = tid < used ? (mine > chunk_edges ? (mine + chunk_edges - 1) / chunk_edges : 1) : 0;
        const bool counted = PART != kPartAll && mine > kRecountMost;
        rows_mine = counted ? chunks : 0;
        if (COUNTED) row_of[tid] = block_excl_scan<kBucketWaves>(rows_mine, &total, lds);
        item_of[tid] = block_excl_scan<kBucketWaves>(COUNTED ? rows_mine << range_bits : counted ? chunks : chunks << range_bits, &items, lds);
        if (tid == 0) item_of[kOrderDigits] = items;
    }
    __syncthreads();
    constexpr int U = 8;
    constexpr int kNone = -(1 << 16);                      // in no range
    for (int item = static_cast<int>(blockIdx.x); item < items; item += grid) {
        int b = 0;                                         // the last bucket that begins at or before the item
#pragma unroll
        for (int h = kOrderDigits / 2; h > 0; h >>= 1)
            if (item_of[b + h] <= item) b += h;
        b = __builtin_amdgcn_readfirstlane(b);
        const int k = item - item_of[b];
        const int start = start_of[b], n = start_of[b + 1] - start;
        const uint16_t *bk = keys + start;
        if (PART == kPartFirst && n > kRecountMost) {      // counts of chunk k, all ranges
            int rows_before = 0;
            (void)block_excl_scan<kBucketWaves>(tid < b ? rows_mine : 0, &rows_before, lds);
            if (tid == 0) totals[kOrderDigits] = 1;        // (any workgroup that counts)
            uint32_t *counts = &pairs[0][0];
            for (int q = tid; q < 2 * stride; q += kBucketThreads) counts[q] = 0;
            __syncthreads();
            const int c0 = k * chunk_edges, c1 = n - c0 < chunk_edges ? n : c0 + chunk_edges;
            for_keys(keys, start + c0, start + c1, tid, kBucketThreads, [&](int, int key, bool hot) {
                add_each(hot, key, key >= 0, [&](int v) { atomicAdd(&counts[key], static_cast<uint32_t>(v)); });
            });
            __syncthreads();
            const int64_t row = rows_before + k;
            for (int q = tid; q < stride; q += kBucketThreads) table[row * stride + q] = counts[2 * q] | counts[2 * q + 1] << 16;
            int before = 0;
            for (int r = 0; r < 1 << range_bits; ++r) {    // first edge of every range among the chunk's
                if (tid == 0) range_first[row * kMostRanges + r] = before;
                int mine = 0, total;
                for (int q = tid; q < subs; q += kBucketThreads) mine += static_cast<int>(counts[r * kSub + q]);
                (void)block_excl_scan<kBucketWaves>(mine, &total, lds);
                before += total;
            }
            __syncthreads();                               // counts[] is the next item's
            continue;
        }
        const int range = k & ((1 << range_bits) - 1), chunk = k >> range_bits;
        const bool whole = !COUNTED && n <= chunk_edges;
        for (int q = lane; 2 * q < subs + 2; q += kWave) pairs[wave][q < kSub / 2 ? q : 0] = 0;
        for (int q = tid; !COUNTED && !whole && q < subs; q += kBucketThreads) base_of[q] = stage[q] = 0;
        __syncthreads();
        const int c0 = chunk * chunk_edges, c1 = n - c0 < chunk_edges ? n : c0 + chunk_edges;
        const int share = ((c1 - c0 + kBucketWaves - 1) / kBucketWaves + kWave - 1) / kWave * kWave;
        const int my0 = c0 + wave * share < c1 ? c0 + wave * share : c1, my1 = my0 + share < c1 ? my0 + share : c1;
        int below = 0;                                     // edges of the ranges before
        for (int i0 = my0; i0 < my1; i0 += U * kWave) {
            int key[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * kWave + lane;
                key[u] = i < my1 ? bk[i] : kNone;
            }
            const bool hot = many_alike(key[0], key[0] >= 0);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int r = key[u] >> kSubBits, d = key[u] & (kSub - 1);
                add_each(hot, d, r == range, [&](int v) { atomicAdd(&pairs[wave][d >> 1], static_cast<uint32_t>(v) << ((d & 1) << 4)); });
                below += r >= 0 && r < range ? 1 : 0;
            }
        }
        if constexpr (COUNTED) {
            below = 0;
            const int chunks = (n + chunk_edges - 1) / chunk_edges;
            for (int c = tid; c < chunks; c += kBucketThreads) below += range_first[int64_t(row_of[b] + c) * kMostRanges + range];
        }
        if (!COUNTED && !whole) {                          // the other chunks
            for_keys(keys, start, start + n, tid, kBucketThreads, [&](int i, int key, bool hot) {
                const int r = i < start + c0 || i >= start + c1 ? key >> kSubBits : -1, d = key & (kSub - 1);
                add_each(hot, d, r == range, [&](int v) { atomicAdd(i < start + c0 ? &stage[d] : &base_of[d], v); });
                below += r >= 0 && r < range ? 1 : 0;
            });
        }
        below = wave_sum(below);
        if (lane == 0) below_of[wave] = below;
        __syncthreads();
        int held, first = start;                           // the range's edges and the first one's place
        {
            const int d = 4 * tid;
            int all[4] = {0, 0, 0, 0}, ahead[4] = {0, 0, 0, 0};
            if (d < subs) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    uint32_t run = 0;                      // both halves: a chunk's edges fit 16 bits
#pragma unroll
                    for (int v = 0; v < kBucketWaves; ++v) {
                        const uint32_t c = pairs[v][2 * tid + h];
                        pairs[v][2 * tid + h] = run;
                        run += c;
                    }
                    all[2 * h] = static_cast<int>(run & 0xFFFF);
                    all[2 * h + 1] = static_cast<int>(run >> 16);
                }
                if constexpr (COUNTED) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) all[q] = 0;
                    const int chunks = (n + chunk_edges - 1) / chunk_edges;
                    const uint2 *column = reinterpret_cast<const uint2 *>(table + int64_t(row_of[b]) * stride + range * (kSub / 2)) + tid;
                    int c = 0;
                    for (; c + U <= chunks; c += U) {
                        uint2 v[U];
#pragma unroll
                        for (int u = 0; u < U; ++u) v[u] = column[int64_t(c + u) * (stride / 2)];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const int x[4] = {static_cast<int>(v[u].x & 0xFFFF), static_cast<int>(v[u].x >> 16), static_cast<int>(v[u].y & 0xFFFF),
                                              static_cast<int>(v[u].y >> 16)};
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                all[q] += x[q];
                                ahead[q] += c + u < chunk ? x[q] : 0;
                            }
                        }
                    }
                    for (; c < chunks; ++c) {
                        const uint2 v = column[int64_t(c) * (stride / 2)];
                        const int x[4] = {static_cast<int>(v.x & 0xFFFF), static_cast<int>(v.x >> 16), static_cast<int>(v.y & 0xFFFF), static_cast<int>(v.y >> 16)};
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            all[q] += x[q];
                            ahead[q] += c < chunk ? x[q] : 0;
                        }
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {                  // (ranges of one or two sources)
                if (d + q >= subs) all[q] = 0;
                else if (!COUNTED && !whole) all[q] += base_of[d + q] + stage[d + q];
            }
            int at = block_excl_scan<kBucketWaves>((all[0] + all[1]) + (all[2] + all[3]), &held, lds);
#pragma unroll
            for (int v = 0; v < kBucketWaves; ++v) first += below_of[v];
            const int64_t source = (int64_t(b) << shift) + (int64_t(range) << kSubBits) + d;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (d + q < subs) {
                    if (chunk == 0 && source + q < num_src) col_ptr[source + q] = first + at;
                    base_of[d + q] = at + (COUNTED ? ahead[q] : whole ? 0 : stage[d + q]);
                }
                at += all[q];
            }
        }
        __syncthreads();
        // every wavefront its own edges, in order
        const bool staged = whole && held <= kStage;
        const int32_t *br = rows + start;
        const float *bw = w + start;
        for (int i0 = my0; i0 < my1; i0 += U * kWave) {
            int key[U];
            int32_t row[U];
            float weight[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * kWave + lane;
                key[u] = i < my1 ? bk[i] : kNone;
                row[u] = i < my1 ? br[i] : 0;
                weight[u] = WEIGHTED && i < my1 ? bw[i] : 0.f;
            }
            const bool hot = many_alike(key[0], (key[0] >> kSubBits) == range);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                // The lanes of the first lane's source, if they are many, take their places together.  Every other lane takes the next
                // place of its source; lanes of the same source take them in any order: a lane that did not get the first place free
                // tells that there are some, and then ballots put them in order - one source after the other, or,
                // from the third on, all by the bits of their sources.
                bool in = (key[u] >> kSubBits) == range;
                const bool mine = in;
                const uint64_t live = ballot64(in);
                if (!live) continue;
                const int d = key[u] & (kSub - 1), half = (d & 1) << 4;
                int o = 0;
                uint32_t so_far = 0;
                if (in) {
                    so_far = pairs[wave][d >> 1] >> half & 0xFFFF;
                    o = base_of[d] + static_cast<int>(so_far);
                }
                wave_lds_sync();
                if (hot) {
                    const uint64_t same = lanes_like_first(d, live);
                    if ((same >> lane) & 1) {
                        if ((same & lanes_below(lane)) == 0) (void)atomicAdd(&pairs[wave][d >> 1], static_cast<uint32_t>(popc64(same)) << half);
                        o += popc64(same & lanes_below(lane));
                        in = false;
                    }
                }
                bool later = false;
                if (in) {
                    const uint32_t got = atomicAdd(&pairs[wave][d >> 1], 1u << half) >> half & 0xFFFF;
                    later = got != so_far;
                }
                uint64_t left = ballot64(later);
                for (int round = 0; left && round < 2; ++round) {
                    const int source = static_cast<int>(readlane32(static_cast<uint32_t>(d), __ffsll(static_cast<long long>(left)) - 1));
                    const uint64_t peers = ballot64(in && d == source);
                    if (in && d == source) {
                        o += popc64(peers & lanes_below(lane));
                        in = false;
                    }
                    left &= ~peers;
                }
                if (left) {
                    uint64_t peers = ballot64(in);         // of the same source
                    for (int bit = 0; bit < sub_bits; ++bit) {
                        const int v = __builtin_amdgcn_sbfe(d, bit, 1);         // all ones or zero
                        peers &= ~(ballot64(v != 0) ^ static_cast<uint64_t>(int64_t(v)));
                    }
                    if (in) o += popc64(peers & lanes_below(lane));
                }
                if (mine && staged) {
                    stage[o] = row[u];
                    if (WEIGHTED) stage[kStage + o] = __float_as_int(weight[u]);
                } else if (mine) {
                    row_out[first + o] = row[u];
                    if (WEIGHTED) w_out[first + o] = weight[u];
                }
            }
        }
        __syncthreads();
        if (staged) {
            for (int q = tid; q < held; q += kBucketThreads) {
                row_out[first + q] = stage[q];
                if (WEIGHTED) w_out[first + q] = __int_as_float(stage[kStage + q]);
            }
            __syncthreads();                               // stage[] is the next item's
        }
    }
}

}  // namespace

// Sources up to which the order is made this way: kMostRanges ranges a bucket, each of which reads the bucket's keys.
bool can_order_edges(int64_t src_cap) { return src_cap <= (int64_t(kMostRanges) << (kSubBits + kOrderBits)); }

// entries of bwd.hist for blocks of at most nnz_cap edges
int64_t order_hist_len(int64_t nnz_cap) { return kOrderDigits * std::max<int64_t>(radix_blocks(nnz_cap), kRadixSelfBlocks); }

// Edges of block b by source into rows_out (destination rows), w_out (weights, if edge_w is given) and col_ptr.
int order_edges_by_source(mqg_ctx *ctx, const mqg_block *b, const float *edge_w, int32_t *col_ptr, int32_t *rows_out, float *w_out, hipStream_t s) {
    const int64_t cap = b->cap_nnz;
    const RadixBufs &t = ctx->bwd;
    uint16_t *keys = reinterpret_cast<uint16_t *>(t.keys[0]);
    int32_t *rows = t.vals[0];
    float *w = reinterpret_cast<float *>(t.keys[1]);
    // up to kRadixSelfBlocks tiles: no scan launch
    const bool self = cap <= int64_t(kRadixTile) * kRadixSelfBlocks, large = cap > kLargeOrder;
    const int threads = large ? kOrderThreads : kBlock;
    const int items = radix_items(cap);
    const int nblocks = static_cast<int>(std::max<int64_t>(1, ceil_div(cap, int64_t(threads) * items)));
    const int grid = self ? nblocks : xcd_grid(nblocks);
    if (large)
        MQG_LAUNCH(ctx, "k_order_hist", s, (k_order_hist<kOrderThreads><<<grid, threads, 0, s>>>(b->indices, b->sizes, cap, t.hist, nblocks, items, 0, t.totals)));
    else
        MQG_LAUNCH(ctx, "k_order_hist", s, (k_order_hist<kBlock><<<grid, threads, 0, s>>>(b->indices, b->sizes, cap, t.hist, nblocks, items, self ? 1 : 0, t.totals)));
    if (!self) {
        int rc = launch_radix_scan(ctx, t.hist, nblocks, kOrderDigits, t.totals, cap, &b->sizes[2], threads * items, s);
        if (rc != MQG_OK) return rc;
    }
#define MQG_ORDER(SELF, T)                                                                                                                  \
    do {                                                                                                                                    \
        if (edge_w)                                                                                                                         \
            MQG_LAUNCH(ctx, "k_order_scatter", s,                                                                                           \
                       (k_order_scatter<SELF, true, T><<<grid, T, 0, s>>>(b->indices, b->indptr, edge_w, b->sizes, cap, t.hist, t.totals,    \
                                                                          nblocks, items, keys, rows, w)));                                 \
        else                                                                                                                                \
            MQG_LAUNCH(ctx, "k_order_scatter", s,                                                                                           \
                       (k_order_scatter<SELF, false, T><<<grid, T, 0, s>>>(b->indices, b->indptr, edge_w, b->sizes, cap, t.hist, t.totals,   \
                                                                           nblocks, items, keys, rows, w)));                                \
    } while (0)
    if (self) MQG_ORDER(true, kBlock);
    else if (large) MQG_ORDER(false, kOrderThreads);
    else MQG_ORDER(false, kBlock);
#undef MQG_ORDER
    // one workgroup per bucket, range and chunk if there are fewer of them than kBucketGrid
    const int shift = order_shift(b->cap_src);
    const int chunk = order_chunk(cap, shift);
    const int64_t pieces = (int64_t(kOrderDigits) + cap / chunk) << (shift > kSubBits ? shift - kSubBits : 0);
    const int bgrid = static_cast<int>(std::min<int64_t>(pieces, kBucketGrid));
    // The table of the counted buckets' chunks and where their ranges begin lie in vals[1], of four bytes an edge: a chunk's row
    // takes 2 bytes a source and 16 more, and a bucket of n has at most n / chunk + n / kRecountMost chunks.
    uint32_t *table = reinterpret_cast<uint32_t *>(t.vals[1]);
    const int64_t table_rows = cap / chunk + cap / kRecountMost;
    int32_t *range_first = t.vals[1] + table_rows * order_table_stride(shift);
#define MQG_BUCKETS(NAME, W, C)                                                                                                             \
    MQG_LAUNCH(ctx, NAME, s,                                                                                                                \
               (k_order_buckets<W, C><<<bgrid, kBucketThreads, 0, s>>>(keys, rows, w, b->sizes, cap, t.totals, chunk, bgrid, table, range_first, \
                                                                       col_ptr, rows_out, w_out)))
    if (cap <= kRecountMost) {
        if (edge_w) MQG_BUCKETS("k_order_buckets", true, kPartAll);
        else MQG_BUCKETS("k_order_buckets", false, kPartAll);
    } else {
        if (edge_w) MQG_BUCKETS("k_order_buckets", true, kPartFirst);
        else MQG_BUCKETS("k_order_buckets", false, kPartFirst);
        if (edge_w) MQG_BUCKETS("k_order_counted", true, kPartCounted);
        else MQG_BUCKETS("k_order_counted", false, kPartCounted);
    }
#undef MQG_BUCKETS
    return MQG_OK;
}

}  // namespace mqg
