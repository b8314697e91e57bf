// Feature gather through the hot-node cache (paper Sec. III "Feature Cache", Sec. IV
// "Mini-Batch Transfer To GPU"): out[i] = F[ids[i]], a row coming from the HBM cache when the
// node is cached and from the full feature matrix (pinned host memory, read over the host link
// by the kernel itself) when it is not.
//
//   k_classify        slot_of lookup, ballot-compacted (output row, source row) lists for hits and
//                     misses, one atomic per tile of ids
//   k_gather_rows     hits: HBM cache -> HBM output, widest aligned loads; rows of up to 64 vectors
//                     as one flat sequence of vectors (every lane carries one), longer rows two at a
//                     time by a wavefront; misses: feature matrix -> HBM output.  One launch for both, the few
//                     workgroups that keep the host link busy first; in halves, and while profiling, a launch
//                     each (<., 0> hits, <., 1> misses, so that profiles tell the HBM-bound from the link-bound)
//   k_gather_slots    a cache that holds every node: slot lookup and copy in one launch, but for many narrow rows
//   k_gather_direct   no cache: every row straight from the feature matrix
// The last two count the rows for the statistics in a few workgroups beside the copy.
#include <hip/hip_ext.h>

#include <algorithm>
#include <mutex>

#include "common.h"
#include "device_utils.h"

namespace mqg {

namespace {

// Words of a context's (or the static array's) counters; all but the last two are zero between gathers.
constexpr int kCountSplit = 0;         // hits, misses and tiles so far, see classify_tiles
constexpr int kCountRare = 1;          // misses of a gather from a cache that holds every node, see count_ids
constexpr int kCountTiles = 3;         // tiles of a split into more than its word can count
constexpr int kCountMissed = 2;        // finished workgroups that copy misses
constexpr int kCountHits = 4, kCountMisses = 5;    // entries of the lists of the last split; misses are zero again once they are copied

// Stats of a gather of no ids.
__global__ void k_direct_stats(int64_t *stats) {
    if (blockIdx.x == 0 && threadIdx.x < 2) stats[threadIdx.x] = 0;
}

// Splits the ids into a hit list (output row, cache slot) and a miss list (output row, node id).
// A workgroup classifies a tile of 256 * ITEMS ids and reserves its share of both lists with one atomic.  Atomics on one
// address are served one after the other, at 13 ns, so more than 512 k ids go in tiles of
// 4,096 (1.35 M ids: 41 -> 20 us); fewer keep tiles of 1,024, enough workgroups to hide the slot lookups (100 k ids
// 7.9 us, in tiles of 4,096 14.3; level at 500 k with 16.5 and 17.5), and up to 32 k ids go in tiles of 256.
// The number of ids decides, which only
// the device knows; the capacity is often twice that and more.  Positions inside a share come from ballots, so that
// a wavefront writes consecutive entries.  The order of the list entries is arbitrary; the gather does not depend on
// it.  An id outside [0, num_nodes) is never used as an index: it goes on neither list, so its output row stays
// untouched and hits + misses fall short of the number of ids.
// The word that the atomics go to holds the hits and the misses so far, BITS bits each, and above them the tiles: whoever adds the last
// tile hands the numbers on.  2^25 ids and more leave no bits for the tiles: they are counted in a word of their own.
constexpr int64_t kClassifyLarge = int64_t(1) << 19, kClassifyHuge = int64_t(1) << 25;
constexpr int64_t kClassifySmall = int64_t(1) << 15;
struct ClassifyLds {
    int hits[kWavesPerBlock], misses[kWavesPerBlock];
    unsigned long long base[2];
};
template <int ITEMS, int BITS, typename IdxT>
__device__ __forceinline__ void classify_tiles(const IdxT *__restrict__ ids, int64_t n, const int32_t *__restrict__ slot_of, int64_t num_nodes,
                                               int2 *__restrict__ hit_list, int2 *__restrict__ miss_list,
                                               unsigned long long *__restrict__ counters, int64_t *__restrict__ stats, ClassifyLds &lds, int grid) {
    constexpr int kTile = kBlock * ITEMS;
    constexpr bool kTilesApart = BITS == 32;
    constexpr unsigned long long kMask = (1ull << BITS) - 1;
    const int lane = lane_id();
    const int wave = static_cast<int>(threadIdx.x) >> 6;
    const int64_t tiles = n > 0 ? (n + kTile - 1) / kTile : 1;             // of no ids one, for the numbers
    for (int64_t tile = blockIdx.x; tile < tiles; tile += grid) {
        const int64_t t0 = tile * kTile;
        int32_t id[ITEMS], slot[ITEMS];
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            const int64_t i = t0 + q * kBlock + threadIdx.x;
            const int64_t raw = i < n ? static_cast<int64_t>(ids[i]) : -1;
            id[q] = raw >= 0 && raw < num_nodes ? static_cast<int32_t>(raw) : -1;
        }
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) slot[q] = id[q] >= 0 ? slot_of[id[q]] : -1;
        int h = 0, m = 0;
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            h += popc64(ballot64(slot[q] >= 0));
            m += popc64(ballot64(slot[q] < 0 && id[q] >= 0));
        }
        if (lane == 0) {
            lds.hits[wave] = h;
            lds.misses[wave] = m;
        }
        __syncthreads();
        unsigned long long th = 0, tm = 0, before = 0;     // of thread 0
        if (threadIdx.x == 0) {
#pragma unroll
            for (int w = 0; w < kWavesPerBlock; ++w) {
                th += static_cast<unsigned>(lds.hits[w]);
                tm += static_cast<unsigned>(lds.misses[w]);
            }
            before = atomicAdd(&counters[kCountSplit], th | tm << BITS | (kTilesApart ? 0ull : 1ull << (2 * BITS & 63)));
            lds.base[0] = before & kMask;
            lds.base[1] = before >> BITS & kMask;
        }
        __syncthreads();
        int64_t ph = static_cast<int64_t>(lds.base[0]), pm = static_cast<int64_t>(lds.base[1]);
        for (int w = 0; w < wave; ++w) {
            ph += lds.hits[w];
            pm += lds.misses[w];
        }
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            const int i = static_cast<int>(t0 + q * kBlock + threadIdx.x);
            const bool hit = slot[q] >= 0, miss = slot[q] < 0 && id[q] >= 0;
            const uint64_t hb = ballot64(hit), mb = ballot64(miss);
            if (hit) hit_list[ph + popc64(hb & lanes_below(lane))] = make_int2(i, slot[q]);
            if (miss) miss_list[pm + popc64(mb & lanes_below(lane))] = make_int2(i, id[q]);
            ph += popc64(hb);
            pm += popc64(mb);
        }
        if (threadIdx.x == 0) {
            // (tiles apart: a tile is counted once its share is reserved, so whoever counts the last finds all reserved)
            bool last;
            unsigned long long all = before + (th | tm << BITS);
            if (kTilesApart) {
                __threadfence();
                last = atomicAdd(&counters[kCountTiles], 1ull) == static_cast<unsigned long long>(tiles - 1);
                if (last) all = atomicAdd(&counters[kCountSplit], 0ull);
            } else {
                last = static_cast<int64_t>(before >> (2 * BITS & 63)) == tiles - 1;
            }
            if (last) {
                // the words are left at zero, so that the call is self-contained and can be replayed from a recorded graph
                counters[kCountSplit] = 0;
                if (kTilesApart) counters[kCountTiles] = 0;
                counters[kCountHits] = all & kMask;
                counters[kCountMisses] = all >> BITS & kMask;
                if (stats) {
                    stats[0] = static_cast<int64_t>(all & kMask);
                    stats[1] = static_cast<int64_t>(all >> BITS & kMask);
                }
            }
        }
        __syncthreads();                                // hits[], misses[] and base are rewritten by the next tile
    }
}

template <typename IdxT>
__global__ void __launch_bounds__(kBlock)
k_classify(const IdxT *__restrict__ ids, const int64_t *__restrict__ num_ids, int64_t cap,
           const int32_t *__restrict__ slot_of, int64_t num_nodes, int2 *__restrict__ hit_list,
           int2 *__restrict__ miss_list, unsigned long long *__restrict__ counters, int64_t *__restrict__ stats, int grid) {
    __shared__ ClassifyLds lds;
    int64_t n = *num_ids;
    if (n > cap) n = cap;
    // 4,096 ids a tile: fewer than 2^25 ids in at most 2^13 tiles, 25 + 25 + 14 bits; otherwise at most 2^19 ids and 2^9 tiles
    if (n >= kClassifyHuge) classify_tiles<16, 32>(ids, n, slot_of, num_nodes, hit_list, miss_list, counters, stats, lds, grid);
    else if (n > kClassifyLarge) classify_tiles<16, 25>(ids, n, slot_of, num_nodes, hit_list, miss_list, counters, stats, lds, grid);
    else if (n > kClassifySmall) classify_tiles<4, 21>(ids, n, slot_of, num_nodes, hit_list, miss_list, counters, stats, lds, grid);
    else classify_tiles<1, 21>(ids, n, slot_of, num_nodes, hit_list, miss_list, counters, stats, lds, grid);
}

// Which rows to copy: entry r of a (output row, source row) list, or row ids[r] to output row r.
// get() returns false for a row that must not be written (an id outside the feature matrix); the
// source row is then 0, so that a load issued before the check stays inside the matrix.
struct ListRows {
    const int2 *list;
    __device__ __forceinline__ bool get(int64_t r, int64_t *src_row, int64_t *dst_row) const {
        int2 e = list[r];
        *src_row = e.y;
        *dst_row = e.x;
        return true;
    }
    __device__ __forceinline__ const char *at(int64_t row, const char *src, int64_t stride) const { return src + row * stride; }
};
template <typename IdxT>
struct DirectRows {
    const IdxT *ids;
    int64_t num_rows;                    // rows of the source matrix
    __device__ __forceinline__ bool get(int64_t r, int64_t *src_row, int64_t *dst_row) const {
        const int64_t id = static_cast<int64_t>(ids[r]);
        const bool ok = id >= 0 && id < num_rows;
        *src_row = ok ? id : 0;
        *dst_row = r;
        return ok;
    }
    __device__ __forceinline__ const char *at(int64_t row, const char *src, int64_t stride) const { return src + row * stride; }
};

// Row ids[r] to output row r, from the cache if it has a slot there and else from the feature matrix (row -1 - id).
template <typename IdxT>
struct SlotRows {
    const IdxT *ids;
    const int32_t *slot_of;
    int64_t num_nodes;                   // at least 1, and so has the cache a row
    const char *feats;
    int64_t feat_stride_bytes;
    __device__ __forceinline__ bool get(int64_t r, int64_t *src_row, int64_t *dst_row) const {
        const int64_t id = static_cast<int64_t>(ids[r]);
        const bool ok = id >= 0 && id < num_nodes;
        const int32_t slot = slot_of[ok ? id : 0];
        *src_row = !ok ? 0 : slot >= 0 ? slot : -1 - id;
        *dst_row = r;
        return ok;
    }
    __device__ __forceinline__ const char *at(int64_t row, const char *src, int64_t stride) const {
        return row >= 0 ? src + row * stride : feats + (-1 - row) * feat_stride_bytes;
    }
};

// A 16-byte load that is not kept in the caches on its way (STREAM: read-once data of a launch too
// large for the last-level cache); narrower vectors are loaded normally.
typedef unsigned int uint4_native __attribute__((ext_vector_type(4)));
template <bool STREAM, typename VecT>
__device__ __forceinline__ VecT load_vec(const VecT *p) {
    if constexpr (STREAM && sizeof(VecT) == 16) {
        const uint4_native v = __builtin_nontemporal_load(reinterpret_cast<const uint4_native *>(p));
        VecT out;
        __builtin_memcpy(&out, &v, 16);
        return out;
    } else {
        return *p;
    }
}

constexpr int kRowUnroll = 4;                            // row loads in flight per lane (rows of up to 64 vectors)
// Longer rows: all 64 lanes walk WR rows at a time, NCH 64-vector chunks of each, so that up to
// eight loads per lane are issued before the first store (a row's last, partial chunk rides along
// instead of trailing alone).  NCH is the number of chunks a row needs, at most four; loads are
// unconditional (an index past the row re-reads its last vector), only the stores are predicated.
template <typename VecT, int NCH, int WR, bool STREAM, typename Rows>
__device__ __forceinline__ void copy_rows_wide(const Rows &rows, int64_t n, const char *__restrict__ src,
                                               int64_t src_stride_bytes, char *__restrict__ dst,
                                               int64_t dst_stride_bytes, int vecs, int vb, int nb) {
    const int lane = lane_id();
    const int64_t wave0 = int64_t(vb) * kWavesPerBlock + (threadIdx.x >> 6);
    const int64_t nwaves = int64_t(nb) * kWavesPerBlock;
    for (int64_t r0 = wave0 * WR; r0 < n; r0 += nwaves * WR) {
        const VecT *sp[WR];
        VecT *dp[WR];
        bool rok[WR];
#pragma unroll
        for (int q = 0; q < WR; ++q) {
            const int64_t r = r0 + q;
            int64_t srow, drow;
            const bool valid = rows.get(r < n ? r : n - 1, &srow, &drow);          // a row past the end re-reads the last one
            rok[q] = r < n && valid;
            sp[q] = reinterpret_cast<const VecT *>(rows.at(srow, src, src_stride_bytes));
            dp[q] = reinterpret_cast<VecT *>(dst + drow * dst_stride_bytes);
        }
        for (int c0 = lane; c0 < vecs; c0 += NCH * kWave) {
            VecT v[WR][NCH];
#pragma unroll
            for (int q = 0; q < WR; ++q)
#pragma unroll
                for (int k = 0; k < NCH; ++k) {
                    const int c = c0 + k * kWave;
                    v[q][k] = load_vec<STREAM>(&sp[q][c < vecs ? c : vecs - 1]);
                }
#pragma unroll
            for (int q = 0; q < WR; ++q)
#pragma unroll
                for (int k = 0; k < NCH; ++k) {
                    const int c = c0 + k * kWave;
                    if (rok[q] && c < vecs) dp[q][c] = v[q][k];
                }
        }
    }
}

// chunks per row and rows per wavefront of the long-row copy
inline __host__ __device__ int wide_chunks(int vecs) { return vecs > 3 * kWave ? 4 : (vecs > 2 * kWave ? 3 : 2); }
inline __host__ __device__ int wide_rows(int vecs) { return vecs > 2 * kWave ? 2 : 4; }

// (All copies: workgroup vb of nb.)  Row copies by one wavefront (the grouped copy).  Rows of up to 64 vectors: the wavefront is split
// into 64/LPR groups of LPR lanes (LPR = 2^log2_lpr >= vecs), every group copies one row per step
// and kRowUnroll steps are in flight, so a wavefront moves 4*64/LPR short rows at a time.  Longer
// rows: copy_rows_wide.
template <typename VecT, bool STREAM, typename Rows>
__device__ __forceinline__ void copy_rows(const Rows &rows, int64_t n, const char *__restrict__ src,
                                          int64_t src_stride_bytes, char *__restrict__ dst,
                                          int64_t dst_stride_bytes, int vecs, int log2_lpr, int vb, int nb) {
    if (vecs > kWave) {
        switch (wide_chunks(vecs)) {
            case 2: copy_rows_wide<VecT, 2, 4, STREAM>(rows, n, src, src_stride_bytes, dst, dst_stride_bytes, vecs, vb, nb); break;
            case 3: copy_rows_wide<VecT, 3, 2, STREAM>(rows, n, src, src_stride_bytes, dst, dst_stride_bytes, vecs, vb, nb); break;
            default: copy_rows_wide<VecT, 4, 2, STREAM>(rows, n, src, src_stride_bytes, dst, dst_stride_bytes, vecs, vb, nb); break;
        }
        return;
    }
    const int lane = lane_id();
    const int64_t wave0 = int64_t(vb) * kWavesPerBlock + (threadIdx.x >> 6);
    const int64_t nwaves = int64_t(nb) * kWavesPerBlock;
    const int groups = kWave >> log2_lpr;
    const int g = lane >> log2_lpr;
    const int gl = lane & ((1 << log2_lpr) - 1);
    const int64_t per_wave = int64_t(groups) * kRowUnroll;
    for (int64_t base = wave0 * per_wave; base < n; base += nwaves * per_wave) {
        const VecT *sp[kRowUnroll];
        VecT *dp[kRowUnroll];
        bool ok[kRowUnroll];
        VecT v[kRowUnroll];
#pragma unroll
        for (int u = 0; u < kRowUnroll; ++u) {
            const int64_t r = base + u * groups + g;
            int64_t srow = 0, drow = 0;
            bool valid = false;
            if (r < n) {
                valid = rows.get(r, &srow, &drow);
            }
            ok[u] = valid && gl < vecs;
            sp[u] = reinterpret_cast<const VecT *>(rows.at(srow, src, src_stride_bytes)) + gl;
            dp[u] = reinterpret_cast<VecT *>(dst + drow * dst_stride_bytes) + gl;
        }
#pragma unroll
        for (int u = 0; u < kRowUnroll; ++u)
            if (ok[u]) v[u] = *sp[u];
#pragma unroll
        for (int u = 0; u < kRowUnroll; ++u)
            if (ok[u]) *dp[u] = v[u];
    }
}

// The rows of a launch as one flat sequence of vectors: vector t belongs to row t / vecs (a
// multiplication by magic = ceil(2^64 / vecs), exact for t < 2^32).  Every lane carries a vector
// whatever the row length - no idle lanes in a row's last, partial chunk - and kFlatUnroll
// consecutive 256-vector spans are in flight per workgroup.

constexpr int kFlatUnroll = 4;
// Read plus written bytes of one hit-gather launch above which the source rows are loaded with the
// non-temporal hint: the chip's last-level cache holds 256 MB; measured on 512-byte rows, 453 MB per
// launch 77.5 -> 72.0 us and 889 MB 159.7 -> 139.2 us with the hint, while launches of 125-180 MB
// lose 5-15 % with it.
constexpr int64_t kStreamingBytes = int64_t(320) << 20;

template <typename VecT, bool STREAM, typename Rows>
__device__ __forceinline__ void copy_rows_flat(const Rows &rows, int64_t n, const char *__restrict__ src,
                                               int64_t src_stride_bytes, char *__restrict__ dst,
                                               int64_t dst_stride_bytes, int vecs, unsigned long long magic, int vb, int nb) {
    const int64_t total = n * vecs;
    const int64_t span = int64_t(kBlock) * kFlatUnroll;
    for (int64_t b0 = int64_t(vb) * span; b0 < total; b0 += int64_t(nb) * span) {
        const VecT *sp[kFlatUnroll];
        VecT *dp[kFlatUnroll];
        bool ok[kFlatUnroll];
        VecT v[kFlatUnroll];
#pragma unroll
        for (int u = 0; u < kFlatUnroll; ++u) {
            const int64_t t = b0 + u * kBlock + threadIdx.x;
            ok[u] = t < total;
            const unsigned long long tc = static_cast<unsigned long long>(ok[u] ? t : total - 1);   // past the end: re-read the last vector
            const int64_t row = static_cast<int64_t>(__umul64hi(tc, magic));
            const int64_t col = static_cast<int64_t>(tc) - row * vecs;
            int64_t srow, drow;
            const bool valid = rows.get(row, &srow, &drow);
            ok[u] = ok[u] && valid;
            sp[u] = reinterpret_cast<const VecT *>(rows.at(srow, src, src_stride_bytes)) + col;
            dp[u] = reinterpret_cast<VecT *>(dst + drow * dst_stride_bytes) + col;
        }
#pragma unroll
        for (int u = 0; u < kFlatUnroll; ++u) v[u] = load_vec<STREAM>(sp[u]);
#pragma unroll
        for (int u = 0; u < kFlatUnroll; ++u)
            if (ok[u]) *dp[u] = v[u];
    }
}

// Rows by a list of (output row, source row) whose length the host knows.
template <typename VecT>
__global__ void __launch_bounds__(kBlock)
k_gather_listed(const int2 *__restrict__ list, int64_t n, const char *__restrict__ src, int64_t src_stride_bytes, char *__restrict__ dst,
                int64_t dst_stride_bytes, int vecs, int log2_lpr, unsigned long long magic, int grid) {
    if (magic) copy_rows_flat<VecT, false>(ListRows{list}, n, src, src_stride_bytes, dst, dst_stride_bytes, vecs, magic, static_cast<int>(blockIdx.x), grid);
    else copy_rows<VecT, false>(ListRows{list}, n, src, src_stride_bytes, dst, dst_stride_bytes, vecs, log2_lpr, static_cast<int>(blockIdx.x), grid);
}

// One side of a gather: entries of a list, copied from src.
struct RowSide {
    const int2 *list;
    const char *src;
    int64_t src_stride_bytes;
    int blocks;                  // workgroups
    int vecs, log2_lpr;
    unsigned long long magic;    // flat copy, see copy_rows_flat; 0: grouped
};
// WHAT: 0 = hits (rows from the HBM cache), 1 = misses (rows from the feature matrix in pinned host memory), 2 = both: the
// workgroups of the misses come first, so that the link is busy from the start, and the hits pass beside them.  (As two
// launches, one after the other: 179 MB over the link and 50 k cached rows of 400 bytes 1,862 us, 1.35 M cached rows and no
// missed ones 268; in one 1,816 and 265.)  The misses' workgroup that ends last, every one having read their number by
// then, sets it to zero: a second half on its own copies nothing.
template <typename VecT, int WHAT>
__global__ void __launch_bounds__(kBlock)
k_gather_rows(RowSide hit, RowSide miss, char *__restrict__ dst, int64_t dst_stride_bytes, unsigned long long *counters) {
    const int b = static_cast<int>(blockIdx.x);
    if (WHAT == 0 || (WHAT == 2 && b >= miss.blocks)) {
        const int vb = WHAT == 0 ? b : b - miss.blocks;
        const int64_t n = static_cast<int64_t>(counters[kCountHits]);
        // a launch that moves more than the last-level cache holds reads its source rows past the caches
        const bool streaming = sizeof(VecT) == 16 && 2 * n * hit.vecs * int64_t(sizeof(VecT)) > kStreamingBytes;
        const ListRows rows{hit.list};
        if (streaming) {                                   // one uniform branch; the copies themselves are straight code
            if (hit.magic) copy_rows_flat<VecT, true>(rows, n, hit.src, hit.src_stride_bytes, dst, dst_stride_bytes, hit.vecs, hit.magic, vb, hit.blocks);
            else copy_rows<VecT, true>(rows, n, hit.src, hit.src_stride_bytes, dst, dst_stride_bytes, hit.vecs, hit.log2_lpr, vb, hit.blocks);
        } else {
            if (hit.magic) copy_rows_flat<VecT, false>(rows, n, hit.src, hit.src_stride_bytes, dst, dst_stride_bytes, hit.vecs, hit.magic, vb, hit.blocks);
            else copy_rows<VecT, false>(rows, n, hit.src, hit.src_stride_bytes, dst, dst_stride_bytes, hit.vecs, hit.log2_lpr, vb, hit.blocks);
        }
        return;
    }
    if (WHAT == 0) return;
    const int64_t n = static_cast<int64_t>(counters[kCountMisses]);
    copy_rows<VecT, false>(ListRows{miss.list}, n, miss.src, miss.src_stride_bytes, dst, dst_stride_bytes, miss.vecs, miss.log2_lpr, b, miss.blocks);
    __syncthreads();                                       // every thread of the workgroup has read the number
    if (threadIdx.x == 0) {
        __threadfence();
        if (atomicAdd(&counters[kCountMissed], 1ull) == static_cast<unsigned long long>(miss.blocks - 1)) {
            counters[kCountMisses] = 0;
            counters[kCountMissed] = 0;
        }
    }
}

// The statistics of a gather without lists: count_blocks workgroups beside the copying ones count the hits and misses, and the one that
// ends last writes them.  (Without a cache, in a recorded graph: 192 workgroups of 64 rows of 256 bytes 4.6 us with a launch for the
// statistics, 5.5 where every copying workgroup counted its own rows, 13 ns for each one's atomic, 3.0 so; 400 k rows 28.3 -> 26.5.)
struct CountLds {
    int hits[kWavesPerBlock], misses[kWavesPerBlock];
};
inline int count_blocks_of(int64_t cap) { return static_cast<int>(std::min<int64_t>(std::max<int64_t>(1, ceil_div(cap, kBlock * 8)), 256)); }
// SLOTS: a hit has a slot; otherwise no id is a hit.
template <bool SLOTS, typename IdxT>
__device__ __forceinline__ void count_ids(const IdxT *__restrict__ ids, int64_t n, const int32_t *__restrict__ slot_of, int64_t num_nodes, int count_blocks,
                                          unsigned long long *counters, int64_t *__restrict__ stats, CountLds &lds) {
    constexpr int U = 4;
    int h = 0, m = 0;
    for (int64_t i0 = int64_t(blockIdx.x) * kBlock + threadIdx.x; i0 < n; i0 += int64_t(count_blocks) * kBlock * U) {
        int64_t id[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = i0 + int64_t(u) * count_blocks * kBlock;
            const int64_t raw = i < n ? static_cast<int64_t>(ids[i]) : -1;
            id[u] = raw >= 0 && raw < num_nodes ? raw : -1;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool hit = SLOTS && id[u] >= 0 && slot_of[id[u]] >= 0;
            h += hit ? 1 : 0;
            m += id[u] >= 0 && !hit ? 1 : 0;
        }
    }
    h = wave_sum(h);
    m = wave_sum(m);
    const int wave = static_cast<int>(threadIdx.x) >> 6;
    if (lane_id() == 0) {
        lds.hits[wave] = h;
        lds.misses[wave] = m;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long th = 0, tm = 0;
#pragma unroll
        for (int w = 0; w < kWavesPerBlock; ++w) {
            th += static_cast<unsigned>(lds.hits[w]);
            tm += static_cast<unsigned>(lds.misses[w]);
        }
        // the common ones and the workgroups in one word; the others, counted before their workgroup is, in another
        const unsigned long long common = SLOTS ? th : tm, rare = SLOTS ? tm : 0;
        if (rare) {
            atomicAdd(&counters[kCountRare], rare);
            __threadfence();
        }
        const unsigned long long mine = common | 1ull << 32, all = atomicAdd(&counters[kCountSplit], mine) + mine;
        if (static_cast<int>(all >> 32) == count_blocks) {
            const int64_t others = SLOTS ? static_cast<int64_t>(atomicExch(&counters[kCountRare], 0ull)) : 0;
            counters[kCountSplit] = 0;
            counters[kCountHits] = SLOTS ? all & 0xFFFFFFFFu : 0;
            counters[kCountMisses] = 0;                    // they are copied
            if (stats) {
                stats[0] = SLOTS ? static_cast<int64_t>(all & 0xFFFFFFFFu) : 0;
                stats[1] = SLOTS ? others : static_cast<int64_t>(all & 0xFFFFFFFFu);
            }
        }
    }
}

// No cache.  The first count_blocks workgroups count.
template <typename VecT, typename IdxT>
__global__ void __launch_bounds__(kBlock)
k_gather_direct(const IdxT *__restrict__ ids, const int64_t *__restrict__ num_ids, int64_t cap, int64_t src_rows,
                const char *__restrict__ src, int64_t src_stride_bytes, char *__restrict__ dst,
                int64_t dst_stride_bytes, int vecs, int log2_lpr, unsigned long long magic, int count_blocks, int copy_blocks,
                unsigned long long *counters, int64_t *__restrict__ stats) {
    __shared__ CountLds lds;
    int64_t n = *num_ids;
    if (n > cap) n = cap;
    const int vb = static_cast<int>(blockIdx.x) - count_blocks;
    if (vb < 0) {
        count_ids<false>(ids, n, nullptr, src_rows, count_blocks, counters, stats, lds);
        return;
    }
    const DirectRows<IdxT> rows{ids, src_rows};
    if (magic) copy_rows_flat<VecT, false>(rows, n, src, src_stride_bytes, dst, dst_stride_bytes, vecs, magic, vb, copy_blocks);
    else copy_rows<VecT, false>(rows, n, src, src_stride_bytes, dst, dst_stride_bytes, vecs, log2_lpr, vb, copy_blocks);
}

// A cache that holds every node: no lists.  A row finds its slot while it is copied, in one launch; the first count_blocks
// workgroups count the hits and misses beside it (as a split and a copy 1.35 M rows of 512 bytes 18 + 247 us, 247 in all; a few thousand rows 14.5 and 8).
template <typename VecT, typename IdxT>
__global__ void __launch_bounds__(kBlock)
k_gather_slots(SlotRows<IdxT> rows, const int64_t *__restrict__ num_ids, int64_t cap, const char *__restrict__ cache, int64_t cache_stride_bytes,
               char *__restrict__ dst, int64_t dst_stride_bytes, int vecs, int log2_lpr, unsigned long long magic, int count_blocks, int copy_blocks,
               unsigned long long *counters, int64_t *__restrict__ stats) {
    __shared__ CountLds lds;
    const int b = static_cast<int>(blockIdx.x);
    int64_t n = *num_ids;
    if (n > cap) n = cap;
    if (b >= count_blocks) {
        const int vb = b - count_blocks;
        const bool streaming = sizeof(VecT) == 16 && 2 * n * vecs * int64_t(sizeof(VecT)) > kStreamingBytes;
        if (streaming) {
            if (magic) copy_rows_flat<VecT, true>(rows, n, cache, cache_stride_bytes, dst, dst_stride_bytes, vecs, magic, vb, copy_blocks);
            else copy_rows<VecT, true>(rows, n, cache, cache_stride_bytes, dst, dst_stride_bytes, vecs, log2_lpr, vb, copy_blocks);
        } else {
            if (magic) copy_rows_flat<VecT, false>(rows, n, cache, cache_stride_bytes, dst, dst_stride_bytes, vecs, magic, vb, copy_blocks);
            else copy_rows<VecT, false>(rows, n, cache, cache_stride_bytes, dst, dst_stride_bytes, vecs, log2_lpr, vb, copy_blocks);
        }
        return;
    }
    count_ids<true>(rows.ids, n, rows.slot_of, rows.num_nodes, count_blocks, counters, stats, lds);
}

// Widest power-of-two access (16, 8, 4 or 2 bytes) that keeps every row of both sides aligned.
int pick_vec_bytes(int64_t row_bytes, int64_t a_stride, int64_t b_stride, const void *a, const void *b) {
    uint64_t bits = static_cast<uint64_t>(row_bytes) | static_cast<uint64_t>(a_stride) | static_cast<uint64_t>(b_stride) |
                    reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b);
    for (int v = 16; v > 2; v >>= 1)
        if ((bits & static_cast<uint64_t>(v - 1)) == 0) return v;
    return 2;
}

// Bytes to move per row.  When both sides keep rows 16-byte aligned and have room for it, the row
// is rounded up to whole 16-byte words so that 128-bit accesses can be used; an HBM-to-HBM copy
// (whole_lines) whose rows are 64-byte aligned on both sides is rounded up to whole 64-byte lines,
// so that no line of the destination is written in part (2,408-byte rows: 47.7 -> 46.7 us).  The
// few bytes past the row that are then copied come from the source row's own padding and land in
// the destination row's own padding.  Copies over the host link move no more than they must.
int64_t copy_bytes(int64_t row_bytes, int64_t a_stride, int64_t b_stride, const void *a, const void *b,
                   bool whole_lines) {
    uint64_t bits = static_cast<uint64_t>(a_stride) | static_cast<uint64_t>(b_stride) |
                    reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b);
    int64_t r64 = (row_bytes + 63) & ~int64_t(63);
    if (whole_lines && (bits & 63) == 0 && r64 <= a_stride && r64 <= b_stride) return r64;
    int64_t r16 = (row_bytes + 15) & ~int64_t(15);
    if ((bits & 15) == 0 && r16 <= a_stride && r16 <= b_stride) return r16;
    return row_bytes;
}

// Geometry of a row-copy launch.
struct RowGeom {
    int vb;          // bytes per vector
    int vecs;        // vectors per row
    int log2_lpr;    // lanes per row group (rows of at most 64 vectors)
    int64_t rows_per_wave;       // rows a wavefront has in flight
    int64_t bytes_per_wave;      // bytes a wavefront has in flight
};

RowGeom row_geom(int64_t row_bytes, int64_t a_stride, int64_t b_stride, const void *a, const void *b) {
    RowGeom g;
    g.vb = pick_vec_bytes(row_bytes, a_stride, b_stride, a, b);
    g.vecs = static_cast<int>(row_bytes / g.vb);
    g.log2_lpr = 0;
    while ((1 << g.log2_lpr) < g.vecs && g.log2_lpr < 6) ++g.log2_lpr;
    if (g.vecs <= kWave) {
        g.rows_per_wave = int64_t(kWave >> g.log2_lpr) * kRowUnroll;
        g.bytes_per_wave = g.rows_per_wave * row_bytes;
    } else {
        g.rows_per_wave = wide_rows(g.vecs);
        g.bytes_per_wave = g.rows_per_wave * std::min<int64_t>(row_bytes, int64_t(wide_chunks(g.vecs)) * kWave * g.vb);
    }
    return g;
}

// HBM-side copies: enough wavefronts to cover the rows, capped at several per SIMD of 256 CUs.
int hbm_grid(int64_t rows, const RowGeom &g) {
    int64_t waves = ceil_div(rows, g.rows_per_wave);
    // measured on "medium": the copy rate stops rising at about 2,048 workgroups
    return static_cast<int>(std::min<int64_t>(std::max<int64_t>(1, ceil_div(waves, kWavesPerBlock)), 256 * 16));
}

// Which HBM-side copies go flat: rows of 2..64 vectors, where the grouped copy leaves lanes idle
// (25 vectors occupy a 32-lane group) and keeps fewer bytes in flight; measured 3.8 -> 5.1 TB/s for
// 400-byte rows, 4.0 -> 5.4 for 256-byte rows, 4.4 -> 5.7 for 512-byte rows.  Longer rows stay with
// the two-rows-at-a-time copy (2,408-byte rows: 49.3 us grouped, 50.1 us flat inside the whole
// step).  Copies over the host link stay grouped too: with 1 MiB of reads outstanding the grouped
// copy is as fast or faster on its own (256-byte rows 54.6 vs 54.2 GB/s flat, 400-byte rows 43.8 vs
// 42.6) and the flat one slows the pipelined step (0.69 -> 0.84 ms per "xlarge" mini-batch).
// Returns ceil(2^64 / vecs), or 0 for the grouped copy.
unsigned long long flat_magic(int64_t rows, const RowGeom &g) {
    if (g.vecs < 2 || g.vecs > kWave || rows * g.vecs >= (int64_t(1) << 32)) return 0;
    return ~0ull / static_cast<unsigned long long>(g.vecs) + 1;
}
// one workgroup per span of 4 x 256 vectors, up to 32 K workgroups (measured: no difference between
// 8 K and 128 K, and between 2, 4 and 8 spans in flight)
int flat_grid(int64_t rows, const RowGeom &g) {
    const int64_t spans = ceil_div(rows * g.vecs, int64_t(kBlock) * kFlatUnroll);
    return static_cast<int>(std::min<int64_t>(std::max<int64_t>(1, spans), 32 * 1024));
}

// Host-link copies: only as many wavefronts as keep `inflight_bytes` of reads outstanding.  The
// link is saturated by little more than a hundred kilobytes in flight; more only queues up in
// the memory system in front of the HBM traffic of whatever runs beside this kernel.
int link_grid(int64_t rows, const RowGeom &g, int64_t inflight_bytes) {
    int64_t waves = std::max<int64_t>(1, ceil_div(inflight_bytes, g.bytes_per_wave));
    int64_t blocks = ceil_div(waves, kWavesPerBlock);
    return static_cast<int>(std::min<int64_t>(blocks, hbm_grid(rows, g)));
}

RowSide row_side(const int2 *list, const void *src, int64_t src_stride_bytes, const void *dst, int64_t dst_stride_bytes, int64_t row_bytes, int64_t cap,
                 bool miss, int64_t inflight_bytes, int *vec_bytes) {
    row_bytes = copy_bytes(row_bytes, src_stride_bytes, dst_stride_bytes, src, dst, !miss);
    const RowGeom g = row_geom(row_bytes, src_stride_bytes, dst_stride_bytes, src, dst);
    RowSide r;
    r.list = list;
    r.src = static_cast<const char *>(src);
    r.src_stride_bytes = src_stride_bytes;
    r.vecs = g.vecs;
    r.log2_lpr = g.log2_lpr;
    r.magic = miss ? 0 : flat_magic(cap, g);
    r.blocks = miss ? link_grid(cap, g, inflight_bytes) : r.magic ? flat_grid(cap, g) : hbm_grid(cap, g);
    *vec_bytes = g.vb;
    return r;
}

template <int WHAT>
int launch_rows(mqg_ctx *ctx, const char *name, int vec_bytes, const RowSide &hit, const RowSide &miss, void *dst, int64_t dst_stride_bytes,
                unsigned long long *counters, hipStream_t s) {
    const int grid = (WHAT != 1 ? hit.blocks : 0) + (WHAT != 0 ? miss.blocks : 0);
    char *dp = static_cast<char *>(dst);
    if (ctx->profile && vec_bytes == 16) {
        // the two kernels the rooflines are quoted on: timed by the dispatch's own start and end
        hipEvent_t e0, e1;
        prof_begin_ext(ctx, name, &e0, &e1);
        hipExtLaunchKernelGGL((k_gather_rows<uint4, WHAT>), dim3(grid), dim3(kBlock), 0, s, e0, e1, 0, hit, miss, dp, dst_stride_bytes, counters);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(ctx, MQG_ERR_HIP, std::string(name) + ": " + hipGetErrorString(e));
        return MQG_OK;
    }
    switch (vec_bytes) {
        case 16: MQG_LAUNCH(ctx, name, s, (k_gather_rows<uint4, WHAT><<<grid, kBlock, 0, s>>>(hit, miss, dp, dst_stride_bytes, counters))); break;
        case 8: MQG_LAUNCH(ctx, name, s, (k_gather_rows<uint2, WHAT><<<grid, kBlock, 0, s>>>(hit, miss, dp, dst_stride_bytes, counters))); break;
        case 4: MQG_LAUNCH(ctx, name, s, (k_gather_rows<uint32_t, WHAT><<<grid, kBlock, 0, s>>>(hit, miss, dp, dst_stride_bytes, counters))); break;
        default: MQG_LAUNCH(ctx, name, s, (k_gather_rows<uint16_t, WHAT><<<grid, kBlock, 0, s>>>(hit, miss, dp, dst_stride_bytes, counters))); break;
    }
    return MQG_OK;
}

// from_host: the source is host memory, so the launch is sized for the link
template <typename IdxT>
int launch_direct(mqg_ctx *ctx, const IdxT *ids, const int64_t *num_ids, int64_t cap, int64_t src_rows, const void *src,
                  int64_t src_stride_bytes, void *dst, int64_t dst_stride_bytes, int64_t row_bytes, bool from_host, int64_t *stats, hipStream_t s) {
    row_bytes = copy_bytes(row_bytes, src_stride_bytes, dst_stride_bytes, src, dst, !from_host);
    const RowGeom g = row_geom(row_bytes, src_stride_bytes, dst_stride_bytes, src, dst);
    int grid = from_host ? link_grid(cap, g, ctx->miss_inflight_bytes) : hbm_grid(cap, g);
    const unsigned long long magic = from_host ? 0 : flat_magic(cap, g);
    if (magic) grid = flat_grid(cap, g);
    const char *sp = static_cast<const char *>(src);
    char *dp = static_cast<char *>(dst);
    const int count_blocks = stats ? count_blocks_of(cap) : 0;
#define MQG_DIRECT(V)                                                                                                                       \
    MQG_LAUNCH(ctx, "k_gather_direct", s,                                                                                                   \
               (k_gather_direct<V, IdxT><<<count_blocks + grid, kBlock, 0, s>>>(ids, num_ids, cap, src_rows, sp, src_stride_bytes, dp, dst_stride_bytes, \
                                                                                g.vecs, g.log2_lpr, magic, count_blocks, grid, ctx->counters, stats)))
    switch (g.vb) {
        case 16: MQG_DIRECT(uint4); break;
        case 8: MQG_DIRECT(uint2); break;
        case 4: MQG_DIRECT(uint32_t); break;
        default: MQG_DIRECT(uint16_t); break;
    }
#undef MQG_DIRECT
    return MQG_OK;
}

// Up to how many ids a gather from a cache that holds every node goes without lists.  There every lane looks up the slot of its own
// vector's row, and the counting workgroups once more: what that costs grows with the vectors, what the lists cost with the ids, and they take a
// launch more.  Rows of 128 bytes and more in 16-byte vectors: always (with and without lists, 1 M rows of 128 bytes 64 and 63 us,
// 2.5 M of 256 290 and 262); narrower ones up to 512 k ids (64 bytes: 500 k ids 30 and 28 us, 1 M 47 and 53, 2.5 M 110 and 132); rows that
// take narrower vectors, or a single one, up to 128 k (300 bytes in 4-byte vectors: 130 k ids 25 and 23 us, 260 k 37 and 41, 2.5 M 414 and 584).
int64_t most_ids_by_slots(const RowGeom &g) {
    if (g.vb < 16 || g.vecs < 2) return int64_t(1) << 17;
    return g.vecs >= 8 ? int64_t(1) << 62 : int64_t(1) << 19;
}

// *done: false if the two sources' rows cannot be copied with the same vectors, or the lists are faster; nothing is launched then.
template <typename IdxT>
int launch_slots(mqg_ctx *ctx, const mqg_cache *c, const IdxT *ids, const int64_t *num_ids, int64_t cap, void *out, int64_t out_stride_bytes,
                 int64_t row_bytes, int64_t elt, int64_t *stats, bool *done, hipStream_t s) {
    const int64_t cs = c->cache_stride * elt, fs = c->feat_stride * elt;
    // whole lines only where the feature matrix would be read no further than its own misses are
    const int64_t feat_bytes = copy_bytes(row_bytes, fs, out_stride_bytes, c->feats, out, false);
    int64_t bytes = copy_bytes(row_bytes, cs, out_stride_bytes, c->cache_rows, out, true);
    if (bytes > feat_bytes) bytes = copy_bytes(row_bytes, cs, out_stride_bytes, c->cache_rows, out, false);
    const RowGeom g = row_geom(bytes, cs, out_stride_bytes, c->cache_rows, out);
    *done = bytes <= feat_bytes && pick_vec_bytes(bytes, fs, out_stride_bytes, c->feats, out) == g.vb && cap <= most_ids_by_slots(g);
    if (!*done) return MQG_OK;
    const unsigned long long magic = flat_magic(cap, g);
    const int copy_blocks = magic ? flat_grid(cap, g) : hbm_grid(cap, g);
    const int count_blocks = stats ? count_blocks_of(cap) : 0;
    const SlotRows<IdxT> rows{ids, c->slot_of, c->num_nodes, static_cast<const char *>(c->feats), fs};
#define MQG_SLOTS(V)                                                                                                                        \
    MQG_LAUNCH(ctx, "k_gather_slots", s,                                                                                                    \
               (k_gather_slots<V, IdxT><<<count_blocks + copy_blocks, kBlock, 0, s>>>(rows, num_ids, cap, static_cast<const char *>(c->cache_rows), cs, \
                                                                                      static_cast<char *>(out), out_stride_bytes, g.vecs, g.log2_lpr,   \
                                                                                      magic, count_blocks, copy_blocks, ctx->counters, stats)))
    switch (g.vb) {
        case 16: MQG_SLOTS(uint4); break;
        case 8: MQG_SLOTS(uint2); break;
        case 4: MQG_SLOTS(uint32_t); break;
        default: MQG_SLOTS(uint16_t); break;
    }
#undef MQG_SLOTS
    return MQG_OK;
}

// Is p host memory (as opposed to memory of a GPU)?  Unknown pointers count as host.
bool is_host_memory(const void *p) {
    hipPointerAttribute_t attr;
    hipError_t e = hipPointerGetAttributes(&attr, p);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    return attr.type != hipMemoryTypeDevice;
}

}  // namespace

// The rows of a list of (output row, source row), every one of them valid, from `src` (used by the cache build to fill the cache).
int gather_listed(mqg_ctx *ctx, const int2 *list, int64_t n, const void *src, int64_t src_stride_bytes, void *dst, int64_t dst_stride_bytes,
                  int64_t row_bytes, hipStream_t s) {
    const bool from_host = is_host_memory(src);
    row_bytes = copy_bytes(row_bytes, src_stride_bytes, dst_stride_bytes, src, dst, !from_host);
    const RowGeom g = row_geom(row_bytes, src_stride_bytes, dst_stride_bytes, src, dst);
    const unsigned long long magic = from_host ? 0 : flat_magic(n, g);
    const int grid = from_host ? link_grid(n, g, ctx->miss_inflight_bytes) : magic ? flat_grid(n, g) : hbm_grid(n, g);
    const char *sp = static_cast<const char *>(src);
    char *dp = static_cast<char *>(dst);
#define MQG_LISTED(V)                                                                                                                       \
    MQG_LAUNCH(ctx, "k_gather_listed", s,                                                                                                   \
               (k_gather_listed<V><<<grid, kBlock, 0, s>>>(list, n, sp, src_stride_bytes, dp, dst_stride_bytes, g.vecs, g.log2_lpr, magic, grid)))
    switch (g.vb) {
        case 16: MQG_LISTED(uint4); break;
        case 8: MQG_LISTED(uint2); break;
        case 4: MQG_LISTED(uint32_t); break;
        default: MQG_LISTED(uint16_t); break;
    }
#undef MQG_LISTED
    return MQG_OK;
}

// Host-side argument checks shared by the gather entry points.  max_ids bounds cap_ids when the
// rows go through the cache (the hit and miss lists hold one entry per id); what_max names it.
int check_gather_args(mqg_ctx *ctx, const mqg_cache *cache, int32_t idx_type, const void *ids_dev,
                      const int64_t *num_ids_dev, int64_t cap_ids, const void *out_dev, int64_t out_stride,
                      int64_t max_ids, const char *what_max) {
    if (!cache || !num_ids_dev) return fail(ctx, MQG_ERR_INVALID_ARG, "mqg_gather_features: NULL cache or num_ids_dev");
    if ((idx_type != MQG_I32 && idx_type != MQG_I64) || (cache->dtype != MQG_F32 && cache->dtype != MQG_F16) || cache->dim < 1)
        return fail(ctx, MQG_ERR_INVALID_ARG, "mqg_gather_features: bad idx_type, dtype or dim");
    if (cap_ids < 0) return fail(ctx, MQG_ERR_INVALID_ARG, "mqg_gather_features: negative cap_ids");
    if (cap_ids > 0 && (!ids_dev || !out_dev)) return fail(ctx, MQG_ERR_INVALID_ARG, "mqg_gather_features: NULL ids or out");
    if (!cache->feats) return fail(ctx, MQG_ERR_INVALID_ARG, "mqg_gather_features: feats is NULL");
    if (out_stride < cache->dim || cache->feat_stride < cache->dim)
        return fail(ctx, MQG_ERR_INVALID_ARG, "mqg_gather_features: stride below dim");
    if (cache->slot_of != nullptr) {
        if (cache->num_cached > 0 && !cache->cache_rows) return fail(ctx, MQG_ERR_INVALID_ARG, "mqg_gather_features: slot_of without cache_rows");
        if (cache->cache_stride < cache->dim) return fail(ctx, MQG_ERR_INVALID_ARG, "mqg_gather_features: cache_stride below dim");
        if (cap_ids > max_ids)
            return fail(ctx, MQG_ERR_CAPACITY, std::string("mqg_gather_features: cap_ids above ") + what_max + " (" +
                        std::to_string(max_ids) + ")");
    } else if (cache->cache_rows) {
        return fail(ctx, MQG_ERR_INVALID_ARG, "mqg_gather_features: cache_rows without slot_of");
    }
    return MQG_OK;
}

// phases: bit 0 = classify the ids and copy the rows found in the cache, bit 1 = copy the others
// from the feature matrix.  Without a cache every row counts as one of the others.
int run_gather(mqg_ctx *ctx, const mqg_cache *c, int32_t idx_type, const void *ids, const int64_t *num_ids,
               int64_t cap_ids, void *out, int64_t out_stride, int64_t *stats, int phases, hipStream_t s) {
    const int64_t elt = c->dtype == MQG_F16 ? 2 : 4;
    const int64_t row_bytes = int64_t(c->dim) * elt;
    if (cap_ids == 0) {
        if (stats && (phases & kGatherMissed)) MQG_LAUNCH(ctx, "k_direct_stats", s, (k_direct_stats<<<1, 64, 0, s>>>(stats)));
        return MQG_OK;
    }

    if (!c->slot_of) {                                   // no cache: everything from feats
        if (!(phases & kGatherMissed)) return MQG_OK;
        const bool from_host = is_host_memory(c->feats);
        if (idx_type == MQG_I64)
            return launch_direct<int64_t>(ctx, static_cast<const int64_t *>(ids), num_ids, cap_ids, c->num_nodes, c->feats, c->feat_stride * elt, out,
                                          out_stride * elt, row_bytes, from_host, stats, s);
        return launch_direct<int32_t>(ctx, static_cast<const int32_t *>(ids), num_ids, cap_ids, c->num_nodes, c->feats, c->feat_stride * elt, out,
                                      out_stride * elt, row_bytes, from_host, stats, s);
    }

    if (phases == (kGatherCached | kGatherMissed) && c->num_cached == c->num_nodes && c->num_nodes > 0 && !ctx->profile) {
        bool done = false;
        const int rc = idx_type == MQG_I64 ? launch_slots(ctx, c, static_cast<const int64_t *>(ids), num_ids, cap_ids, out, out_stride * elt, row_bytes, elt, stats, &done, s)
                                           : launch_slots(ctx, c, static_cast<const int32_t *>(ids), num_ids, cap_ids, out, out_stride * elt, row_bytes, elt, stats, &done, s);
        if (rc != MQG_OK || done) return rc;
    }
    unsigned long long *counters = ctx->counters;
    int hit_vec, miss_vec;
    const RowSide hit = row_side(ctx->hit_list, c->cache_rows, c->cache_stride * elt, out, out_stride * elt, row_bytes, cap_ids, false, 0, &hit_vec);
    const RowSide miss = row_side(ctx->miss_list, c->feats, c->feat_stride * elt, out, out_stride * elt, row_bytes, cap_ids, true,
                                  ctx->miss_inflight_bytes, &miss_vec);
    if (phases & kGatherCached) {
        const int cgrid = static_cast<int>(std::min<int64_t>(std::max<int64_t>(1, ceil_div(cap_ids, cap_ids <= 4 * kClassifySmall ? kBlock : kBlock * 4)), 1024));
#define MQG_CLASSIFY(IT)                                                                                               \
    MQG_LAUNCH(ctx, "k_classify", s,                                                                                   \
               (k_classify<IT><<<cgrid, kBlock, 0, s>>>(static_cast<const IT *>(ids), num_ids, cap_ids, c->slot_of, c->num_nodes, \
                                                        ctx->hit_list, ctx->miss_list, counters, stats, cgrid)))
        if (idx_type == MQG_I64) MQG_CLASSIFY(int64_t);
        else MQG_CLASSIFY(int32_t);
#undef MQG_CLASSIFY
    }
    // both sides in one launch if they move vectors of the same width
    if (phases == (kGatherCached | kGatherMissed) && hit_vec == miss_vec && !ctx->profile)
        return launch_rows<2>(ctx, "k_gather_both", hit_vec, hit, miss, out, out_stride * elt, counters, s);
    if (phases & kGatherCached) {
        int rc = launch_rows<0>(ctx, "k_gather_hit", hit_vec, hit, miss, out, out_stride * elt, counters, s);
        if (rc != MQG_OK) return rc;
    }
    if (phases & kGatherMissed) return launch_rows<1>(ctx, "k_gather_miss", miss_vec, hit, miss, out, out_stride * elt, counters, s);
    return MQG_OK;
}

}  // namespace mqg

// ---- the gather for callers that cannot allocate ------------------------------------------------
//
// mqg_gather_features keeps its hit and miss lists and its counters in a context, and a context is
// hipMalloc'ed.  The entry point below needs no context: the same lists live in a device array of
// fixed size that is part of the code object, so nothing is allocated when it is called (or ever).
// Layout of the array, in 8-byte words: [0, kMax) hit list, [kMax, 2 kMax) miss list, then the
// eight counter words of run_gather.

namespace mqg {
namespace {

constexpr int64_t kStaticMaxIds = MQG_GATHER_STATIC_MAX_IDS;
constexpr int kStaticMaxDevices = 64;

static __device__ __align__(256) unsigned long long scratch[2 * kStaticMaxIds + 8];

// What the host knows about a device's copy of the array: its address there, and a context object
// (host memory only) that points run_gather at it.  Filled at the first call on the device.
struct StaticGather {
    bool ready = false;
    unsigned long long *ptr = nullptr;
    mqg_ctx ctx;
};
StaticGather g_static[kStaticMaxDevices];
std::mutex g_static_mutex;

__global__ void k_clear_words(unsigned long long *p, int n) {
    if (static_cast<int>(threadIdx.x) < n) p[threadIdx.x] = 0;
}

}  // namespace
}  // namespace mqg

extern "C" int mqg_gather_features_static(const mqg_cache *cache, int32_t idx_type, const void *ids_dev,
                                          const int64_t *num_ids_dev, int64_t cap_ids, void *out_dev,
                                          int64_t out_stride, int64_t *stats_dev, mqg_stream stream) {
    using namespace mqg;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(nullptr, MQG_ERR_HIP, std::string("mqg_gather_features_static: hipGetDevice: ") + hipGetErrorString(e));
    if (dev < 0 || dev >= kStaticMaxDevices)
        return fail(nullptr, MQG_ERR_UNSUPPORTED, "mqg_gather_features_static: device index above 63");
    StaticGather &sg = g_static[dev];
    {
        std::lock_guard<std::mutex> lock(g_static_mutex);
        if (!sg.ready) {
            // `scratch` is a host-side stand-in here; the device's copy of the array is at the
            // address this call returns, with that device current
            void *p = nullptr;
            e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
            if (e != hipSuccess || !p)
                return fail(nullptr, MQG_ERR_HIP, std::string("mqg_gather_features_static: hipGetSymbolAddress: ") + hipGetErrorString(e));
            sg.ptr = static_cast<unsigned long long *>(p);
            sg.ctx.device = dev;
            sg.ctx.max_src = kStaticMaxIds;
            sg.ctx.hit_list = reinterpret_cast<int2 *>(sg.ptr);
            sg.ctx.miss_list = reinterpret_cast<int2 *>(sg.ptr + kStaticMaxIds);
            sg.ctx.counters = sg.ptr + 2 * kStaticMaxIds;
            sg.ready = true;
        }
    }
    mqg_ctx *ctx = &sg.ctx;
    int rc = check_gather_args(ctx, cache, idx_type, ids_dev, num_ids_dev, cap_ids, out_dev, out_stride, kStaticMaxIds,
                               "MQG_GATHER_STATIC_MAX_IDS");
    if (rc == MQG_OK) {
        hipStream_t s = static_cast<hipStream_t>(stream);
        // the array keeps what the last call left; the counters have to start at zero (a fill
        // kernel rather than a memset, so that the call can also be recorded into a graph)
        if (cap_ids > 0) {
            k_clear_words<<<1, 64, 0, s>>>(ctx->counters, 8);
            e = hipGetLastError();
            if (e != hipSuccess) return fail(nullptr, MQG_ERR_HIP, std::string("mqg_gather_features_static: k_clear_words: ") + hipGetErrorString(e));
        }
        rc = run_gather(ctx, cache, idx_type, ids_dev, num_ids_dev, cap_ids, out_dev, out_stride, stats_dev, kGatherCached | kGatherMissed, s);
    }
    if (rc != MQG_OK) return fail(nullptr, rc, ctx->last_error);      // no context handle: the message goes where mqg_last_error(NULL) reads
    return MQG_OK;
}
