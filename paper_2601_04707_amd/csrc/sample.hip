// L-hop fixed-fanout neighbour sampling into bipartite blocks (paper Sec. III-A, GraphSAGE
// paragraph; block layout after Sec. IV "Mini-Batch Transfer To GPU" and Eq. 16).
//
// Per block, outward from the seeds (two or three launches, four on graphs of more than 3 M nodes; the first block's row
// information is a launch of its own there, for many seeds and for a single block, otherwise part of its k_sample):
//   row info       adjacency start/degree of every destination, copy of the destinations into the
//                  block's source list, per-tile sums of min(fanout, degree), list of the hubs
//   k_sample       a wavefront takes destinations one by one: smallest-k random keys, then for a few
//                  destinations together the neighbours, written in ascending adjacency slot at
//                  row * fanout (no offsets needed yet), first-seen nodes marked in an N-bit bitmap
//                  (destinations whose degree exceeds heavy_degree are taken by whole workgroups in the
//                  same launch, so that a hub's key evaluation is spread over four wavefronts instead of
//                  stretching the kernel's tail); workgroups of their own relabel the block before meanwhile, copy its
//                  sources, which are this block's destinations, into this block's source list and add up the row tiles
//   k_offsets_count  two independent jobs in one launch: indptr from the row tile sums (every
//                  workgroup adds up the sums of the tiles before its own; only above 8,192 tiles
//                  does one k_scan_tiles launch scan them first) and the popcount of every tile
//                  of the bitmap
//   k_bitmap_emit  popcount-rank the bitmap: new source nodes come out ascending by id, get their
//                  position recorded in local_of[], the bitmap is cleared on the way; the new sources' row information
//                  for the next block outward, whose destinations they are, is recorded with them
//   k_emit_offsets  graphs of up to half a million nodes: the two launches above in one - every
//                  tile's workgroup counts the bits of the tiles before its own itself (the relabel
//                  clears the bitmap then, while the next block is marked in another)
//   k_relabel      indices[indptr[row] + j] = local_of[neighbour j of row] of the outermost block
//   k_relabel_rowinfo  graphs of more than 3 M nodes: that of every other block, and in the same
//                  launch the row information of the next block outward
// The hash-table dedup (an option) keeps the older order: offsets first, neighbours written compactly.
// All sizes that depend on the data stay on the device; grids are sized by worst-case bounds.
#include <type_traits>

#include "common.h"
#include "device_utils.h"

namespace mqg {

namespace {

constexpr uint64_t kGolden = 0x9E3779B97F4A7C15ULL;
constexpr uint64_t kMaxKey = ~uint64_t(0);
constexpr int kBusyWaves = 8192;          // wavefronts that the chip runs at once: 256 CUs x 4 SIMDs x 8
constexpr int kBatchRows = 8;             // destinations per wavefront and batch in k_sample, at most
constexpr int kHubBlocks = 2048;          // workgroups for the hubs, at most
constexpr int kSeedRows = 2 * kBusyWaves; // seeds below this are sampled without row information of an earlier launch, see RowSource
static_assert(kSeedRows <= kWave * kHubBlocks, "a workgroup's seeds fit its lanes");

uint64_t host_mix64(uint64_t z) {
    z ^= z >> 30;
    z *= 0xBF58476D1CE4E5B9ULL;
    z ^= z >> 27;
    z *= 0x94D049BB133111EBULL;
    z ^= z >> 31;
    return z;
}

// ------------------------------------------------------------------------------------------

// Destinations of more than heavy_degree slots, hubs, are listed for the sampling kernels.
struct HubList {
    int32_t *rows;
    int32_t *count;
    int heavy_degree;
    // places for what the threads of a workgroup have (all call it; lds as for block_excl_scan): one atomic per workgroup that has any
    // (one per wavefront queued up at the counter: the row information of 295 k destinations 32 -> 21 us, of 43 k 10.2 -> 5.7 us)
    __device__ __forceinline__ int take(int mine, int *lds) const {
        int total;
        const int ex = block_excl_scan<kWavesPerBlock>(mine, &total, lds);
        if (total == 0) return 0;                          // workgroup-uniform
        __syncthreads();
        if (threadIdx.x == 0) lds[0] = atomicAdd(count, total);
        __syncthreads();
        return lds[0] + ex;
    }
};

// the last launch of a call: counts and seed flags back to zero for the next one
__device__ __forceinline__ void clear_hubs(int32_t *__restrict__ hub_count) {
    if (threadIdx.x <= MQG_MAX_LAYERS) hub_count[threadIdx.x] = 0;
}

// Arguments of the row-information step of one block.
template <typename PtrT, typename IdxT>
struct RowInfoArgs {
    const PtrT *row_ptr;
    const IdxT *dst;             // the block's destinations (the caller's seeds, or the previous block's sources)
    const int64_t *sizes;        // this block's sizes: [0] = number of destinations (unless n_seeds >= 0)
    IdxT *src_out;
    int fanout;
    int64_t *row_start;
    int32_t *row_deg;
    int32_t *tile_sums;
    int64_t *sizes_rw;
    HubList hubs;
    int64_t n_seeds;             // >= 0: innermost block
    int32_t *local_of;
    int32_t pos_base;            // see take_positions
    int64_t num_nodes;
    int32_t *seed_flags;
};

// LIST: hubs are listed, too.  seed_bits not null: a bit is set for every seed, too.
template <bool LIST, typename PtrT, typename IdxT>
__device__ __forceinline__ void row_info_tile(const RowInfoArgs<PtrT, IdxT> &a, int tile, int *lds, uint32_t *seed_bits = nullptr) {
    // innermost block (n_seeds >= 0): the destinations are the caller's seeds; their number comes
    // from the host and their positions are entered into local_of here
    const int64_t n = a.n_seeds >= 0 ? a.n_seeds : a.sizes[0];
    const int64_t i = int64_t(tile) * kBlock + threadIdx.x;
    int cnt = 0;
    int64_t d = 0;
    if (i < n) {
        IdxT v = a.dst[i];
        if (a.n_seeds >= 0) {
            // caller-supplied ids: an id outside the graph is flagged and replaced by node 0, so that
            // nothing downstream ever indexes with it; a repeated id is flagged (its rows are kept and
            // share one position in the source lists)
            if (v < 0 || static_cast<int64_t>(v) >= a.num_nodes) {
                v = 0;
                atomicOr(a.seed_flags, 1);
            }
            if (a.local_of && atomicMax(&a.local_of[v], a.pos_base + static_cast<int32_t>(i)) >= a.pos_base) atomicOr(a.seed_flags, 2);
            if (seed_bits) (void)atomicOr(&seed_bits[v >> 5], 1u << (v & 31));
        }
        int64_t s = static_cast<int64_t>(a.row_ptr[v]);
        d = static_cast<int64_t>(a.row_ptr[v + 1]) - s;
        a.row_start[i] = s;
        a.row_deg[i] = static_cast<int32_t>(d);
        a.src_out[i] = v;
        cnt = d < a.fanout ? static_cast<int>(d) : a.fanout;
    }
    const int w = wave_sum(cnt);
    if (lane_id() == 0) lds[threadIdx.x >> 6] = w;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
#pragma unroll
        for (int k = 0; k < kWavesPerBlock; ++k) t += lds[k];
        a.tile_sums[tile] = t;
        if (tile == 0 && a.n_seeds >= 0) a.sizes_rw[0] = a.n_seeds;
    }
    if constexpr (LIST) {
        const bool hub = i < n && d > a.hubs.heavy_degree;
        const int place = a.hubs.take(hub ? 1 : 0, lds);
        if (hub) a.hubs.rows[place] = static_cast<int32_t>(i);
    }
}

// What the sampling of the next block needs of its new destinations, recorded as they are listed: their adjacency, and
// which of them are hubs.  row_ptr null: there is no next block.
template <typename PtrT>
struct NewRows {
    const PtrT *row_ptr;
    int64_t *row_start;
    int32_t *row_deg;
    HubList hubs;
};

template <typename PtrT, typename IdxT>
__global__ void __launch_bounds__(kBlock)
k_row_info(RowInfoArgs<PtrT, IdxT> a) {
    __shared__ int lds[kWavesPerBlock];
    row_info_tile<true>(a, static_cast<int>(blockIdx.x), lds);
}

// One workgroup of 1024 threads: vals[0..n) -> exclusive scan in place; totals, `most` at most, stored.
__global__ void __launch_bounds__(1024)
k_scan_tiles(int32_t *__restrict__ vals, int64_t n, const int64_t *__restrict__ addend,
             int64_t *__restrict__ total_a, int64_t *__restrict__ total_b, int64_t most) {
    __shared__ int lds[16];
    int64_t carry = 0;
    for (int64_t base = 0; base < n; base += 1024) {
        int64_t i = base + threadIdx.x;
        int v = i < n ? vals[i] : 0;
        int total;
        int ex = block_excl_scan<16>(v, &total, lds);
        if (i < n) vals[i] = static_cast<int32_t>(carry + ex);
        carry += total;
    }
    if (threadIdx.x == 0) {
        int64_t t = carry + (addend ? *addend : 0);
        t = t < most ? t : most;
        if (total_a) *total_a = t;
        if (total_b) *total_b = t;
    }
}

// scanned: tile_vals holds the exclusive scan of the tile sums (k_scan_tiles ran, and stored nnz);
// otherwise it holds the sums themselves, every workgroup adds up its own base and the last one
// stores nnz.
__device__ __forceinline__ void row_offsets_tile(const int32_t *__restrict__ row_deg, int fanout, int64_t *sizes,
                                                 const int32_t *__restrict__ tile_vals, int scanned,
                                                 int32_t *__restrict__ indptr, const int32_t *__restrict__ seed_flags,
                                                 int tile, int ntiles, int *lds) {
    const int64_t n = sizes[0];
    // the block's flags word: what the seed check found (innermost block), 0 otherwise
    if (tile == 0 && threadIdx.x == 0) sizes[3] = seed_flags ? *seed_flags : 0;
    const int tile_base = scanned ? tile_vals[tile] : tiles_before(tile_vals, lds, tile);
    const int64_t i = int64_t(tile) * kBlock + threadIdx.x;
    int cnt = 0;
    if (i < n) {
        int d = row_deg[i];
        cnt = d < fanout ? d : fanout;
    }
    int total;
    int ex = block_excl_scan<kWavesPerBlock>(cnt, &total, lds);
    int off = tile_base + ex;
    if (i < n) {
        indptr[i] = off;
        if (i == n - 1) indptr[n] = off + cnt;
    }
    if (n == 0 && i == 0) indptr[0] = 0;
    if (!scanned && tile == ntiles - 1 && threadIdx.x == 0) sizes[2] = tile_base + total;
}

__global__ void __launch_bounds__(kBlock)
k_row_offsets(const int32_t *__restrict__ row_deg, int fanout, int64_t *sizes,
              const int32_t *__restrict__ tile_vals, int scanned, int32_t *__restrict__ indptr,
              const int32_t *__restrict__ seed_flags) {
    __shared__ int lds[kWavesPerBlock];
    row_offsets_tile(row_deg, fanout, sizes, tile_vals, scanned, indptr, seed_flags, static_cast<int>(blockIdx.x),
                     static_cast<int>(gridDim.x), lds);
}

// ------------------------------------------------------------------------------------------

// Neighbour j of row r sits at nbr[r * fanout + j]; its edge position is indptr[r] + j.  Workgroups
// vb of nb walk the num_dst * fanout slots.
__device__ __forceinline__ void relabel_slots(const int32_t *__restrict__ nbr, const int64_t *__restrict__ sizes,
                                              const int32_t *__restrict__ indptr, int fanout,
                                              const int32_t *__restrict__ local_of, int32_t pos_base, int32_t *__restrict__ indices, int vb, int nb) {
    const uint32_t total = static_cast<uint32_t>(sizes[0] * fanout);
    const uint32_t stride = static_cast<uint32_t>(nb) * kBlock;
    for (uint64_t t64 = uint64_t(vb) * kBlock + threadIdx.x; t64 < total; t64 += stride) {
        const uint32_t t = static_cast<uint32_t>(t64);
        const uint32_t row = t / static_cast<uint32_t>(fanout);
        const int j = static_cast<int>(t - row * static_cast<uint32_t>(fanout));
        const int b = indptr[row];
        if (j < indptr[row + 1] - b) {
            const int32_t u = nbr[t];
            const int32_t p = u < 0 ? ~u : local_of[u] - pos_base;
            indices[b + j] = p < 0 ? 0 : p;                // below 0: left out of the sources, see store_num_src
        }
    }
}

// (clear: the frontier bitmap, when the emit launch left its words set; vb of nb workgroups)
__device__ __forceinline__ void clear_words(uint32_t *__restrict__ clear, int64_t clear_words, int vb, int nb) {
    if (!clear) return;
    for (int64_t w = int64_t(vb) * kBlock + threadIdx.x; w < clear_words; w += int64_t(nb) * kBlock) clear[w] = 0;
}

// What the launch that samples a block does beside that, in workgroups of its own: the relabel of the block before, whose
// sources are this block's destinations, their copy into this block's source list, and the sums of the rows' tiles.
// (In a launch of its own before this one: 4 us of a batch of 1,024 seeds' 54, 25 of 8,192 seeds' 253.)
template <typename IdxT>
struct SideWork {
    int relabel_blocks, row_tiles;                         // workgroups; both 0: nothing to do
    const int32_t *nbr;                                    // of the block before
    const int64_t *sizes;
    const int32_t *indptr;
    int fanout;
    const int32_t *local_of;
    int32_t pos_base;
    int32_t *indices;
    uint32_t *clear;
    int64_t nclear;
    uint32_t *seed_bits;                                   // not null: the block before is the innermost; its seeds' bits are set back
    const IdxT *dst;                                       // this block's destinations: the block before's sources
    const int64_t *dst_count;
    const int32_t *row_deg;
    int row_fanout;                                        // this block's
    IdxT *src_out;
    int32_t *tile_sums;
};

template <typename IdxT>
__device__ __forceinline__ void side_work(const SideWork<IdxT> &w, int b, int *lds) {
    if (b < w.relabel_blocks) {
        clear_words(w.clear, w.nclear, b, w.relabel_blocks);
        if (w.seed_bits)
            for (int64_t i = int64_t(b) * kBlock + threadIdx.x; i < w.sizes[0]; i += int64_t(w.relabel_blocks) * kBlock) w.seed_bits[w.dst[i] >> 5] = 0;
        relabel_slots(w.nbr, w.sizes, w.indptr, w.fanout, w.local_of, w.pos_base, w.indices, b, w.relabel_blocks);
        return;
    }
    const int tile = b - w.relabel_blocks;
    const int64_t n = *w.dst_count;
    const int64_t i = int64_t(tile) * kBlock + threadIdx.x;
    int cnt = 0;
    if (i < n) {
        const int d = w.row_deg[i];
        w.src_out[i] = w.dst[i];
        cnt = d < w.row_fanout ? d : w.row_fanout;
    }
    cnt = wave_sum(cnt);
    if (lane_id() == 0) lds[threadIdx.x >> 6] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
#pragma unroll
        for (int k = 0; k < kWavesPerBlock; ++k) t += lds[k];
        w.tile_sums[tile] = t;
    }
}

// ------------------------------------------------------------------------------------------
// Neighbour selection.  A wavefront takes destinations one by one, a workgroup the hubs.

struct SampleArgs {
    const int64_t *row_start; // (the seeds' own launch: see RowSource)
    const int32_t *row_deg;
    const int32_t *indptr;    // null: row r's neighbours go to nbr[r * fanout ...) and are compacted by the relabel
    const int64_t *sizes;
    int32_t *nbr;
    const int32_t *local_of;  // null: no position is looked up
    int32_t pos_base;
    uint32_t *bitmap;         // null: no mark is set (the hash path dedups)
    uint64_t layer_hash;      // mix(mix(rng_seed + golden) ^ block index), used when seed_dev is null
    const uint64_t *seed_dev; // the sampling seed in device memory (calls recorded into a HIP graph)
    int layer;                // block index, for seed_dev
    int fanout;
    int force_slow;
    int heavy_degree;         // rows longer than this are sampled by whole workgroups
};

__device__ __forceinline__ int32_t out_base_of(const SampleArgs &a, int64_t row) {
    return a.indptr ? a.indptr[row] : static_cast<int32_t>(row * a.fanout);
}

__device__ __forceinline__ uint64_t layer_hash_of(const SampleArgs &a) {
    if (!a.seed_dev) return a.layer_hash;
    return mix64(mix64(*a.seed_dev + 0x9E3779B97F4A7C15ULL) ^ static_cast<uint64_t>(a.layer));
}

// The neighbour's id goes to nbr, or, if it is one of the block's destinations, the complement of its position: the
// relabel then has no position to look up (a third of the edges of large batches; the relabel of 4.3 M edges 43 -> 28 us).
template <typename IdxT>
__device__ __forceinline__ void emit_neighbour(const IdxT *__restrict__ col_idx, int64_t start, int slot,
                                               int32_t out_pos, const SampleArgs &a) {
    int32_t u = static_cast<int32_t>(col_idx[start + slot]);
    const int32_t p = a.local_of ? a.local_of[u] - a.pos_base : -1;
    if (p >= 0) {
        u = ~p;
    } else if (a.bitmap) {
        uint32_t bit = 1u << (u & 31);
        uint32_t *w = a.bitmap + (u >> 5);
        (void)__hip_atomic_fetch_or(w, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    a.nbr[out_pos] = u;
}

// The same for a wavefront that has one neighbour per lane after the other, in two steps that overlap with what it does in
// between: the id is loaded when it is pushed, its position at the next push, and the one after that stores it.
template <typename IdxT>
struct NeighbourPipe {
    const SampleArgs &a;
    bool in1 = false, in2 = false;
    int32_t out1 = 0, out2 = 0, u2 = 0, p2 = -1;
    IdxT u1 = 0;
    __device__ __forceinline__ explicit NeighbourPipe(const SampleArgs &args) : a(args) {}
    __device__ __forceinline__ void advance() {
        if (in2) {
            int32_t u = u2;
            if (p2 >= a.pos_base) u = ~(p2 - a.pos_base);
            else if (a.bitmap) (void)__hip_atomic_fetch_or(a.bitmap + (u >> 5), 1u << (u & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            a.nbr[out2] = u;
        }
        in2 = in1;
        out2 = out1;
        u2 = static_cast<int32_t>(u1);
        p2 = -1;
        if (a.local_of && in2) p2 = a.local_of[u2];
    }
    __device__ __forceinline__ void push(const IdxT *__restrict__ col_idx, bool in, int64_t pos, int32_t out) {
        advance();
        in1 = in;
        out1 = out;
        if (in) u1 = col_idx[pos];
    }
    __device__ __forceinline__ void drain() {
        advance();
        in1 = false;
        advance();
    }
};

// Where a sampling launch takes its rows' adjacency from: recorded by a launch before, or, SEEDS, the innermost block of
// graphs of few bitmap tiles, from the seeds themselves, while workgroups of their own record it (a launch of its own for that: 4 us of
// the 54 of a call for 1,024 seeds, one launch of nine).  The seeds' positions are not known meanwhile: all neighbours are marked, and the launch
// that lists the new sources leaves out the seeds, which have a bitmap of their own.
template <typename PtrT, typename IdxT, bool SEEDS>
struct RowSource {
    const SampleArgs &a;
    const IdxT *dst;
    const RowInfoArgs<PtrT, IdxT> &seeds;
    __device__ __forceinline__ void row(int64_t r, int64_t &start, int &deg, IdxT &node) const {
        if constexpr (SEEDS) {
            IdxT v = seeds.dst[r];
            if (v < 0 || static_cast<int64_t>(v) >= seeds.num_nodes) v = 0;
            start = static_cast<int64_t>(seeds.row_ptr[v]);
            deg = static_cast<int>(static_cast<int64_t>(seeds.row_ptr[v + 1]) - start);
            node = v;
        } else {
            start = a.row_start[r];
            deg = a.row_deg[r];
            node = dst[r];
        }
    }
};

// A candidate: the upper 31 bits of its key and its slot.
struct alignas(8) Candidate {
    uint32_t word;
    int32_t slot;
};

// The distance of a row's keys on average, in upper 31 bits.
__device__ __forceinline__ uint32_t key_gap(int d) {
    const float g = 2147483648.0f * __builtin_amdgcn_rcpf(static_cast<float>(d));
    return g >= 1.0f ? static_cast<uint32_t>(g < 2147483520.0f ? g : 2147483520.0f) : 1u;
}
// About `expect` of the d slots have keys whose upper 31 bits lie below this.
__device__ __forceinline__ uint32_t key_limit(int expect, int d, uint32_t gap) {
    return d <= expect ? kNoWord : static_cast<uint32_t>(expect) * gap;
}

// The slots of a row of d whose keys lie below limit, as candidates in `out` in slot order; returns their number (more than
// the list's `cap`, a power of two: not all are there).  row_candidates: of a row of up to 2^30.  hub_candidates: a wavefront's
// share of a long row, every fourth part of CHUNKS * 64 slots, most of which have few candidates or none in 64.
constexpr int kHubChunks = 4;
constexpr int kHubChunksFrom = 16 * kHubChunks * kWave;    // slots, four parts per wavefront; of shorter rows one would hold too large a share (2,300 slots 99 -> 106 us)
template <bool EMPTY>
__device__ __forceinline__ void keep_candidates(uint32_t z, int slot, bool c, Candidate *out, int cap, int &cnt) {
    const uint64_t m = ballot64(c);
    if (EMPTY && !m) return;
    if (c) out[rank_below(m, cnt) & (cap - 1)] = Candidate{z >> 1, slot};
    cnt += popc64(m);
}
__device__ __forceinline__ int row_candidates(uint32_t low, uint32_t hi_term, int d, uint32_t limit, Candidate *out, int cap) {
    const uint32_t above = limit << 1;                     // of the whole upper word, whose bit 0 is not known yet
    const WaveKeys<1> keys(low, hi_term);
    int cnt = 0, slot = lane_id(), base = 0;
    for (; base + kWave <= d; base += kWave, slot += kWave) {
        const uint32_t z = keys.upper(keys.row_part(base));
        keep_candidates<false>(z, slot, z < above, out, cap, cnt);
    }
    if (base < d) {
        const uint32_t z = keys.upper(keys.row_part(base));
        keep_candidates<false>(z, slot, z < above && slot < d, out, cap, cnt);
    }
    return cnt;
}
template <int CHUNKS>
__device__ __forceinline__ int hub_candidates(uint64_t hv, int d, uint32_t limit, int wave, Candidate *out, int cap) {
    constexpr uint32_t kPart = CHUNKS * kWave, kStride = kPart * kWavesPerBlock;
    const uint32_t above = limit << 1;
    const int lane = lane_id();
    int cnt = 0;
    for (uint32_t range = 0; range < static_cast<uint32_t>(d); range += 0x40000000u) {
        const WaveKeys<CHUNKS> keys(__builtin_amdgcn_readfirstlane(key_low(hv, range)), __builtin_amdgcn_readfirstlane(key_hi_term(hv)));
        const uint32_t end = static_cast<uint32_t>(d) - range < 0x40000000u ? static_cast<uint32_t>(d) : range + 0x40000000u;
        uint32_t base = range + wave * kPart;
        for (; base + kPart <= end; base += kStride) {
            const uint64_t part = keys.row_part(base);
            uint32_t z[CHUNKS];
#pragma unroll
            for (int u = 0; u < CHUNKS; ++u) z[u] = keys.upper(part, u);
#pragma unroll
            for (int u = 0; u < CHUNKS; ++u)
                keep_candidates<true>(z[u], static_cast<int>(base + u * kWave) + lane, z[u] < above, out, cap, cnt);
        }
        if (base < end) {
            const uint64_t part = keys.row_part(base);
#pragma unroll
            for (int u = 0; u < CHUNKS; ++u) {
                if (base + u * kWave >= end) break;
                const uint32_t z = keys.upper(part, u);
                keep_candidates<true>(z, static_cast<int>(base + u * kWave) + lane, z < above && base + u * kWave + lane < end, out, cap, cnt);
            }
        }
    }
    return cnt;
}

// The chosen of candidates that are in no particular order: their slots are listed in sel_slot (LDS, 64
// entries) and emitted in ascending order.
template <int NCH, typename IdxT>
__device__ __forceinline__ void emit_by_slot(const uint32_t (&slot)[NCH], const uint64_t (&sel)[NCH], int k, int32_t *sel_slot,
                                             const IdxT *__restrict__ col_idx, int64_t start, int32_t out_base, const SampleArgs &a) {
    const int lane = lane_id();
    int pos = 0;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        if ((sel[c] >> lane) & 1) sel_slot[pos + popc64(sel[c] & lanes_below(lane))] = static_cast<int32_t>(slot[c] & 0x7FFFFFFFu);
        pos += popc64(sel[c]);
    }
    wave_lds_sync();
    const int my_slot = lane < k ? sel_slot[lane] : 0x7FFFFFFF;
    int rank = 0;
    for (int t = 0; t < k; ++t) {
        int other = static_cast<int>(readlane32(static_cast<uint32_t>(my_slot), t));
        rank += (other < my_slot) ? 1 : 0;
    }
    if (lane < k) emit_neighbour(col_idx, start, my_slot, out_base + rank, a);
}

// ------------------------------------------------------------------------------------------
// Cache-prioritised selection (the paper's Sec. I on global neighbour sampling: neighbours that are
// in the feature cache are preferred, so that fewer distinct uncached rows enter a mini-batch).
// The k slots of a row are the first k in the order (not cached, key, slot): with c cached
// neighbours the row keeps min(k, c) of them, drawn uniformly, and fills up from the uncached ones,
// drawn uniformly.  `prio` is a bitmap over the nodes, bit set = cached; prio_count tabulates c.
struct PrioArgs {
    const uint32_t *prio;
    const int32_t *prio_count;
};

template <typename IdxT>
__device__ __forceinline__ bool is_cached(const IdxT *__restrict__ row, int j, const uint32_t *__restrict__ prio) {
    const uint32_t u = static_cast<uint32_t>(row[j]);
    return (prio[u >> 5] >> (u & 31)) & 1u;
}

// lexicographic (key, slot) order
__device__ __forceinline__ bool pair_less(uint64_t ka, int sa, uint64_t kb, int sb) {
    return ka < kb || (ka == kb && sa < sb);
}

// Unconditional selection among d: k rounds, each finding the smallest (key, index) pair above the previous round's,
// whose index it takes: take(round, index).  O(k*d/64) key evaluations.
template <typename KeyAt, typename Take>
__device__ __forceinline__ void take_one_by_one(int d, int k, const KeyAt &key_at, const Take &take) {
    uint64_t prev_key = 0;
    int prev_slot = -1;
    for (int r = 0; r < k; ++r) {
        uint64_t best_key = kMaxKey;
        int best_slot = 0x7FFFFFFF;
        uint32_t next = lane_id();
        for (int left = d; left > 0; left -= kWave, next += kWave) {
            if (lane_id() < left) {
                const int j = static_cast<int>(next);
                const uint64_t key = key_at(j);
                const bool above = (r == 0) || pair_less(prev_key, prev_slot, key, j);
                if (above && pair_less(key, j, best_key, best_slot)) {
                    best_key = key;
                    best_slot = j;
                }
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const uint64_t ok = __shfl_xor(best_key, off, 64);
            const int os = __shfl_xor(best_slot, off, 64);
            if (pair_less(ok, os, best_key, best_slot)) {
                best_key = ok;
                best_slot = os;
            }
        }
        prev_key = best_key;
        prev_slot = best_slot;
        take(r, best_slot);
    }
}

__device__ __forceinline__ bool prio_less(bool ua, uint64_t ka, int sa, bool ub, uint64_t kb, int sb) {
    return ua != ub ? !ua : pair_less(ka, sa, kb, sb);
}

// The same in the (late, key, index) order.
template <typename KeyAt, typename LateAt, typename Take>
__device__ __forceinline__ void take_one_by_one_prio(int d, int k, const KeyAt &key_at, const LateAt &late_at, const Take &take) {
    bool prev_late = false;
    uint64_t prev_key = 0;
    int prev_slot = -1;
    for (int r = 0; r < k; ++r) {
        bool best_late = true;
        uint64_t best_key = kMaxKey;
        int best_slot = 0x7FFFFFFF;
        uint32_t next = lane_id();
        for (int left = d; left > 0; left -= kWave, next += kWave) {
            if (lane_id() < left) {
                const int j = static_cast<int>(next);
                const uint64_t key = key_at(j);
                const bool late = late_at(j);
                const bool above = (r == 0) || prio_less(prev_late, prev_key, prev_slot, late, key, j);
                if (above && prio_less(late, key, j, best_late, best_key, best_slot)) {
                    best_late = late;
                    best_key = key;
                    best_slot = j;
                }
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const uint64_t ok = __shfl_xor(best_key, off, 64);
            const int os = __shfl_xor(best_slot, off, 64);
            const bool ol = __shfl_xor(static_cast<int>(best_late), off, 64) != 0;
            if (prio_less(ol, ok, os, best_late, best_key, best_slot)) {
                best_late = ol;
                best_key = ok;
                best_slot = os;
            }
        }
        prev_late = best_late;
        prev_key = best_key;
        prev_slot = best_slot;
        take(r, best_slot);
    }
}

// A row's k slots one by one, where the faster selections found no bound or too many or too few candidates, and in tests.
template <bool PRIO, typename IdxT>
__device__ void select_by_repeated_min(const IdxT *__restrict__ col_idx, int64_t start, int d, int k, uint64_t hv,
                                       int32_t out_base, const SampleArgs &a, const uint32_t *__restrict__ prio) {
    const int lane = lane_id();
    const RowKeys key_of(hv);
    const IdxT *row = col_idx + start;
    int my_slot = -1;                                // lane r keeps the r-th selected slot
    auto take = [&](int r, int slot) { if (lane == r) my_slot = slot; };
    if constexpr (PRIO) take_one_by_one_prio(d, k, key_of, [&](int j) { return !is_cached(row, j, prio); }, take);
    else take_one_by_one(d, k, key_of, take);
    // order the k chosen slots ascending
    int rank = 0;
    for (int t = 0; t < k; ++t) {
        int other = static_cast<int>(readlane32(static_cast<uint32_t>(my_slot), t));
        rank += (other < my_slot) ? 1 : 0;
    }
    if (lane < k) emit_neighbour(col_idx, start, my_slot, out_base + rank, a);
}

// Which of a row's d slots compete for how many of its k places: without priority all of them; with at least k cached
// ones these, and only they are looked for; otherwise the uncached ones, for what the cached ones leave.
struct Contest {
    bool cached;                 // the competing slots are the cached ones
    int want, pool;              // places and competitors
    __device__ __forceinline__ Contest(bool prio, int d, int k, int c) {
        cached = prio && c >= k;
        want = prio && !cached ? k - c : k;
        pool = !prio ? d : cached ? c : d - c;
    }
};

// (Every slot was looked up, by k_sample's rules before: a mini-batch of 8,192 seeds on 300 k nodes of 300 neighbours, one in five cached,
// 536 -> 272 us, of 1,024 on 1 M nodes of 50 267 -> 133: the keys are cheap, a look-up is two dependent random accesses.)
// Candidates of a row with cached neighbours, from the slots first + lane, first + stride + lane, ... on (multiples of 64), in slot
// order; bit 31 of the slot says that it is not cached.  Only cached ones: a slot whose key is not below the limit is not looked
// up.  Otherwise every slot is, and the cached ones are candidates whatever their keys.
constexpr int kPrioUnroll = 4;   // chunks of 64 slots whose loads are issued together
template <typename IdxT>
__device__ __forceinline__ int prio_candidates(uint64_t hv, const IdxT *__restrict__ row, int d, uint32_t limit, bool only_cached,
                                               const uint32_t *__restrict__ prio, int first, int stride, Candidate *out, int cap) {
    const uint32_t above = limit << 1;
    const uint32_t lane = static_cast<uint32_t>(lane_id());
    int cnt = 0;
    for (uint32_t range = 0; range < static_cast<uint32_t>(d); range += 0x40000000u) {
        const WaveKeys<1> keys(__builtin_amdgcn_readfirstlane(key_low(hv, range)), __builtin_amdgcn_readfirstlane(key_hi_term(hv)));
        const uint32_t end = static_cast<uint32_t>(d) - range < 0x40000000u ? static_cast<uint32_t>(d) : range + 0x40000000u;
        for (uint32_t base = range + first; base < end; base += kPrioUnroll * stride) {
            uint32_t z[kPrioUnroll], u[kPrioUnroll], bits[kPrioUnroll];
            bool look[kPrioUnroll];
#pragma unroll
            for (int q = 0; q < kPrioUnroll; ++q) {
                z[q] = keys.upper(keys.row_part(base + q * stride));
                look[q] = base + q * stride + lane < end && (!only_cached || z[q] < above);
                u[q] = bits[q] = 0;
            }
#pragma unroll
            for (int q = 0; q < kPrioUnroll; ++q)
                if (look[q]) u[q] = static_cast<uint32_t>(row[base + q * stride + lane]);
#pragma unroll
            for (int q = 0; q < kPrioUnroll; ++q)
                if (look[q]) bits[q] = prio[u[q] >> 5];
#pragma unroll
            for (int q = 0; q < kPrioUnroll; ++q) {
                const bool hit = (bits[q] >> (u[q] & 31)) & 1u;                // (not looked up: no bits)
                const uint32_t slot = base + q * stride + lane;
                keep_candidates<true>(z[q], static_cast<int>(slot | (hit ? 0u : 0x80000000u)), only_cached ? hit : hit || (look[q] && z[q] < above),
                                      out, cap, cnt);
            }
        }
    }
    return cnt;
}

// What a wavefront keeps in LDS: the candidates of the row at hand, and the slots that its batch of rows has selected
// (slot; row of the batch, and number among the row's slots from bit 8 on).
struct SampleLds {
    Candidate cand[kWavesPerBlock][kCandidates];
    uint2 pick[kWavesPerBlock][kWave];
    int32_t slot[kWavesPerBlock][kWave];
};

// Hubs (degree > heavy_degree, listed with the row information): the four wavefronts of a workgroup walk
// one row together, 64 slots each in turn, each with a list of its own for 64 candidates.  About 2k + 32 are
// expected in all, but no more than k + 48: a list that overflows, or too few candidates, costs k walks of the
// row by one wavefront, milliseconds for a long one.  At k = 64 that is one row in 10^7 from 600 slots on, and
// 2 in 10,000 of the short rows that only a low heavy_degree brings here; with 160 expected it was 6 in 10,000
// (4,000 rows of 20,000 slots at k = 60: 2.3 ms instead of 0.08).  The k winners are selected by (key, slot) and then ordered by slot.  The wavefronts take
// turns at that, while the others go on with the next hub into the second set of lists: one barrier per hub.
// With priority the cached slots, which may lie close together, are candidates without a limit: lists for 256 each, one set of them.
template <typename PtrT, typename IdxT, bool PRIO, bool SEEDS>
__device__ __forceinline__ void sample_hubs(const IdxT *__restrict__ col_idx, const RowSource<PtrT, IdxT, SEEDS> &rows, const SampleArgs &a,
                            const PrioArgs &pa, const HubList &hubs, int first, int step, SampleLds &lds, int (&counts)[2][kWavesPerBlock]) {
    // SEEDS: there is no list yet; a workgroup looks its rows over itself, one per lane (kSeedRows bounds them)
    uint64_t heavy = 0;
    int64_t my_start = 0;
    int my_deg = 0;
    IdxT my_node = 0;
    if constexpr (SEEDS) {
        const int64_t r = first + int64_t(lane_id()) * step;
        if (r < rows.seeds.n_seeds) rows.row(r, my_start, my_deg, my_node);
        heavy = ballot64(my_deg > a.heavy_degree);
    }
    const int nheavy = SEEDS ? first + popc64(heavy) * step : *hubs.count;
    static_assert(kWavesPerBlock * kWave == kCandidates, "one chunk of candidates per wavefront");
    constexpr int NCH = kWavesPerBlock;
    constexpr int kList = PRIO ? kCandidates : kWave;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    const int k = a.fanout;
    const uint64_t layer_hash = layer_hash_of(a);
    int turn = 0;
    for (int h = first; h < nheavy; h += step, ++turn) {   // the same for all four
        int row, deg;
        int64_t start;
        IdxT node;
        if constexpr (SEEDS) {
            const int l = __ffsll(static_cast<long long>(heavy)) - 1;
            heavy &= heavy - 1;
            row = first + l * step;
            start = static_cast<int64_t>(readlane64(static_cast<uint64_t>(my_start), l));
            deg = static_cast<int>(readlane32(static_cast<uint32_t>(my_deg), l));
            node = static_cast<IdxT>(readlane64(static_cast<uint64_t>(my_node), l));
        } else {
            row = __builtin_amdgcn_readfirstlane(hubs.rows[h]);
            rows.row(row, start, deg, node);
        }
        const int d = __builtin_amdgcn_readfirstlane(deg);
        const uint64_t hv = readlane64(mix64(layer_hash ^ uint64_t(node)), 0);
        const int c_row = PRIO ? __builtin_amdgcn_readfirstlane(pa.prio_count[node]) : 0;
        const Contest contest(PRIO, d, k, c_row);
        Candidate *cand = &lds.cand[0][0] + (PRIO ? 0 : (turn & 1) * kCandidates);
        const uint32_t gap = __builtin_amdgcn_readfirstlane(key_gap(contest.pool));
        const uint32_t limit = key_limit(contest.want + (contest.want < 16 ? contest.want + 32 : 48), contest.pool, gap);
        Candidate *list = cand + wave * kList;
        const int mine = PRIO && c_row > 0 ? prio_candidates(hv, col_idx + start, d, limit, contest.cached, pa.prio, wave * kWave, kBlock, list, kList)
                         : d >= kHubChunksFrom ? hub_candidates<kHubChunks>(hv, d, limit, wave, list, kList)
                                               : hub_candidates<1>(hv, d, limit, wave, list, kList);
        if (lane == 0) counts[turn & 1][wave] = mine;
        __syncthreads();
        if (wave == (turn & 3)) {
            const int32_t out_base = out_base_of(a, row);
            uint64_t sel[NCH];
            uint32_t word[NCH], slot[NCH], bound = 0;
            int n[NCH], most = 0;
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                n[c] = __builtin_amdgcn_readfirstlane(counts[turn & 1][c]);
                most = n[c] > most ? n[c] : most;
            }
            if constexpr (PRIO) {                          // the four lists end to end
                int end[NCH];
                end[0] = n[0];
#pragma unroll
                for (int c = 1; c < NCH; ++c) end[c] = end[c - 1] + n[c];
                bool sure[NCH];
                const bool fits = most <= kList && end[NCH - 1] <= kCandidates;
#pragma unroll
                for (int c = 0; c < NCH; ++c) {
                    const int i = c * kWave + lane;
                    const int w = (i >= end[0] ? 1 : 0) + (i >= end[1] ? 1 : 0) + (i >= end[2] ? 1 : 0);
                    const int before = w == 0 ? 0 : w == 1 ? end[0] : w == 2 ? end[1] : end[2];
                    const bool live = fits && i < end[NCH - 1];
                    const Candidate v = live ? cand[w * kList + i - before] : Candidate{kNoWord, 0};
                    const bool hit = c_row > 0 && v.slot >= 0;
                    word[c] = live && hit == contest.cached ? v.word : kNoWord;
                    slot[c] = static_cast<uint32_t>(v.slot);
                    sure[c] = live && hit && !contest.cached;
                }
                if (fits) bound = word_bound(word, contest.want, gap);
#pragma unroll
                for (int c = 0; c < NCH; ++c) sel[c] = ballot64(word[c] < bound || sure[c]);
            } else {
#pragma unroll
                for (int c = 0; c < NCH; ++c) {
                    const Candidate v = cand[c * kWave + lane];
                    word[c] = lane < n[c] ? v.word : kNoWord;
                    slot[c] = static_cast<uint32_t>(v.slot);
                }
                if (most <= kWave) bound = word_bound(word, k, gap);
#pragma unroll
                for (int c = 0; c < NCH; ++c) sel[c] = ballot64(word[c] < bound);
            }
            if (bound != 0) emit_by_slot<NCH>(slot, sel, k, lds.slot[wave], col_idx, start, out_base, a);
            // a list ran over, or equal words: practically never
            else select_by_repeated_min<PRIO>(col_idx, start, d, k, hv, out_base, a, pa.prio);
        }
        if (SEEDS && threadIdx.x == 0) hubs.rows[atomicAdd(hubs.count, 1)] = row;     // the next blocks' too
        if (PRIO) __syncthreads();                         // the lists are the next hub's
    }
}

static_assert(kCandidates % kWave == 0, "candidates are selected in chunks of one per lane");

// The slots of the lanes with `in`, of row r of the batch, appended to the batch's list.
__device__ __forceinline__ int push_slots(bool in, int slot, int r, int held, int before, uint2 *pick) {
    const uint64_t m = ballot64(in);
    if (in) {
        const int p = rank_below(m, before);
        pick[held + p] = make_uint2(static_cast<uint32_t>(slot), static_cast<uint32_t>(r | p << 8));
    }
    return before + popc64(m);
}
// The `want` smallest of a row's competing candidates, and with priority those that need not compete (flagged: the candidates say
// whether they are cached); false if that takes more than their words.
template <int NCH, bool PRIO>
__device__ __forceinline__ bool push_smallest(const Candidate *cand, int cnt, int want, uint32_t gap, int r, int held, uint2 *pick, bool flagged, bool cached) {
    const int lane = lane_id();
    uint32_t word[NCH];
    int slot[NCH];
    bool sure[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        const Candidate v = cand[c * kWave + lane];
        const bool live = c * kWave + lane < cnt;
        const bool hit = PRIO && flagged && v.slot >= 0;
        word[c] = live && (!PRIO || hit == cached) ? v.word : kNoWord;
        sure[c] = PRIO && live && hit && !cached;
        slot[c] = PRIO ? v.slot & 0x7FFFFFFF : v.slot;
    }
    const uint32_t bound = word_bound(word, want, gap);
    if (bound == 0) return false;
    int n = 0;
#pragma unroll
    for (int c = 0; c < NCH; ++c) n = push_slots(word[c] < bound || sure[c], slot[c], r, held, n, pick);
    return true;
}

// The same for any number of candidates.
template <bool PRIO>
__device__ __forceinline__ bool push_candidates(const Candidate *cand, int cnt, int want, uint32_t gap, int r, int held, uint2 *pick, bool flagged, bool cached) {
    if (cnt <= kWave) return push_smallest<1, PRIO>(cand, cnt, want, gap, r, held, pick, flagged, cached);
    if (cnt <= 2 * kWave) return push_smallest<2, PRIO>(cand, cnt, want, gap, r, held, pick, flagged, cached);
    return push_smallest<kCandidates / kWave, PRIO>(cand, cnt, want, gap, r, held, pick, flagged, cached);
}

// The selection that k_sample makes from a row's candidates, on candidates of the caller's (mqg_select_row_candidates), one wavefront: the
// bound on the keys' upper words, and one by one where there is none.  Late candidates are those that are not cached.  The candidates are first
// put in the order of their slot words' low 31 bits (ordered: they are), which tell equal keys apart, as a row's slots do.
template <bool PRIO>
__global__ void __launch_bounds__(kWave)
k_select_candidates(const uint64_t *__restrict__ keys, const uint32_t *__restrict__ slot_words, int cnt, int k, int ordered,
                    uint32_t *__restrict__ out_mask) {
    __shared__ int from[kCandidates];                      // the caller's index of a candidate
    __shared__ Candidate cand[kCandidates];
    __shared__ uint2 pick[kCandidates];
    __shared__ uint32_t mask[kCandidates / 32];
    const int lane = lane_id();
    if (lane < kCandidates / 32) mask[lane] = 0;
    for (int i = lane; i < cnt; i += kWave) {
        const uint32_t slot = slot_words[i] & 0x7FFFFFFFu;
        int rank = ordered ? i : 0;
        for (int o = 0; o < cnt && !ordered; ++o) {
            const uint32_t other = slot_words[o] & 0x7FFFFFFFu;
            rank += other < slot || (other == slot && o < i) ? 1 : 0;
        }
        from[rank] = i;
    }
    wave_lds_sync();
    auto key_at = [&](int j) { return keys[from[j]]; };
    auto late_at = [&](int j) { return (slot_words[from[j]] >> 31) != 0; };
    int hits = 0;
    for (int base = 0; base < cnt; base += kWave) {
        const int j = base + lane;
        const bool hit = PRIO && j < cnt && !late_at(j);
        if (j < cnt) cand[j] = Candidate{static_cast<uint32_t>(key_at(j) >> 33), PRIO && !hit ? static_cast<int32_t>(static_cast<uint32_t>(j) | 0x80000000u) : j};
        hits += popc64(ballot64(hit));
    }
    wave_lds_sync();
    const Contest contest(PRIO, cnt, k, hits);
    auto choose = [&](int j) { (void)atomicOr(&mask[from[j] >> 5], 1u << (from[j] & 31)); };
    auto take = [&](int, int j) { if (lane == 0) choose(j); };
    if (push_candidates<PRIO>(cand, cnt, contest.want, key_gap(contest.pool), 0, 0, pick, hits > 0, contest.cached)) {
        wave_lds_sync();
        for (int i = lane; i < k; i += kWave) choose(static_cast<int>(pick[i].x));
    } else if constexpr (PRIO) {
        take_one_by_one_prio(cnt, k, key_at, late_at, take);
    } else {
        take_one_by_one(cnt, k, key_at, take);
    }
    wave_lds_sync();
    if (lane < kCandidates / 32) out_mask[lane] = mask[lane];
}

// The first hub_blocks workgroups take the hubs (they are dispatched first and run the longest; 1,024 of them
// instead of 2,048: 10 % slower where hubs hold most of the slots); the others' wavefronts take batches of
// consecutive destinations, as many as leave a batch for every wavefront of the chip and select at most 64
// slots: their row information is loaded by one instruction, and their neighbours' ids, positions and
// marks - a chain of three dependent accesses - are fetched once for all.
// Bound by instruction issue, vector and scalar alike (stress: 35 M and 41 M instructions in 114 us): hence eight
// wavefronts per SIMD, which takes a bound on the registers (without it 106 scalar registers leave room for seven: the three
// sampling cases 2 to 7 % slower; with it 18 to 29 scalar registers, prioritised 99 to 107, are kept in lanes of vector ones),
// candidates of half a word of the key, the k smallest of them by a bound (word_bound), and divisions made once per batch, in its lanes.  92 M keys of 43 k rows (graph of 111 M nodes), ten vector instructions
// per 64 keys, three of them quarter-rate multiplications: 80 -> 61 us; 23 M keys of 10 k rows 32 -> 24; 65 M keys
// of 284 k rows 147 -> 114, of 44 k rows 45 -> 34.  While a batch is selected, the row information of the next one and the
// neighbours of the last two are on their way (4 us of the 147).
template <typename PtrT, typename IdxT, bool PRIO, bool SEEDS>
__global__ void __launch_bounds__(kBlock, 8)
k_sample(const IdxT *__restrict__ col_idx, const IdxT *__restrict__ dst_ids, SampleArgs a, PrioArgs pa,
         HubList hubs, int hub_blocks, int row_blocks, SideWork<IdxT> side, RowInfoArgs<PtrT, IdxT> seeds) {
    __shared__ SampleLds lds;
    __shared__ int counts[2][kWavesPerBlock];
    const RowSource<PtrT, IdxT, SEEDS> rows{a, dst_ids, seeds};
    if (static_cast<int>(blockIdx.x) < hub_blocks) {
        sample_hubs<PtrT, IdxT, PRIO, SEEDS>(col_idx, rows, a, pa, hubs, static_cast<int>(blockIdx.x), hub_blocks, lds, counts);
        return;
    }
    const int row_block = static_cast<int>(blockIdx.x) - hub_blocks - (side.relabel_blocks + side.row_tiles);
    if (row_block < 0) {
        if constexpr (SEEDS) row_info_tile<false>(seeds, static_cast<int>(blockIdx.x) - hub_blocks, counts[0], side.seed_bits);
        else side_work(side, static_cast<int>(blockIdx.x) - hub_blocks, counts[0]);
        return;
    }
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    const int64_t n = SEEDS ? seeds.n_seeds : a.sizes[0];
    const int k = a.fanout;
    const int64_t share = n / kBusyWaves;
    const int most = kWave / k < kBatchRows ? kWave / k : kBatchRows;
    const int batch = share < 1 ? 1 : share < most ? static_cast<int>(share) : most;
    const int64_t step = int64_t(row_blocks) * kWavesPerBlock * batch;
    auto expected = [](int want) { return want + 4 * static_cast<int>(__builtin_sqrtf(static_cast<float>(want))) + 8; };   // candidates of a long row
    const int first_expect = expected(k);
    const uint64_t layer_hash = layer_hash_of(a);
    Candidate *cand = lds.cand[wave];
    uint2 *pick = lds.pick[wave];
    const int64_t first_row = (int64_t(row_block) * kWavesPerBlock + wave) * batch;
    if (first_row >= n) return;
    // row information of the batch at hand, one row per lane, loaded a batch ahead
    auto row_of_lane = [&](int64_t row0) {
        const int64_t last = n - 1;
        const int64_t r = row0 + (lane < batch ? lane : 0);
        return r < n ? r : last;
    };
    int64_t next_start;
    int next_deg;
    IdxT next_node;
    {
        const int64_t r = row_of_lane(first_row);
        rows.row(r, next_start, next_deg, next_node);
    }
    // neighbours on their way: ids of the batch before, positions of the one before that
    NeighbourPipe<IdxT> pipe(a);
    for (int64_t row0 = first_row; row0 < n; row0 += step) {
        const int m = n - row0 < batch ? static_cast<int>(n - row0) : batch;
        const int64_t my_row = row_of_lane(row0);
        const int64_t my_start = next_start;
        const int my_deg = next_deg;
        const int32_t my_out = out_base_of(a, my_row);
        const uint64_t my_hv = mix64(layer_hash ^ uint64_t(next_node));
        const int my_cached = PRIO ? pa.prio_count[next_node] : 0;
        if (!SEEDS || row0 + step < n) {
            const int64_t r = row_of_lane(row0 + step);
            rows.row(r, next_start, next_deg, next_node);
        }
        const Contest my_contest(PRIO, my_deg, k, my_cached);
        const int my_expect = PRIO ? expected(my_contest.want) : 0;
        const uint32_t my_gap = key_gap(my_contest.pool > 0 ? my_contest.pool : 1), my_low = key_low(my_hv), my_hi_term = key_hi_term(my_hv);
        int held = 0;                                      // slots selected so far
        for (int r = 0; r < m; ++r) {
            const int d = static_cast<int>(readlane32(static_cast<uint32_t>(my_deg), r));
            if (d > a.heavy_degree && d > k) continue;     // a hub: sampled by the first workgroups
            if (d <= k) {                                  // the whole row, no randomness
                held += push_slots(lane < d, lane, r, held, 0, pick);
                continue;
            }
            const uint32_t gap = readlane32(my_gap, r), low = readlane32(my_low, r), hi_term = readlane32(my_hi_term, r);
            const Contest contest(PRIO, d, k, PRIO ? static_cast<int>(readlane32(static_cast<uint32_t>(my_cached), r)) : 0);
            const bool flagged = PRIO && (contest.cached || contest.want < k);             // the row has cached neighbours
            const IdxT *nbrs = PRIO ? col_idx + static_cast<int64_t>(readlane64(static_cast<uint64_t>(my_start), r)) : nullptr;
            bool done = false;
            if (d <= kWave) {                              // one key per lane
                const uint32_t x = low ^ static_cast<uint32_t>(lane);
                const uint32_t z = key_upper(uint64_t(x) * RowKeys::kC1Lo + (uint64_t(x * RowKeys::kC1Hi + hi_term) << 32));
                bool hit = false;
                if (flagged && lane < d) hit = is_cached(nbrs, lane, pa.prio);
                const uint32_t word[1] = {lane < d && (!PRIO || hit == contest.cached) ? z >> 1 : kNoWord};
                const uint32_t bound = a.force_slow ? 0 : word_bound(word, contest.want, gap);
                done = bound != 0;
                if (done) (void)push_slots(word[0] < bound || (PRIO && hit && !contest.cached), lane, r, held, 0, pick);
            } else if (!a.force_slow) {
                // Longer rows: the slots whose keys lie under a limit are candidates, stored in ascending slot order; too
                // few (3 rows in 100,000): again with a higher one.
                const int expect = PRIO ? static_cast<int>(readlane32(static_cast<uint32_t>(my_expect), r)) : first_expect;
                auto candidates = [&](int e) {
                    const uint32_t limit = key_limit(e, contest.pool, gap);
                    if (flagged) return prio_candidates(readlane64(my_hv, r), nbrs, d, limit, contest.cached, pa.prio, 0, kWave, cand, kCandidates);
                    return row_candidates(low, hi_term, d, limit, cand, kCandidates);
                };
                int cnt = candidates(expect);
                if (cnt < k) cnt = candidates(2 * expect + 32);
                wave_lds_sync();
                done = cnt >= k && cnt <= kCandidates && push_candidates<PRIO>(cand, cnt, contest.want, gap, r, held, pick, flagged, contest.cached);
                wave_lds_sync();                           // the candidates' place is the next row's
            }
            if (done) {
                held += k;
            } else {
                const int64_t start = static_cast<int64_t>(readlane64(static_cast<uint64_t>(my_start), r));
                const int32_t out_base = static_cast<int32_t>(readlane32(static_cast<uint32_t>(my_out), r));
                select_by_repeated_min<PRIO>(col_idx, start, d, k, readlane64(my_hv, r), out_base, a, pa.prio);
            }
        }
        wave_lds_sync();
        const uint2 mine = pick[lane];
        const int of = lane < held ? static_cast<int>(mine.y & 0xFF) : 0;
        const int64_t slot_pos = __shfl(my_start, of, kWave) + static_cast<int32_t>(mine.x);
        const int32_t out_pos = __shfl(my_out, of, kWave) + static_cast<int32_t>(mine.y >> 8);
        pipe.push(col_idx, lane < held, slot_pos, out_pos);
        wave_lds_sync();                                   // pick is the next batch's
    }
    pipe.drain();
}

// prio_count[v] = number of cached neighbours of node v.  A lane owns a node; rows of up to 32 slots
// are walked by their lane, longer rows by the whole wavefront, one after the other.
template <typename PtrT, typename IdxT>
__global__ void __launch_bounds__(kBlock)
k_prio_counts(const PtrT *__restrict__ row_ptr, const IdxT *__restrict__ col_idx, int64_t n,
              const uint32_t *__restrict__ prio, int32_t *__restrict__ prio_count) {
    const int lane = lane_id();
    const int64_t v = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    int64_t start = 0;
    int d = 0;
    if (v < n) {
        start = static_cast<int64_t>(row_ptr[v]);
        d = static_cast<int>(static_cast<int64_t>(row_ptr[v + 1]) - start);
    }
    int c = 0;
    if (d <= 32)
        for (int j = 0; j < d; ++j) c += is_cached(col_idx + start, j, prio) ? 1 : 0;
    uint64_t big = ballot64(d > 32);
    while (big) {
        const int l = __ffsll(static_cast<long long>(big)) - 1;
        big &= big - 1;
        const int dl = static_cast<int>(readlane32(static_cast<uint32_t>(d), l));
        const int64_t sl = static_cast<int64_t>(readlane64(static_cast<uint64_t>(start), l));
        int m = 0;
        for (int base = 0; base < dl; base += kWave) {
            const int j = base + lane;
            m += popc64(ballot64(j < dl && is_cached(col_idx + sl, j, prio)));
        }
        if (lane == l) c = m;
    }
    if (v < n) prio_count[v] = c;
}

// bit v of the bitmap = node v is cached (slot_of[v] >= 0); one lane per node
__global__ void __launch_bounds__(kBlock)
k_prio_bitmap(const int32_t *__restrict__ slot_of, int64_t n, uint32_t *__restrict__ prio) {
    const int64_t v = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    const uint64_t m = ballot64(v < n && slot_of[v] >= 0);
    if (lane_id() == 0) {                                  // v is a multiple of 64 here; padding words get zeros
        prio[v >> 5] = static_cast<uint32_t>(m);
        prio[(v >> 5) + 1] = static_cast<uint32_t>(m >> 32);
    }
}

// ------------------------------------------------------------------------------------------
// Bitmap -> ascending list of new source nodes.

// Two tile shapes.  Dense bitmaps (up to 32 M nodes): one word per thread, 256 words per
// workgroup, ids staged through LDS so that the source list is written coalesced.  Larger graphs:
// four words per thread (one 16-byte load), ids written straight from the bit loop - their bitmaps
// are sparse, a thread rarely has more than a bit or two.
// (except, where it is not null: the seeds' bits, which do not count, see RowSource)
__device__ __forceinline__ uint32_t new_bits(const uint32_t *__restrict__ bitmap, const uint32_t *__restrict__ except, int64_t w) {
    return except ? bitmap[w] & ~except[w] : bitmap[w];
}
template <int WPT>
__device__ __forceinline__ void bitmap_count_tile(const uint32_t *__restrict__ bitmap, const uint32_t *__restrict__ except, int32_t *__restrict__ tile_sums,
                                                  int tile, int *lds) {
    const int64_t w0 = (int64_t(tile) * kBlock + threadIdx.x) * WPT;
    int c;
    if (WPT == 4) {
        uint4 w = *reinterpret_cast<const uint4 *>(bitmap + w0);
        c = __popc(w.x) + __popc(w.y) + __popc(w.z) + __popc(w.w);
    } else {
        c = __popc(new_bits(bitmap, except, w0));
    }
    int s = wave_sum(c);
    if (lane_id() == 0) lds[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
#pragma unroll
        for (int k = 0; k < kWavesPerBlock; ++k) t += lds[k];
        tile_sums[tile] = t;
    }
}

// The first row_tiles workgroups turn the row tile sums into indptr, the others count the bits of
// one bitmap tile each: both only need what the launches before produced.
template <int WPT>
__global__ void __launch_bounds__(kBlock)
k_offsets_count(const int32_t *__restrict__ row_deg, int fanout, int64_t *sizes, const int32_t *__restrict__ row_tile_vals,
                int rows_scanned, int32_t *__restrict__ indptr, const int32_t *__restrict__ seed_flags, int row_tiles,
                const uint32_t *__restrict__ bitmap, const uint32_t *__restrict__ except, int32_t *__restrict__ bitmap_tile_sums) {
    __shared__ int lds[kWavesPerBlock];
    const int b = static_cast<int>(blockIdx.x);
    if (b < row_tiles) row_offsets_tile(row_deg, fanout, sizes, row_tile_vals, rows_scanned, indptr, seed_flags, b, row_tiles, lds);
    else bitmap_count_tile<WPT>(bitmap, except, bitmap_tile_sums, b - row_tiles, lds);
}

// num_src of a block is also num_dst of the next block outward.  A call's bounds count distinct seeds; repeated ones, which are
// flagged but keep their rows, can leave more new sources than that.  The last of those, beyond `most`, are not listed.
__device__ __forceinline__ void store_num_src(int64_t *sizes, int64_t *next_num_dst, int64_t num_src, int64_t most) {
    num_src = num_src < most ? num_src : most;
    sizes[1] = num_src;
    if (next_num_dst) *next_num_dst = num_src;
}

// The ids staged in LDS, ascending, to the source list from place `base` on, up to place `most`.  Four a thread at a time, the two row
// offsets of an id being a random access: a listing of 9 tiles of 22 k nodes 4.6 us, 5.3 one at a time, a call for 179 seeds there 39.7 and 40.5; the
// listings of 2.4 M nodes, whose 300 tiles hide each other's, 8.5 to 12 us both ways.
template <typename PtrT, typename IdxT>
__device__ __forceinline__ void store_staged(int32_t *staged, int total, int64_t base, int64_t most, IdxT *__restrict__ src_ids,
                                             int32_t *__restrict__ local_of, int32_t pos_base, const NewRows<PtrT> &next, int *lds) {
    constexpr int U = 4;
    if (base + total > most) total = base < most ? static_cast<int>(most - base) : 0;      // workgroup-uniform
    int hubs = 0;
    for (int k0 = threadIdx.x; k0 < total; k0 += U * kBlock) {
        int32_t v[U];
        int64_t begin[U], degree[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = staged[k0 + u * kBlock < total ? k0 + u * kBlock : k0];
        if (next.row_ptr) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                begin[u] = static_cast<int64_t>(next.row_ptr[v[u]]);
                degree[u] = static_cast<int64_t>(next.row_ptr[int64_t(v[u]) + 1]) - begin[u];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + u * kBlock;
            if (k >= total) break;
            src_ids[base + k] = static_cast<IdxT>(v[u]);
            local_of[v[u]] = pos_base + static_cast<int32_t>(base + k);
            if (next.row_ptr) {
                next.row_start[base + k] = begin[u];
                next.row_deg[base + k] = static_cast<int32_t>(degree[u]);
                const int hub = degree[u] > next.hubs.heavy_degree ? 1 : 0;
                staged[k] = hub;                           // this thread's own entry
                hubs += hub;
            }
        }
    }
    if (!next.row_ptr) return;
    int place = next.hubs.take(hubs, lds);
    if (hubs)
        for (int k = threadIdx.x; k < total; k += kBlock)
            if (staged[k]) next.hubs.rows[place++] = static_cast<int32_t>(base + k);
}

// BOUNDED: repeated seeds can leave more sources than `most`, see store_num_src; false where the rows' neighbours cannot fill the graph: num_dst + nnz
// then bounds the sources however often seeds repeat.  (The test costs 0.3 us in each of the three listings of a graph of 111 M nodes, 9.7 us on average.)
template <typename IdxT, bool BOUNDED>
__global__ void __launch_bounds__(kBlock)
k_bitmap_emit4(uint32_t *__restrict__ bitmap, const int32_t *__restrict__ tile_vals, int scanned, int32_t most,
               int64_t *__restrict__ sizes, int64_t *__restrict__ next_num_dst, IdxT *__restrict__ src_ids,
               int32_t *__restrict__ local_of, int32_t pos_base) {
    __shared__ int lds[kWavesPerBlock];
    const int tile_base = scanned ? tile_vals[blockIdx.x] : tiles_before(tile_vals, lds);
    const int64_t w0 = (int64_t(blockIdx.x) * kBlock + threadIdx.x) * 4;
    uint4 w = *reinterpret_cast<const uint4 *>(bitmap + w0);
    int c = __popc(w.x) + __popc(w.y) + __popc(w.z) + __popc(w.w);
    int total;
    int ex = block_excl_scan<kWavesPerBlock>(c, &total, lds);
    const int64_t num_dst = sizes[0];
    if (!scanned && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) store_num_src(sizes, next_num_dst, num_dst + tile_base + total, most);
    if (c == 0) return;
    int64_t pos = num_dst + tile_base + ex;
    uint32_t words[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        uint32_t bits = words[q];
        while (bits) {
            int b = __ffs(bits) - 1;
            bits &= bits - 1;
            int32_t v = static_cast<int32_t>((w0 + q) * 32 + b);
            if (!BOUNDED || pos < most) {
                src_ids[pos] = static_cast<IdxT>(v);
                local_of[v] = pos_base + static_cast<int32_t>(pos);
            }
            ++pos;
        }
    }
    *reinterpret_cast<uint4 *>(bitmap + w0) = make_uint4(0, 0, 0, 0);
}

template <typename PtrT, typename IdxT>
__global__ void __launch_bounds__(kBlock)
k_bitmap_emit1(uint32_t *__restrict__ bitmap, const uint32_t *__restrict__ except, const int32_t *__restrict__ tile_vals, int scanned, int32_t most,
               int64_t *__restrict__ sizes, int64_t *__restrict__ next_num_dst, IdxT *__restrict__ src_ids,
               int32_t *__restrict__ local_of, int32_t pos_base, NewRows<PtrT> next) {
    __shared__ int lds[kWavesPerBlock];
    __shared__ int32_t staged[kBlock * 32];                // every id of the tile, ascending
    const int tile_base = scanned ? tile_vals[blockIdx.x] : tiles_before(tile_vals, lds);
    const int64_t w0 = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    uint32_t bits = new_bits(bitmap, except, w0);
    const int c = __popc(bits);
    int total;
    int ex = block_excl_scan<kWavesPerBlock>(c, &total, lds);
    const int64_t num_dst = sizes[0];
    if (!scanned && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) store_num_src(sizes, next_num_dst, num_dst + tile_base + total, most);
    if (c || except) bitmap[w0] = 0;                       // (seeds are marked too)
    if (total == 0) return;                                // workgroup-uniform
    if (c) {
        const int32_t v0 = static_cast<int32_t>(w0 * 32);
        while (bits) {
            int b = __ffs(bits) - 1;
            bits &= bits - 1;
            staged[ex++] = v0 + b;
        }
    }
    __syncthreads();
    store_staged(staged, total, num_dst + tile_base, most, src_ids, local_of, pos_base, next, lds);
}

// Small bitmaps (at most kSelfCountTiles tiles of 256 words, i.e. graphs of up to half a million
// nodes): no counting launch.  Every tile's workgroup counts the set bits of the tiles before its own
// itself, so the words must stay as they are until every workgroup has read them: the relabel clears
// them, which, of all blocks but the outermost, runs beside the sampling of the next block; so that marks
// its nodes in another bitmap.  The same launch turns the row tile sums into indptr (the
// workgroups past the bitmap's tiles), as k_offsets_count does on larger graphs.
constexpr int kSelfCountTiles = 64;
template <typename PtrT, typename IdxT>
__global__ void __launch_bounds__(kBlock)
k_emit_offsets(const uint32_t *__restrict__ bitmap, const uint32_t *__restrict__ except, int bitmap_tiles, int32_t most, int64_t *sizes, int64_t *__restrict__ next_num_dst,
               IdxT *__restrict__ src_ids, int32_t *__restrict__ local_of, int32_t pos_base, const int32_t *__restrict__ row_deg, int fanout,
               const int32_t *__restrict__ row_tile_vals, int rows_scanned, int32_t *__restrict__ indptr,
               const int32_t *__restrict__ seed_flags, int row_tiles, NewRows<PtrT> next) {
    __shared__ int lds[kWavesPerBlock];
    __shared__ int32_t staged[kBlock * 32];                // every id of the tile, ascending
    const int tile = static_cast<int>(blockIdx.x);
    if (tile >= bitmap_tiles) {
        row_offsets_tile(row_deg, fanout, sizes, row_tile_vals, rows_scanned, indptr, seed_flags, tile - bitmap_tiles, row_tiles, lds);
        return;
    }
    // (16 bytes a load and four of them at a time: of 28 tiles 6.8 -> 5.8 us, with the seeds' bits 11.9 -> 5.9)
    int part = 0;
    auto count_before = [&](auto with_except) {
        constexpr int U = 4;
        const uint4 *marked = reinterpret_cast<const uint4 *>(bitmap), *left_out = reinterpret_cast<const uint4 *>(except);
        const int end = tile * (kBlock / 4);
        for (int q0 = threadIdx.x; q0 < end; q0 += U * kBlock) {
            uint4 v[U], e[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int q = q0 + u * kBlock < end ? q0 + u * kBlock : q0;
                v[u] = marked[q];
                e[u] = decltype(with_except)::value ? left_out[q] : make_uint4(0, 0, 0, 0);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = __popc(v[u].x & ~e[u].x) + __popc(v[u].y & ~e[u].y) + __popc(v[u].z & ~e[u].z) + __popc(v[u].w & ~e[u].w);
                part += q0 + u * kBlock < end ? c : 0;
            }
        }
    };
    if (except) count_before(std::true_type());
    else count_before(std::false_type());
    part = wave_sum(part);
    if (lane_id() == 0) lds[threadIdx.x >> 6] = part;
    __syncthreads();
    int tile_base = 0;
#pragma unroll
    for (int k = 0; k < kWavesPerBlock; ++k) tile_base += lds[k];
    const int64_t w0 = int64_t(tile) * kBlock + threadIdx.x;
    uint32_t bits = new_bits(bitmap, except, w0);
    const int c = __popc(bits);
    int total;
    int ex = block_excl_scan<kWavesPerBlock>(c, &total, lds);
    const int64_t num_dst = sizes[0];
    if (tile == bitmap_tiles - 1 && threadIdx.x == 0) store_num_src(sizes, next_num_dst, num_dst + tile_base + total, most);
    if (total == 0) return;                                // workgroup-uniform
    if (c) {
        const int32_t v0 = static_cast<int32_t>(w0 * 32);
        while (bits) {
            int b = __ffs(bits) - 1;
            bits &= bits - 1;
            staged[ex++] = v0 + b;
        }
    }
    __syncthreads();
    store_staged(staged, total, num_dst + tile_base, most, src_ids, local_of, pos_base, next, lds);
}

__global__ void __launch_bounds__(kBlock)
k_relabel(const int32_t *__restrict__ nbr, const int64_t *__restrict__ sizes, const int32_t *__restrict__ indptr, int fanout,
          const int32_t *__restrict__ local_of, int32_t pos_base, int32_t *__restrict__ indices, uint32_t *__restrict__ clear, int64_t nclear,
          int32_t *__restrict__ hub_count) {
    if (blockIdx.x == 0) clear_hubs(hub_count);
    clear_words(clear, nclear, static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x));
    relabel_slots(nbr, sizes, indptr, fanout, local_of, pos_base, indices, static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x));
}

// The relabel of one block and, in the same launch, the row information of the next block outward
// (its destinations are this block's sources, complete since k_bitmap_emit).
template <typename PtrT, typename IdxT>
__global__ void __launch_bounds__(kBlock)
k_relabel_rowinfo(const int32_t *__restrict__ nbr, const int64_t *__restrict__ sizes, const int32_t *__restrict__ indptr,
                  int fanout, const int32_t *__restrict__ local_of, int32_t pos_base, int32_t *__restrict__ indices, int relabel_blocks,
                  RowInfoArgs<PtrT, IdxT> next) {
    __shared__ int lds[kWavesPerBlock];
    const int b = static_cast<int>(blockIdx.x);
    if (b < relabel_blocks) {
        relabel_slots(nbr, sizes, indptr, fanout, local_of, pos_base, indices, b, relabel_blocks);
    } else {
        row_info_tile<true>(next, b - relabel_blocks, lds);
    }
}

__global__ void __launch_bounds__(kBlock)
k_fill_i32(int32_t *__restrict__ p, int64_t n, int32_t value, int grid) {
    for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += int64_t(grid) * kBlock) p[i] = value;
}

// Calls that are being recorded take their positions back, see take_positions.
template <typename IdxT>
__global__ void __launch_bounds__(kBlock)
k_reset_local(const IdxT *__restrict__ src_ids, const int64_t *__restrict__ sizes, int32_t *__restrict__ local_of) {
    const int64_t n = sizes[1];
    const int64_t stride = int64_t(gridDim.x) * kBlock;
    for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += stride) {
        local_of[src_ids[i]] = -1;
    }
}

__global__ void __launch_bounds__(kBlock)
k_clear_hubs(int32_t *__restrict__ hub_count) {
    clear_hubs(hub_count);
}

template <typename PtrT, typename IdxT>
int sample_blocks_impl(mqg_ctx *ctx, const mqg_graph *g, const void *seeds_v, int32_t num_seeds, const uint64_t *seed_dev,
                       const int32_t *fanouts, int32_t L, uint64_t rng_seed, mqg_block *blocks, hipStream_t s) {
    const PtrT *row_ptr = static_cast<const PtrT *>(g->row_ptr);
    const IdxT *col_idx = static_cast<const IdxT *>(g->col_idx);
    const IdxT *seeds = static_cast<const IdxT *>(seeds_v);
    const uint64_t seed_hash = host_mix64(rng_seed + kGolden);

    const bool use_hash = ctx->dedup_hash;
    int32_t *local_of = use_hash ? nullptr : ctx->local_of;
    int32_t pos_base = 0;
    bool take_back = false;
    if (!use_hash) {
        int rc = take_positions(ctx, ctx->max_src, s, &pos_base, &take_back);
        if (rc != MQG_OK) return rc;
    }
    int64_t need_dst = num_seeds;
    const int bitmap_wpt = ctx->bitmap_words <= (int64_t(1) << 20) ? 1 : 4;     // words per thread, see k_bitmap_emit*
    const int bitmap_tiles = static_cast<int>(std::max<int64_t>(1, ctx->bitmap_words / (int64_t(kBlock) * bitmap_wpt)));
    const bool self_count = !use_hash && bitmap_wpt == 1 && bitmap_tiles <= kSelfCountTiles;    // see k_emit_offsets
    // (rows that are no hubs are walked in one range of 2^30 slots)
    const int heavy_degree = ctx->force_slow_select ? 0x7FFFFFFF : std::min(ctx->heavy_degree, 1 << 30);
    const bool one_list = !use_hash && ctx->records_rows;                  // of hubs for all blocks: they stay destinations
    auto hub_list = [&](int l) {
        return HubList{ctx->heavy_rows, ctx->heavy_count + (one_list ? 0 : l), heavy_degree};
    };
    auto row_info_args = [&](int l, int64_t dst_count) {
        RowInfoArgs<PtrT, IdxT> r;
        r.row_ptr = row_ptr;
        r.dst = (l == L - 1) ? seeds : static_cast<const IdxT *>(blocks[l + 1].src_ids);
        r.sizes = blocks[l].sizes;
        r.src_out = static_cast<IdxT *>(blocks[l].src_ids);
        r.fanout = fanouts[l];
        r.row_start = ctx->row_start;
        r.row_deg = ctx->row_deg;
        r.tile_sums = ctx->tile_vals;
        r.sizes_rw = blocks[l].sizes;
        r.hubs = hub_list(l);
        r.n_seeds = l == L - 1 ? dst_count : int64_t(-1);
        r.local_of = local_of;
        r.pos_base = pos_base;
        r.num_nodes = g->num_nodes;
        r.seed_flags = ctx->heavy_count + MQG_MAX_LAYERS;
        return r;
    };
    auto tiles_of = [](int64_t rows) { return static_cast<int>(std::max<int64_t>(1, ceil_div(rows, kBlock))); };
    // The innermost block's row information; that of the others is recorded as their destinations are listed.  With the sampling, see
    // RowSource, if there is a next block, whose launch sets the seeds' bits back, and up to where every wavefront has one row (from there on
    // rows come in batches, whose information is loaded a batch ahead; a launch less counts for less, too).
    const bool with_seeds = one_list && L > 1 && num_seeds < kSeedRows;
    uint32_t *seed_bits = with_seeds ? ctx->bitmap + 2 * ctx->bitmap_words : nullptr;
    if (!with_seeds)
        MQG_LAUNCH(ctx, "k_row_info", s, (k_row_info<PtrT, IdxT><<<tiles_of(need_dst), kBlock, 0, s>>>(row_info_args(L - 1, need_dst))));
    SideWork<IdxT> side{};                                 // what the next sampling launch does for the block before
    for (int l = L - 1; l >= 0; --l) {
        mqg_block &b = blocks[l];
        const int k = fanouts[l];
        IdxT *src_ids = static_cast<IdxT *>(b.src_ids);
        const int64_t need_nnz = need_dst * k;
        const int row_tiles = tiles_of(need_dst);
        // where a block is relabelled while the next one is sampled, they take the two ends of the room in turn (two neighbouring blocks
        // fit it side by side), at whole lines
        int32_t *nbr = ctx->nbr + (one_list && (l & 1) ? (ctx->nbr_room - need_nnz) & ~int64_t(31) : 0);
        const int64_t next_dst = std::max(need_dst, std::min<int64_t>(g->num_nodes, need_dst + need_nnz));
        // Where repeated seeds leave more sources than the bound, an inner block's end there, the next block's scratch being sized by
        // it, the outermost one's with the room that there is.  (32 bits, where the listings' arguments had a gap: as a 64-bit argument more
        // it made each 0.25 us longer, 4.2 -> 4.5 us on 22 k nodes.)
        const int32_t most_src = static_cast<int32_t>(l > 0 ? next_dst : std::min(b.cap_src, ctx->max_src));
        // marks of this block, and the other half of the words, which the side work clears meanwhile, see k_emit_offsets
        uint32_t *bitmap = ctx->bitmap + (self_count ? (l & 1) * ctx->bitmap_words : 0);

        // few tiles: every workgroup of the consumer adds up the tile sums before its own; many: one scan launch
        const int rows_scanned = row_tiles > kSelfPrefixTiles ? 1 : 0;
        auto scan_rows = [&]() {
            return rows_scanned ? launch_scan_tiles(ctx, ctx->tile_vals, row_tiles, nullptr, &b.sizes[2], nullptr, s, "k_scan_tiles(rows)") : int(MQG_OK);
        };
        int rc = MQG_OK;
        const int32_t *seed_flags = l == L - 1 ? ctx->heavy_count + MQG_MAX_LAYERS : nullptr;
        if (use_hash) {
            rc = scan_rows();
            if (rc != MQG_OK) return rc;
            if (l == L - 1) {                              // the seeds enter the table (and repeated ones are flagged) first
                rc = hash_put_seeds(ctx, b.src_ids, g->idx_type, need_dst, b.sizes, s);   // ids as the row info checked them
                if (rc != MQG_OK) return rc;
            }
            MQG_LAUNCH(ctx, "k_row_offsets", s,
                       (k_row_offsets<<<row_tiles, kBlock, 0, s>>>(ctx->row_deg, k, b.sizes, ctx->tile_vals, rows_scanned, b.indptr, seed_flags)));
        }

        SampleArgs a;
        a.row_start = ctx->row_start;
        a.row_deg = ctx->row_deg;
        a.indptr = use_hash ? b.indptr : nullptr;
        a.sizes = b.sizes;
        a.nbr = nbr;
        const bool seeds_here = with_seeds && l == L - 1;
        a.local_of = seeds_here ? nullptr : local_of;
        a.pos_base = pos_base;
        a.bitmap = use_hash ? nullptr : bitmap;
        a.layer_hash = host_mix64(seed_hash ^ uint64_t(l));
        a.seed_dev = seed_dev;
        a.layer = l;
        a.fanout = k;
        a.force_slow = ctx->force_slow_select ? 1 : 0;
        a.heavy_degree = heavy_degree;
        // (where the side work copies the destinations, this block's own source list is not complete yet)
        const IdxT *dst_ids = !one_list || l == L - 1 ? src_ids : static_cast<const IdxT *>(blocks[l + 1].src_ids);
        const int hub_blocks = static_cast<int>(std::min<int64_t>(std::max<int64_t>(1, need_dst), kHubBlocks));
        // k_sample's wavefronts loop over their batches: no more workgroups than fill the chip four times
        // (the bound is often twice the number of destinations, and an idle workgroup costs a dispatch)
        const int row_blocks = static_cast<int>(std::min<int64_t>(std::max<int64_t>(1, ceil_div(need_dst, kWavesPerBlock)), 8192));
        if (side.relabel_blocks) {
            side.row_tiles = row_tiles;
            side.dst = dst_ids;
            side.dst_count = b.sizes;
            side.row_deg = ctx->row_deg;
            side.row_fanout = k;
            side.src_out = src_ids;
            side.tile_sums = ctx->tile_vals;
        }
        if (seeds_here) {
            side.row_tiles = row_tiles;
            side.seed_bits = seed_bits;
        }
        const int sample_grid = hub_blocks + side.relabel_blocks + side.row_tiles + row_blocks;
        const PrioArgs prio = ctx->prio_enabled ? PrioArgs{ctx->prio_bitmap, ctx->prio_count} : PrioArgs{};
#define MQG_SAMPLE(NAME, PT, PRIO, SEEDS, INFO)                                                                                                \
        MQG_LAUNCH(ctx, NAME, s,                                                                                                                \
                   (k_sample<PT, IdxT, PRIO, SEEDS><<<sample_grid, kBlock, 0, s>>>(col_idx, dst_ids, a, prio, hub_list(l), hub_blocks, row_blocks, side, INFO)))
        if (seeds_here && ctx->prio_enabled) MQG_SAMPLE("k_sample_prio", PtrT, true, true, row_info_args(l, need_dst));
        else if (seeds_here) MQG_SAMPLE("k_sample", PtrT, false, true, row_info_args(l, need_dst));
        else if (ctx->prio_enabled) MQG_SAMPLE("k_sample_prio", int32_t, true, false, (RowInfoArgs<int32_t, IdxT>{}));
        else MQG_SAMPLE("k_sample", int32_t, false, false, (RowInfoArgs<int32_t, IdxT>{}));
#undef MQG_SAMPLE
        const uint32_t *except = seeds_here ? seed_bits : nullptr;

        if (use_hash) {
            rc = hash_dedup_block(ctx, nbr, need_nnz, g->num_nodes, g->idx_type, b.src_ids, b.sizes,
                                  l > 0 ? blocks[l - 1].sizes : nullptr, most_src, b.indices, s);
            if (rc != MQG_OK) return rc;
            need_dst = next_dst;
            if (l > 0) MQG_LAUNCH(ctx, "k_row_info", s, (k_row_info<PtrT, IdxT><<<tiles_of(need_dst), kBlock, 0, s>>>(row_info_args(l - 1, need_dst))));
            continue;
        }
        rc = scan_rows();
        if (rc != MQG_OK) return rc;
        // num_src = num_dst + number of new nodes; it is also the next block's num_dst
        int64_t *next_num_dst = l > 0 ? &blocks[l - 1].sizes[0] : nullptr;
        const NewRows<PtrT> next{l > 0 && one_list ? row_ptr : nullptr, ctx->row_start, ctx->row_deg, hub_list(l)};
        if (self_count) {
            // indptr from the row tile sums and the new sources from the bitmap, one launch
            MQG_LAUNCH(ctx, "k_emit_offsets", s,
                       (k_emit_offsets<PtrT, IdxT><<<bitmap_tiles + row_tiles, kBlock, 0, s>>>(bitmap, except, bitmap_tiles, most_src, b.sizes, next_num_dst, src_ids,
                                                                                              ctx->local_of, pos_base, ctx->row_deg, k, ctx->tile_vals, rows_scanned,
                                                                                              b.indptr, seed_flags, row_tiles, next)));
        } else {
            // indptr from the row tile sums, and the bitmap's tile popcounts
            if (bitmap_wpt == 1) {
                MQG_LAUNCH(ctx, "k_offsets_count", s,
                           (k_offsets_count<1><<<row_tiles + bitmap_tiles, kBlock, 0, s>>>(ctx->row_deg, k, b.sizes, ctx->tile_vals, rows_scanned, b.indptr,
                                                                                          seed_flags, row_tiles, bitmap, except, ctx->bitmap_tile_vals)));
            } else {
                MQG_LAUNCH(ctx, "k_offsets_count", s,
                           (k_offsets_count<4><<<row_tiles + bitmap_tiles, kBlock, 0, s>>>(ctx->row_deg, k, b.sizes, ctx->tile_vals, rows_scanned, b.indptr,
                                                                                          seed_flags, row_tiles, bitmap, except, ctx->bitmap_tile_vals)));
            }
            const int bits_scanned = bitmap_tiles > kSelfPrefixTiles ? 1 : 0;
            if (bits_scanned) rc = launch_scan_tiles(ctx, ctx->bitmap_tile_vals, bitmap_tiles, &b.sizes[0], &b.sizes[1], next_num_dst, s, "k_scan_tiles(bitmap)", most_src);
            if (rc != MQG_OK) return rc;
            if (bitmap_wpt == 1) {
                MQG_LAUNCH(ctx, "k_bitmap_emit", s,
                           (k_bitmap_emit1<PtrT, IdxT><<<bitmap_tiles, kBlock, 0, s>>>(bitmap, except, ctx->bitmap_tile_vals, bits_scanned, most_src, b.sizes, next_num_dst, src_ids, ctx->local_of, pos_base, next)));
            } else {
                const bool bounded = need_dst + need_nnz > g->num_nodes;
#define MQG_EMIT4(BOUNDED)                                                                                                                   \
                MQG_LAUNCH(ctx, "k_bitmap_emit", s,                                                                                          \
                           (k_bitmap_emit4<IdxT, BOUNDED><<<bitmap_tiles, kBlock, 0, s>>>(bitmap, ctx->bitmap_tile_vals, bits_scanned, most_src, b.sizes, next_num_dst, src_ids, ctx->local_of, pos_base)))
                if (bounded) MQG_EMIT4(true);
                else MQG_EMIT4(false);
#undef MQG_EMIT4
            }
        }
        const int relabel_grid = static_cast<int>(std::min<int64_t>(std::max<int64_t>(1, ceil_div(need_nnz, kBlock)), 4096));
        uint32_t *clear = self_count ? bitmap : nullptr;
        if (l > 0 && !one_list) {
            MQG_LAUNCH(ctx, "k_relabel_rowinfo", s,
                       (k_relabel_rowinfo<PtrT, IdxT><<<relabel_grid + tiles_of(next_dst), kBlock, 0, s>>>(nbr, b.sizes, b.indptr, k, ctx->local_of, pos_base, b.indices,
                                                                                                          relabel_grid, row_info_args(l - 1, next_dst))));
        } else if (l > 0) {
            side.relabel_blocks = relabel_grid;
            side.seed_bits = seeds_here ? seed_bits : nullptr;
            side.nbr = nbr;
            side.sizes = b.sizes;
            side.indptr = b.indptr;
            side.fanout = k;
            side.local_of = ctx->local_of;
            side.pos_base = pos_base;
            side.indices = b.indices;
            side.clear = clear;
            side.nclear = ctx->bitmap_words;
        } else {
            MQG_LAUNCH(ctx, "k_relabel", s, (k_relabel<<<relabel_grid, kBlock, 0, s>>>(nbr, b.sizes, b.indptr, k, ctx->local_of, pos_base, b.indices,
                                                                                       clear, ctx->bitmap_words, ctx->heavy_count)));
        }
        need_dst = next_dst;
    }
    if (take_back) {
        int grid = static_cast<int>(std::min<int64_t>(std::max<int64_t>(1, ceil_div(need_dst, kBlock)), 4096));
        MQG_LAUNCH(ctx, "k_reset_local", s,
                   (k_reset_local<IdxT><<<grid, kBlock, 0, s>>>(static_cast<const IdxT *>(blocks[0].src_ids), blocks[0].sizes, local_of)));
    }
    if (use_hash) MQG_LAUNCH(ctx, "k_clear_hubs", s, (k_clear_hubs<<<1, kBlock, 0, s>>>(ctx->heavy_count)));
    if (use_hash) return hash_clear(ctx, s);
    return MQG_OK;
}

}  // namespace

// Positions of nodes in a block's source list are kept in local_of with an offset that grows from call to call, so that
// what earlier calls left there is told from this call's by its size: a node of which local_of holds less than
// the call's offset is not in the list.  (Before, the last launch of every call set the entries back: 8 of 183 us on a
// graph of 111 M nodes, 14 of 318 for 1.35 M sources, one launch of eight for small calls.)  When the offsets run out,
// after 2^31 / count calls, the table is cleared once.  A call that is being recorded into a graph is replayed with the
// same offset again: it gets the range above all others and sets its entries back at its end, as does every call
// where two ranges do not fit.
int take_positions(mqg_ctx *ctx, int64_t count, hipStream_t s, int32_t *base, bool *take_back) {
    const int64_t end = int64_t(1) << 31;
    const int64_t most = std::max<int64_t>(ctx->num_nodes, ctx->max_src);   // no call needs more
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    const bool known = hipStreamIsCapturing(s, &status) == hipSuccess;
    if (!known) (void)hipGetLastError();
    if (!known || status != hipStreamCaptureStatusNone || 2 * most > end) {
        *base = static_cast<int32_t>(end - most);
        *take_back = true;
        return MQG_OK;
    }
    *take_back = false;
    if (ctx->pos_next + count > end - most) {
        const int grid = static_cast<int>(std::min<int64_t>(std::max<int64_t>(1, ceil_div(ctx->num_nodes, kBlock)), 8192));
        MQG_LAUNCH(ctx, "k_fill_i32", s, (k_fill_i32<<<grid, kBlock, 0, s>>>(ctx->local_of, ctx->num_nodes, -1, grid)));
        ctx->pos_next = 0;
    }
    *base = static_cast<int32_t>(ctx->pos_next);
    ctx->pos_next += count;
    return MQG_OK;
}

int launch_scan_tiles(mqg_ctx *ctx, int32_t *vals, int64_t n, const int64_t *addend, int64_t *total_a,
                      int64_t *total_b, hipStream_t s, const char *name, int64_t most) {
    MQG_LAUNCH(ctx, name, s, (k_scan_tiles<<<1, 1024, 0, s>>>(vals, n, addend, total_a, total_b, most)));
    return MQG_OK;
}

int run_sample_blocks(mqg_ctx *ctx, const mqg_graph *g, const void *seeds, int32_t num_seeds, const int32_t *fanouts,
                      int32_t L, uint64_t rng_seed, const uint64_t *seed_dev, mqg_block *blocks, hipStream_t s) {
    const bool p64 = g->ptr_type == MQG_I64, i64 = g->idx_type == MQG_I64;
    if (p64 && i64) return sample_blocks_impl<int64_t, int64_t>(ctx, g, seeds, num_seeds, seed_dev, fanouts, L, rng_seed, blocks, s);
    if (p64 && !i64) return sample_blocks_impl<int64_t, int32_t>(ctx, g, seeds, num_seeds, seed_dev, fanouts, L, rng_seed, blocks, s);
    if (!p64 && i64) return sample_blocks_impl<int32_t, int64_t>(ctx, g, seeds, num_seeds, seed_dev, fanouts, L, rng_seed, blocks, s);
    return sample_blocks_impl<int32_t, int32_t>(ctx, g, seeds, num_seeds, seed_dev, fanouts, L, rng_seed, blocks, s);
}

int run_select_row_candidates(mqg_ctx *ctx, const uint64_t *keys, const uint32_t *slot_words, int32_t cnt, int32_t k,
                              int32_t prioritised, int32_t ordered, uint32_t *out_mask, hipStream_t s) {
    if (prioritised) MQG_LAUNCH(ctx, "k_select_candidates", s, (k_select_candidates<true><<<1, kWave, 0, s>>>(keys, slot_words, cnt, k, ordered, out_mask)));
    else MQG_LAUNCH(ctx, "k_select_candidates", s, (k_select_candidates<false><<<1, kWave, 0, s>>>(keys, slot_words, cnt, k, ordered, out_mask)));
    return MQG_OK;
}

// the membership bitmap and the table of cached-neighbour counts
int ensure_priority_scratch(mqg_ctx *ctx) {
    if (ctx->prio_bitmap) return MQG_OK;
    bool ok = hipMalloc(reinterpret_cast<void **>(&ctx->prio_bitmap), static_cast<size_t>(ctx->bitmap_words) * sizeof(uint32_t)) == hipSuccess &&
              hipMalloc(reinterpret_cast<void **>(&ctx->prio_count), static_cast<size_t>(std::max<int64_t>(ctx->num_nodes, 1)) * sizeof(int32_t)) == hipSuccess;
    if (!ok) {
        (void)hipFree(ctx->prio_bitmap);
        (void)hipFree(ctx->prio_count);
        ctx->prio_bitmap = nullptr;
        ctx->prio_count = nullptr;
        return fail(ctx, MQG_ERR_HIP, "mqg_ctx_set_sampling_priority: allocation failed");
    }
    return MQG_OK;
}

// cache == nullptr switches the priority off; otherwise the membership bitmap is (re)built from cache->slot_of
int run_set_sampling_priority(mqg_ctx *ctx, const mqg_graph *g, const mqg_cache *cache, hipStream_t s) {
    if (!cache) {
        ctx->prio_enabled = false;
        return MQG_OK;
    }
    int rc0 = ensure_priority_scratch(ctx);
    if (rc0 != MQG_OK) return rc0;
    const int grid = static_cast<int>(ctx->bitmap_words * 32 / kBlock);
    MQG_LAUNCH(ctx, "k_prio_bitmap", s, (k_prio_bitmap<<<grid, kBlock, 0, s>>>(cache->slot_of, ctx->num_nodes, ctx->prio_bitmap)));
    const int64_t n = ctx->num_nodes;
    const int ngrid = static_cast<int>(std::max<int64_t>(1, ceil_div(n, kBlock)));
#define MQG_PRIOC(PT, IT)                                                                                        \
    MQG_LAUNCH(ctx, "k_prio_counts", s,                                                                          \
               (k_prio_counts<PT, IT><<<ngrid, kBlock, 0, s>>>(static_cast<const PT *>(g->row_ptr),               \
                                                              static_cast<const IT *>(g->col_idx), n, ctx->prio_bitmap, \
                                                              ctx->prio_count)))
    if (g->ptr_type == MQG_I64 && g->idx_type == MQG_I64) MQG_PRIOC(int64_t, int64_t);
    else if (g->ptr_type == MQG_I64) MQG_PRIOC(int64_t, int32_t);
    else if (g->idx_type == MQG_I64) MQG_PRIOC(int32_t, int64_t);
    else MQG_PRIOC(int32_t, int32_t);
#undef MQG_PRIOC
    ctx->prio_enabled = true;
    return MQG_OK;
}

}  // namespace mqg
