// Layer-wise sampling after LADIES (paper Sec. III-B, Eq. 6-9): the nodes of the next layer are
// drawn from the neighbours of the current layer's nodes (and these nodes themselves: A + I) with
// probability proportional to the squared column norm of the row-selected normalised adjacency
// P = D^-1/2 (A + I) D^-1/2, and a drawn node's column is scaled by 1 / (s p) (Eq. 8).
//
// Per block, for the rows D (the seeds, then the previous block's drawn nodes):
//   k_lw_mass        mass[i] += floor(2^40 / (deg_v + 1)) for every row v and every i in N(v) or
//                    i == v: integer atomics, so the sums do not depend on the schedule.
//                    q_i = mass[i] / (deg_i + 1) is 2^40 times the squared column norm of Eq. 7.
//                    Touched nodes are marked in the context's node bitmap - slot by slot on graphs
//                    above kMassScanNodes nodes, otherwise by k_lw_mass_bits from the masses.
//   bitmap -> list   the candidates (Eq. 6), ascending: set bits counted per tile (by k_lw_mass_bits
//                    itself, else k_lw_tile_counts), then k_lw_emit, whose workgroups add up the
//                    counts of the tiles before their own
//   k_lw_keys        exponential race: key = ticket * (deg_i + 1) / mass[i] in doubles (the "flat"
//                    variants, Eq. 10, draw in proportion to sqrt(q_i): ticket^2 in place of ticket), ticket from
//                    exp_ticket64; partial sums of q per workgroup, added up in a fixed order
//   layers of up to kPickMost nodes:
//   k_lw_list        the keys' leading bits, sixteen bins to the octave, are counted by k_lw_keys itself; this
//                    launch finds the threshold's bin and lists the nodes of the bins before it and of the bin
//   k_lw_pick        ranks the bin's nodes by (key, id) and all that are drawn by id: the block's sources,
//                    their positions into local_of[], their columns' share of the weights
//   larger layers:
//   k_lw_select      radix select of the s-th smallest 64-bit key pattern, most significant digit
//                    first: the leading 12 bits are counted by k_lw_keys itself, the next 13 by
//                    this launch, whose workgroups derive the digit found so far from the
//                    histogram before
//   k_lw_mark        derives the threshold's 25 leading bits; keys below them are marked in the
//                    bitmap, keys that share them (a few dozen) are listed (all candidates are
//                    marked if there are at most s)
//   k_lw_finish      one workgroup ranks the listed keys by (key, id) and marks as many as are
//                    still wanted (a long list - many equal keys - by a radix select of its own)
//   bitmap -> list   the drawn nodes ascending = the block's sources, positions into local_of[]
//   k_lw_count/fill  row v lists the drawn nodes among v and its adjacency row (self edge first,
//                    then slot order) with weight P_vi / (s p_i), optionally divided by the row sum;
//                    k_lw_fill also writes indptr and the block's sizes, k_lw_count sets the masses and the
//                    histogram back to zero
// A row is shared by kRowChunks wavefronts, each with a contiguous range of adjacency slots, so
// that a hub does not become a kernel's tail.
//   k_lw_drawn_keys / k_lw_draw_order / k_lw_debias   (the "+debias" variants, Eq. 12) the drawn nodes in
//                    the order of the race and their debiased coefficients, three scans in one workgroup
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "device_utils.h"
#include "radix.h"

namespace mqg {

namespace {

constexpr uint64_t kGolden = 0x9E3779B97F4A7C15ULL;
constexpr int kLayerwiseTag = 64;
constexpr int64_t kMassScanNodes = int64_t(8) << 20;   // up to here the candidates are read off the masses
constexpr int64_t kDenseNodes = int64_t(1) << 20;      // up to here every node has a key slot: no candidate list

uint64_t host_mix64(uint64_t z) {
    z ^= z >> 30;
    z *= 0xBF58476D1CE4E5B9ULL;
    z ^= z >> 27;
    z *= 0x94D049BB133111EBULL;
    z ^= z >> 31;
    return z;
}

__device__ __forceinline__ void set_bit(uint32_t *bitmap, uint32_t i) {
    uint32_t *w = bitmap + (i >> 5);
    const uint32_t bit = 1u << (i & 31);
    if (!(__hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit))
        (void)__hip_atomic_fetch_or(w, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// the caller's seeds, checked: an id outside the graph is replaced by node 0 and flagged (FastGCN; the other
// methods do it in k_lw_mass)
template <typename IdxT>
__global__ void __launch_bounds__(kBlock)
k_lw_seeds(const IdxT *__restrict__ seeds, int64_t n, int64_t num_nodes, IdxT *__restrict__ dst, int64_t *sizes,
           int32_t *__restrict__ flags) {
    const int64_t t = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (t == 0) sizes[0] = n;
    if (t >= n) return;
    IdxT v = seeds[t];
    if (v < 0 || static_cast<int64_t>(v) >= num_nodes) {
        v = 0;
        atomicOr(flags, 1);
    }
    dst[t] = v;
}

// A row is shared by kRowChunks wavefronts, each with a contiguous range of adjacency slots: LEAST, or
// more where the row is longer than all chunks of that size.
constexpr int kRowChunks = 16;
constexpr int kSlotUnroll = 4;      // groups of 64 slots whose loads are issued together

template <int LEAST>
__device__ __forceinline__ void chunk_range(int64_t d, int c, int64_t *begin, int64_t *end) {
    int64_t len = ((d + kRowChunks - 1) / kRowChunks + kWave - 1) / kWave * kWave;
    len = len < LEAST ? LEAST : len;
    *begin = len * c < d ? len * c : d;
    *end = len * (c + 1) < d ? len * (c + 1) : d;
}

// The ticket of node i (integer below 2^39, exact in a double).
__device__ __forceinline__ double lw_ticket(uint64_t tag_hash, int64_t i) {
    return static_cast<double>(exp_ticket64(mix64(mix64(tag_hash ^ static_cast<uint64_t>(i)))));
}

// The rows are the seeds (n_seeds >= 0: checked here and written to `checked`), a block's destinations, or, without
// a list, every node of the graph.  Bound by the atomics (23 G/s); a hub's chunk of more than a thousand slots is a
// chain of loads, four groups at a time.  The workgroups past `grid` make the tickets of all nodes, 32 squarings each, while the
// atomics of the others are under way: they add nothing (first in the grid 2 us) and take 3.5 of k_lw_keys' 11.7 us away.
template <typename PtrT, typename IdxT>
__global__ void __launch_bounds__(kBlock)
k_lw_mass(const PtrT *__restrict__ row_ptr, const IdxT *__restrict__ col_idx, const IdxT *__restrict__ dst,
          int64_t *sizes, int64_t n_seeds, int64_t num_nodes, IdxT *__restrict__ checked, int32_t *__restrict__ flags,
          unsigned long long *__restrict__ mass, uint32_t *__restrict__ bitmap, int64_t *__restrict__ zero_me, int grid,
          uint64_t tag_hash, double *__restrict__ tickets) {
    const int lane = lane_id();
    const int block = static_cast<int>(blockIdx.x);
    if (block >= grid) {
        const int64_t i = int64_t(block - grid) * kBlock + threadIdx.x;
        if (i < num_nodes) tickets[i] = lw_ticket(tag_hash, i);
        return;
    }
    if (block == 0 && threadIdx.x == 0) {
        if (zero_me) *zero_me = 0;                         // the candidate count k_lw_keys adds up
        if (n_seeds >= 0) sizes[0] = n_seeds;
    }
    const int64_t n = (n_seeds >= 0 ? n_seeds : sizes[0]) * kRowChunks;
    const int64_t wave0 = int64_t(block) * kWavesPerBlock + (threadIdx.x >> 6);
    const int64_t nwaves = int64_t(grid) * kWavesPerBlock;
    for (int64_t u = wave0; u < n; u += nwaves) {
        const int64_t t = u / kRowChunks;
        const int c = static_cast<int>(u % kRowChunks);
        int64_t v = dst ? static_cast<int64_t>(dst[t]) : t;
        if (n_seeds >= 0) {
            const bool bad = v < 0 || v >= num_nodes;
            if (bad) v = 0;
            if (c == 0 && lane == 0) {
                checked[t] = static_cast<IdxT>(v);
                if (bad) atomicOr(flags, 1);
            }
        }
        const int64_t start = static_cast<int64_t>(row_ptr[v]);
        const int64_t d = static_cast<int64_t>(row_ptr[v + 1]) - start;
        const unsigned long long add = (1ull << 40) / static_cast<unsigned long long>(d + 1);
        if (c == 0 && lane == 0) {
            atomicAdd(&mass[v], add);
            if (bitmap) set_bit(bitmap, static_cast<uint32_t>(v));
        }
        int64_t jb, je;
        chunk_range<kWave>(d, c, &jb, &je);
        for (int64_t j0 = jb + lane; j0 < je; j0 += kSlotUnroll * kWave) {
            uint32_t id[kSlotUnroll];
#pragma unroll
            for (int q = 0; q < kSlotUnroll; ++q) {
                const int64_t j = j0 + q * kWave;
                id[q] = static_cast<uint32_t>(col_idx[start + (j < je ? j : j0)]);
            }
#pragma unroll
            for (int q = 0; q < kSlotUnroll; ++q) {
                if (j0 + q * kWave >= je) continue;
                atomicAdd(&mass[id[q]], add);
                if (bitmap) set_bit(bitmap, id[q]);
            }
        }
    }
}

// Bitmap -> ascending list, two launches: the set bits of every tile are counted, then every tile's
// workgroup adds up the counts of the tiles before its own and writes its ids.  A tile is
// kBlock * WPT words (WPT = 1 up to 32 M nodes, ids staged through LDS and written coalesced;
// otherwise 4, one 16-byte load per thread, ids written from the bit loop: those bitmaps are sparse).
constexpr int kMassTileNodes = kBlock * 32;          // nodes behind one tile of kBlock words
constexpr int kEmitFewTiles = 32, kEmitParts = 8;    // see k_lw_emit

// The touched nodes from the masses themselves (bit i = mass[i] != 0), for graphs small enough that
// reading every mass costs less than marking a bit per adjacency slot in k_lw_mass; the same launch
// counts the tile (WPT = 1).  In round r thread t looks at node tile * 8192 + r * 256 + t, so the
// ballot of a wavefront is the word pair r * 8 + 2 * wave of the tile.
__global__ void __launch_bounds__(kBlock)
k_lw_mass_bits(const unsigned long long *__restrict__ mass, int64_t n, uint32_t *__restrict__ bitmap,
               int32_t *__restrict__ tile_sums) {
    __shared__ unsigned long long pairs[kBlock / 2];
    __shared__ int lds[kWavesPerBlock];
    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    const int64_t base = int64_t(blockIdx.x) * kMassTileNodes + tid;
    unsigned long long v[32];
#pragma unroll
    for (int r = 0; r < 32; ++r) {
        const int64_t i = base + r * kBlock;
        v[r] = i < n ? mass[i] : 0ull;
    }
    int cnt = 0;
#pragma unroll
    for (int r = 0; r < 32; ++r) {
        const uint64_t m = ballot64(v[r] != 0);
        cnt += popc64(m);
        if (lane_id() == 0) pairs[r * kWavesPerBlock + wave] = m;
    }
    if (lane_id() == 0) lds[wave] = cnt;
    __syncthreads();
    bitmap[int64_t(blockIdx.x) * kBlock + tid] = reinterpret_cast<const uint32_t *>(pairs)[tid];
    if (tid == 0) {
        int t = 0;
#pragma unroll
        for (int k = 0; k < kWavesPerBlock; ++k) t += lds[k];
        tile_sums[blockIdx.x] = t;
    }
}

template <int WPT>
__global__ void __launch_bounds__(kBlock)
k_lw_tile_counts(const uint32_t *__restrict__ bitmap, int32_t *__restrict__ tile_sums) {
    __shared__ int lds[kWavesPerBlock];
    const int64_t w0 = (int64_t(blockIdx.x) * kBlock + threadIdx.x) * WPT;
    int c;
    if (WPT == 4) {
        const uint4 w = *reinterpret_cast<const uint4 *>(bitmap + w0);
        c = __popc(w.x) + __popc(w.y) + __popc(w.z) + __popc(w.w);
    } else {
        c = __popc(bitmap[w0]);
    }
    const int s = wave_sum(c);
    if (lane_id() == 0) lds[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
#pragma unroll
        for (int k = 0; k < kWavesPerBlock; ++k) t += lds[k];
        tile_sums[blockIdx.x] = t;
    }
}

// What a drawn node's column contributes to the weights of its edges: Eq. 8 with p_i = q_i / q_total,
// q_i = mass_i / di, gives P_vi / (s p_i) = (q_total / s) / sqrt(dv) * f_i with f_i = di / (mass_i sqrt(di)); flat
// (p_i = sqrt(q_i) / total): f_i = 1 / (sqrt(q_i) sqrt(di)).  With debiased coefficients (paper Eq. 12) the weight is
// beta_i / sqrt(dv di): 1 / sqrt(di) here, and k_lw_debias multiplies by beta_i.
struct LwColumns {
    const void *row_ptr;                 // of PtrT
    const unsigned long long *mass;
    int flat, debias;
    double *factor;                      // [sources]; null: a list of candidates, no factors
    template <typename PtrT, int U>
    __device__ __forceinline__ void values(const int32_t (&i)[U], double (&f)[U]) const {
        const PtrT *rp = static_cast<const PtrT *>(row_ptr);
        PtrT begin[U], end[U];
        unsigned long long m[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            begin[u] = rp[i[u]];
            end[u] = rp[int64_t(i[u]) + 1];
            m[u] = mass[i[u]];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double di = static_cast<double>(static_cast<int64_t>(end[u]) - static_cast<int64_t>(begin[u]) + 1);
            const double mi = static_cast<double>(m[u]);
            f[u] = debias ? 1.0 / sqrt(di) : flat ? 1.0 / (sqrt(mi / di) * sqrt(di)) : di / (mi * sqrt(di));
        }
    }
    template <typename PtrT>
    __device__ __forceinline__ double value(int64_t i) const {
        const int32_t node[1] = {static_cast<int32_t>(i)};
        double f[1];
        values<PtrT, 1>(node, f);
        return f[0];
    }
};

template <typename PtrT, int U, typename OutT>
__device__ __forceinline__ void lw_emit_nodes(const int32_t *staged, int total, int part, int parts, int tile_base, OutT *__restrict__ out,
                                              int32_t *__restrict__ local_of, int32_t pos_base, const LwColumns &columns) {
    const int step = parts * kBlock;
    for (int k0 = part * kBlock + threadIdx.x; k0 < total; k0 += U * step) {
        int32_t v[U];
        double f[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = staged[k0 + u * step < total ? k0 + u * step : k0];
        if (columns.factor) columns.values<PtrT, U>(v, f);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + u * step;
            if (k >= total) break;
            out[tile_base + k] = static_cast<OutT>(v[u]);
            if (local_of) local_of[v[u]] = pos_base + tile_base + k;
            if (columns.factor) columns.factor[tile_base + k] = f[u];
        }
    }
}

// ids of the set bits, ascending, into out[0..total); the words are cleared (with several workgroups a tile: later, by
// k_lw_count); total to count_a/b.
// parts (WPT = 1): workgroups that share a tile's ids: on small graphs there are few tiles, and a node's factor is two loads and a
// double division and square root (10 k of 20 k nodes in 3 workgroups 11 us).
// scanned: tile_vals holds the exclusive scan of the tile counts, otherwise the counts themselves.
template <typename PtrT, typename OutT, int WPT>
__global__ void __launch_bounds__(kBlock)
k_lw_emit(uint32_t *__restrict__ bitmap, const int32_t *__restrict__ tile_vals, int scanned, OutT *__restrict__ out,
          int32_t *__restrict__ local_of, int32_t pos_base, LwColumns columns, int64_t *count_a, int64_t *count_b, int tiles, int parts) {
    __shared__ int lds[kWavesPerBlock];
    __shared__ int32_t staged[WPT == 1 ? kBlock * 32 : 1];   // every id of the tile, ascending
    const int tile = WPT == 1 ? static_cast<int>(blockIdx.x) / parts : static_cast<int>(blockIdx.x);
    const int part = static_cast<int>(blockIdx.x) - tile * parts;
    const int tile_base = scanned ? tile_vals[tile] : tiles_before(tile_vals, lds, tile);
    const int64_t w0 = (int64_t(tile) * kBlock + threadIdx.x) * WPT;
    uint32_t words[WPT];
    if constexpr (WPT == 4) {
        const uint4 w = *reinterpret_cast<const uint4 *>(bitmap + w0);
        words[0] = w.x;
        words[1] = w.y;
        words[2] = w.z;
        words[3] = w.w;
    } else {
        words[0] = bitmap[w0];
    }
    int c = 0;
#pragma unroll
    for (int q = 0; q < WPT; ++q) c += __popc(words[q]);
    int total;
    int ex = block_excl_scan<kWavesPerBlock>(c, &total, lds);
    if (tile == tiles - 1 && part == 0 && threadIdx.x == 0) {
        const int64_t all = int64_t(tile_base) + total;
        if (count_a) *count_a = all;
        if (count_b) *count_b = all;
    }
    if (total == 0) return;                                // workgroup-uniform
    if constexpr (WPT == 1) {
        if (c) {
            if (parts == 1) bitmap[w0] = 0;
            const int32_t v0 = static_cast<int32_t>(w0 * 32);
            uint32_t bits = words[0];
            while (bits) {
                const int b = __ffs(bits) - 1;
                bits &= bits - 1;
                staged[ex++] = v0 + b;
            }
        }
        __syncthreads();
        // nodes whose loads are issued together, where the tile has as many
        if (total > parts * kBlock) lw_emit_nodes<PtrT, 4>(staged, total, part, parts, tile_base, out, local_of, pos_base, columns);
        else lw_emit_nodes<PtrT, 1>(staged, total, part, parts, tile_base, out, local_of, pos_base, columns);
    } else {
        if (c == 0) return;
        int32_t pos = tile_base + ex;
#pragma unroll
        for (int q = 0; q < WPT; ++q) {
            uint32_t bits = words[q];
            if (!bits) continue;
            bitmap[w0 + q] = 0;
            while (bits) {
                const int b = __ffs(bits) - 1;
                bits &= bits - 1;
                const int64_t v = (w0 + q) * 32 + b;
                out[pos] = static_cast<OutT>(v);
                if (local_of) local_of[v] = pos_base + pos;
                if (columns.factor) columns.factor[pos] = columns.value<PtrT>(v);
                ++pos;
            }
        }
    }
}

// The race key of a candidate and the measure its probability is proportional to.  Plain: rate
// q = mass / (deg + 1).  Flat (paper Eq. 10: in proportion to the column norm, not its square): rate
// sqrt(q); the race compares ticket / sqrt(q), and squaring that keeps the order with nothing but
// multiplications and one division, each rounded once, as the CPU statement of the same steps does.
__device__ __forceinline__ double lw_race_key(double ticket, double deg1, double m, int flat) {
    return flat ? ((ticket * ticket) * deg1) / m : (ticket * deg1) / m;
}
__device__ __forceinline__ double lw_measure(double m, double deg1, int flat) {
    const double q = m / deg1;
    return flat ? sqrt(q) : q;
}

// Radix select of the s-th smallest 64-bit key pattern: kSelPasses counting passes over all keys, most
// significant digit first - the top 12 bits (sign and exponent of a double), then 13 bits; what
// is left undecided after these 25 bits is a short list (k_lw_mark, k_lw_finish).
constexpr int kSelPasses = 2;
constexpr int kSelBins = 8192;
constexpr int kSelHistLen = kSelPasses * kSelBins;
__host__ __device__ constexpr int sel_shift(int pass) { return 52 - 13 * pass; }

// Layers of up to kPickMost nodes take k_lw_list and k_lw_pick, two launches (6.6 and 6.4 us for 512 of 233 k nodes) in place of
// five (select 7.1, mark 6.8, finish 3.9, tile counts 2.7, list 3.4).  k_lw_pick compares every id with every other: whole calls
// with two layers of 2,048 nodes 0.90 to 0.98 of the time of the other way, of 4,096 1.0 to 1.16.  Bins of a sixteenth of an octave, so that the threshold's bin holds at most
// about a sixteenth of the nodes drawn.  The bin ascends with the key whatever the key; the race keys lie in
// 2^-62 .. 2^98, well inside.
constexpr int kPickMost = 2048;
constexpr int kFineBins = 4096;
__device__ __forceinline__ int fine_bin(uint64_t key) {
    const int b = static_cast<int>(key >> 48) - ((1023 - 128) << 4);
    return b < 0 ? 0 : b < kFineBins ? b : kFineBins - 1;
}

// Race keys of the candidates and the per-workgroup partial sums of q (a fixed launch shape, so the
// sums are the same from run to run); the keys are counted into hist[0..4096): by fine_bin (fine), or by
// their leading 12 bits, the first pass of the radix select.  have_tickets: key64[i] holds node i's ticket.  (A wavefront per SIMD, 256 workgroups of 256, left
// the 32 squarings of a ticket a bare chain.  233 k nodes 11.7 us, 8.1 with the tickets at hand; what is left is the chain of loads,
// the LDS counts and their way into hist.)  Candidates: cand[0..n) if given, otherwise the nodes 0..n-1
// themselves, of which those with no mass are none (key = all ones, not counted); their number is
// added to *count_out then.  n = *n_dev if given, else n_fixed.  hist must be clear.
constexpr uint64_t kNoKey = ~uint64_t(0);
constexpr int kKeyThreads = 1024;          // at most; `threads` of them: as many wavefronts per SIMD as the nodes give all compute units
template <typename PtrT>
__global__ void __launch_bounds__(kKeyThreads)
k_lw_keys(const PtrT *__restrict__ row_ptr, const int32_t *__restrict__ cand, const int64_t *__restrict__ n_dev, int64_t n_fixed,
          const unsigned long long *__restrict__ mass, uint64_t tag_hash, int flat, uint64_t *__restrict__ key64,
          double *__restrict__ q_part, int32_t *__restrict__ hist, int64_t *__restrict__ count_out,
          unsigned long long *__restrict__ state, int64_t layer_size, unsigned long long *__restrict__ bcount, int fine, int grid, int threads, int have_tickets,
          int32_t *__restrict__ row_count, int64_t row_counts) {
    constexpr int kWaves = kKeyThreads / kWave;
    __shared__ double lds[kWaves];
    __shared__ int cnt_lds[kWaves];
    __shared__ int h[4096];
    if (blockIdx.x == 0 && threadIdx.x == 0) {             // the select's state before its first pass
        state[0] = 0;
        state[1] = static_cast<unsigned long long>(layer_size);
        *bcount = 0;                                       // the boundary list is empty
    }
    const int64_t n = n_dev ? *n_dev : n_fixed;
    const int64_t stride = int64_t(grid) * threads;
    for (int64_t k = int64_t(blockIdx.x) * threads + threadIdx.x; k < row_counts; k += stride) row_count[k] = 0;      // for k_lw_count
    for (int d = threadIdx.x; d < 4096; d += threads) h[d] = 0;
    __syncthreads();
    double q = 0.0;
    int cnt = 0;
    for (int64_t c = int64_t(blockIdx.x) * threads + threadIdx.x; c < n; c += stride) {
        const int64_t i = cand ? cand[c] : c;
        const unsigned long long mi = mass[i];
        if (mi == 0) {
            key64[c] = kNoKey;
            continue;
        }
        const double deg1 = static_cast<double>(static_cast<int64_t>(row_ptr[i + 1]) - static_cast<int64_t>(row_ptr[i]) + 1);
        const double m = static_cast<double>(mi);
        const double ticket = have_tickets ? __longlong_as_double(static_cast<long long>(key64[c])) : lw_ticket(tag_hash, i);
        const uint64_t key = static_cast<uint64_t>(__double_as_longlong(lw_race_key(ticket, deg1, m, flat)));
        key64[c] = key;
        atomicAdd(&h[fine ? fine_bin(key) : static_cast<int>(key >> 52)], 1);
        q += lw_measure(m, deg1, flat);
        ++cnt;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) q += __shfl_xor(q, off, 64);
    cnt = wave_sum(cnt);
    if (lane_id() == 0) {
        lds[threadIdx.x >> 6] = q;
        cnt_lds[threadIdx.x >> 6] = cnt;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double sum = 0.0;
        int total = 0;
        for (int w = 0; w < threads / kWave; ++w) {
            sum += lds[w];
            total += cnt_lds[w];
        }
        q_part[blockIdx.x] = sum;
        if (count_out && total) atomicAdd(reinterpret_cast<unsigned long long *>(count_out), static_cast<unsigned long long>(total));
    }
    for (int d = threadIdx.x; d < 4096; d += threads)
        if (h[d]) atomicAdd(&hist[d], h[d]);
}

// q_total = sum of the partial sums, in a fixed order (one workgroup; `lds` needs kBlock doubles)
__device__ __forceinline__ void lw_sum_parts(const double *__restrict__ q_part, int parts, double *__restrict__ q_total, double *lds) {
    double a = 0.0;
    for (int k = threadIdx.x; k < parts; k += kBlock) a += q_part[k];
    lds[threadIdx.x] = a;
    __syncthreads();
    for (int off = kBlock / 2; off > 0; off >>= 1) {
        if (static_cast<int>(threadIdx.x) < off) lds[threadIdx.x] += lds[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) *q_total = lds[0];
}

// The state of the select before pass `pass`:
//   st[0] = the digits chosen in the passes before, most significant first, as the low bits of a word
//   st[1] = how many of the keys with that prefix are still wanted
// derived from the state before the previous pass (state[2(pass-1)], state[2(pass-1)+1]) and that
// pass's histogram: the first digit at which the running count reaches the wanted number.  Every
// thread of the workgroup calls it; st[] is valid after the next __syncthreads().  If fewer keys
// exist than are wanted no digit qualifies and st stays {0, 0}.
__device__ __forceinline__ void sel_derive(const unsigned long long *__restrict__ state, const int32_t *__restrict__ hist,
                                           int64_t layer_size, int pass, unsigned long long *st, int *lds) {
    const int tid = threadIdx.x;
    if (pass == 0) {
        if (tid == 0) {
            st[0] = 0;
            st[1] = static_cast<unsigned long long>(layer_size);
        }
        return;
    }
    if (tid == 0) {
        st[0] = 0;
        st[1] = 0;
    }
    const unsigned long long prefix = state[2 * (pass - 1)];
    const long long want = static_cast<long long>(state[2 * (pass - 1) + 1]);
    constexpr int kPer = kSelBins / kBlock;                // consecutive digits per thread
    const int4 *hp = reinterpret_cast<const int4 *>(hist + int64_t(pass - 1) * kSelBins + tid * kPer);
    int v[kPer];
    int c = 0;
#pragma unroll
    for (int q = 0; q < kPer / 4; ++q) {
        const int4 x = hp[q];
        v[4 * q] = x.x;
        v[4 * q + 1] = x.y;
        v[4 * q + 2] = x.z;
        v[4 * q + 3] = x.w;
        c += x.x + x.y + x.z + x.w;
    }
    int total;
    const int before = block_excl_scan<kWavesPerBlock>(c, &total, lds);   // its barriers order the stores to st[] above
    // exactly one digit has before < want <= before + count (if 1 <= want <= total)
    if (before < want && want <= static_cast<long long>(before) + c) {
        long long run = before;
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            if (run < want && want <= run + v[q]) {
                st[0] = (prefix << 13) | static_cast<unsigned long long>(tid * kPer + q);
                st[1] = static_cast<unsigned long long>(want - run);
            }
            run += v[q];
        }
    }
}

// Counting pass `pass` of the select: the keys that carry the prefix found so far are counted by
// their next digit, per workgroup in LDS and then into hist[pass].  Workgroup 0 stores the state.
__global__ void __launch_bounds__(kBlock)
k_lw_select(const uint64_t *__restrict__ key64, const int64_t *__restrict__ n_dev, int64_t n_fixed, int64_t layer_size,
            unsigned long long *__restrict__ state, int32_t *__restrict__ hist, int pass) {
    __shared__ int lds[kWavesPerBlock];
    __shared__ int h[kSelBins];
    __shared__ unsigned long long st[2];
    const int tid = threadIdx.x;
    sel_derive(state, hist, layer_size, pass, st, lds);
#pragma unroll
    for (int q = 0; q < kSelBins / kBlock; ++q) h[q * kBlock + tid] = 0;
    __syncthreads();
    if (blockIdx.x == 0 && tid == 0) {
        state[2 * pass] = st[0];
        state[2 * pass + 1] = st[1];
    }
    const unsigned long long prefix = st[0];
    const int shift = sel_shift(pass);
    const int64_t n = n_dev ? *n_dev : n_fixed;
    const int64_t stride = int64_t(gridDim.x) * kBlock;
    int mine = 0;
    for (int64_t c = int64_t(blockIdx.x) * kBlock + tid; c < n; c += stride) {
        const uint64_t k = key64[c];
        if (pass == 0 || (k >> (shift + 13)) == prefix) {
            atomicAdd(&h[(k >> shift) & (kSelBins - 1)], 1);
            mine = 1;
        }
    }
    if (!__syncthreads_or(mine)) return;                   // no key of this workgroup carries the prefix
#pragma unroll
    for (int q = 0; q < kSelBins / kBlock; ++q) {
        const int d = q * kBlock + tid;
        if (h[d]) atomicAdd(&hist[pass * kSelBins + d], h[d]);
    }
}

// n keys (*n_dev if given, else n_fixed), of which *n_cand are candidates (all of them without
// n_cand; with skip_no_key the keys equal to kNoKey are none).
// After the two counting passes 25 leading bits of the threshold are known (every workgroup derives
// them from the second histogram; workgroup 0 stores them and the number of keys still wanted among
// those that share them in state[4], state[5]).  Keys with smaller leading bits are marked.  Keys with
// these leading bits - a few dozen of random keys - go to the boundary list (key, position), which
// k_lw_finish settles.  Workgroup 0 also adds up the partial sums of q, if there are any.
constexpr int kSelKnownShift = 39;                        // bits below the two counted digits
__global__ void __launch_bounds__(kBlock)
k_lw_mark(const int32_t *__restrict__ cand, const uint64_t *__restrict__ key64, const int64_t *__restrict__ n_dev, int64_t n_fixed,
          const int64_t *__restrict__ n_cand, int skip_no_key, int64_t layer_size, unsigned long long *__restrict__ state,
          const int32_t *__restrict__ hist, uint32_t *__restrict__ bitmap, const double *__restrict__ q_part, int parts,
          double *__restrict__ q_total, uint64_t *__restrict__ bkey, int32_t *__restrict__ bpos,
          unsigned long long *__restrict__ bcount) {
    __shared__ double qlds[kBlock];
    __shared__ int lds[kWavesPerBlock];
    __shared__ unsigned long long st[2];
    if (q_part && blockIdx.x == 0) lw_sum_parts(q_part, parts, q_total, qlds);
    const int64_t n = n_dev ? *n_dev : n_fixed;            // keys
    const int64_t stride = int64_t(gridDim.x) * kBlock;
    if ((n_cand ? *n_cand : n) <= layer_size) {            // every candidate is drawn
        for (int64_t c = int64_t(blockIdx.x) * kBlock + threadIdx.x; c < n; c += stride)
            if (!skip_no_key || key64[c] != kNoKey) set_bit(bitmap, cand ? static_cast<uint32_t>(cand[c]) : static_cast<uint32_t>(c));
        return;
    }
    sel_derive(state, hist, layer_size, 2, st, lds);
    __syncthreads();
    const uint64_t lead = st[0];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        state[4] = st[0];
        state[5] = st[1];
    }
    const int lane = lane_id();
    const int64_t first = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    for (int64_t c0 = first - lane; c0 < n; c0 += stride) {          // whole wavefronts: the ballot below
        const int64_t c = c0 + lane;
        const uint64_t k = c < n ? key64[c] : kNoKey;
        const uint64_t kl = k >> kSelKnownShift;
        if (c < n && kl < lead) set_bit(bitmap, cand ? static_cast<uint32_t>(cand[c]) : static_cast<uint32_t>(c));
        const bool edge = c < n && kl == lead;
        const uint64_t m = ballot64(edge);
        if (m) {
            unsigned long long at = 0;
            if (lane == 0) at = atomicAdd(bcount, static_cast<unsigned long long>(popc64(m)));
            at = __shfl(at, 0, 64);
            if (edge) {
                const unsigned long long o = at + popc64(m & lanes_below(lane));
                bkey[o] = k;
                bpos[o] = static_cast<int32_t>(c);
            }
        }
    }
}

// Of the m (key, position) pairs of a list in memory, whose keys equal kp from bit `known` on (known = 64:
// nothing is known), the last of the `want` first ones in (key, position) order: 1 <= want <= m.  A radix select,
// eight bits at a time, over the key bits and, among the keys equal to the threshold, over the 32 position
// bits.  Every thread of the workgroup (256) calls it; h: 256 ints, lds: kWavesPerBlock, pick: 2.
__device__ __forceinline__ void lw_select_pairs(const uint64_t *__restrict__ bkey, const int32_t *__restrict__ bpos, int64_t m, long long want,
                                                uint64_t &kp, int known, uint32_t &pp, int *h, int *lds, long long *pick) {
    const int tid = threadIdx.x;
    int pknown = 32;
    pp = 0;
    while (known > 0 || pknown > 0) {
        const bool on_key = known > 0;
        const int shift = on_key ? ((known - 1) & ~7) : pknown - 8;
        h[tid] = 0;
        __syncthreads();
        for (int64_t e = tid; e < m; e += kBlock) {
            const uint64_t k = bkey[e];
            if (on_key) {
                if (known == 64 || (k >> known) == (kp >> known)) atomicAdd(&h[(k >> shift) & ((1 << (known - shift)) - 1)], 1);
            } else if (k == kp) {
                const uint32_t ps = static_cast<uint32_t>(bpos[e]);
                if (pknown == 32 || (ps >> pknown) == (pp >> pknown)) atomicAdd(&h[(ps >> shift) & 255], 1);
            }
        }
        __syncthreads();
        const int c = h[tid];
        int total;
        const int before = block_excl_scan<kWavesPerBlock>(c, &total, lds);
        if (before < want && want <= static_cast<long long>(before) + c) {      // exactly one digit
            pick[0] = tid;
            pick[1] = want - before;
        }
        __syncthreads();
        const uint64_t digit = static_cast<uint64_t>(pick[0]);
        want = pick[1];
        if (on_key) {
            kp |= digit << shift;
            known = shift;
        } else {
            pp |= static_cast<uint32_t>(digit) << shift;
            pknown = shift;
        }
        __syncthreads();                                   // pick[] and h[] are rewritten by the next pass
    }
}

// The boundary list: m keys that share the 25 known leading bits, of which the state[5] smallest in
// (key, position) order are drawn (positions ascend with the ids).  One workgroup.  Up to
// kBoundaryRanked entries: every entry counts the entries ahead of it.  More (many equal keys): lw_select_pairs.
constexpr int kBoundaryRanked = 1024;
__global__ void __launch_bounds__(kBlock)
k_lw_finish(const int32_t *__restrict__ cand, const int64_t *__restrict__ n_dev, int64_t n_fixed,
            const int64_t *__restrict__ n_cand, int64_t layer_size, const unsigned long long *__restrict__ state,
            const uint64_t *__restrict__ bkey, const int32_t *__restrict__ bpos, const unsigned long long *__restrict__ bcount,
            uint32_t *__restrict__ bitmap) {
    __shared__ uint64_t lk[kBoundaryRanked];
    __shared__ int32_t lp[kBoundaryRanked];
    __shared__ int h[256];
    __shared__ int lds[kWavesPerBlock];
    __shared__ long long pick[2];
    const int tid = threadIdx.x;
    const int64_t n = n_dev ? *n_dev : n_fixed;
    if ((n_cand ? *n_cand : n) <= layer_size) return;      // every candidate was drawn by k_lw_mark
    const int64_t m = static_cast<int64_t>(*bcount);
    const long long want = static_cast<long long>(state[5]);
    if (m <= kBoundaryRanked) {
        for (int e = tid; e < m; e += kBlock) {
            lk[e] = bkey[e];
            lp[e] = bpos[e];
        }
        __syncthreads();
        constexpr int PER = kBoundaryRanked / kBlock;
        uint64_t mk[PER];
        int32_t mp[PER];
        int rank[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int e = q * kBlock + tid;
            mk[q] = e < m ? lk[e] : 0;
            mp[q] = e < m ? lp[e] : 0;
            rank[q] = 0;
        }
        for (int j = 0; j < m; ++j) {
            const uint64_t ok = lk[j];
            const int32_t op = lp[j];
#pragma unroll
            for (int q = 0; q < PER; ++q) rank[q] += (ok < mk[q] || (ok == mk[q] && op < mp[q])) ? 1 : 0;
        }
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int e = q * kBlock + tid;
            if (e < m && rank[q] < want) set_bit(bitmap, cand ? static_cast<uint32_t>(cand[mp[q]]) : static_cast<uint32_t>(mp[q]));
        }
        return;
    }
    uint64_t kp = state[4] << kSelKnownShift;
    uint32_t pp;
    lw_select_pairs(bkey, bpos, m, want, kp, kSelKnownShift, pp, h, lds, pick);
    // kp, pp: the last drawn entry
    for (int64_t e = tid; e < m; e += kBlock) {
        const uint64_t k = bkey[e];
        const int32_t ps = bpos[e];
        if (k < kp || (k == kp && static_cast<uint32_t>(ps) <= pp)) set_bit(bitmap, cand ? static_cast<uint32_t>(cand[ps]) : static_cast<uint32_t>(ps));
    }
}

__global__ void __launch_bounds__(kBlock)
k_lw_zero_i32(int32_t *__restrict__ p, int64_t n) {
    const int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (i < n) p[i] = 0;
}

// Layers of up to kPickMost nodes.  hist holds the candidates' keys by fine_bin.  Every workgroup finds the threshold's
// bin (the first at which the running count reaches layer_size; past all bins if there are no more candidates
// than that) and classifies tiles of 1,024 keys: nodes of the bins before it are drawn and listed in `sure`,
// nodes of the bin go to the boundary list (key, id), of which *want are drawn.  One atomic per tile that
// has any: count = listed as sure | listed as boundary << 32 (zero before).  Workgroup 0 also adds up the partial
// sums of q and stores the number of candidates.
constexpr int kListItems = 4;
__global__ void __launch_bounds__(kBlock)
k_lw_list(const int32_t *__restrict__ cand, const uint64_t *__restrict__ key64, const int64_t *__restrict__ n_dev, int64_t n_fixed, int layer_size,
          const int32_t *__restrict__ hist, const double *__restrict__ q_part, int parts, double *__restrict__ q_total,
          int64_t *__restrict__ n_cand, int32_t *__restrict__ sure, uint64_t *__restrict__ bkey, int32_t *__restrict__ bpos,
          unsigned long long *__restrict__ count, unsigned long long *__restrict__ want, int grid) {
    __shared__ double qlds[kBlock];
    __shared__ int lds[kWavesPerBlock];
    __shared__ int totals[2][kWavesPerBlock];
    __shared__ unsigned long long base;
    __shared__ int threshold[2];
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    if (blockIdx.x == 0) lw_sum_parts(q_part, parts, q_total, qlds);
    const int64_t n = n_dev ? *n_dev : n_fixed;
    constexpr int kTile = kBlock * kListItems;
    uint64_t key[kListItems];                              // of the first tile, on their way already
    auto load = [&](int64_t t0) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < kListItems; ++q) {
            const int64_t c = t0 + q * kBlock + tid;
            key[q] = c < n ? key64[c] : kNoKey;
        }
    };
    load(int64_t(blockIdx.x) * kTile);
    {
        constexpr int kPer = kFineBins / kBlock;           // consecutive bins per thread
        const int4 *hp = reinterpret_cast<const int4 *>(hist + tid * kPer);
        int v[kPer], c = 0, all;
#pragma unroll
        for (int q = 0; q < kPer / 4; ++q) {
            const int4 x = hp[q];
            v[4 * q] = x.x;
            v[4 * q + 1] = x.y;
            v[4 * q + 2] = x.z;
            v[4 * q + 3] = x.w;
            c += x.x + x.y + x.z + x.w;
        }
        int run = block_excl_scan<kWavesPerBlock>(c, &all, lds);
        if (all <= layer_size) {
            if (tid == 0) {
                threshold[0] = kFineBins;
                threshold[1] = 0;
            }
        } else if (run < layer_size && layer_size <= run + c) {      // exactly one thread, and one of its bins
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                if (run < layer_size && layer_size <= run + v[q]) {
                    threshold[0] = tid * kPer + q;
                    threshold[1] = layer_size - run;
                }
                run += v[q];
            }
        }
        __syncthreads();
        if (blockIdx.x == 0 && tid == 0) {
            *n_cand = all;
            *want = static_cast<unsigned long long>(threshold[1]);
        }
    }
    const int bin = threshold[0];
    for (int64_t t0 = int64_t(blockIdx.x) * kTile; t0 < n; t0 += int64_t(grid) * kTile) {
        uint64_t sm[kListItems], bm[kListItems];
        int ns = 0, nb = 0;
#pragma unroll
        for (int q = 0; q < kListItems; ++q) {
            const int b = fine_bin(key[q]);
            sm[q] = ballot64(key[q] != kNoKey && b < bin);
            bm[q] = ballot64(key[q] != kNoKey && b == bin);
            ns += popc64(sm[q]);
            nb += popc64(bm[q]);
        }
        if (lane == 0) {
            totals[0][wave] = ns;
            totals[1][wave] = nb;
        }
        __syncthreads();
        if (tid == 0) {
            unsigned long long all = 0;
#pragma unroll
            for (int w = 0; w < kWavesPerBlock; ++w)
                all += static_cast<unsigned long long>(totals[0][w]) | static_cast<unsigned long long>(totals[1][w]) << 32;
            if (all) base = atomicAdd(count, all);
        }
        __syncthreads();
        uint32_t ps = static_cast<uint32_t>(base), pb = static_cast<uint32_t>(base >> 32);
        for (int w = 0; w < wave; ++w) {
            ps += totals[0][w];
            pb += totals[1][w];
        }
#pragma unroll
        for (int q = 0; q < kListItems; ++q) {
            const int64_t c = t0 + q * kBlock + tid;
            if ((sm[q] >> lane) & 1) sure[ps + popc64(sm[q] & lanes_below(lane))] = cand ? cand[c] : static_cast<int32_t>(c);
            if ((bm[q] >> lane) & 1) {
                const uint32_t o = pb + popc64(bm[q] & lanes_below(lane));
                bkey[o] = key[q];
                bpos[o] = cand ? cand[c] : static_cast<int32_t>(c);
            }
            ps += popc64(sm[q]);
            pb += popc64(bm[q]);
        }
        load(t0 + int64_t(grid) * kTile);
        __syncthreads();                                   // totals[] and base are rewritten by the next tile
    }
}

// The drawn nodes, ascending, are the block's sources.  Every workgroup ranks the boundary list by (key, id) for
// itself, which completes the list of drawn ids in LDS; then four threads count the ids below each.
constexpr int kPickThreads = 4;
template <typename PtrT, typename IdxT>
__global__ void __launch_bounds__(kBlock)
k_lw_pick(const int32_t *__restrict__ sure, const uint64_t *__restrict__ bkey, const int32_t *__restrict__ bpos,
          const unsigned long long *__restrict__ count, const unsigned long long *__restrict__ want_dev, int layer_size, int64_t list_cap,
          IdxT *__restrict__ src_ids, int32_t *__restrict__ local_of, int32_t pos_base, LwColumns columns, int64_t *count_a, int64_t *count_b) {
    __shared__ __align__(16) int32_t ids[kPickMost + 8];
    __shared__ __align__(16) uint64_t lk[kBoundaryRanked + 4];
    __shared__ __align__(16) int32_t lp[kBoundaryRanked + 4];
    __shared__ int h[256];
    __shared__ int lds[kWavesPerBlock];
    __shared__ long long pick[2];
    const int tid = threadIdx.x;
    // the lists' first entries are loaded whether they are filled or not, together with the counts
    for (int e = tid; e < layer_size; e += kBlock) ids[e] = sure[e];
    lk[tid] = tid < list_cap ? bkey[tid] : 0;
    lp[tid] = tid < list_cap ? bpos[tid] : 0;
    const unsigned long long cnt = *count;
    const int ns = static_cast<int>(cnt & 0xFFFFFFFFu), want = static_cast<int>(*want_dev);
    const int64_t m = static_cast<int64_t>(cnt >> 32);
    const int total = ns + want;                           // at most the layer's size, and that at most kPickMost
    __syncthreads();
    if (want > 0 && m <= kBoundaryRanked) {
        for (int e = kBlock + tid; e < m; e += kBlock) {
            lk[e] = bkey[e];
            lp[e] = bpos[e];
        }
        if (tid < 4) {                                     // ahead of none
            lk[m + tid] = ~uint64_t(0);
            lp[m + tid] = 0x7FFFFFFF;
        }
        __syncthreads();
        for (int e = tid; e < m; e += kBlock) {
            const uint64_t k = lk[e];
            const int32_t p = lp[e];
            int rank = 0;
#pragma unroll 2
            for (int j = 0; j < m; j += 4) {
                const ulonglong2 a = *reinterpret_cast<const ulonglong2 *>(lk + j), b = *reinterpret_cast<const ulonglong2 *>(lk + j + 2);
                const int4 o = *reinterpret_cast<const int4 *>(lp + j);
                rank += (a.x < k || (a.x == k && o.x < p)) + (a.y < k || (a.y == k && o.y < p)) + (b.x < k || (b.x == k && o.z < p)) +
                        (b.y < k || (b.y == k && o.w < p));
            }
            if (rank < want) ids[ns + rank] = p;
        }
    } else if (want > 0) {                                 // many keys of nearly the same size
        uint64_t kp = 0;
        uint32_t pp;
        lw_select_pairs(bkey, bpos, m, want, kp, 64, pp, h, lds, pick);
        int at = ns;                                       // in the list's order, which is the same for all workgroups
        for (int64_t e0 = 0; e0 < m; e0 += kBlock) {
            const int64_t e = e0 + tid;
            const uint64_t k = e < m ? bkey[e] : 0;
            const int32_t p = e < m ? bpos[e] : 0;
            const bool in = e < m && (k < kp || (k == kp && static_cast<uint32_t>(p) <= pp));
            int found;
            const int o = block_excl_scan<kWavesPerBlock>(in ? 1 : 0, &found, lds);
            if (in) ids[at + o] = p;
            at += found;
        }
    }
    if (tid < 4) ids[total + tid] = 0x7FFFFFFF;
    if (blockIdx.x == 0 && tid == 0) {
        if (count_a) *count_a = total;
        if (count_b) *count_b = total;
    }
    __syncthreads();
    const int e = (static_cast<int>(blockIdx.x) * kBlock + tid) / kPickThreads;
    const int part = tid % kPickThreads;
    if (e >= total) return;
    const int32_t id = ids[e];
    const double f = columns.value<PtrT>(id);              // its loads ahead of the counting
    int pos = 0;
#pragma unroll 8
    for (int j = 4 * part; j < total; j += 4 * kPickThreads) {
        const int4 o = *reinterpret_cast<const int4 *>(ids + j);
        pos += (o.x < id) + (o.y < id) + (o.z < id) + (o.w < id);
    }
    pos += __shfl_xor(pos, 1, 64);
    pos += __shfl_xor(pos, 2, 64);
    if (part == 0) {
        src_ids[pos] = static_cast<IdxT>(id);
        local_of[id] = pos_base + pos;
        columns.factor[pos] = f;
    }
}

// Rows up to which k_lw_fill adds up the edges of the rows before its own; more are scanned in launches of their own.
constexpr int64_t kSelfOffsetRows = 2048;

// A wavefront per (row, chunk): the number of drawn nodes in the chunk's slots (chunk 0 also counts the self edge) and the
// sum of their columns' factors; the rows' edges (row_count is zero before).  `cleared` workgroups more set
// the masses of the candidates (of all nodes without a list of them), the histogram and (bitmap_words) the bitmap back to zero; the
// block's flags word.  Bound by the lookups behind its caches: the two layers of a batch of 1,024 seeds on a graph of 233 k
// nodes and mean degree 490 15.8 + 12.9 us, then 5.8 + 4.2
// for a scan of the counts -> 13.6 + 9.1 (a workgroup per row 20 + 15: a hub's lookups take a 128-byte line each, and a compute
// unit fetches 64 bytes per cycle).
template <typename PtrT, typename IdxT>
__global__ void __launch_bounds__(kBlock)
k_lw_count(const PtrT *__restrict__ row_ptr, const IdxT *__restrict__ col_idx, const IdxT *__restrict__ dst,
           int64_t *sizes, const int32_t *__restrict__ local_of, int32_t pos_base, const double *__restrict__ factor,
           int32_t *__restrict__ counts, double *__restrict__ psum, int32_t *__restrict__ row_count, int row_blocks, int cleared,
           const int32_t *__restrict__ cand, const int64_t *__restrict__ n_cand, int64_t all_nodes, unsigned long long *__restrict__ mass,
           int32_t *__restrict__ sel_hist, int hist_len, uint32_t *__restrict__ bitmap, int64_t bitmap_words, int32_t *__restrict__ seed_flags) {
    const int lane = lane_id();
    if (static_cast<int>(blockIdx.x) >= row_blocks) {
        const int64_t first = int64_t(static_cast<int>(blockIdx.x) - row_blocks) * kBlock + threadIdx.x;
        const int64_t stride = int64_t(cleared) * kBlock;
        for (int64_t k = first; k < hist_len; k += stride) sel_hist[k] = 0;
        for (int64_t k = first; k < bitmap_words; k += stride) bitmap[k] = 0;
        if (cand) {
            const int64_t nc = *n_cand;
            for (int64_t k = first; k < nc; k += stride) mass[cand[k]] = 0;
        } else {
            for (int64_t k = first; k < all_nodes; k += stride) mass[k] = 0;
        }
        return;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sizes[3] = seed_flags ? *seed_flags : 0;
        if (seed_flags) *seed_flags = 0;                   // for the next call
    }
    const int64_t rows = sizes[0];
    const int64_t wave0 = int64_t(blockIdx.x) * kWavesPerBlock + (threadIdx.x >> 6);
    const int64_t nwaves = int64_t(row_blocks) * kWavesPerBlock;
    for (int64_t u = wave0; u < rows * kRowChunks; u += nwaves) {
        const int64_t t = u / kRowChunks;
        const int c = static_cast<int>(u % kRowChunks);
        const int64_t v = static_cast<int64_t>(dst[t]);
        const int64_t start = static_cast<int64_t>(row_ptr[v]);
        const int64_t d = static_cast<int64_t>(row_ptr[v + 1]) - start;
        int cnt = 0;
        double acc = 0.0;
        if (c == 0) {
            const int32_t li = local_of[v] - pos_base;
            if (li >= 0) {
                cnt = 1;
                if (lane == 0) acc = factor[li];
            }
        }
        int64_t jb, je;
        chunk_range<kSlotUnroll * kWave>(d, c, &jb, &je);
        // a batch's ids are on their way while the positions of the batch before are looked up, and a batch's
        // factors while the next one's are
        IdxT id[kSlotUnroll];
        double f[kSlotUnroll];
        auto load = [&](int64_t j0) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < kSlotUnroll; ++q) {
                const int64_t j = j0 + q * kWave + lane;
                if (j0 + q * kWave < je) id[q] = col_idx[start + (j < je ? j : jb)];         // uniform
            }
        };
#pragma unroll
        for (int q = 0; q < kSlotUnroll; ++q) f[q] = 0.0;
        if (jb < je) load(jb);
        for (int64_t j0 = jb; j0 < je; j0 += kSlotUnroll * kWave) {
            int32_t li[kSlotUnroll];
#pragma unroll
            for (int q = 0; q < kSlotUnroll; ++q)
                if (j0 + q * kWave < je) li[q] = local_of[id[q]];
            if (j0 + kSlotUnroll * kWave < je) load(j0 + kSlotUnroll * kWave);
#pragma unroll
            for (int q = 0; q < kSlotUnroll; ++q) {
                if (j0 + q * kWave >= je) break;           // uniform
                li[q] -= pos_base;
                const bool in = li[q] >= 0 && j0 + q * kWave + lane < je;
                cnt += popc64(ballot64(in));
                acc += f[q];
                f[q] = 0.0;
                if (in) f[q] = factor[li[q]];
            }
        }
#pragma unroll
        for (int q = 0; q < kSlotUnroll; ++q) acc += f[q];
        if (cnt > 0) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
        }
        if (lane == 0) {
            counts[u] = cnt;
            psum[u] = acc;
            if (cnt > 0) atomicAdd(&row_count[t], cnt);
        }
    }
}

// scanned: row_count holds its exclusive scan, one entry past the last row too; otherwise every wavefront that needs a
// row's first edge position adds up the counts before it (a launch of its own for that took 4 to 6 us per block).
template <typename PtrT, typename IdxT>
__global__ void __launch_bounds__(kBlock)
k_lw_fill(const PtrT *__restrict__ row_ptr, const IdxT *__restrict__ col_idx, const IdxT *__restrict__ dst,
          int64_t *sizes, const int32_t *__restrict__ local_of, int32_t pos_base, const double *__restrict__ q_total,
          const double *__restrict__ factor, int debias, const int32_t *__restrict__ counts, const int32_t *__restrict__ row_count, int scanned,
          const double *__restrict__ psum, int32_t *__restrict__ indptr, int32_t *__restrict__ indices,
          float *__restrict__ edge_w, int normalise, int64_t cap_nnz, int grid) {
    const int lane = lane_id();
    const int64_t rows = sizes[0];
    const int64_t wave0 = int64_t(blockIdx.x) * kWavesPerBlock + (threadIdx.x >> 6);
    const int64_t nwaves = int64_t(grid) * kWavesPerBlock;
    if (rows == 0 && wave0 == 0 && lane == 0) {
        indptr[0] = 0;
        sizes[2] = 0;
    }
    for (int64_t u = wave0; u < rows * kRowChunks; u += nwaves) {
        const int64_t t = u / kRowChunks;
        const int c = static_cast<int>(u % kRowChunks);
        // the row's chunks, one per lane
        const int of_chunk = lane < kRowChunks ? counts[t * kRowChunks + lane] : 0;
        const int mine = static_cast<int>(readlane32(static_cast<uint32_t>(of_chunk), c));
        if (mine == 0 && c != 0) continue;                 // nothing drawn in this chunk
        int64_t pos = 0;                                   // first edge position of the row
        if (scanned) {
            pos = row_count[t];
        } else {
            int part = 0;
#pragma unroll 2
            for (int64_t k = 4 * lane; k < t; k += 4 * kWave) {
                const int4 x = *reinterpret_cast<const int4 *>(row_count + k);
                part += x.x + (k + 1 < t ? x.y : 0) + (k + 2 < t ? x.z : 0) + (k + 3 < t ? x.w : 0);
            }
            pos = wave_sum(part);
        }
        if (c == 0 && lane == 0) indptr[t] = static_cast<int32_t>(pos);
        if (c == 0 && t == rows - 1) {                     // the end of indptr, the block's nnz, its flags
            const int64_t nnz = pos + wave_sum(of_chunk);
            if (lane == 0) {
                indptr[rows] = static_cast<int32_t>(nnz);
                sizes[2] = nnz < cap_nnz ? nnz : cap_nnz;
                if (nnz > cap_nnz) sizes[3] |= 4;
            }
        }
        if (mine == 0) continue;
        pos += wave_sum(lane < c ? of_chunk : 0);
        const int64_t end = pos + mine;
        const int64_t v = static_cast<int64_t>(dst[t]);
        const int64_t start = static_cast<int64_t>(row_ptr[v]);
        const int64_t d = static_cast<int64_t>(row_ptr[v + 1]) - start;
        double scale;
        if (normalise) {                                   // the row's sum: its chunks' partial sums in order
            const double part = lane < kRowChunks ? psum[t * kRowChunks + lane] : 0.0;
            double row_sum = 0.0;
            for (int k = 0; k < kRowChunks; ++k) row_sum += __shfl(part, k, 64);
            scale = 1.0 / row_sum;
        } else {
            scale = (debias ? 1.0 : *q_total / static_cast<double>(sizes[1])) / sqrt(static_cast<double>(d + 1));
        }
        if (c == 0) {
            const int32_t self_pos = local_of[v] - pos_base;
            if (self_pos >= 0) {
                if (lane == 0 && pos < cap_nnz) {
                    indices[pos] = self_pos;
                    edge_w[pos] = static_cast<float>(factor[self_pos] * scale);
                }
                pos += 1;
            }
        }
        int64_t jb, je;
        chunk_range<kSlotUnroll * kWave>(d, c, &jb, &je);
        IdxT id[kSlotUnroll];
        auto load = [&](int64_t j0) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < kSlotUnroll; ++q) {
                const int64_t j = j0 + q * kWave + lane;
                if (j0 + q * kWave < je) id[q] = col_idx[start + (j < je ? j : jb)];         // uniform
            }
        };
        if (jb < je) load(jb);
        for (int64_t j0 = jb; j0 < je && pos < end; j0 += kSlotUnroll * kWave) {
            int32_t li[kSlotUnroll];
#pragma unroll
            for (int q = 0; q < kSlotUnroll; ++q)
                if (j0 + q * kWave < je) li[q] = local_of[id[q]];
            if (j0 + kSlotUnroll * kWave < je) load(j0 + kSlotUnroll * kWave);
#pragma unroll
            for (int q = 0; q < kSlotUnroll; ++q) {
                if (j0 + q * kWave >= je) break;           // uniform
                li[q] -= pos_base;
                const bool in = li[q] >= 0 && j0 + q * kWave + lane < je;
                const uint64_t m = ballot64(in);
                if (in) {
                    const int64_t p = pos + popc64(m & lanes_below(lane));
                    if (p < cap_nnz) {
                        indices[p] = li[q];
                        edge_w[p] = static_cast<float>(factor[li[q]] * scale);
                    }
                }
                pos += popc64(m);
            }
        }
    }
}

// ---- debiased coefficients (paper Eq. 12) of the drawn nodes

// race key and q = mass / (deg + 1) of every drawn node, by source position
template <typename PtrT, typename IdxT>
__global__ void __launch_bounds__(kBlock)
k_lw_drawn_keys(const PtrT *__restrict__ row_ptr, const IdxT *__restrict__ src_ids, const int64_t *__restrict__ sizes,
                const unsigned long long *__restrict__ mass, uint64_t tag_hash, int flat, uint64_t *__restrict__ dkey,
                double *__restrict__ dq) {
    const int64_t ns = sizes[1];
    const int64_t pos = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (pos >= ns) return;
    const int64_t i = static_cast<int64_t>(src_ids[pos]);
    const double deg1 = static_cast<double>(static_cast<int64_t>(row_ptr[i + 1]) - static_cast<int64_t>(row_ptr[i]) + 1);
    const double m = static_cast<double>(mass[i]);
    const double ticket = lw_ticket(tag_hash, i);
    dkey[pos] = static_cast<uint64_t>(__double_as_longlong(lw_race_key(ticket, deg1, m, flat)));
    dq[pos] = lw_measure(m, deg1, flat);
}

// order[r] = source position of the r-th drawn node: the race order is ascending (key, id), and
// positions ascend with the ids.  Every thread counts the drawn nodes ahead of its own.
__global__ void __launch_bounds__(kBlock)
k_lw_draw_order(const uint64_t *__restrict__ dkey, const int64_t *__restrict__ sizes, int32_t *__restrict__ order) {
    const int64_t ns = sizes[1];
    const int64_t pos = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (pos >= ns) return;
    const uint64_t k = dkey[pos];
    int rank = 0;
    for (int64_t t = 0; t < ns; ++t) {
        const uint64_t o = dkey[t];
        rank += (o < k || (o == k && t < pos)) ? 1 : 0;
    }
    order[rank] = static_cast<int32_t>(pos);
}

// Inclusive scan over the 256 threads of a workgroup with a binary operation on doubles (sum or
// product); *total gets the workgroup's result.  `lds` needs kWavesPerBlock doubles.
template <bool PRODUCT>
__device__ __forceinline__ double lw_block_scan_incl(double v, double *total, double *lds) {
    const int lane = lane_id();
    const int wave = static_cast<int>(threadIdx.x) >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const double t = __shfl_up(v, off, 64);
        if (lane >= off) v = PRODUCT ? v * t : v + t;
    }
    __syncthreads();                                       // lds may still be read from an earlier use
    if (lane == 63) lds[wave] = v;
    __syncthreads();
    double before = PRODUCT ? 1.0 : 0.0, all = PRODUCT ? 1.0 : 0.0;
#pragma unroll
    for (int k = 0; k < kWavesPerBlock; ++k) {
        const double t = lds[k];
        if (k < wave) before = PRODUCT ? before * t : before + t;
        all = PRODUCT ? all * t : all + t;
    }
    *total = all;
    return PRODUCT ? before * v : before + v;
}

// The recursion of Eq. 12 in closed form.  With a_r = n / ((n - r)(r + 1)) (r = 0 for the first draw)
// and b0_r = a_r (1 - sum of the p drawn before) / p_r the coefficient an item gets when it is
// drawn, later steps turn a coefficient b into (1 - a_u) b + a_u, so the final one is
//   beta_r = b0_r G_r + H_r,  G_r = prod_{u > r} (1 - a_u),  H_r = sum_{u > r} a_u G_u.
// One workgroup: a prefix sum over the draws for b0, then, from the last draw backwards, a prefix
// product for G and a prefix sum of a_u G_u for H, 256 draws at a time with running carries.
// Every candidate drawn: beta = 1.  The coefficients go into the drawn nodes' factors (LwColumns).
__global__ void __launch_bounds__(kBlock)
k_lw_debias(const int32_t *__restrict__ order, const double *__restrict__ dq, const double *__restrict__ q_total,
            const int64_t *__restrict__ sizes, const int64_t *__restrict__ n_cand, double *__restrict__ b0,
            double *__restrict__ factor) {
    __shared__ double lds[kWavesPerBlock];
    __shared__ double incl_of[kBlock];
    const int64_t s = sizes[1];
    const int64_t n = *n_cand;
    if (s >= n) return;
    const double total = *q_total;
    const double nd = static_cast<double>(n);
    double drawn = 0.0;                                    // probability mass of the draws before this chunk
    for (int64_t base = 0; base < s; base += kBlock) {
        const int64_t r = base + threadIdx.x;
        const bool in = r < s;
        const double p = in ? dq[order[r]] / total : 0.0;
        double chunk;
        const double incl = lw_block_scan_incl<false>(p, &chunk, lds);
        if (in) {
            const double alpha = nd / (static_cast<double>(n - r) * static_cast<double>(r + 1));
            b0[r] = alpha * (1.0 - (drawn + (incl - p))) / p;
        }
        drawn += chunk;
    }
    __syncthreads();
    double G = 1.0, H = 0.0;                               // over the draws after this chunk
    for (int64_t top = s; top > 0; top -= kBlock) {        // thread t takes draw top - 1 - t
        const int64_t r = top - 1 - threadIdx.x;
        const bool in = r >= 0;
        const double alpha = in ? nd / (static_cast<double>(n - r) * static_cast<double>(r + 1)) : 0.0;
        const double x = 1.0 - alpha;
        const int32_t at = in ? order[r] : 0;              // on its way during the scans
        const double f = in ? factor[at] : 0.0, b = in ? b0[r] : 0.0;
        double gprod, hsum;
        const double g_incl = lw_block_scan_incl<true>(x, &gprod, lds);
        incl_of[threadIdx.x] = g_incl;                     // the exclusive product is the previous thread's inclusive one
        __syncthreads();
        const double Gr = G * (threadIdx.x == 0 ? 1.0 : incl_of[threadIdx.x - 1]);
        const double term = alpha * Gr;
        const double h_incl = lw_block_scan_incl<false>(term, &hsum, lds);
        if (in) factor[at] = f * (b * Gr + (H + (h_incl - term)));
        H += hsum;
        G *= gprod;
        __syncthreads();                                   // incl_of[] is rewritten by the next chunk
    }
}

// Calls that are being recorded take their positions back, see take_positions.
template <typename IdxT>
__global__ void __launch_bounds__(kBlock)
k_lw_reset(const IdxT *__restrict__ src_ids, const int64_t *__restrict__ sizes, int32_t *__restrict__ local_of) {
    const int64_t ns = sizes[1];
    const int64_t k = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (k < ns) local_of[src_ids[k]] = -1;
}

__global__ void k_lw_store_i64(int64_t *p, int64_t v, int64_t *zero) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *p = v;
        if (zero) *zero = 0;
    }
}


template <typename T>
bool dev_alloc(T **p, int64_t count) {
    return hipMalloc(reinterpret_cast<void **>(p), static_cast<size_t>(std::max<int64_t>(count, 1)) * sizeof(T)) == hipSuccess;
}

}  // namespace

void free_layerwise_scratch(mqg_ctx *ctx) {
    LayerwiseScratch &w = ctx->lw;
    void *ptrs[] = {w.mass, w.cand, w.key64, w.bkey, w.bpos, w.xkey, w.xpos, w.word_offs, w.scan_tiles, w.q_part, w.counters, w.q_total, w.seeds_copy, w.flags,
                    w.sel_state, w.sel_hist, w.sure, w.chunk_counts, w.row_count, w.chunk_sum, w.fg_mass, w.dkey, w.dq, w.order, w.factor};
    for (void *p : ptrs) (void)hipFree(p);
    w = LayerwiseScratch{};
}

// scratch of the layer-wise sampler: about 32 bytes per graph node, allocated at the first call
int ensure_layerwise_scratch(mqg_ctx *ctx, int64_t rows_cap, hipStream_t s) {
    LayerwiseScratch &w = ctx->lw;
    if (w.mass && rows_cap <= w.rows_cap) return MQG_OK;
    hipError_t e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail(ctx, MQG_ERR_HIP, std::string("mqg_sample_layerwise: ") + hipGetErrorString(e));
    free_layerwise_scratch(ctx);
    const int64_t n = std::max<int64_t>(ctx->num_nodes, 1);
    const int64_t chunks = rows_cap * kRowChunks;
    const int64_t scan_len = std::max<int64_t>(ctx->bitmap_words + 1, rows_cap + 1);
    bool ok = dev_alloc(&w.mass, n) && dev_alloc(&w.cand, n) && dev_alloc(&w.key64, n) && dev_alloc(&w.bkey, n) && dev_alloc(&w.bpos, n) && dev_alloc(&w.word_offs, ctx->bitmap_words + 1) &&
              dev_alloc(&w.scan_tiles, ceil_div(scan_len, kScanTile) + 2) && dev_alloc(&w.q_part, ceil_div(n, kBlock) + 1) &&
              dev_alloc(&w.counters, 4) && dev_alloc(&w.q_total, 1) && dev_alloc(&w.seeds_copy, rows_cap) && dev_alloc(&w.flags, 1) &&
              dev_alloc(&w.sel_state, 18) && dev_alloc(&w.sel_hist, kSelHistLen) && dev_alloc(&w.sure, kPickMost) && dev_alloc(&w.chunk_counts, chunks) &&
              dev_alloc(&w.row_count, rows_cap + 4) && dev_alloc(&w.chunk_sum, chunks) && dev_alloc(&w.dkey, rows_cap) && dev_alloc(&w.dq, rows_cap) &&
              dev_alloc(&w.order, rows_cap) && dev_alloc(&w.factor, rows_cap);
    if (ok) ok = hipMemset(w.mass, 0, static_cast<size_t>(n) * sizeof(unsigned long long)) == hipSuccess &&
                 hipMemset(w.flags, 0, sizeof(int32_t)) == hipSuccess &&
                 hipMemset(w.sel_hist, 0, kSelHistLen * sizeof(int32_t)) == hipSuccess && hipDeviceSynchronize() == hipSuccess;
    if (!ok) {
        free_layerwise_scratch(ctx);
        return fail(ctx, MQG_ERR_HIP, "mqg_sample_layerwise: scratch allocation failed");
    }
    w.rows_cap = rows_cap;
    return MQG_OK;
}

template <typename PtrT, typename IdxT>
static int sample_layerwise_impl(mqg_ctx *ctx, const mqg_graph *g, const void *seeds_v, int32_t num_seeds,
                                 const int32_t *layer_sizes, int32_t L, uint64_t rng_seed, int32_t normalise, bool fastgcn, bool debias, bool flat_p,
                                 mqg_block *blocks, float *const *edge_w, hipStream_t s) {
    LayerwiseScratch &w = ctx->lw;
    const int flat = flat_p ? 1 : 0;
    const PtrT *row_ptr = static_cast<const PtrT *>(g->row_ptr);
    const IdxT *col_idx = static_cast<const IdxT *>(g->col_idx);
    const int64_t n = ctx->num_nodes;
    // bitmap -> list: tiles of kBlock * wpt words, counted by the launch before (w.word_offs)
    const int wpt = ctx->bitmap_words <= (int64_t(1) << 20) ? 1 : 4;
    const int tiles = static_cast<int>(ctx->bitmap_words / (int64_t(kBlock) * wpt));
    const int tiles_scanned = tiles > kSelfPrefixTiles ? 1 : 0;
    const int emit_parts = tiles <= kEmitFewTiles ? kEmitParts : 1;
    auto count_tiles = [&]() -> int {
        if (wpt == 1) MQG_LAUNCH(ctx, "k_lw_tile_counts", s, (k_lw_tile_counts<1><<<tiles, kBlock, 0, s>>>(ctx->bitmap, w.word_offs)));
        else MQG_LAUNCH(ctx, "k_lw_tile_counts", s, (k_lw_tile_counts<4><<<tiles, kBlock, 0, s>>>(ctx->bitmap, w.word_offs)));
        return MQG_OK;
    };
    auto emit_list = [&](auto *out, int32_t *local_of, int32_t pos_base, LwColumns columns, int64_t *count_a, int64_t *count_b, int parts) -> int {
        using OutT = std::remove_pointer_t<decltype(out)>;
        if (tiles_scanned) {
            int rc = device_scan(ctx, w.word_offs, tiles, w.scan_tiles, s);
            if (rc != MQG_OK) return rc;
        }
        if (wpt == 1)
            MQG_LAUNCH(ctx, "k_lw_emit", s, (k_lw_emit<PtrT, OutT, 1><<<tiles * parts, kBlock, 0, s>>>(ctx->bitmap, w.word_offs, tiles_scanned, out, local_of, pos_base, columns, count_a, count_b, tiles, parts)));
        else
            MQG_LAUNCH(ctx, "k_lw_emit", s, (k_lw_emit<PtrT, OutT, 4><<<tiles, kBlock, 0, s>>>(ctx->bitmap, w.word_offs, tiles_scanned, out, local_of, pos_base, columns, count_a, count_b, tiles, 1)));
        return MQG_OK;
    };
    const int cand_grid = static_cast<int>(std::max<int64_t>(1, ceil_div(n, kBlock)));
    const uint64_t seed_hash = host_mix64(rng_seed + kGolden);
    // Three ways to the candidates.  FastGCN: every node, with batch-independent masses.  Graphs of up
    // to kDenseNodes nodes: every node gets a key slot and the nodes without mass hold no key - no
    // candidate list, a node's key sits at its id (on "medium" 200 k of the 233 k nodes are candidates
    // anyway).  Otherwise: the list of touched nodes, ascending.
    const int how = ctx->layerwise_candidates;
    const bool dense = !fastgcn && (how == 0 ? n <= kDenseNodes : how == 1);
    const bool keyed_by_id = fastgcn || dense;
    int64_t *n_cand = fastgcn ? w.counters + 2 : w.counters;
    const int32_t *cand = keyed_by_id ? nullptr : w.cand;
    const int64_t *n_keys_dev = keyed_by_id ? nullptr : w.counters;       // keyed by id: n keys
    const unsigned long long *mass = fastgcn ? w.fg_mass : w.mass;
    unsigned long long *bcount = reinterpret_cast<unsigned long long *>(w.counters + 3);
    if (fastgcn && !w.fg_ready) {
        // the batch-independent masses: the mass kernel over every row of the graph, once per context
        MQG_LAUNCH(ctx, "k_lw_store_i64", s, (k_lw_store_i64<<<1, 64, 0, s>>>(w.counters + 2, n, nullptr)));
        const int grid = static_cast<int>(std::min<int64_t>(std::max<int64_t>(1, ceil_div(n * kRowChunks, kWavesPerBlock)), 256 * 64));
        MQG_LAUNCH(ctx, "k_lw_mass", s,
                   (k_lw_mass<PtrT, IdxT><<<grid, kBlock, 0, s>>>(row_ptr, col_idx, nullptr, w.counters + 2, -1, n, nullptr, nullptr, w.fg_mass, nullptr, nullptr, grid, 0, nullptr)));
        w.fg_ready = true;
    }

    IdxT *dst0 = reinterpret_cast<IdxT *>(w.seeds_copy);
    if (fastgcn) {
        const int grid = static_cast<int>(std::max<int64_t>(1, ceil_div(num_seeds, kBlock)));
        MQG_LAUNCH(ctx, "k_lw_seeds", s,
                   (k_lw_seeds<IdxT><<<grid, kBlock, 0, s>>>(static_cast<const IdxT *>(seeds_v), num_seeds, n, dst0, blocks[L - 1].sizes, w.flags)));
    }
    for (int l = L - 1; l >= 0; --l) {
        mqg_block &b = blocks[l];
        const IdxT *dst = l == L - 1 ? dst0 : static_cast<const IdxT *>(blocks[l + 1].src_ids);
        IdxT *src_ids = static_cast<IdxT *>(b.src_ids);
        const int64_t rows_cap = l == L - 1 ? num_seeds : std::min<int64_t>(n, layer_sizes[l + 1]);
        const uint64_t tag_hash = host_mix64(seed_hash ^ static_cast<uint64_t>(int64_t(kLayerwiseTag + l)));

        const int64_t src_cap = std::min<int64_t>(n, layer_sizes[l]);
        int32_t pos_base = 0;
        bool take_back = false;
        int rc = take_positions(ctx, src_cap, s, &pos_base, &take_back);
        if (rc != MQG_OK) return rc;
        // tickets in the shadow of the masses' atomics, if the rows have more slots than the graph has nodes (most nodes
        // are candidates then; fewer would make their tickets themselves)
        const bool shadow = dense && g->num_edges / std::max<int64_t>(n, 1) * rows_cap >= n;
        const int ticket_blocks = shadow ? cand_grid : 0;
        if (!fastgcn) {
            const int mass_grid = static_cast<int>(std::min<int64_t>(std::max<int64_t>(1, ceil_div(rows_cap * kRowChunks, kWavesPerBlock)), 256 * 64));
            // list of candidates: marked slot by slot in the node bitmap, or, on graphs of up to
            // kMassScanNodes nodes, read off the masses afterwards
            const bool scan_masses = how == 0 ? n <= kMassScanNodes : how == 2;
            MQG_LAUNCH(ctx, "k_lw_mass", s,
                       (k_lw_mass<PtrT, IdxT><<<mass_grid + ticket_blocks, kBlock, 0, s>>>(row_ptr, col_idx, l == L - 1 ? static_cast<const IdxT *>(seeds_v) : dst, b.sizes,
                                                                           l == L - 1 ? int64_t(num_seeds) : int64_t(-1), n, dst0, w.flags, w.mass,
                                                                           dense || scan_masses ? nullptr : ctx->bitmap,
                                                                           dense ? w.counters : nullptr, mass_grid, tag_hash,
                                                                           reinterpret_cast<double *>(w.key64))));
            if (!dense) {
                if (scan_masses)
                    MQG_LAUNCH(ctx, "k_lw_mass_bits", s, (k_lw_mass_bits<<<tiles, kBlock, 0, s>>>(w.mass, n, ctx->bitmap, w.word_offs)));
                else
                    rc = count_tiles();
                if (rc == MQG_OK) rc = emit_list(w.cand, nullptr, 0, LwColumns{}, n_cand, nullptr, 1);
                if (rc != MQG_OK) return rc;
            }
        }
        // Race keys and the first digit's counts, then the drawn nodes.  (Few workgroups: every one of them adds its
        // counts to the same words - 911 workgroups spent 9 us of 15 queueing there.)
        const bool pick = layer_sizes[l] <= kPickMost;
        const int key_threads = n <= 256 * 256 ? 256 : n <= 256 * 512 ? 512 : kKeyThreads;
        const int key_grid = static_cast<int>(std::min<int64_t>(std::max<int64_t>(1, ceil_div(n, key_threads)), n <= (int64_t(1) << 22) ? 256 : 512));
        MQG_LAUNCH(ctx, "k_lw_keys", s,
                   (k_lw_keys<PtrT><<<key_grid, key_threads, 0, s>>>(row_ptr, cand, n_keys_dev, n, mass, tag_hash, flat, w.key64, w.q_part, w.sel_hist,
                                                                    dense && !pick ? w.counters : nullptr, w.sel_state, layer_sizes[l], bcount,
                                                                    pick ? 1 : 0, key_grid, key_threads, ticket_blocks > 0 ? 1 : 0, w.row_count, rows_cap + 1)));
        const LwColumns columns{row_ptr, mass, flat, debias ? 1 : 0, w.factor};
        int64_t *next_rows = l > 0 ? &blocks[l - 1].sizes[0] : nullptr;
        if (pick) {
            const int list_grid = static_cast<int>(std::min<int64_t>(std::max<int64_t>(1, ceil_div(n, kBlock * kListItems)), 1024));
            MQG_LAUNCH(ctx, "k_lw_list", s,
                       (k_lw_list<<<list_grid, kBlock, 0, s>>>(cand, w.key64, n_keys_dev, n, layer_sizes[l], w.sel_hist, w.q_part, key_grid, w.q_total,
                                                               w.counters + 1, w.sure, w.bkey, w.bpos, bcount, w.sel_state + 5, list_grid)));
            MQG_LAUNCH(ctx, "k_lw_pick", s,
                       (k_lw_pick<PtrT, IdxT><<<static_cast<int>(std::max<int64_t>(1, ceil_div(src_cap * kPickThreads, kBlock))), kBlock, 0, s>>>(
                           w.sure, w.bkey, w.bpos, bcount, w.sel_state + 5, layer_sizes[l], std::max<int64_t>(n, 1), src_ids, ctx->local_of, pos_base, columns, &b.sizes[1], next_rows)));
        } else {
            // Every workgroup adds up 32 KB of digit counts first, so no more of them than the keys need.  Whole calls (two
            // layers of 512) with 256 / 512 / 1,024: 233 k nodes 115 / 116 / 121 us, 524 k 137 / 137 / 141, 1 M 170 / 167 / 170,
            // 2 M 131 / 131 / 135; layers of 2,048 on 1 M nodes 206 / 200 / 202.
            const int sel_grid = static_cast<int>(std::min<int64_t>(cand_grid, n <= (int64_t(1) << 19) ? 256 : 512));
            for (int pass = 1; pass < kSelPasses; ++pass)
                MQG_LAUNCH(ctx, "k_lw_select", s,
                           (k_lw_select<<<sel_grid, kBlock, 0, s>>>(w.key64, n_keys_dev, n, layer_sizes[l], w.sel_state, w.sel_hist, pass)));
            MQG_LAUNCH(ctx, "k_lw_mark", s,
                       (k_lw_mark<<<sel_grid, kBlock, 0, s>>>(cand, w.key64, n_keys_dev, n, n_cand, dense ? 1 : 0, layer_sizes[l], w.sel_state,
                                                              w.sel_hist, ctx->bitmap, w.q_part, key_grid, w.q_total, w.bkey, w.bpos, bcount)));
            MQG_LAUNCH(ctx, "k_lw_finish", s,
                       (k_lw_finish<<<1, kBlock, 0, s>>>(cand, n_keys_dev, n, n_cand, layer_sizes[l], w.sel_state, w.bkey, w.bpos, bcount,
                                                         ctx->bitmap)));
            rc = count_tiles();
            if (rc == MQG_OK) rc = emit_list(src_ids, ctx->local_of, pos_base, columns, &b.sizes[1], next_rows, emit_parts);
            if (rc != MQG_OK) return rc;
        }
        if (debias) {
            const int sgrid = static_cast<int>(std::max<int64_t>(1, ceil_div(src_cap, kBlock)));
            MQG_LAUNCH(ctx, "k_lw_drawn_keys", s,
                       (k_lw_drawn_keys<PtrT, IdxT><<<sgrid, kBlock, 0, s>>>(row_ptr, src_ids, b.sizes, mass, tag_hash, flat, w.dkey, w.dq)));
            MQG_LAUNCH(ctx, "k_lw_draw_order", s, (k_lw_draw_order<<<sgrid, kBlock, 0, s>>>(w.dkey, b.sizes, w.order)));
            MQG_LAUNCH(ctx, "k_lw_debias", s,
                       (k_lw_debias<<<1, kBlock, 0, s>>>(w.order, w.dq, w.q_total, b.sizes, pick ? w.counters + 1 : n_cand, w.chunk_sum, w.factor)));
        }
        // rows: edges and weight sums per (row, chunk), then the edges
        const int row_grid = static_cast<int>(std::min<int64_t>(std::max<int64_t>(1, ceil_div(rows_cap * kRowChunks, kWavesPerBlock)), 256 * 64));
        const int clear_grid = static_cast<int>(std::min<int64_t>(ceil_div(fastgcn ? 0 : n, kBlock * 8) + 8, 1024));
        MQG_LAUNCH(ctx, "k_lw_count", s,
                   (k_lw_count<PtrT, IdxT><<<row_grid + clear_grid, kBlock, 0, s>>>(row_ptr, col_idx, dst, b.sizes, ctx->local_of, pos_base, w.factor,
                                                                                   w.chunk_counts, w.chunk_sum, w.row_count, row_grid, clear_grid, cand, n_cand,
                                                                                   dense ? n : 0, w.mass, w.sel_hist, pick ? kFineBins : kSelHistLen, ctx->bitmap,
                                                                                   !pick && emit_parts > 1 ? ctx->bitmap_words : 0,
                                                                                   l == L - 1 ? w.flags : nullptr)));
        const int scanned = rows_cap > kSelfOffsetRows ? 1 : 0;
        if (scanned) {
            rc = device_scan(ctx, w.row_count, rows_cap + 1, w.scan_tiles, s);
            if (rc != MQG_OK) return rc;
        }
        MQG_LAUNCH(ctx, "k_lw_fill", s,
                   (k_lw_fill<PtrT, IdxT><<<row_grid, kBlock, 0, s>>>(row_ptr, col_idx, dst, b.sizes, ctx->local_of, pos_base, w.q_total, w.factor,
                                                                     debias ? 1 : 0, w.chunk_counts, w.row_count, scanned, w.chunk_sum, b.indptr,
                                                                     b.indices, edge_w[l], normalise, b.cap_nnz, row_grid)));
        if (take_back)
            MQG_LAUNCH(ctx, "k_lw_reset", s,
                       (k_lw_reset<IdxT><<<static_cast<int>(std::max<int64_t>(1, ceil_div(src_cap, kBlock))), kBlock, 0, s>>>(src_ids, b.sizes, ctx->local_of)));
    }
    return MQG_OK;
}

// the selection step on its own: bit c of out_bitmap = key c is among the k smallest (key, index) pairs
int run_select_smallest_keys(mqg_ctx *ctx, const uint64_t *keys, int64_t n, int64_t k, uint32_t *out_bitmap, hipStream_t s) {
    int rc = ensure_layerwise_scratch(ctx, 1, s);
    if (rc != MQG_OK) return rc;
    LayerwiseScratch &w = ctx->lw;
    // the boundary list may hold every key: the sampler's own list has room for one per graph node
    uint64_t *bkey = w.bkey;
    int32_t *bpos = w.bpos;
    if (n > std::max<int64_t>(ctx->num_nodes, 1)) {
        if (n > w.xcap) {
            hipError_t e = hipStreamSynchronize(s);
            if (e != hipSuccess) return fail(ctx, MQG_ERR_HIP, std::string("mqg_select_smallest_keys: ") + hipGetErrorString(e));
            (void)hipFree(w.xkey);
            (void)hipFree(w.xpos);
            w.xkey = nullptr;
            w.xpos = nullptr;
            w.xcap = 0;
            if (!dev_alloc(&w.xkey, n) || !dev_alloc(&w.xpos, n)) {
                (void)hipFree(w.xkey);
                w.xkey = nullptr;
                return fail(ctx, MQG_ERR_HIP, "mqg_select_smallest_keys: scratch allocation failed");
            }
            w.xcap = n;
        }
        bkey = w.xkey;
        bpos = w.xpos;
    }
    int64_t *n_dev = w.counters + 1;
    const int64_t words = ceil_div(n, 32);
    MQG_LAUNCH(ctx, "k_lw_store_i64", s, (k_lw_store_i64<<<1, 64, 0, s>>>(n_dev, n, w.counters + 3)));
    if (words > 0)
        MQG_LAUNCH(ctx, "k_lw_zero_i32", s,
                   (k_lw_zero_i32<<<static_cast<int>(ceil_div(words, kBlock)), kBlock, 0, s>>>(reinterpret_cast<int32_t *>(out_bitmap), words)));
    const int grid = static_cast<int>(std::min<int64_t>(std::max<int64_t>(1, ceil_div(n, kBlock)), 1024));
    for (int pass = 0; pass < kSelPasses; ++pass)
        MQG_LAUNCH(ctx, "k_lw_select", s, (k_lw_select<<<grid, kBlock, 0, s>>>(keys, n_dev, 0, k, w.sel_state, w.sel_hist, pass)));
    unsigned long long *bcount = reinterpret_cast<unsigned long long *>(w.counters + 3);
    MQG_LAUNCH(ctx, "k_lw_mark", s,
               (k_lw_mark<<<grid, kBlock, 0, s>>>(nullptr, keys, n_dev, 0, nullptr, 0, k, w.sel_state, w.sel_hist, out_bitmap, nullptr, 0, nullptr,
                                                  bkey, bpos, bcount)));
    MQG_LAUNCH(ctx, "k_lw_finish", s,
               (k_lw_finish<<<1, kBlock, 0, s>>>(nullptr, n_dev, 0, nullptr, k, w.sel_state, bkey, bpos, bcount, out_bitmap)));
    // the histogram is clear between calls
    MQG_LAUNCH(ctx, "k_lw_zero_i32", s, (k_lw_zero_i32<<<kSelHistLen / kBlock, kBlock, 0, s>>>(w.sel_hist, kSelHistLen)));
    return MQG_OK;
}

int run_sample_layerwise(mqg_ctx *ctx, const mqg_graph *g, const void *seeds, int32_t num_seeds, const int32_t *layer_sizes,
                         int32_t L, uint64_t rng_seed, int32_t normalise, int32_t method, mqg_block *blocks, float *const *edge_w,
                         hipStream_t s) {
    const bool fg = (method & MQG_LAYERWISE_FASTGCN) != 0;
    const bool db = (method & MQG_LAYERWISE_DEBIAS) != 0;
    const bool fl = (method & MQG_LAYERWISE_FLAT) != 0;
    int64_t rows_cap = num_seeds;
    for (int l = 0; l < L; ++l) rows_cap = std::max<int64_t>(rows_cap, std::min<int64_t>(ctx->num_nodes, layer_sizes[l]));
    int rc = ensure_layerwise_scratch(ctx, rows_cap, s);
    if (rc != MQG_OK) return rc;
    if (fg && !ctx->lw.fg_mass) {
        const int64_t n = std::max<int64_t>(ctx->num_nodes, 1);
        if (!dev_alloc(&ctx->lw.fg_mass, n) ||
            hipMemsetAsync(ctx->lw.fg_mass, 0, static_cast<size_t>(n) * sizeof(unsigned long long), s) != hipSuccess) {
            (void)hipFree(ctx->lw.fg_mass);
            ctx->lw.fg_mass = nullptr;
            return fail(ctx, MQG_ERR_HIP, "mqg_sample_layerwise: scratch allocation failed");
        }
        ctx->lw.fg_ready = false;
    }
    const bool p64 = g->ptr_type == MQG_I64, i64 = g->idx_type == MQG_I64;
    if (p64 && i64) return sample_layerwise_impl<int64_t, int64_t>(ctx, g, seeds, num_seeds, layer_sizes, L, rng_seed, normalise, fg, db, fl, blocks, edge_w, s);
    if (p64) return sample_layerwise_impl<int64_t, int32_t>(ctx, g, seeds, num_seeds, layer_sizes, L, rng_seed, normalise, fg, db, fl, blocks, edge_w, s);
    if (i64) return sample_layerwise_impl<int32_t, int64_t>(ctx, g, seeds, num_seeds, layer_sizes, L, rng_seed, normalise, fg, db, fl, blocks, edge_w, s);
    return sample_layerwise_impl<int32_t, int32_t>(ctx, g, seeds, num_seeds, layer_sizes, L, rng_seed, normalise, fg, db, fl, blocks, edge_w, s);
}

}  // namespace mqg
