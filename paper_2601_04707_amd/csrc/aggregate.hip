// GraphSAGE mean aggregation over one block and its backward (paper Eq. 16: Z_agg(v) =
// Mean(H(v)), the GA step "AH" of Sec. IV "Computation"; the backward of GA is the transposed
// product "AG").  Both are segmented reductions over rows of a sparse operator: HBM-bound, no
// dense contraction, hence no matrix cores.
//
//   k_segment_flat   one wavefront per run of up to kRunRows consecutive output rows, its 64 lanes side by
//                    side over the columns (wider rows: several vectors per lane, or slabs of 64 vectors, each a
//                    share of the grid).  The entries of the run are walked as one sequence across the row ends:
//                    64 of them are fetched at a time, one per lane, and U input rows are loaded before the
//                    first of them is added, however few entries the rows have.  Entry numbers, row ends and
//                    addresses are the same in all lanes and live in scalar registers: per entry the vector
//                    unit sees one load and VEC additions.
//   reduce_long_row  rows of many entries and few columns: the lanes are split into groups, each takes a share
//                    of the row's entries.
// Forward: output row i reduces x[indices[e]] over the edges e of destination i and divides by
// their number.  Backward: output row s reduces grad_out[i] / n_i over the edges that point to
// source s, taken from the block's edge list sorted by source (stable radix sort, so a row's terms
// always come in ascending destination order).  A row's sum is made of partial sums that take its terms
// in turn; which takes which depends on the row's own terms and on the width, strides and alignment of the
// call, not on the rows around it: the result is reproducible bit for bit.
// Sums are fp32; fp16 output is rounded once (to nearest even) at the store.
#include <hip/hip_fp16.h>

#include <algorithm>
#include <type_traits>

#include "common.h"
#include "device_utils.h"
#include "radix.h"

namespace mqg {

namespace {

template <typename T, int VEC>
struct alignas(sizeof(T) * VEC) Pack {
    T v[VEC];
};

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(_Float16 x) { return static_cast<float>(x); }
__device__ __forceinline__ void from_f32(float x, float *o) { *o = x; }
__device__ __forceinline__ void from_f32(float x, _Float16 *o) { *o = static_cast<_Float16>(x); }

// Forward: entries of output row i are the block's edges of destination i.
struct ForwardRows {
    static constexpr bool kFewEntries = false;
    static constexpr bool kWeighted = false;
    static constexpr bool kSelf = false;
    __device__ __forceinline__ int64_t self_rows(int64_t) const { return 0; }
    __device__ __forceinline__ float self_weight(int64_t) const { return 0.f; }
    const int32_t *indptr;
    const int32_t *indices;
    __device__ __forceinline__ int begin(int64_t i) const { return indptr[i]; }
    __device__ __forceinline__ int input_row(int p) const { return indices[p]; }
    __device__ __forceinline__ float weight(int) const { return 1.f; }
    __device__ __forceinline__ float finish(float acc, int count) const { return count > 0 ? acc / static_cast<float>(count) : 0.f; }
};

// Backward: entries of output row s are the edges pointing to source s; each contributes the
// gradient row of its destination scaled by one over that destination's edge count.
struct BackwardRows {
    static constexpr bool kFewEntries = true;
    static constexpr bool kWeighted = true;
    static constexpr bool kSelf = false;
    __device__ __forceinline__ int64_t self_rows(int64_t) const { return 0; }
    __device__ __forceinline__ float self_weight(int64_t) const { return 0.f; }
    const int32_t *col_ptr;     // [num_src + 1] offsets into dst_rows
    const int32_t *dst_rows;    // [nnz] destination row of every edge, edges ordered by source
    const int32_t *indptr;      // the block's forward offsets, for the edge counts
    __device__ __forceinline__ int begin(int64_t s) const { return col_ptr[s]; }
    __device__ __forceinline__ int input_row(int p) const { return dst_rows[p]; }
    __device__ __forceinline__ float weight(int p) const {
        const int i = dst_rows[p];
        return 1.f / static_cast<float>(indptr[i + 1] - indptr[i]);
    }
    __device__ __forceinline__ float finish(float acc, int) const { return acc; }
};

// Weighted forward (the sampled estimator of the graph convolution, paper Eq. 1-3, or any other
// per-edge weights): out[i] = self_w[i] x[i] + sum over the edges p of row i of edge_w[p] x[indices[p]].
struct WeightedRows {
    static constexpr bool kFewEntries = false;
    static constexpr bool kWeighted = true;
    static constexpr bool kSelf = true;
    const int32_t *indptr;
    const int32_t *indices;
    const float *edge_w;
    const float *self_w;        // may be null: no diagonal term
    __device__ __forceinline__ int begin(int64_t i) const { return indptr[i]; }
    __device__ __forceinline__ int input_row(int p) const { return indices[p]; }
    __device__ __forceinline__ float weight(int p) const { return edge_w[p]; }
    __device__ __forceinline__ int64_t self_rows(int64_t n) const { return self_w ? n : 0; }
    __device__ __forceinline__ float self_weight(int64_t i) const { return self_w[i]; }
    __device__ __forceinline__ float finish(float acc, int) const { return acc; }
};

// Its transpose: output row s reduces edge_w * grad_out[destination] over the edges pointing to
// source s (ordered by source, stable), plus self_w[s] * grad_out[s] where s is a destination.
struct WeightedBackwardRows {
    static constexpr bool kFewEntries = true;
    static constexpr bool kWeighted = true;
    static constexpr bool kSelf = true;
    const int32_t *col_ptr;
    const int32_t *dst_rows;
    const float *w_sorted;      // edge weights in the by-source order
    const float *self_w;
    const int64_t *sizes;
    __device__ __forceinline__ int begin(int64_t s) const { return col_ptr[s]; }
    __device__ __forceinline__ int input_row(int p) const { return dst_rows[p]; }
    __device__ __forceinline__ float weight(int p) const { return w_sorted[p]; }
    __device__ __forceinline__ int64_t self_rows(int64_t) const { return self_w ? sizes[0] : 0; }
    __device__ __forceinline__ float self_weight(int64_t s) const { return self_w[s]; }
    __device__ __forceinline__ float finish(float acc, int) const { return acc; }
};

// One row of many entries and few columns (at most eight vectors of LV elements): the lanes are split into groups of
// 2^log2_lpr that cover the columns, group g takes the row's entries g, g + G, ..., and the G partial sums (8 to 64)
// are folded across the groups.  ws: the weight of the diagonal term, 0 if there is none.  G rows per load and, in
// long rows, four loads in flight, where the walk below has 16 rows in flight and most lanes idle: 2,000 rows of 300
// entries and 16 fp32 columns 22.5 -> 6.7 us (8.7 with one load at a time), of 2,000 entries 139 -> 33 (60); and
// more partial sums keep the error down (300 entries 1.7e-7 -> 1.0e-7 of the result, 2,000 entries 4.0e-7 -> 2.1e-7).
// Four loads where one or two will do cost 5 to 40 % on rows of G entries and fewer.
template <typename T, int LV, typename Rows>
__device__ __forceinline__ void reduce_long_row(const Rows &rows, int64_t i, int b, int e, float ws, const T *__restrict__ x, int64_t x_stride,
                                                T *__restrict__ out, int64_t out_stride, int dim, int log2_lpr) {
    using P = Pack<T, LV>;
    const int lane = lane_id();
    const int lpr = 1 << log2_lpr;
    const int groups = kWave >> log2_lpr;
    const int g = lane >> log2_lpr;
    const int col0 = (lane & (lpr - 1)) * LV;
    const bool live = col0 < dim;
    float acc[LV];
#pragma unroll
    for (int q = 0; q < LV; ++q) acc[q] = 0.f;
    if (Rows::kSelf && ws != 0.f && live && g == 0) {
        const P v = *reinterpret_cast<const P *>(x + i * x_stride + col0);
#pragma unroll
        for (int q = 0; q < LV; ++q) acc[q] = ws * to_f32(v.v[q]);
    }
    // F entries of every group from position p0 on: all their loads, then their additions
    auto batch = [&](int p0, auto flight) __attribute__((always_inline)) {
        constexpr int F = decltype(flight)::value;
        const int p = p0 + g;
        if (p >= e) return;
        int r[F];
        float w[F];
        P v[F];
#pragma unroll
        for (int u = 0; u < F; ++u) {
            const int pu = p + u * groups < e ? p + u * groups : p;        // past the end: the first again, not added
            r[u] = rows.input_row(pu);
            w[u] = Rows::kWeighted ? rows.weight(pu) : 1.f;
        }
#pragma unroll
        for (int u = 0; u < F; ++u) v[u] = *reinterpret_cast<const P *>(x + r[u] * x_stride + (live ? col0 : 0));
#pragma unroll
        for (int u = 0; u < F; ++u)
            if (p + u * groups < e) {
#pragma unroll
                for (int q = 0; q < LV; ++q) {
                    if (Rows::kWeighted) acc[q] += w[u] * to_f32(v[u].v[q]);
                    else acc[q] += to_f32(v[u].v[q]);
                }
            }
    };
    int p0 = b;
    for (; e - p0 > 2 * groups; p0 += 4 * groups) batch(p0, std::integral_constant<int, 4>());
    if (e - p0 > groups) batch(p0, std::integral_constant<int, 2>());
    else if (e - p0 > 0) batch(p0, std::integral_constant<int, 1>());
    for (int off = lpr; off < kWave; off <<= 1) {
#pragma unroll
        for (int q = 0; q < LV; ++q) acc[q] += __shfl_xor(acc[q], off, 64);
    }
    if (live && g == 0) {
        P o;
#pragma unroll
        for (int q = 0; q < LV; ++q) from_f32(rows.finish(acc[q], e - b), &o.v[q]);
        *reinterpret_cast<P *>(out + i * out_stride + col0) = o;
    }
}

// The segmented reduction.  What bounds it is the traffic behind the L2s: random 512-byte rows are read at
// 7.5 TB/s from a table that the memory-side cache holds and at 6.6 TB/s from a larger one (measured with a
// kernel that does nothing else).  A loop over one row after the other, the wavefront split into groups of
// lanes that share a row's entries, came near that only for long rows.  Measured, such a loop -> this: the three
// blocks of a mini-batch of 8,192 seeds (512-byte rows; 347 k output rows, 4.7 M entries) 0.432 -> 0.338 ms,
// the reductions of their backward (1.7 M output rows of 3 entries) 0.89 -> 0.49 ms; 2,408-byte rows (10 k
// rows of 25 entries: 612 MB read in 83 us = 7.4 TB/s) as before.
// Few short rows are bound by the instructions of a wavefront and the chain of loads in it: the last entries of
// a run take a batch of 4 or 8 rows if that will do (3,000 rows of 3 entries, 128 fp32 columns: 4.3 us with 16
// loads for three entries, 3.3 now; the loop 3.3).
// Measured and dropped: slabs of 128 to 512 bytes dealt to the XCDs so that every L2 keeps its slab of the
// hot rows (L2 hits 13 -> 24 %, time unchanged or worse); 4 or 16 instead of 8 vectors of 16 bytes in flight;
// lanes past the row left out of the loads (wide fp16 rows 1.3 to 1.7 times slower).
constexpr int kRunRows = 16;
// LV > 0 (rows of at most eight vectors of LV elements): rows of kLongRow entries and more go to reduce_long_row,
// the shorter ones are walked.  fp32, 16 columns, walk and groups: 100 k rows of 10 entries 24 and 28 us, of 15 32 and 28;
// in blocks of a few thousand rows the groups are ahead from 5 or 6 entries.  fp16, 32 columns, where a vector of 16 bytes
// has more additions: 100 k rows of 15 entries 32 and 43 us, 30 k of 20 20.6 and 16.6.
template <typename T>
constexpr int kLongRow = sizeof(T) == 4 ? 12 : 16;

struct FlatShape {
    int dim;
    uint32_t row_blocks;          // workgroups per slab
    int one_slab;                 // (the grid's size, which would tell, is an argument that the launch has to fill in)
    uint32_t busy;                // wavefronts to hand rows to before any gets a second one, up to four rows (run below)
    int mostly_long;              // rows are expected to have kLongRow entries or more: a wavefront takes one at a time
    int log2_lpr;                 // lanes per row in reduce_long_row
};

template <typename T, int VEC, int NV, int LV, typename Rows>
__global__ void __launch_bounds__(kBlock)
k_segment_flat(Rows rows, const int64_t *__restrict__ n_rows, const T *__restrict__ x, int64_t x_stride,
               T *__restrict__ out, int64_t out_stride, FlatShape sh) {
    const int dim = sh.dim, log2_lpr = sh.log2_lpr;
    const uint32_t row_blocks = sh.row_blocks;
    const bool mostly_long = LV > 0 && sh.mostly_long;
    constexpr int kLong = kLongRow<T>;
    using P = Pack<T, VEC>;
    constexpr int U = NV == 1 ? (sizeof(P) == 16 ? 8 : 16) : NV <= 3 ? 4 : 2;    // input rows in flight: 4 to 12 KB per wavefront
    // Partial sums that take the entries in turn.  The turn counts from the start of the run, so a row may begin
    // at any of them; opposite ones are added first, which gives the same bits wherever it began.
    constexpr int NACC = U < 2 ? 1 : VEC <= 2 ? (U < 4 ? U : 4) : NV <= 2 ? 2 : 1;
    const int lane = lane_id();
    const int64_t n = *n_rows;
    const uint32_t slab = sh.one_slab ? 0 : blockIdx.x / row_blocks;
    const uint32_t row_block = blockIdx.x - slab * row_blocks;
    bool live[NV];
    uint32_t lane_off[NV];                                 // lanes past the row read its start and store nothing
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const uint32_t col = ((slab * NV + k) * kWave + lane) * VEC;
        live[k] = col < static_cast<uint32_t>(dim);
        lane_off[k] = (live[k] ? col : 0u) * sizeof(T);
    }
    const int64_t self_rows = Rows::kSelf ? rows.self_rows(n) : 0;         // rows with a diagonal term: the first ones
    const int64_t nwaves = int64_t(row_blocks) * kWavesPerBlock;
    const int64_t wave0 = __builtin_amdgcn_readfirstlane(static_cast<int>(row_block) * kWavesPerBlock + static_cast<int>(threadIdx.x >> 6));
    int run = 1;                                           // rows per wavefront and run
    while (run < kRunRows && run * (run < 4 ? int64_t(sh.busy) : nwaves) < n && !mostly_long) ++run;
    const char *xb = reinterpret_cast<const char *>(x);
    const int64_t x_bytes = x_stride * int64_t(sizeof(T)), out_bytes = out_stride * int64_t(sizeof(T));
    for (int64_t c0 = wave0 * run; c0 < n; c0 += nwaves * run) {
        if constexpr (LV > 0) {
            if (mostly_long) {
                const int b = rows.begin(c0), e = rows.begin(c0 + 1);
                const bool own = c0 < self_rows;
                const float ws = Rows::kSelf && own ? rows.self_weight(c0) : 0.f;      // on its way with the two offsets
                if (e - b >= kLong) {
                    reduce_long_row<T, LV>(rows, c0, b, e, ws, x, x_stride, out, out_stride, dim, log2_lpr);
                    continue;
                }
            }
        }
        const int m = n - c0 < run ? static_cast<int>(n - c0) : run;       // rows of this run
        // diagonal terms in this run: one more entry, its first, for each of the run's first `diag` rows
        const int diag = self_rows > c0 ? static_cast<int>(self_rows - c0 < m ? self_rows - c0 : m) : 0;
        const int t = lane < m ? lane : m;                 // lane t keeps the first position of row c0 + t
        const uint32_t off = static_cast<uint32_t>(rows.begin(c0 + t)) + static_cast<uint32_t>(t < diag ? t : diag);
        uint64_t longs = 0;                                // the run's long rows, if they go by themselves
        if constexpr (LV > 0) {
            const int entries = static_cast<int>(__shfl_down(off, 1) - off) - (lane < diag ? 1 : 0);
            longs = ballot64(lane < m && entries >= kLong);
        }
        for (int cur = 0;;) {
            const int stop = LV > 0 && longs ? __ffsll(static_cast<long long>(longs)) - 1 : m;
            const uint32_t begin = readlane32(off, cur), end = readlane32(off, stop);
            uint32_t row_begin = begin, row_end = readlane32(off, cur + 1);
            float acc[NACC][NV][VEC];
#pragma unroll
            for (int a = 0; a < NACC; ++a)
#pragma unroll
                for (int k = 0; k < NV; ++k)
#pragma unroll
                    for (int q = 0; q < VEC; ++q) acc[a][k][q] = 0.f;
            auto finish_row = [&]() __attribute__((always_inline)) {
                char *orow = reinterpret_cast<char *>(out) + (c0 + cur) * out_bytes;
#pragma unroll
                for (int k = 0; k < NV; ++k) {
                    P o;
#pragma unroll
                    for (int q = 0; q < VEC; ++q) {
                        float sum = acc[0][k][q];
                        if constexpr (NACC == 2) sum += acc[1][k][q];
                        if constexpr (NACC == 4) sum = (sum + acc[2][k][q]) + (acc[1][k][q] + acc[3][k][q]);
                        from_f32(rows.finish(sum, static_cast<int>(row_end - row_begin)), &o.v[q]);
#pragma unroll
                        for (int a = 0; a < NACC; ++a) acc[a][k][q] = 0.f;
                    }
                    if (live[k]) *reinterpret_cast<P *>(orow + lane_off[k]) = o;
                }
                ++cur;
                row_begin = row_end;
                row_end = readlane32(off, cur + 1);
            };
            // the entries e0 ... of the walk, one per lane: input row, weight, and whether it is a diagonal term
            struct Entry {
                int row;
                float w;
                bool own;
            };
            auto fetch = [&](uint32_t e0) __attribute__((always_inline)) {
                Entry en;
                en.w = 1.f;
                en.own = false;
                const uint32_t p = e0 + lane < end ? e0 + lane : end - 1;      // past the end: the last entry again, loaded but not added
                if (Rows::kSelf && diag > 0) {
                    int k = 0;                             // the entry's row: the last that begins at or before it
                    uint32_t first = begin;
                    if (m > 1) {
#pragma unroll
                        for (int h = kRunRows / 2; h > 0; h >>= 1)
                            if (static_cast<uint32_t>(__shfl(static_cast<int>(off), k + h)) <= p) k += h;
                        first = static_cast<uint32_t>(__shfl(static_cast<int>(off), k));
                    }
                    en.own = k < diag && p == first;
                    const int q = static_cast<int>(p - (k < diag ? k + 1 : diag));
                    if (en.own) {
                        en.w = rows.self_weight(c0 + k);
                        en.row = en.w != 0.f ? static_cast<int>(c0) + k : -1;
                    } else {
                        en.row = rows.input_row(q);
                        en.w = rows.weight(q);
                    }
                } else {
                    en.row = rows.input_row(static_cast<int>(p));
                    if (Rows::kWeighted) en.w = rows.weight(static_cast<int>(p));
                }
                return en;
            };
            // W entries from position b of the 64 on: all their loads, then their additions
            auto batch = [&](const Entry &en, uint32_t e0, int cnt, int b, auto width) __attribute__((always_inline)) {
                constexpr int W = decltype(width)::value;
                P v[W][NV];
#pragma unroll
                for (int u = 0; u < W; ++u) {
                    const int r = static_cast<int>(readlane32(static_cast<uint32_t>(en.row), b + u));
                    const char *row = xb + (Rows::kSelf && r < 0 ? 0 : r) * x_bytes;
#pragma unroll
                    for (int k = 0; k < NV; ++k) v[u][k] = *reinterpret_cast<const P *>(row + lane_off[k]);
                }
#pragma unroll
                for (int u = 0; u < W; ++u) {
                    if (b + u >= cnt) continue;
                    while (e0 + static_cast<uint32_t>(b + u) >= row_end) finish_row();
                    if (Rows::kSelf && static_cast<int>(readlane32(static_cast<uint32_t>(en.row), b + u)) < 0) continue;
                    const float w = __uint_as_float(readlane32(__float_as_uint(en.w), b + u));
#pragma unroll
                    for (int k = 0; k < NV; ++k)
#pragma unroll
                        for (int q = 0; q < VEC; ++q) {
                            float &a = acc[u % NACC][k][q];
                            if (Rows::kWeighted) a += w * to_f32(v[u][k].v[q]);
                            else a += to_f32(v[u][k].v[q]);
                        }
                }
            };
            auto walk = [&](auto width) __attribute__((always_inline)) {
                constexpr int W = decltype(width)::value;
                for (uint32_t e0 = begin; e0 < end; e0 += kWave) {
                    const int cnt = end - e0 < kWave ? static_cast<int>(end - e0) : kWave;
                    const Entry en = fetch(e0);
                    int b = 0;
                    for (; b + W <= cnt; b += W) batch(en, e0, cnt, b, width);
                    const int left = cnt - b;
                    if (left > 8 && W > 8) batch(en, e0, cnt, b, width);
                    else if (left > 4 && W > 4) batch(en, e0, cnt, b, std::integral_constant<int, W < 8 ? W : 8>());
                    else if (left > 0) batch(en, e0, cnt, b, std::integral_constant<int, W < 4 ? W : 4>());
                }
            };
            if (begin < end) walk(std::integral_constant<int, U>());
            while (cur < stop) finish_row();
            if (stop == m) break;
            const int b = static_cast<int>(readlane32(off, stop)) - (stop < diag ? stop : diag);
            const int e = static_cast<int>(readlane32(off, stop + 1)) - (stop + 1 < diag ? stop + 1 : diag);
            const float ws = Rows::kSelf && stop < diag ? rows.self_weight(c0 + stop) : 0.f;
            if constexpr (LV > 0) reduce_long_row<T, LV>(rows, c0 + stop, b, e, ws, x, x_stride, out, out_stride, dim, log2_lpr);
            longs &= longs - 1;
            cur = stop + 1;
            if (cur == m) break;
        }
    }
}

// columns [0, shape.dim) of all rows, nv vectors of vec elements per lane; long_vec: the kernel's LV
template <typename T, typename Rows>
int launch_columns(mqg_ctx *ctx, const char *name, const Rows &rows, const int64_t *n_rows, const T *x,
                   int64_t x_stride, T *out, int64_t out_stride, FlatShape shape, int vec, int nv, int long_vec, hipStream_t s) {
    const int64_t slabs = ceil_div(ceil_div(shape.dim, vec), int64_t(nv) * kWave);
    shape.one_slab = slabs == 1 ? 1 : 0;
    const int grid = static_cast<int>(shape.row_blocks * slabs);
#define MQG_AGG_LV(V, NV, LV)                                                                                          \
    MQG_LAUNCH(ctx, name, s,                                                                                    \
               (k_segment_flat<T, V, NV, LV, Rows><<<grid, kBlock, 0, s>>>(rows, n_rows, x, x_stride, out, out_stride, shape)))
#define MQG_AGG(V, NV) MQG_AGG_LV(V, NV, 0)
#define MQG_AGG_PICK(V)                        \
    switch (nv) {                              \
        case 1: MQG_AGG(V, 1); break;          \
        case 2: MQG_AGG(V, 2); break;          \
        case 3: MQG_AGG(V, 3); break;          \
        case 4: MQG_AGG(V, 4); break;          \
        case 5: if constexpr (Rows::kFewEntries) MQG_AGG(V, 5); break;          /* the others' are filled: slabs */ \
        default: if constexpr (Rows::kFewEntries) MQG_AGG(V, 6); break;         \
    }
    constexpr int kWidest = 16 / static_cast<int>(sizeof(T));
    if (long_vec == 8) {
        if constexpr (kWidest == 8) MQG_AGG_LV(1, 1, 8);
    } else if (long_vec == 4) {
        MQG_AGG_LV(1, 1, 4);
    } else if (long_vec == 2) {
        MQG_AGG_LV(1, 1, 2);
    } else if (long_vec == 1) {
        MQG_AGG_LV(1, 1, 1);
    } else if (vec == kWidest) {
        MQG_AGG_PICK(kWidest);
    } else if (vec == kWidest / 2) {
        MQG_AGG_PICK(kWidest / 2);
    } else if (vec == 2 && kWidest == 8) {
        MQG_AGG(2, 1);
    } else {
        MQG_AGG(1, 1);
    }
#undef MQG_AGG_PICK
#undef MQG_AGG
#undef MQG_AGG_LV
    return MQG_OK;
}

template <typename T, typename Rows>
int launch(mqg_ctx *ctx, const char *name, const Rows &rows, const int64_t *n_rows, int64_t cap_rows, int64_t cap_nnz, const T *x,
           int64_t x_stride, T *out, int64_t out_stride, int dim, hipStream_t s) {
    // widest vector (<= 16 bytes) that divides dim and both strides and keeps the bases aligned.
    // When both strides leave room, dim is first rounded up to whole 16-byte words: the extra
    // columns are read from the input rows' padding and written to the output rows' padding.
    int vec = 16 / static_cast<int>(sizeof(T));
    {
        const int dim16 = static_cast<int>(ceil_div(dim, vec)) * vec;
        if (dim16 <= x_stride && dim16 <= out_stride && x_stride % vec == 0 && out_stride % vec == 0) dim = dim16;
    }
    auto ok = [&](int v) {
        int64_t bytes = int64_t(v) * sizeof(T);
        return dim % v == 0 && x_stride % v == 0 && out_stride % v == 0 &&
               reinterpret_cast<uintptr_t>(x) % bytes == 0 && reinterpret_cast<uintptr_t>(out) % bytes == 0;
    };
    while (vec > 1 && !ok(vec)) vec >>= 1;
    // Up to eight of these vectors: rows of many entries go by themselves, see k_segment_flat.
    const int wide_lanes = static_cast<int>(ceil_div(dim, vec));
    const int long_vec = wide_lanes <= 8 ? vec : 0;
    int log2_lpr = 0;
    while ((1 << log2_lpr) < wide_lanes && log2_lpr < 3) ++log2_lpr;
    // the narrowest vector with which the 64 lanes still cover the row (wider rows: the widest, in slabs)
    while (vec > 1 && ceil_div(dim, vec / 2) <= kWave) vec >>= 1;
    // Rows of more than 64 vectors: NV vectors per lane, or slabs of 64 vectors with a wavefront each.  More
    // vectors per lane share the walk over the entries, slabs spread few rows over more wavefronts and
    // leave a row's last, partly filled vector to a wavefront of its own.  Output rows of few entries (the
    // backward) want the first up to six vectors (513 to 800 fp32 columns: 236 to 345 us against 295 to
    // 367 us).  Output rows of many entries want slabs if the vectors are well filled, in time over that with
    // vectors per lane, three mini-batches of fanouts 4 to 25: 67 % filled 1.14 to 1.16, 71 to 75 % 0.97 to 1.07,
    // 77 % 1.01 to 1.05, 79 to 84 % 0.90 to 1.03, full 0.88 to 0.97.  Two vectors only if both are full: two slabs
    // share the cache lines in the middle of a row (500 columns 1.05 to 1.07, 512 0.93 to 0.98).
    const int64_t lanes = ceil_div(dim, vec);
    const int64_t units = ceil_div(lanes, kWave);
    const bool filled = units == 2 ? lanes == 2 * kWave : units > 2 && lanes * 100 >= units * kWave * 78;
    const bool spread = units > 6 || vec < 8 / static_cast<int>(sizeof(T)) || (!Rows::kFewEntries && filled);
    const int nv = spread ? 1 : static_cast<int>(units);
    const int64_t row_blocks = std::min<int64_t>(std::max<int64_t>(1, ceil_div(cap_rows, kWavesPerBlock)), 256 * 32);
    // Narrow rows of few entries are handed out two to four at a time once the chip's 8,192 wavefronts have one
    // each (10 k rows of 5 entries, 16 fp32 columns: 5.1 -> 4.6 us, 30 k of 10: 13.2 -> 9.6; rows of 25: the other
    // way round).  Their expected length is what the block's capacities say, a sampled block's fanout.
    const bool mostly_long = cap_nnz >= kLongRow<T> * cap_rows;
    FlatShape shape;
    shape.dim = dim;
    shape.row_blocks = static_cast<uint32_t>(row_blocks);
    shape.busy = long_vec && !mostly_long ? 8192 : static_cast<uint32_t>(row_blocks * kWavesPerBlock);
    shape.mostly_long = mostly_long ? 1 : 0;
    shape.log2_lpr = log2_lpr;
    // A launch has fewer than 2^32 threads and the kernel's column offsets are 32 bits: very wide rows take
    // several launches over pieces of their columns, 64 MB of a row at most each.
    const int64_t slabs_at_once = std::min<int64_t>((int64_t(1) << 22) / row_blocks, int64_t(1) << 16);
    if (nv == 1 && units > slabs_at_once) {
        const int64_t piece = slabs_at_once * kWave * vec;
        for (int64_t c0 = 0; c0 < dim; c0 += piece) {
            shape.dim = static_cast<int>(std::min<int64_t>(piece, dim - c0));
            int rc = launch_columns(ctx, name, rows, n_rows, x + c0, x_stride, out + c0, out_stride, shape, vec, nv, 0, s);
            if (rc != MQG_OK) return rc;
        }
        return MQG_OK;
    }
    return launch_columns(ctx, name, rows, n_rows, x, x_stride, out, out_stride, shape, vec, nv, long_vec, s);
}

// ---------------------------------------------------------------- edges ordered by source

// payload of edge e = its destination row (the keys are `indices`).  A wavefront takes a run of consecutive edges,
// 64 or as many more as give every wavefront of the chip one run (runs of 512 left 38 k edges to 74 wavefronts:
// 5.9 us, 2.4 in runs of 64; a bisection per edge 3.4); its lanes hold the offsets of 64 consecutive rows, and every edge finds its row among them.  The
// window of rows only moves forward and ends at the last row, which takes every edge past the last offset
// (the number of edges comes from another array than the offsets): the loop ends whatever the block holds.
// Bound by its 4-byte store per edge; a bisection of all of indptr per edge (19 dependent loads) took 57
// instead of 13 us for 4.3 M edges of 295 k rows.
constexpr int kEdgeWaves = 8192;
constexpr int64_t kPickRowsEdges = int64_t(3) << 19;     // see run_aggregate_backward
__global__ void __launch_bounds__(kBlock)
k_edge_dst_rows(const int32_t *__restrict__ indptr, const int64_t *__restrict__ sizes, int32_t *__restrict__ dst_row) {
    const int lane = lane_id();
    const int64_t num_dst = sizes[0], nnz = sizes[2];
    const int64_t run = nnz > kEdgeWaves * kWave ? (nnz + kEdgeWaves * kWave - 1) / (kEdgeWaves * kWave) * kWave : kWave;
    const int64_t step = int64_t(gridDim.x) * kWavesPerBlock * run;
    for (int64_t e0 = (int64_t(blockIdx.x) * kWavesPerBlock + (threadIdx.x >> 6)) * run; e0 < nnz; e0 += step) {
        const int64_t e1 = e0 + run < nnz ? e0 + run : nnz;
        auto row_of = [&](int64_t e) {
            const int64_t r = wave_count_below<false>(indptr, num_dst, e) - 1;
            return r > 0 ? r : 0;
        };
        int64_t r0 = row_of(e0);
        auto offset = [&](int64_t r) { return indptr[r < num_dst ? r : num_dst]; };
        int off = offset(r0 + lane), end = offset(r0 + kWave);                  // of rows r0 ..., and where they end
        for (int64_t c0 = e0; c0 < e1; c0 += kWave) {
            const int64_t e = c0 + lane;
            bool open = e < e1;
            for (;;) {
                int k = 0;                                 // the last of the 64 rows that begins at or before e
#pragma unroll
                for (int h = 32; h > 0; h >>= 1)
                    if (__shfl(off, k + h, 64) <= e) k += h;
                if (open && (e < end || r0 + kWave >= num_dst)) {
                    const int64_t r = r0 + k < num_dst ? r0 + k : num_dst - 1;
                    dst_row[e] = static_cast<int32_t>(r > 0 ? r : 0);
                    open = false;
                }
                const uint64_t left = ballot64(open);
                if (!left) break;
                // the next 64 rows, or, past a stretch of empty ones, the row of the first edge that is left
                r0 += kWave;
                const int64_t first = c0 + __ffsll(static_cast<long long>(left)) - 1;
                if (offset(r0 + kWave) <= first) {
                    const int64_t r = row_of(first);
                    r0 = r > r0 ? r : r0;
                }
                off = offset(r0 + lane);
                end = offset(r0 + kWave);
            }
        }
    }
}

// col_ptr[s] = first position in the sorted key array whose source is >= s, s = 0..num_src.  A wavefront
// takes 64 consecutive sources, finds the positions they span, and every lane bisects that span only: its
// loads hit the wavefront's own lines (25.5 -> 23.2 us for 1.35 M sources of 4.3 M edges; four sources per lane: 10 us more).
__global__ void __launch_bounds__(kBlock)
k_col_ptr(const uint32_t *__restrict__ sorted_src, const int64_t *__restrict__ sizes, int32_t *__restrict__ col_ptr) {
    const int64_t num_src = sizes[1], nnz = sizes[2];
    const int64_t stride = int64_t(gridDim.x) * kBlock;
    for (int64_t k0 = int64_t(blockIdx.x) * kBlock + (threadIdx.x & ~63u); k0 <= num_src; k0 += stride) {
        int64_t lo = wave_count_below<true>(sorted_src, nnz, k0);
        int64_t hi = wave_count_below<true>(sorted_src, nnz, k0 + kWave);
        const int64_t k = k0 + lane_id();
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (static_cast<int64_t>(sorted_src[mid]) < k) lo = mid + 1; else hi = mid;
        }
        if (k <= num_src) col_ptr[k] = static_cast<int32_t>(lo);
    }
}

// destination row and weight of every edge in the by-source order; rows: the destination row of every edge in
// the block's own order, or null (then indptr is bisected)
__global__ void __launch_bounds__(kBlock)
k_permute_edges(const int32_t *__restrict__ perm, const int32_t *__restrict__ indptr, const int32_t *__restrict__ rows,
                const float *__restrict__ edge_w, const int64_t *__restrict__ sizes, int32_t *__restrict__ dst_row, float *__restrict__ w_sorted) {
    const int64_t num_dst = sizes[0], nnz = sizes[2];
    const int64_t stride = int64_t(gridDim.x) * kBlock;
    for (int64_t q = int64_t(blockIdx.x) * kBlock + threadIdx.x; q < nnz; q += stride) {
        const int32_t e = perm[q];
        w_sorted[q] = edge_w[e];
        if (rows) {
            dst_row[q] = rows[e];
            continue;
        }
        int64_t lo = 0, hi = num_dst;                      // largest i with indptr[i] <= e
        while (hi - lo > 1) {
            int64_t mid = (lo + hi) >> 1;
            if (indptr[mid] <= e) lo = mid; else hi = mid;
        }
        dst_row[q] = static_cast<int32_t>(lo);
    }
}

// Weights of the sampled estimator of P H, P = D^-1/2 (A + I) D^-1/2 (paper Eq. 1-3): LANES lanes per
// destination row; edge p = (v_i, v_j) gets deg(v_i)/n_i / sqrt((deg(v_i)+1)(deg(v_j)+1)), the
// row's diagonal term is 1/(deg(v_i)+1).  Computed in double, rounded once to float.
// Bound by the double division and square root, which a wavefront pays for whole, and by the chain of four loads: the row's and
// its first edges' are under way together.  (A wavefront per row, one load after the other: 10 k rows of 25 edges 10.3 us, 7.0 so.  Beside
// the weighted sums and their backwards, 306 us, that is within the spread of the runs.)
template <typename PtrT, typename IdxT, int LANES>
__global__ void __launch_bounds__(kBlock)
k_gcn_edge_weights(const PtrT *__restrict__ row_ptr, const IdxT *__restrict__ src_ids, const int32_t *__restrict__ indptr,
                   const int32_t *__restrict__ indices, const int64_t *__restrict__ sizes, float *__restrict__ edge_w,
                   float *__restrict__ self_w, int grid) {
    const int lane = static_cast<int>(threadIdx.x) % LANES;
    const int64_t n = sizes[0];
    const int64_t step = int64_t(grid) * (kBlock / LANES);
    for (int64_t i = int64_t(blockIdx.x) * (kBlock / LANES) + threadIdx.x / LANES; i < n; i += step) {
        const int64_t v = static_cast<int64_t>(src_ids[i]);
        const int b = indptr[i], e = indptr[i + 1];
        int p = b + lane;
        int64_t u = p < e ? static_cast<int64_t>(src_ids[indices[p]]) : v;
        const int64_t v0 = static_cast<int64_t>(row_ptr[v]), v1 = static_cast<int64_t>(row_ptr[v + 1]);
        int64_t u0 = static_cast<int64_t>(row_ptr[u]), u1 = static_cast<int64_t>(row_ptr[u + 1]);
        const double deg_i = static_cast<double>(v1 - v0);
        const double scale = deg_i / static_cast<double>(e - b);
        if (lane == 0) self_w[i] = static_cast<float>(1.0 / (deg_i + 1.0));
        while (p < e) {
            const double deg_j = static_cast<double>(u1 - u0);
            edge_w[p] = static_cast<float>(scale * (1.0 / sqrt((deg_i + 1.0) * (deg_j + 1.0))));
            p += LANES;
            if (p < e) {
                u = static_cast<int64_t>(src_ids[indices[p]]);
                u0 = static_cast<int64_t>(row_ptr[u]);
                u1 = static_cast<int64_t>(row_ptr[u + 1]);
            }
        }
    }
}

}  // namespace

template <typename PtrT, typename IdxT>
static int launch_gcn_edge_weights(mqg_ctx *ctx, const mqg_graph *g, const mqg_block *b, float *edge_w, float *self_w, hipStream_t s) {
    // As many lanes as a row has edges at most, by the block's capacities: what the rows hold is known on the device only.  A block with
    // room for more rows than its edges fill takes several rounds (64 edges a row: 10 k rows 7.7 us in eight, 6.6 in one; 300 rows 5.4 and
    // 4.7), one with room for more edges leaves lanes idle, as a wavefront per row did (10 k rows of 25: 4.9 and 4.6).
    const int64_t most = b->cap_nnz / std::max<int64_t>(b->cap_dst, 1);
#define MQG_GCNW(LANES)                                                                                                                \
    do {                                                                                                                               \
        const int grid = static_cast<int>(std::min<int64_t>(std::max<int64_t>(1, ceil_div(b->cap_dst, kBlock / LANES)), 256 * 32));     \
        MQG_LAUNCH(ctx, "k_gcn_edge_weights", s,                                                                                       \
                   (k_gcn_edge_weights<PtrT, IdxT, LANES><<<grid, kBlock, 0, s>>>(                                                     \
                       static_cast<const PtrT *>(g->row_ptr), static_cast<const IdxT *>(b->src_ids), b->indptr, b->indices, b->sizes,  \
                       edge_w, self_w, grid)));                                                                                        \
    } while (0)
    if (most <= 8) MQG_GCNW(8);
    else if (most <= 16) MQG_GCNW(16);
    else if (most <= 32) MQG_GCNW(32);
    else MQG_GCNW(64);
#undef MQG_GCNW
    return MQG_OK;
}

int run_gcn_edge_weights(mqg_ctx *ctx, const mqg_graph *g, const mqg_block *b, float *edge_w, float *self_w, hipStream_t s) {
    if (g->ptr_type == MQG_I64 && g->idx_type == MQG_I64) return launch_gcn_edge_weights<int64_t, int64_t>(ctx, g, b, edge_w, self_w, s);
    if (g->ptr_type == MQG_I64) return launch_gcn_edge_weights<int64_t, int32_t>(ctx, g, b, edge_w, self_w, s);
    if (g->idx_type == MQG_I64) return launch_gcn_edge_weights<int32_t, int64_t>(ctx, g, b, edge_w, self_w, s);
    return launch_gcn_edge_weights<int32_t, int32_t>(ctx, g, b, edge_w, self_w, s);
}

int run_weighted_aggregate(mqg_ctx *ctx, const mqg_block *b, const float *edge_w, const float *self_w, const void *x,
                           int64_t x_stride, void *out, int64_t out_stride, int32_t dim, int32_t dtype, hipStream_t s) {
    WeightedRows rows{b->indptr, b->indices, edge_w, self_w};
    if (dtype == MQG_F16)
        return launch<_Float16>(ctx, "k_weighted_aggregate", rows, &b->sizes[0], b->cap_dst, b->cap_nnz, static_cast<const _Float16 *>(x),
                                x_stride, static_cast<_Float16 *>(out), out_stride, dim, s);
    return launch<float>(ctx, "k_weighted_aggregate", rows, &b->sizes[0], b->cap_dst, b->cap_nnz, static_cast<const float *>(x), x_stride,
                         static_cast<float *>(out), out_stride, dim, s);
}

int run_mean_aggregate(mqg_ctx *ctx, const mqg_block *b, const void *x, int64_t x_stride, void *out,
                       int64_t out_stride, int32_t dim, int32_t dtype, hipStream_t s) {
    ForwardRows rows{b->indptr, b->indices};
    if (dtype == MQG_F16)
        return launch<_Float16>(ctx, "k_mean_aggregate", rows, &b->sizes[0], b->cap_dst, b->cap_nnz, static_cast<const _Float16 *>(x),
                                x_stride, static_cast<_Float16 *>(out), out_stride, dim, s);
    return launch<float>(ctx, "k_mean_aggregate", rows, &b->sizes[0], b->cap_dst, b->cap_nnz, static_cast<const float *>(x), x_stride,
                         static_cast<float *>(out), out_stride, dim, s);
}

// Scratch of the backward: room for blocks of nnz_cap edges and src_cap sources (never less than the
// context's own bounds).  Growing it waits for the stream first: earlier work may still use the old one.
int ensure_backward_scratch(mqg_ctx *ctx, int64_t nnz_cap, int64_t src_cap, hipStream_t s, const char *who) {
    if (nnz_cap <= ctx->bwd_nnz_cap && src_cap <= ctx->bwd_src_cap) return MQG_OK;
    hipError_t e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail(ctx, MQG_ERR_HIP, std::string(who) + hipGetErrorString(e));
    free_backward_scratch(ctx);
    const int64_t nn = std::max<int64_t>(std::max(nnz_cap, ctx->max_nnz), 1);
    const int64_t ns = std::max<int64_t>(std::max(src_cap, ctx->max_src), 1);
    auto alloc = [&](void **p, int64_t bytes) { return hipMalloc(p, static_cast<size_t>(std::max<int64_t>(bytes, 4))) == hipSuccess; };
    bool ok = alloc(reinterpret_cast<void **>(&ctx->bwd.keys[0]), nn * 4 + 16) && alloc(reinterpret_cast<void **>(&ctx->bwd.keys[1]), nn * 4) &&
              alloc(reinterpret_cast<void **>(&ctx->bwd.vals[0]), nn * 4) && alloc(reinterpret_cast<void **>(&ctx->bwd.vals[1]), nn * 4) &&
              alloc(reinterpret_cast<void **>(&ctx->bwd.hist), std::max(radix_hist_len_max(nn), order_hist_len(nn)) * 4) &&
              alloc(reinterpret_cast<void **>(&ctx->bwd.totals), kRadixTotals * 4) &&
              alloc(reinterpret_cast<void **>(&ctx->bwd_dst_row), nn * 4) &&
              alloc(reinterpret_cast<void **>(&ctx->bwd_w_sorted), nn * 4) &&
              alloc(reinterpret_cast<void **>(&ctx->bwd_col_ptr), (ns + 2) * 4);
    if (!ok) {
        free_backward_scratch(ctx);
        return fail(ctx, MQG_ERR_HIP, std::string(who) + "scratch allocation failed");
    }
    ctx->bwd_nnz_cap = nn;
    ctx->bwd_src_cap = ns;
    return MQG_OK;
}

// edge_w == nullptr: the mean aggregation's backward; otherwise the weighted one (self_w may be null)
int run_aggregate_backward(mqg_ctx *ctx, const mqg_block *b, const float *edge_w, const float *self_w, const void *grad_out,
                           int64_t go_stride, void *grad_x, int64_t gx_stride, int32_t dim, int32_t dtype, hipStream_t s) {
    const char *who = edge_w ? "mqg_weighted_aggregate_backward: " : "mqg_sage_mean_aggregate_backward: ";
    // scratch for the by-source ordering of the edges (reserved, or allocated at the first backward call)
    const int64_t nnz_cap = b->cap_nnz, src_cap = b->cap_src;
    int rc0 = ensure_backward_scratch(ctx, nnz_cap, src_cap, s, who);
    if (rc0 != MQG_OK) return rc0;

    auto reduce_weighted = [&](const int32_t *dst_sorted) -> int {
        WeightedBackwardRows rows{ctx->bwd_col_ptr, dst_sorted, ctx->bwd_w_sorted, self_w, b->sizes};
        if (dtype == MQG_F16)
            return launch<_Float16>(ctx, "k_weighted_aggregate_backward", rows, &b->sizes[1], src_cap, nnz_cap,
                                    static_cast<const _Float16 *>(grad_out), go_stride, static_cast<_Float16 *>(grad_x), gx_stride, dim, s);
        return launch<float>(ctx, "k_weighted_aggregate_backward", rows, &b->sizes[1], src_cap, nnz_cap, static_cast<const float *>(grad_out),
                             go_stride, static_cast<float *>(grad_x), gx_stride, dim, s);
    };
    auto reduce_mean = [&](const int32_t *dst_sorted) -> int {
        BackwardRows rows{ctx->bwd_col_ptr, dst_sorted, b->indptr};
        if (dtype == MQG_F16)
            return launch<_Float16>(ctx, "k_mean_aggregate_backward", rows, &b->sizes[1], src_cap, nnz_cap,
                                    static_cast<const _Float16 *>(grad_out), go_stride, static_cast<_Float16 *>(grad_x), gx_stride, dim, s);
        return launch<float>(ctx, "k_mean_aggregate_backward", rows, &b->sizes[1], src_cap, nnz_cap, static_cast<const float *>(grad_out),
                             go_stride, static_cast<float *>(grad_x), gx_stride, dim, s);
    };

    if (can_order_edges(src_cap)) {
        // bwd.vals[0] and bwd.keys hold the partitioned edges on the way
        rc0 = order_edges_by_source(ctx, b, edge_w, ctx->bwd_col_ptr, ctx->bwd_dst_row, ctx->bwd_w_sorted, s);
        if (rc0 != MQG_OK) return rc0;
        return edge_w ? reduce_weighted(ctx->bwd_dst_row) : reduce_mean(ctx->bwd_dst_row);
    }
    const int egrid = static_cast<int>(std::min<int64_t>(std::max<int64_t>(1, ceil_div(nnz_cap, kBlock)), 8192));
    // More sources than that: edges by source by a radix sort, stably.  An edge carries its destination row along, or (weighted) its own
    // position, which the sort's first pass makes itself - at least one pass, for that.
    const int rgrid = static_cast<int>(std::min<int64_t>(std::max<int64_t>(1, ceil_div(nnz_cap, kBlock)), kEdgeWaves / kWavesPerBlock));
    if (!edge_w) MQG_LAUNCH(ctx, "k_edge_dst_rows", s, (k_edge_dst_rows<<<rgrid, kBlock, 0, s>>>(b->indptr, b->sizes, ctx->bwd_dst_row)));
    const int bits = std::max(1, radix_key_bits(static_cast<uint64_t>(std::max<int64_t>(src_cap, 1) - 1)));
    int which = -1;
    int rc = radix_sort_pairs(ctx, reinterpret_cast<const uint32_t *>(b->indices), edge_w ? nullptr : ctx->bwd_dst_row, ctx->bwd, nnz_cap,
                              &b->sizes[2], bits, s, &which);
    if (rc != MQG_OK) return rc;
    const uint32_t *sorted_src = ctx->bwd.keys[which];
    const int32_t *sorted_dst = ctx->bwd.vals[which];
    const int cgrid = static_cast<int>(std::min<int64_t>(std::max<int64_t>(1, ceil_div(src_cap + 1, kBlock)), 8192));
    MQG_LAUNCH(ctx, "k_col_ptr", s, (k_col_ptr<<<cgrid, kBlock, 0, s>>>(sorted_src, b->sizes, ctx->bwd_col_ptr)));

    if (edge_w) {
        // the sort's payload was the edge position: turn it into (destination row, weight)
        int32_t *dst_sorted = ctx->bwd_dst_row;
        // the rows of many edges are written once, in order, into the sort's other buffer and picked from there
        // (both kernels against the bisection alone: 1 M edges 55 and 47 us, 2 M 73 and 78, 4 M 112 and 135)
        int32_t *rows_of = nnz_cap > kPickRowsEdges ? ctx->bwd.vals[which ^ 1] : nullptr;
        if (rows_of) MQG_LAUNCH(ctx, "k_edge_dst_rows", s, (k_edge_dst_rows<<<rgrid, kBlock, 0, s>>>(b->indptr, b->sizes, rows_of)));
        MQG_LAUNCH(ctx, "k_permute_edges", s,
                   (k_permute_edges<<<egrid, kBlock, 0, s>>>(sorted_dst, b->indptr, rows_of, edge_w, b->sizes, dst_sorted, ctx->bwd_w_sorted)));
        return reduce_weighted(dst_sorted);
    }
    return reduce_mean(sorted_dst);
}

}  // namespace mqg
