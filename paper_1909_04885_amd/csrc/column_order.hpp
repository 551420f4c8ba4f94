// Long sparse rows: a second copy of the entries, ordered by column inside blocks of rows, for the two passes over the matrix
// that are not the solvers': x_i . w of every row (the gap, and the residuals the next local pass starts from), and the merge of
// the solvers' updates, sum_i coef_i x_i.  Each of the two goes over it where that is the faster way (dots_pay, merge_pays).
//
// By rows a row's thousand entries, spread over twenty million columns, are a thousand lonely 4-byte accesses to the shared
// vector.  Here the rows are divided into blocks of CO_ROWS; a block's entries lie by buckets of neighbouring columns, and inside
// a bucket, a few thousand at a time, by column.  Then everything is a stream:
//   column_dots    a workgroup takes a part of a block's entries and adds val * w[col] up in LDS, one double per row; the entries
//                  of a wavefront lie on a few lines of w;
//   column_merge   a workgroup takes a bucket, and one block after the other: the block's coefficients go into LDS, and
//                  coef[row] * val is added up in LDS, one double per column of the bucket.
// The merge needs no private vectors: the coefficients of the steps are all it reads beside the matrix.  It reads all of a block's
// for every bucket, though, 64 KB: what bounds the dot products is the matrix, eight bytes per entry (and the adds in LDS); the merge
// is bound by these reads of the L2 where a bucket holds few of a block's entries (merge_pays).
#pragma once
#include <hip/hip_runtime.h>
#include "aggregate_gap.hpp"
#include "device_types.hpp"
#include "mem.hpp"

namespace chicle {

constexpr int CO_ROWS_LOG2 = 14, CO_ROWS = 1 << CO_ROWS_LOG2;    // rows of a block: 128 KB of doubles
constexpr int CO_SEG_LOG2 = 32 - CO_ROWS_LOG2;                   // an entry's column is kept relative to its segment's
constexpr int CO_THREADS = 1024;
constexpr int CO_MAX_BUCKET_LOG2 = 13, CO_MIN_BUCKET_LOG2 = 10;  // columns of a bucket (64 KB of doubles at most)
constexpr int CO_LDS_BUCKETS = 16384;                            // so many are counted in LDS
constexpr int CO_PIECE = 4096;                                   // entries that are sorted by column together
constexpr int CO_GROUP_ROWS = 128;                               // rows per workgroup while the copy is made
constexpr int CO_PARTS = 256;                                    // workgroups of the dot products that run side by side: one to a compute unit
constexpr int CO_LEAST_PARTS = 4;                                // parts that a block is given room for, however many blocks there are

struct __align__(8) ColumnEntry { unsigned key; float val; };    // key: column in the segment, row in the block
static_assert(CO_SEG_LOG2 >= CO_MAX_BUCKET_LOG2, "a segment is whole buckets");

struct ColumnOrder {
    const ColumnEntry *entries;
    const long long *off;        // [block * buckets + bucket], and the end
    int buckets, bucket_log2, blocks;
    int64_t n_total;
};

// ---- making the copy, once per data set -----------------------------------------------------------------------------

// A workgroup's rows: CO_GROUP_ROWS of a chunk, as far as they are in one block; f(first row, end, block) for every such part.
template <typename F>
__device__ __forceinline__ void co_row_parts(const ChunkDev &ch, F f)
{
    const int r1 = min(ch.n_rows, ((int)blockIdx.x + 1) * CO_GROUP_ROWS);
    for (int r = (int)blockIdx.x * CO_GROUP_ROWS; r < r1;) {
        const int block = (ch.row_base + r) >> CO_ROWS_LOG2;
        const int end = (int)min((int64_t)r1, ((int64_t)(block + 1) << CO_ROWS_LOG2) - ch.row_base);
        f(r, end, block);
        r = end;
    }
}

// count[block * buckets + bucket] += entries.  Grid: (groups of rows, chunk); dynamic LDS: an int per bucket where these are few.
__global__ __launch_bounds__(256) void co_count(const ChunkDev *__restrict__ chunks, int bucket_log2, int buckets, unsigned long long *count)
{
    extern __shared__ int co_hist[];
    const ChunkDev &ch = chunks[blockIdx.y];
    const bool lds = buckets <= CO_LDS_BUCKETS;
    co_row_parts(ch, [&](int r0, int r1, int block) {
        unsigned long long *mine = count + (int64_t)block * buckets;
        if (lds) {
            for (int i = threadIdx.x; i < buckets; i += 256) co_hist[i] = 0;
            __syncthreads();
        }
        for (int p = ch.row_ptr[r0] + threadIdx.x; p < ch.row_ptr[r1]; p += 256) {
            const int b = ch.col[p] >> bucket_log2;
            if (lds) atomicAdd(&co_hist[b], 1);
            else atomicAdd(mine + b, 1ull);
        }
        __syncthreads();
        if (lds)
            for (int i = threadIdx.x; i < buckets; i += 256)
                if (co_hist[i]) atomicAdd(mine + i, (unsigned long long)co_hist[i]);
        __syncthreads();
    });
}

// off[i] = sum of count[0 .. i), off[n] = all; count becomes a copy of off, to be counted up.  most: the largest bucket, over all
// blocks.  One workgroup.
__global__ __launch_bounds__(1024) void co_scan(unsigned long long *count, long long *off, int64_t n, int buckets, unsigned long long *most)
{
    __shared__ unsigned long long wave_sum[16], carry;
    if (threadIdx.x == 0) carry = 0;
    unsigned long long top = 0;
    for (int b = threadIdx.x; b < buckets; b += 1024) {
        unsigned long long sum = 0;
        for (int64_t i = b; i < n; i += buckets) sum += count[i];
        top = max(top, sum);
    }
    if (top) atomicMax(most, top);
    __syncthreads();
    for (int64_t base = 0; base < n; base += 1024) {
        const int64_t i = base + threadIdx.x;
        const unsigned long long v = i < n ? count[i] : 0;
        unsigned long long incl = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned long long y = __shfl_up(incl, o, 64);
            if ((threadIdx.x & 63) >= o) incl += y;
        }
        if ((threadIdx.x & 63) == 63) wave_sum[threadIdx.x >> 6] = incl;
        __syncthreads();
        unsigned long long at = carry;
        for (int w = 0; w < (int)(threadIdx.x >> 6); ++w) at += wave_sum[w];
        if (i < n) { off[i] = (long long)(at + incl - v); count[i] = at + incl - v; }
        __syncthreads();
        if (threadIdx.x == 1023) carry = at + incl;
        __syncthreads();
    }
    if (threadIdx.x == 0) off[n] = (long long)carry;
}

// Entries into their buckets.  Grid as co_count; a wavefront per row; dynamic LDS: a 64-bit word per bucket where these are few.
__global__ __launch_bounds__(256) void co_scatter(const ChunkDev *__restrict__ chunks, int bucket_log2, int buckets, unsigned long long *next,
                                                  ColumnEntry *entries)
{
    extern __shared__ unsigned long long co_at[];
    const ChunkDev &ch = chunks[blockIdx.y];
    const bool lds = buckets <= CO_LDS_BUCKETS;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    co_row_parts(ch, [&](int r0, int r1, int block) {
        unsigned long long *mine = next + (int64_t)block * buckets;
        if (lds) {
            for (int i = threadIdx.x; i < buckets; i += 256) co_at[i] = 0;
            __syncthreads();
            for (int p = ch.row_ptr[r0] + threadIdx.x; p < ch.row_ptr[r1]; p += 256) atomicAdd(&co_at[ch.col[p] >> bucket_log2], 1ull);
            __syncthreads();
            for (int i = threadIdx.x; i < buckets; i += 256)
                if (co_at[i]) co_at[i] = atomicAdd(mine + i, co_at[i]);
            __syncthreads();
        }
        for (int r = r0 + wave; r < r1; r += 4) {
            const unsigned row = (unsigned)(ch.row_base + r) & (CO_ROWS - 1);
            for (int p = ch.row_ptr[r] + lane; p < ch.row_ptr[r + 1]; p += 64) {
                const int c = ch.col[p], b = c >> bucket_log2;
                const unsigned long long at = atomicAdd(lds ? co_at + b : mine + b, 1ull);
                entries[at] = ColumnEntry{((unsigned)c << CO_ROWS_LOG2) | row, ch.val[p]};
            }
        }
        __syncthreads();
    });
}

// A bucket's entries by column, CO_PIECE of them at a time (the order of equal columns is whichever).  Grid: workgroups over
// (block, bucket).
__global__ __launch_bounds__(1024) void co_sort(const long long *__restrict__ off, int64_t n, int bucket_log2, ColumnEntry *entries)
{
    __shared__ int count[1 << CO_MAX_BUCKET_LOG2];
    __shared__ ColumnEntry piece[CO_PIECE];
    __shared__ int wave_sum[16];
    constexpr int PER = (1 << CO_MAX_BUCKET_LOG2) / 1024;
    const int tid = threadIdx.x;
    const unsigned mask = (1u << bucket_log2) - 1u;
    for (int64_t i = blockIdx.x; i < n; i += gridDim.x)
        for (long long at = off[i]; at < off[i + 1]; at += CO_PIECE) {
            const int m = (int)min((long long)CO_PIECE, off[i + 1] - at);
            if (m <= 64) break;                      // (fewer than lanes of a wavefront)
            for (int c = tid; c < 1 << CO_MAX_BUCKET_LOG2; c += 1024) count[c] = 0;
            __syncthreads();
            ColumnEntry mine[CO_PIECE / 1024];
#pragma unroll
            for (int q = 0; q < CO_PIECE / 1024; ++q)
                if (tid + 1024 * q < m) {
                    mine[q] = entries[at + tid + 1024 * q];
                    atomicAdd(&count[mine[q].key >> CO_ROWS_LOG2 & mask], 1);
                }
            __syncthreads();
            int v[PER], sum = 0;
#pragma unroll
            for (int k = 0; k < PER; ++k) { v[k] = count[tid * PER + k]; sum += v[k]; }
            int incl = sum;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(incl, o, 64);
                if ((tid & 63) >= o) incl += y;
            }
            if ((tid & 63) == 63) wave_sum[tid >> 6] = incl;
            __syncthreads();
            int to = incl - sum;
            for (int w = 0; w < tid >> 6; ++w) to += wave_sum[w];
#pragma unroll
            for (int k = 0; k < PER; ++k) { count[tid * PER + k] = to; to += v[k]; }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < CO_PIECE / 1024; ++q)
                if (tid + 1024 * q < m) piece[atomicAdd(&count[mine[q].key >> CO_ROWS_LOG2 & mask], 1)] = mine[q];
            __syncthreads();
            for (int q = tid; q < m; q += 1024) entries[at + q] = piece[q];
            __syncthreads();
        }
}

// ---- the passes -----------------------------------------------------------------------------------------------------

// The part that a workgroup of column_dots takes.  The workgroups of a part read the same columns of w, and are on one L2 partition
// where there are parts for all of these (whole multiples then).  Fewer parts are dealt out over the whole chip: with each of them on
// a partition of its own the other partitions stood still (110 entries a row: 600000 rows over 2M columns, six parts then and now,
// 270 us and 185; 1.2M rows, three, 667 and 302; 2.2M rows over 20M, one then and three now, 6472 and 1039, by rows 4223).
struct ColumnPart { int block, part; };
__host__ __device__ inline ColumnPart column_part(int group, int blocks, int parts)
{
    if (parts < L2_PARTITIONS) return {group % blocks, group / blocks};
    const int round = group / L2_PARTITIONS;
    return {round % blocks, round / blocks * L2_PARTITIONS + group % L2_PARTITIONS};
}

// Grid: blocks * parts (column_part).  z[part * n_total + row]: the part's share of x_row . w.  Dynamic LDS: a double per row of a
// block.
// (100000 rows of a thousand entries over 20M columns: 250 us, with the rows' ends 296; reading the entries alone 160.  By rows, in
// slices of the columns that an L2 holds, 806 and 40: 26 entries of a row lie in a slice, which use under half of the lines they
// are on.  The next entries asked for before the gathers 260, two workgroups to a compute unit 248.)
template <typename WT>
__global__ __launch_bounds__(CO_THREADS) void column_dots(ColumnOrder C, int parts, const WT *__restrict__ w, double l1, double *z)
{
    extern __shared__ __align__(16) double co_z[];
    const int tid = threadIdx.x;
    const auto [block, part] = column_part((int)blockIdx.x, C.blocks, parts);
    const int64_t row0 = (int64_t)block << CO_ROWS_LOG2;
    const int rows = (int)min((int64_t)CO_ROWS, C.n_total - row0);
    for (int i = tid; i < rows; i += CO_THREADS) co_z[i] = 0.0;
    const long long *off = C.off + (int64_t)block * C.buckets;
    const long long e0 = off[0], all = off[C.buckets] - e0;
    const long long begin = e0 + all * part / parts, end = e0 + all * (part + 1) / parts;
    // the segment the part begins in: the last one that starts at or before it
    const int per_seg = 1 << (CO_SEG_LOG2 - C.bucket_log2), segs = (C.buckets + per_seg - 1) / per_seg;
    int seg = 0;
    for (int hi = segs - 1; seg < hi;) {
        const int mid = (seg + hi + 1) >> 1;
        if (off[mid * per_seg] <= begin) seg = mid; else hi = mid - 1;
    }
    __syncthreads();
    constexpr int AHEAD = 8, STEP = AHEAD * CO_THREADS;
    for (long long at = begin; at < end; ++seg) {
        const long long stop = min(end, off[min((seg + 1) * per_seg, C.buckets)]);
        const WT *ws = w + ((int64_t)seg << CO_SEG_LOG2);
        const long long whole = (stop - at) / STEP;
        const ColumnEntry *p = C.entries + at;
        for (long long i = 0; i < whole; ++i, p += STEP) {
            ColumnEntry e[AHEAD];
            WT x[AHEAD];
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) e[q] = p[tid + q * CO_THREADS];
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) x[q] = shared_at(ws, e[q].key >> CO_ROWS_LOG2, l1);
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) atomicAdd(&co_z[e[q].key & (CO_ROWS - 1)], (double)e[q].val * (double)x[q]);
        }
        const int rest = (int)(stop - at - whole * STEP);
        for (int i = tid; i < rest; i += 2 * CO_THREADS) {
            const ColumnEntry e0 = p[i], e1 = p[min(i + CO_THREADS, rest - 1)];
            const WT x0 = shared_at(ws, e0.key >> CO_ROWS_LOG2, l1), x1 = shared_at(ws, e1.key >> CO_ROWS_LOG2, l1);
            atomicAdd(&co_z[e0.key & (CO_ROWS - 1)], (double)e0.val * (double)x0);
            if (i + CO_THREADS < rest) atomicAdd(&co_z[e1.key & (CO_ROWS - 1)], (double)e1.val * (double)x1);
        }
        at = stop;
    }
    __syncthreads();
    double *out = z + (int64_t)part * C.n_total + row0;
    for (int i = tid; i < rows; i += CO_THREADS) out[i] = co_z[i];
}

// Grid: buckets.  w64 += inv_sigma * sum over the rows of coef[row] * x_row, and its mirror.  Dynamic LDS: a double per column of a
// bucket, then a float per row of a block.  The next block's coefficients and first entries are on their way while this block's
// are added.  (What it costs beside the matrix is the coefficients, which every bucket reads: 100000 rows of a thousand entries
// over 20M columns 341 us, with half as many columns to a bucket and rows to a block 682, half the rows alone 437; as many
// workgroups as compute units that take the buckets in turn, loads two blocks ahead, 368.)
__global__ __launch_bounds__(CO_THREADS) void column_merge(ColumnOrder C, const float *__restrict__ coef, double *w64, float *w32, int64_t d,
                                                           float inv_sigma, double l1)
{
    extern __shared__ __align__(16) double co_sum[];
    const int tid = threadIdx.x, columns = 1 << C.bucket_log2, bucket = (int)blockIdx.x;
    float *s_coef = reinterpret_cast<float *>(co_sum + columns);
    for (int i = tid; i < columns; i += CO_THREADS) co_sum[i] = 0.0;
    constexpr int AHEAD = 8, CQ = CO_ROWS / 4 / CO_THREADS;
    ColumnEntry e[AHEAD];
    float4_v cf[CQ];
    long long at = 0, stop = 0;
    auto request = [&](int block) __attribute__((always_inline)) {
        const long long *off = C.off + (int64_t)min(block, C.blocks - 1) * C.buckets + bucket;
        at = off[0];
        stop = block < C.blocks ? off[1] : at;
        const int64_t row0 = (int64_t)min(block, C.blocks - 1) << CO_ROWS_LOG2;
        // (the coefficients are followed by room up to a multiple of four)
#pragma unroll
        for (int q = 0; q < CQ; ++q) {
            const int64_t r = row0 + 4 * (tid + q * CO_THREADS);
            cf[q] = *(const CHICLE_GLOBAL float4_v *)(coef + (r < C.n_total ? r : row0));
        }
#pragma unroll
        for (int q = 0; q < AHEAD; ++q) {
            const long long i = at + tid + q * CO_THREADS;
            e[q] = ColumnEntry{0u, 0.f};
            if (i < stop) e[q] = C.entries[i];
        }
    };
    auto add = [&](const ColumnEntry &x) __attribute__((always_inline)) {
        atomicAdd(&co_sum[x.key >> CO_ROWS_LOG2 & (columns - 1)], (double)s_coef[x.key & (CO_ROWS - 1)] * (double)x.val);
    };
    request(0);
    for (int block = 0; block < C.blocks; ++block) {
#pragma unroll
        for (int q = 0; q < CQ; ++q) *reinterpret_cast<float4_v *>(s_coef + 4 * (tid + q * CO_THREADS)) = cf[q];
        ColumnEntry now[AHEAD];
#pragma unroll
        for (int q = 0; q < AHEAD; ++q) now[q] = e[q];
        const long long from = at, to = stop;
        __syncthreads();
        request(block + 1);
#pragma unroll
        for (int q = 0; q < AHEAD; ++q)
            if (from + tid + q * CO_THREADS < to) add(now[q]);
        for (long long i = from + tid + AHEAD * CO_THREADS; i < to; i += CO_THREADS) add(C.entries[i]);
        __syncthreads();
    }
    const int64_t c0 = (int64_t)bucket << C.bucket_log2;
    for (int i = tid; i < columns; i += CO_THREADS)
        if (c0 + i < d && co_sum[i] != 0.0) {
            const double x = w64[c0 + i] + co_sum[i] * (double)inv_sigma;
            w64[c0 + i] = x;
            w32[c0 + i] = (float)soft_threshold(x, l1);
        }
}

}  // namespace chicle
