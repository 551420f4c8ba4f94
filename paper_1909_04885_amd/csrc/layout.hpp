// Chunk-store layout kernels: column ids are stored as popularity ranks.
//
// When all chunks are in HBM the columns are renumbered once by how often they occur (most frequent
// column = id 0) and every row is re-sorted by the new ids.  Frequent columns then have small ids, so
// a solver can keep the frequently touched head of its private vector in LDS by a plain range test
// and the rows' frequent entries come first.  The shared vector and the private vectors live in the
// renumbered space; the read/write entry points translate to and from the caller's column ids.
#pragma once
#include <hip/hip_runtime.h>
#include "device_types.hpp"

namespace chicle {

// Words from host memory mapped into the device's address space.
__global__ __launch_bounds__(256) void copy_words(const int32_t *__restrict__ in, int64_t n, int32_t *out)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) out[i] = in[i];
}

// count[col] += 1 for every stored entry.  Grid: (blocks over entries, chunk).
__global__ __launch_bounds__(256) void count_columns(const ChunkDev *__restrict__ chunks, int *count)
{
    const ChunkDev &ch = chunks[blockIdx.y];
    for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < ch.nnz; p += (int64_t)gridDim.x * 256) atomicAdd(&count[ch.col[p]], 1);
}

// The same for every `stride`-th row of a chunk.  Grid: (blocks over rows, chunk).
__global__ __launch_bounds__(256) void count_columns_of_some(const ChunkDev *__restrict__ chunks, int stride, int *count)
{
    const ChunkDev &ch = chunks[blockIdx.y];
    for (int64_t r = (int64_t)blockIdx.x * stride; r < ch.n_rows; r += (int64_t)gridDim.x * stride)
        for (int p = ch.row_ptr[r] + threadIdx.x; p < ch.row_ptr[r + 1]; p += 256) atomicAdd(&count[ch.col[p]], 1);
}

// out[0] += sum of count (count - 1), out[1] += sum of count, over count[0 .. n).
__global__ __launch_bounds__(256) void sum_pairs(const int *__restrict__ count, int64_t n, double *out)
{
    double pairs = 0.0, all = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const double f = (double)count[i];
        pairs += f * (f - 1.0);
        all += f;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { pairs += __shfl_xor(pairs, o, 64); all += __shfl_xor(all, o, 64); }
    if ((threadIdx.x & 63) == 0 && all > 0.0) { atomicAdd(out, pairs); atomicAdd(out + 1, all); }
}

// col <- rank_of[col] and insertion sort of each row by the new ids (values move with their ids).
// One thread per row; rows are short where this is used.  Grid: (blocks over rows, chunk).
__global__ __launch_bounds__(256) void renumber_rows(const ChunkDev *__restrict__ chunks,
                                                     const int32_t *__restrict__ rank_of)
{
    const ChunkDev &ch = chunks[blockIdx.y];
    int32_t *col = const_cast<int32_t *>(ch.col);
    float *val = const_cast<float *>(ch.val);
    for (int r = blockIdx.x * 256 + threadIdx.x; r < ch.n_rows; r += gridDim.x * 256) {
        const int b = ch.row_ptr[r], e = ch.row_ptr[r + 1];
        for (int p = b; p < e; ++p) {
            const int c = rank_of[col[p]];
            const float v = val[p];
            int s = p;
            while (s > b && col[s - 1] > c) {
                col[s] = col[s - 1];
                val[s] = val[s - 1];
                --s;
            }
            col[s] = c;
            val[s] = v;
        }
    }
}

// ---- compact private vectors (sparse rows: a solver touches a small part of the columns) ----
// Per solver a bitmap of the columns its chunks contain and, per 32-column word, the number of set bits
// before it: column c of solver k lives at index pref[k][c >> 5] + popcount(bits[k][c >> 5] below bit c & 31)
// of that solver's compact vector.

// bits[owner[chunk]][c >> 5] |= 1 << (c & 31) for every entry.  Grid: (blocks over entries, chunk).
// multi (may be null): the same layout, a bit is set when a second entry of the solver's chunks holds the column
// (the columns inside a row are distinct, so that is another row).
// What bounds it is contention: with Zipf-distributed columns half of the entries fall into a few words, and an
// atomic (or even a read past the vector cache) per entry queues up at the one cache channel that holds them.  A
// workgroup therefore collects the columns below 32 * MARK_HEAD_WORDS in LDS, where a read shows most bits as
// already set, and adds that bitmap to the solver's once at the end; beyond them a plain read comes first (bits
// are only ever set: a stale read costs an atomic and nothing else).
// 500 000 rows of 40 entries, 32 solvers: 9.2 ms with an atomic per entry, 1.63 ms with only the read in front,
// 0.23 ms with the head in LDS.
constexpr int MARK_HEAD_WORDS = 1024;
__global__ __launch_bounds__(256) void mark_columns(const ChunkDev *__restrict__ chunks, const int32_t *__restrict__ owner,
                                                    unsigned *bits, int64_t words, unsigned *multi)
{
    __shared__ unsigned head[MARK_HEAD_WORDS], head_more[MARK_HEAD_WORDS];
    const ChunkDev &ch = chunks[blockIdx.y];
    unsigned *mine = bits + (int64_t)owner[blockIdx.y] * words;
    unsigned *more = multi ? multi + (int64_t)owner[blockIdx.y] * words : nullptr;
    for (int i = threadIdx.x; i < MARK_HEAD_WORDS; i += 256) head[i] = head_more[i] = 0u;
    __syncthreads();
    for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < ch.nnz; p += (int64_t)gridDim.x * 256) {
        const int c = ch.col[p], j = c >> 5;
        const unsigned bit = 1u << (c & 31);
        if (j < MARK_HEAD_WORDS) {
            unsigned old = head[j];
            if (!(old & bit)) old = atomicOr(&head[j], bit);
            if (more && (old & bit) && !(head_more[j] & bit)) atomicOr(&head_more[j], bit);
        } else {
            unsigned old = mine[j];
            if (!(old & bit)) old = atomicOr(mine + j, bit);
            if (more && (old & bit) && !(more[j] & bit)) atomicOr(more + j, bit);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < MARK_HEAD_WORDS; i += 256) {
        const unsigned h = head[i];
        if (h == 0u) continue;                             // (words past the end are never set)
        unsigned old = mine[i];
        if (h & ~old) old = atomicOr(mine + i, h);
        // a column in this workgroup's bitmap and already in the solver's is held by another row as well
        const unsigned m = more ? head_more[i] | (h & old) : 0u;
        if (m) atomicOr(more + i, m);
    }
}

// Columns [0, n) are present in every solver's vector: sets their bits.  One workgroup per solver.
__global__ __launch_bounds__(256) void force_columns(unsigned *bits, int64_t words, int n)
{
    unsigned *mine = bits + (int64_t)blockIdx.x * words;
    for (int j = threadIdx.x; j * 32 < n; j += 256) {
        const int left = n - j * 32;
        mine[j] |= left >= 32 ? 0xffffffffu : ((1u << left) - 1u);
    }
}

// pref[k][j] = number of set bits in bits[k][0 .. j); count[k] = all of them.  One workgroup of 1024 per solver.
__global__ __launch_bounds__(1024) void prefix_columns(const unsigned *__restrict__ bits, int32_t *pref, int64_t words,
                                                       int32_t *count)
{
    __shared__ int wave_sum[16];
    __shared__ int carry;
    const unsigned *b = bits + (int64_t)blockIdx.x * words;
    int32_t *p = pref + (int64_t)blockIdx.x * words;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int64_t base = 0; base < words; base += 1024) {
        const int64_t j = base + threadIdx.x;
        const int v = j < words ? __popc(b[j]) : 0;
        int incl = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(incl, o, 64);
            if ((threadIdx.x & 63) >= o) incl += y;
        }
        if ((threadIdx.x & 63) == 63) wave_sum[threadIdx.x >> 6] = incl;
        __syncthreads();
        int off = carry;
        for (int w = 0; w < (int)(threadIdx.x >> 6); ++w) off += wave_sum[w];
        if (j < words) p[j] = off + incl - v;
        __syncthreads();
        if (threadIdx.x == 1023) carry = off + incl;
        __syncthreads();
    }
    if (threadIdx.x == 0) count[blockIdx.x] = carry;
}

// The compact index of every entry, written behind the chunk's column ids.  Grid: (blocks over entries, chunk).
// multi (may be null): see mark_columns; an entry whose column no other row of the solver holds gets the sign
// bit (UNIQUE_COLUMN in mem.hpp).
__global__ __launch_bounds__(256) void compact_indices(const ChunkDev *__restrict__ chunks, const int32_t *__restrict__ owner,
                                                       const unsigned *__restrict__ bits, const int32_t *__restrict__ pref,
                                                       int64_t words, const unsigned *__restrict__ multi)
{
    const ChunkDev &ch = chunks[blockIdx.y];
    const int64_t k = owner[blockIdx.y];
    const unsigned *b = bits + k * words;
    const int32_t *pf = pref + k * words;
    int32_t *out = const_cast<int32_t *>(chunk_compact_ids(ch));
    const int64_t n = padded_entries(ch.nnz);
    for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < n; p += (int64_t)gridDim.x * 256) {
        int idx = 0;                                   // the slack behind the last row points at index 0
        if (p < ch.nnz) {
            const int c = ch.col[p];
            idx = pf[c >> 5] + __popc(b[c >> 5] & ((1u << (c & 31)) - 1u));
            if (multi && !(multi[k * words + (c >> 5)] & (1u << (c & 31)))) idx |= (int)0x80000000;
        }
        out[p] = idx;
    }
}

// *out = the largest number of entries any row has at compact indices >= n (the columns the batched solver
// does not keep on chip).  Compact indices ascend inside a row, so a row's count is found by bisection (counting
// entry by entry, one row per thread, read every line of the rows uncoalesced: 0.33 ms for 20 million entries
// against 0.12 ms).  Grid: (blocks over rows, chunk), one thread per row; *out starts at 0.
__global__ __launch_bounds__(256) void max_entries_beyond(const ChunkDev *__restrict__ chunks, int n, int *out)
{
    const ChunkDev &ch = chunks[blockIdx.y];
    const int32_t *cid = chunk_compact_ids(ch);
    int most = 0;
    for (int r = blockIdx.x * 256 + threadIdx.x; r < ch.n_rows; r += gridDim.x * 256) {
        const int e = ch.row_ptr[r + 1];
        int lo = ch.row_ptr[r], hi = e;                    // first entry with an index >= n
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (cid[mid] < n) lo = mid + 1; else hi = mid;
        }
        most = max(most, e - lo);
    }
    if (most > 0) atomicMax(out, most);
}

// Entries [first, first + n) of a row-major matrix with d columns, given in `in`, into rows of ld floats that end in zeros.
__global__ __launch_bounds__(256) void pad_rows(const float *__restrict__ in, int64_t first, int64_t n, int d, int ld, float *out)
{
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) {
        const int64_t r = (first + i) / d;
        const int k = (int)(first + i - r * d);
        float *row = out + r * ld;
        row[k] = in[i];
        if (k == d - 1)
            for (int z = d; z < ld; ++z) row[z] = 0.f;
    }
}

// out[col_of[r]] = in[r] * scale (internal order -> caller's column ids).
template <typename T>
__global__ __launch_bounds__(256) void to_caller_order(const T *__restrict__ in,
                                                       const int32_t *__restrict__ col_of, int64_t d,
                                                       float scale, float *out)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < d; r += stride)
        out[col_of ? col_of[r] : r] = (float)in[r] * scale;
}

// The same into host memory mapped into the device's address space, and the kernels' error flag beside it.
__global__ __launch_bounds__(256) void to_host_in_caller_order(const float *__restrict__ in, const int32_t *__restrict__ rank_of, int64_t d,
                                                               float scale, float *out, const int *err, int *flag)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    if (blockIdx.x == 0 && threadIdx.x == 0) *flag = *err;
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < d; c += stride) out[c] = in[rank_of ? rank_of[c] : c] * scale;
}

// out64[r] = out32[r] = in[col_of[r]] (caller's column ids -> internal order).
__global__ __launch_bounds__(256) void from_caller_order(const float *__restrict__ in,
                                                         const int32_t *__restrict__ col_of, int64_t d,
                                                         double *out64, float *out32)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < d; r += stride) {
        const float x = in[col_of ? col_of[r] : r];
        out64[r] = (double)x;
        out32[r] = x;
    }
}

}  // namespace chicle
