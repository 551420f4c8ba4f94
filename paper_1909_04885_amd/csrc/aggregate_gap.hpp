// Trainer-side kernels: merge of the solvers' updates (paper Section 4.1: "merge updates, broadcast
// model") and the duality gap that solvers report as convergence metric (Section 4.1, Section 5.1).
#pragma once
#include <hip/hip_runtime.h>
#include "device_types.hpp"
#include "mem.hpp"
#include "sdca_rowwise.hpp"

namespace chicle {

// Elastic net (paper Section 2.2: generalised linear models): with the regulariser lambda (|w|^2 / 2 +
// l1 |w|_1) the solvers' updates add up in the dual image v, which is what the double-precision vector
// holds, and the shared vector is w_j = sign(v_j) max(|v_j| - l1, 0).  l1 = 0: w = v.
__device__ __forceinline__ double soft_threshold(double v, double l1)
{
    const double a = fabs(v) - l1;
    return a > 0.0 ? copysign(a, v) : 0.0;
}
// The shared vector as the gap kernels read it: the float mirror holds w itself, the double vector holds v.
__device__ __forceinline__ float shared_at(const float *w, int64_t c, double) { return w[c]; }
__device__ __forceinline__ double shared_at(const double *v, int64_t c, double l1) { return soft_threshold(v[c], l1); }

// u_k <- 0 for k < K (a solver fetching the model starts with no update of its own).
__global__ __launch_bounds__(256) void clear_private(float *u_all, int64_t ld_v, int64_t d4, int K)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < d4; j += stride)
        for (int k = 0; k < K; ++k) reinterpret_cast<float4 *>(u_all + (int64_t)k * ld_v)[j] = z;
}

// w <- w + sum_k Delta w_k with Delta w_k = u_k / sigma, then u_k <- 0 for all k (merge, broadcast).
// The shared vector is kept in double (w64) with a float mirror (w32) for the kernels that gather it.
// One pass: reads K + 1 vectors, writes K + 2 vectors, four columns per thread (ld_v and the
// buffers are 16-byte aligned; d is handled up to its padded length, the padding holds zeros).
__global__ __launch_bounds__(256) void aggregate_broadcast(double *w64, float *w32, float *u_all,
                                                           int64_t ld_v, int64_t d4, int K, float inv_sigma, double l1)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    double2 *wd = reinterpret_cast<double2 *>(w64);
    float4 *wf = reinterpret_cast<float4 *>(w32);
    const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < d4; j += stride) {
        float4 acc = z;
        for (int k = 0; k < K; ++k) {
            float4 *uk = reinterpret_cast<float4 *>(u_all + (int64_t)k * ld_v) + j;
            const float4 x = *uk;
            acc.x += x.x; acc.y += x.y; acc.z += x.z; acc.w += x.w;
            *uk = z;
        }
        double2 lo = wd[2 * j], hi = wd[2 * j + 1];
        lo.x += (double)(acc.x * inv_sigma); lo.y += (double)(acc.y * inv_sigma);
        hi.x += (double)(acc.z * inv_sigma); hi.y += (double)(acc.w * inv_sigma);
        wd[2 * j] = lo; wd[2 * j + 1] = hi;
        wf[j] = make_float4((float)soft_threshold(lo.x, l1), (float)soft_threshold(lo.y, l1),
                            (float)soft_threshold(hi.x, l1), (float)soft_threshold(hi.y, l1));
    }
}

// out <- Delta w_solver, or sum_k Delta w_k when solver < 0 (read-back helper).
__global__ __launch_bounds__(256) void delta_w_out(const float *u_all, int64_t ld_v, int64_t d, int K,
                                                   int solver, float inv_sigma, float *out)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < d; j += stride) {
        float acc = 0.f;
        if (solver >= 0) acc = u_all[(int64_t)solver * ld_v + j];
        else for (int k = 0; k < K; ++k) acc += u_all[(int64_t)k * ld_v + j];
        out[j] = acc * inv_sigma;
    }
}

// The merge where private vectors are stored compactly (see layout.hpp).  A workgroup takes 64 consecutive
// words of 32 columns (2048 columns) and walks the solvers: a solver's entries for these columns are one
// contiguous run of its compact vector, which the workgroup reads (and clears) with coalesced accesses into
// LDS; each thread then picks the entries of its own quarter of a word out of the run, in order, by the word's bits.  (256 words
// to a workgroup, a thread each, left small jobs a few workgroups with long loops: six solvers over 20k columns 18.5 us, and 5
// for the mirror, 7.8 now with it.)  The sums are in double: how many solvers a slice has depends on the number of columns, and
// so would the roundings of a sum in float.
// u_off[k]: where solver k's compact vector starts in u.  Reads and clears only what the solvers touched.
// Where there are few words (few workgroups), the solvers are divided over gridDim.y slices as well; the
// slices then add their sums into the double-precision vector with atomic adds, and the one that is done last refreshes the
// float mirror (tickets[blockIdx.x]: zero, and left so; a pass of its own over the mirror took 5 us, which these 2048 columns
// do not).
constexpr int AGG_THREADS = 256, AGG_WORDS = 64;     // threads and words per workgroup
constexpr int AGG_THIN_WORDS = 256;                  // ... of aggregate_compact_thin
static_assert(AGG_THIN_WORDS == AGG_THREADS, "a thread per word");
__device__ __forceinline__ void mirror_by_last_slice(const double *w64, float *w32, int64_t d, double l1, unsigned *tickets)
{
    __shared__ int last;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // this thread's adds are performed
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(tickets + blockIdx.x, 1u) + 1u == gridDim.y;
    __syncthreads();
    if (!last) return;
    if (threadIdx.x == 0) __hip_atomic_store(tickets + blockIdx.x, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int64_t c0 = (int64_t)blockIdx.x * AGG_WORDS * 32 + threadIdx.x;
    double x[AGG_WORDS * 32 / AGG_THREADS];          // one trip to memory
#pragma unroll
    for (int q = 0; q < AGG_WORDS * 32 / AGG_THREADS; ++q) {
        const int64_t c = c0 + q * AGG_THREADS;
        x[q] = c < d ? __hip_atomic_load(w64 + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0;
    }
#pragma unroll
    for (int q = 0; q < AGG_WORDS * 32 / AGG_THREADS; ++q) {
        const int64_t c = c0 + q * AGG_THREADS;
        if (c < d) w32[c] = (float)soft_threshold(x[q], l1);
    }
}

__global__ __launch_bounds__(AGG_THREADS) void aggregate_compact(double *w64, float *w32, float *u, const int64_t *__restrict__ u_off,
                                                                 const unsigned *__restrict__ bits, const int32_t *__restrict__ pref,
                                                                 int64_t words, int64_t d, int K, float inv_sigma, double l1, unsigned *tickets)
{
    constexpr int PER = 8, PARTS = 32 / PER;         // columns of a thread, threads of a word
    static_assert(AGG_WORDS * PARTS == AGG_THREADS, "a thread per quarter of a word");
    __shared__ __align__(16) double sums[AGG_WORDS * 32];
    float *run = reinterpret_cast<float *>(sums);    // a run is at most all columns of the workgroup; the sums take its place
    __shared__ unsigned touched[AGG_WORDS];
    __shared__ int run_begin, run_end;
    const int tid = threadIdx.x, word = tid / PARTS, part = tid % PARTS;
    const int64_t j = (int64_t)blockIdx.x * AGG_WORDS + word;
    const bool live = j < words;
    const int last = (int)min((int64_t)AGG_WORDS, words - (int64_t)blockIdx.x * AGG_WORDS) - 1;   // last live word
    double acc[PER];
#pragma unroll
    for (int b = 0; b < PER; ++b) acc[b] = 0.0;
    unsigned any = 0;
    // (the next solver's word and prefix are requested before this solver's run is waited for)
    const int per = (K + (int)gridDim.y - 1) / (int)gridDim.y;
    const int k0 = (int)blockIdx.y * per, k1 = min(K, k0 + per);
    unsigned m_next = live && k0 < k1 ? bits[(int64_t)k0 * words + j] : 0u;
    int pf_next = live && k0 < k1 ? pref[(int64_t)k0 * words + j] : 0;
    for (int k = k0; k < k1; ++k) {
        const unsigned m = m_next;
        const int pf = pf_next;
        if (k + 1 < k1 && live) { m_next = bits[(int64_t)(k + 1) * words + j]; pf_next = pref[(int64_t)(k + 1) * words + j]; }
        if (tid == 0) run_begin = pf;
        if (word == last) run_end = pf + __popc(m);
        __syncthreads();
        const int begin = run_begin, len = run_end - begin;
        float *uk = u + u_off[k] + begin;
        float x[AGG_WORDS * 32 / AGG_THREADS];       // all loads in flight
#pragma unroll
        for (int q = 0; q < AGG_WORDS * 32 / AGG_THREADS; ++q) x[q] = tid + q * AGG_THREADS < len ? uk[tid + q * AGG_THREADS] : 0.f;
#pragma unroll
        for (int q = 0; q < AGG_WORDS * 32 / AGG_THREADS; ++q)
            if (tid + q * AGG_THREADS < len) { run[tid + q * AGG_THREADS] = x[q]; uk[tid + q * AGG_THREADS] = 0.f; }
        __syncthreads();
        any |= m;
        int r = pf - begin + __popc(m & ((1u << (PER * part)) - 1u));
#pragma unroll
        for (int b = 0; b < PER; ++b)
            if (m & (1u << (PER * part + b))) acc[b] += (double)run[r++];
        __syncthreads();                             // the run is overwritten by the next solver's
    }
    // the sums go through LDS so that the shared vector is updated with coalesced accesses
    if (part == 0) touched[word] = any;
#pragma unroll
    for (int b = 0; b < PER; b += 2) *reinterpret_cast<double2 *>(sums + tid * PER + b) = make_double2(acc[b], acc[b + 1]);
    __syncthreads();
    const int64_t c0 = (int64_t)blockIdx.x * AGG_WORDS * 32;
#pragma unroll
    for (int q = 0; q < AGG_WORDS * 32 / AGG_THREADS; ++q) {
        const int i = tid + q * AGG_THREADS;
        const int64_t c = c0 + i;
        if (c < d && (touched[i >> 5] & (1u << (i & 31)))) {
            const double add = sums[i] * (double)inv_sigma;
            if (gridDim.y == 1) {
                const double x = w64[c] + add;
                w64[c] = x;
                w32[c] = (float)soft_threshold(x, l1);
            } else {
                atomicAdd(&w64[c], add);
            }
        }
    }
    if (gridDim.y > 1) mirror_by_last_slice(w64, w32, d, l1, tickets);
}

// The same merge for thinly occupied vectors (long rows over many columns: a solver holds a few of every
// hundred columns).  A solver's run for a workgroup's 8192 columns is then a few hundred floats, and staging
// it through LDS costs three workgroup barriers and a dependent trip to memory per solver.  Here every thread
// picks the entries of its own word straight from memory - neighbouring threads read neighbouring short
// pieces of the run, so the lines are shared inside the wavefront - and keeps its 32 sums in LDS (row tid of
// a padded array, touched by that thread alone until the end), with no barrier inside the walk over the
// solvers.  What it waits for are trips to memory, so it takes THIN_SOLVERS solvers at a time, the first THIN_FIRST entries of all
// of them in flight together and the next ones' words and prefixes before that: 64 solvers, 20M columns, 96M entries 537 us
// one solver at a time, 434 now (1.5 GB).  Further entries of a word, which only popular columns have, follow THIN_FIRST at a
// time (one at a time: 96 solvers over 127k columns 90 us, 82 so).  The mirror is a pass of its own here: 8192 columns are
// too many for the one workgroup that is done last (50 solvers over 252k columns 40 us with it, 29.5 so; 42 over 168k 29 and
// 19.5).
constexpr int THIN_SOLVERS = 4, THIN_FIRST = 8;
__global__ __launch_bounds__(AGG_THIN_WORDS) void aggregate_compact_thin(double *w64, float *w32, float *u, const int64_t *__restrict__ u_off,
                                                                    const unsigned *__restrict__ bits, const int32_t *__restrict__ pref,
                                                                    int64_t words, int64_t d, int K, float inv_sigma, double l1)
{
    __shared__ float sums[AGG_THIN_WORDS * 33];
    __shared__ unsigned touched[AGG_THIN_WORDS];
    const int tid = threadIdx.x;
    const int64_t j = (int64_t)blockIdx.x * AGG_THIN_WORDS + tid;
    const bool live = j < words;
    float *mine = sums + tid * 33;
#pragma unroll
    for (int b = 0; b < 32; ++b) mine[b] = 0.f;
    unsigned any = 0;
    const int per = (K + (int)gridDim.y - 1) / (int)gridDim.y;              // slices of solvers, as above
    const int k0 = (int)blockIdx.y * per, k1 = min(K, k0 + per);
    unsigned m_next[THIN_SOLVERS];
    int pf_next[THIN_SOLVERS];
    auto request = [&](int k) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < THIN_SOLVERS; ++s) {
            const bool has = live && k + s < k1;
            m_next[s] = has ? bits[(int64_t)(k + s) * words + j] : 0u;
            pf_next[s] = has ? pref[(int64_t)(k + s) * words + j] : 0;
        }
    };
    request(k0);
    for (int k = k0; k < k1; k += THIN_SOLVERS) {
        unsigned m[THIN_SOLVERS];
        float *uk[THIN_SOLVERS];
        float v[THIN_SOLVERS][THIN_FIRST];
#pragma unroll
        for (int s = 0; s < THIN_SOLVERS; ++s) {
            m[s] = m_next[s];
            uk[s] = u + u_off[min(k + s, k1 - 1)] + pf_next[s];
        }
        request(k + THIN_SOLVERS);
#pragma unroll
        for (int s = 0; s < THIN_SOLVERS; ++s)
#pragma unroll
            for (int q = 0; q < THIN_FIRST; ++q) v[s][q] = q < __popc(m[s]) ? uk[s][q] : 0.f;
#pragma unroll
        for (int s = 0; s < THIN_SOLVERS; ++s) {
            unsigned r = m[s];
            any |= r;
#pragma unroll
            for (int q = 0; q < THIN_FIRST; ++q)
                if (r) {
                    mine[__ffs(r) - 1] += v[s][q];
                    uk[s][q] = 0.f;
                    r &= r - 1;
                }
            for (float *rest = uk[s] + THIN_FIRST; r; rest += THIN_FIRST) {      // (words of popular columns)
                float x[THIN_FIRST];
#pragma unroll
                for (int q = 0; q < THIN_FIRST; ++q) x[q] = q < __popc(r) ? rest[q] : 0.f;
#pragma unroll
                for (int q = 0; q < THIN_FIRST; ++q)
                    if (r) {
                        mine[__ffs(r) - 1] += x[q];
                        rest[q] = 0.f;
                        r &= r - 1;
                    }
            }
        }
    }
    touched[tid] = any;
    __syncthreads();
    const int64_t c0 = (int64_t)blockIdx.x * AGG_THIN_WORDS * 32;
    for (int i = tid; i < AGG_THIN_WORDS * 32; i += AGG_THIN_WORDS) {
        const int64_t c = c0 + i;
        if (c < d && (touched[i >> 5] & (1u << (i & 31)))) {
            const double add = (double)(sums[(i >> 5) * 33 + (i & 31)] * inv_sigma);
            if (gridDim.y == 1) {
                const double x = w64[c] + add;
                w64[c] = x;
                w32[c] = (float)soft_threshold(x, l1);
            } else {
                atomicAdd(&w64[c], add);
            }
        }
    }
}

__global__ __launch_bounds__(256) void mirror_from_double(const double *__restrict__ w64, float *w32, int64_t d, double l1)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < d; c += stride) w32[c] = (float)soft_threshold(w64[c], l1);
}

// Read-back helper for compact private vectors: out <- Delta w_solver, or sum_k Delta w_k when solver < 0.
__global__ __launch_bounds__(256) void delta_w_out_compact(const float *u, const int64_t *__restrict__ u_off,
                                                           const unsigned *__restrict__ bits, const int32_t *__restrict__ pref,
                                                           int64_t words, int64_t d, int K, int solver, float inv_sigma,
                                                           float *out)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < d; c += stride) {
        float acc = 0.f;
        const int64_t j = c >> 5;
        const unsigned bit = 1u << (c & 31);
        for (int k = solver >= 0 ? solver : 0; k < (solver >= 0 ? solver + 1 : K); ++k) {
            const unsigned m = bits[(int64_t)k * words + j];
            if (m & bit) acc += u[u_off[k] + pref[(int64_t)k * words + j] + __popc(m & (bit - 1u))];
        }
        out[c] = acc * inv_sigma;
    }
}

__device__ __forceinline__ double wave_sum_d(double x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

// What the last kernel of the gap does beside its rows.  Its grid has one dimension, whose limit no number of chunks comes
// near: per_chunk workgroups for every chunk, one chunk after the other, then n_w that sum |w|^2 and |w|_1.  Every workgroup
// leaves its two partial sums, and the one that leaves them last adds all of them up in a fixed order: out[0] = sum loss,
// out[1] = sum conj, out[2] = |w|^2, out[3] = the kernels' error flag, out[4] = |w|_1, and when these are there the number of the
// gap, seq, in out[5].  out may be host memory mapped into the device's address space.  (Kernels of their own for the norms and for the end: 500000 x 28 in all 34 us, 17.9 now; 4096 x 256
// 16 and 6.4; sparse rows, 30000 x 20k, 24 and 18.8.)  tickets: nullptr where only the rows' residuals are wanted (n_w is zero
// then); else zero, and left so.  Adds to one address take 13 ns each, so workgroups are counted in GAP_GROUPS groups, and the
// groups that are complete at tickets[GAP_GROUPS * TICKET_LINE].
constexpr int GAP_GROUPS = 32, TICKET_LINE = 32;     // (counters 128 bytes apart)
constexpr int GAP_TICKETS = (GAP_GROUPS + 1) * TICKET_LINE;
struct GapEnd {
    unsigned *tickets;
    const double *v;
    int64_t d;
    double *part_wsq, *part_wabs;
    int n_w, n_chunks, per_chunk;
    const int *err;
    double *out;
    unsigned long long seq;
};
// A row workgroup's chunk (n_chunks and more: a workgroup for the norms), and which of the chunk's workgroups it is.
__device__ __forceinline__ int gap_chunk(const GapEnd &E) { return (int)(blockIdx.x / (unsigned)E.per_chunk); }
__device__ __forceinline__ int gap_slot(const GapEnd &E) { return (int)(blockIdx.x % (unsigned)E.per_chunk); }
// Partial sums go past the caches of the compute units and of their group, so that the last workgroup finds them.
__device__ __forceinline__ void st_part(double *p, double x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ double ld_part(const double *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Workgroup sums of M doubles, in all threads; N: threads.
template <int N, int M>
__device__ __forceinline__ void block_sum(double (&v)[M])
{
    __shared__ double r[M][N / 64];
#pragma unroll
    for (int k = 0; k < M; ++k) v[k] = wave_sum_d(v[k]);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int k = 0; k < M; ++k) r[k][threadIdx.x >> 6] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < M; ++k) {
        v[k] = 0.0;
#pragma unroll
        for (int i = 0; i < N / 64; ++i) v[k] += r[k][i];
    }
}

// A thread's share of the sums of two partial arrays, eight loads of each in flight.
template <int N>
__device__ __forceinline__ void add_parts(const double *pa, const double *pb, int n, double &a, double &b)
{
    for (int i = threadIdx.x; i < n; i += 8 * N) {
        double x[8], y[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            x[q] = i + q * N < n ? ld_part(pa + i + q * N) : 0.0;
            y[q] = i + q * N < n ? ld_part(pb + i + q * N) : 0.0;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) { a += x[q]; b += y[q]; }
    }
}

// The end of a workgroup of a row pass: its sums, and those of all if it is the last.
template <int N>
__device__ __forceinline__ void gap_block_end(double a, double b, double *out_a, double *out_b, double *part_loss, double *part_conj, const GapEnd &E)
{
    __shared__ int last;
    double own[2] = {a, b};
    block_sum<N>(own);
    if (threadIdx.x == 0) {
        st_part(out_a, own[0]);
        st_part(out_b, own[1]);
        if (E.tickets) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            const unsigned all = gridDim.x, group = blockIdx.x % GAP_GROUPS;
            const unsigned members = (all - group + GAP_GROUPS - 1) / GAP_GROUPS, groups = min(all, (unsigned)GAP_GROUPS);
            unsigned *mine = E.tickets + group * TICKET_LINE, *root = E.tickets + GAP_GROUPS * TICKET_LINE;
            last = 0;
            if (atomicAdd(mine, 1u) + 1u == members) {
                __hip_atomic_store(mine, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (atomicAdd(root, 1u) + 1u == groups) {
                    __hip_atomic_store(root, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    last = 1;
                }
            }
        }
    }
    if (!E.tickets) return;
    __syncthreads();
    if (!last) return;
    double sums[4] = {0.0, 0.0, 0.0, 0.0};           // loss, conj, |w|^2, |w|_1
    add_parts<N>(E.part_wsq, E.part_wabs, E.n_w, sums[2], sums[3]);
    add_parts<N>(part_loss, part_conj, (int)gridDim.x - E.n_w, sums[0], sums[1]);
    block_sum<N>(sums);
    if (threadIdx.x == 0) {
        E.out[0] = sums[0];
        E.out[1] = sums[1];
        E.out[2] = sums[2];
        E.out[3] = (double)*E.err;
        E.out[4] = sums[3];
        __hip_atomic_store(reinterpret_cast<unsigned long long *>(E.out + 5), E.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// |w|^2 and |w|_1 partials in double (w = the soft-thresholded image of the double vector).
template <int N>
__device__ __forceinline__ void gap_w_block(double l1, double *part_loss, double *part_conj, const GapEnd &E)
{
    const int part = (int)blockIdx.x - ((int)gridDim.x - E.n_w);
    double s = 0.0, t = 0.0;
    const int64_t stride = (int64_t)E.n_w * N;
    for (int64_t j = (int64_t)part * N + threadIdx.x; j < E.d; j += 4 * stride) {
        double x[4];                                 // four loads in flight per thread
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = j + q * stride < E.d ? E.v[j + q * stride] : 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double y = soft_threshold(x[q], l1);
            s += y * y;
            t += fabs(y);
        }
    }
    gap_block_end<N>(s, t, E.part_wsq + part, E.part_wabs + part, part_loss, part_conj, E);
}

// Per-row loss and conjugate terms of the gap; also leaves the residual rw of every row in the chunk
// for the next local pass (hinge: 1 - y z, squared: y - z with z = x_i . w).  WT is the type the dot
// product is gathered and accumulated in: double for the squared loss, whose steps cancel y - z - alpha
// down to the size of the update near convergence; float for hinge.
// LPR lanes cooperate on one row (LPR divides 64).  Each workgroup writes one partial (loss sum,
// conjugate sum) in double.
//   hinge   : loss = max(0, 1 - y z),   conj = loss^*(-a) = -a
//   squared : loss = (z - y)^2 / 2,     conj = a^2/2 - a y
//   logistic: loss = log(1 + exp(-y z)), conj = a log a + (1 - a) log(1 - a); rw = -y z
template <int LOSS, typename WT>
__device__ __forceinline__ void gap_row_terms(RowState *st, WT z, double &s_loss, double &s_conj)
{
    const float y = st->y, a = st->alpha;
    if (LOSS == 0) {
        const WT rw = (WT)1 - (WT)y * z;
        st->rw = (float)rw;
        s_loss += (double)(rw > (WT)0 ? rw : (WT)0);
        s_conj += (double)(-a);
    } else if (LOSS == 2) {
        const double m = -(double)y * (double)z;
        st->rw = (float)m;
        s_loss += fmax(m, 0.0) + log1p(exp(-fabs(m)));
        const double ad = (double)a, bd = 1.0 - (double)a;
        s_conj += (ad > 0.0 ? ad * log(ad) : 0.0) + (bd > 0.0 ? bd * log(bd) : 0.0);
    } else {
        const WT rw = (WT)y - z;
        st->rw = (float)rw;
        s_loss += 0.5 * (double)rw * (double)rw;
        s_conj += 0.5 * (double)a * (double)a - (double)a * (double)y;
    }
}

// The rows whose dot products a group of lanes has: a lane each, so that their terms (with the logistic loss an exponential and three
// logarithms in double) are formed side by side and their state is one trip to memory, not row by row in one lane of the group.
// (300000 rows of 40 entries, logistic loss: 105 us with the rows one after the other, 64 so; hinge loss, 2M rows, 242 and
// 228; 20011 x 1001, logistic, 34.5 and 25.9; 500000 x 28, squared, 19.0 and 17.5.)
template <typename WT>
struct KeptRow {
    WT z = 0;
    int row = -1;
    __device__ __forceinline__ void keep(bool here, int r, WT v) { if (here) { row = r; z = v; } }
    template <int LOSS>
    __device__ __forceinline__ void terms(RowState *st, double &s_loss, double &s_conj)
    {
        if (row >= 0) gap_row_terms<LOSS, WT>(st + row, z, s_loss, s_conj);
        row = -1;
    }
};

// Grid: see GapEnd.  Every group of LPR lanes walks rows of its chunk with a fixed stride and keeps two rows in flight.
// Partial sums are indexed by the workgroup.  ZT: what dot products are summed in.
template <int LOSS, int LPR, typename WT, typename ZT = WT>
__global__ __launch_bounds__(256) void gap_rows_csr(const ChunkDev *__restrict__ chunks,
                                                    const WT *__restrict__ w, double l1,
                                                    double *part_loss, double *part_conj, GapEnd E)
{
    if (gap_chunk(E) >= E.n_chunks) return gap_w_block<256>(l1, part_loss, part_conj, E);
    constexpr int GROUPS = 256 / LPR;
    const int sub = threadIdx.x % LPR;
    const int grp = threadIdx.x / LPR;
    const ChunkDev &ch = chunks[gap_chunk(E)];
    const int n_rows = ch.n_rows;
    const int32_t *__restrict__ rp = ch.row_ptr;
    const int32_t *__restrict__ col = ch.col;
    const float *__restrict__ val = ch.val;
    const int stride = E.per_chunk * GROUPS;
    double s_loss = 0.0, s_conj = 0.0;
    KeptRow<ZT> kept;
    int at = 0;                                  // the lane of the group that keeps the next row
    for (int r0 = gap_slot(E) * GROUPS + grp; r0 < n_rows; r0 += 2 * stride) {
        const int r1 = r0 + stride;
        const bool two = r1 < n_rows;
        const int b0 = rp[r0], e0 = rp[r0 + 1];
        const int b1 = two ? rp[r1] : 0, e1 = two ? rp[r1 + 1] : 0;
        ZT z0 = 0, z1 = 0;
        int p0 = b0 + sub, p1 = b1 + sub;
        while (p0 < e0 || p1 < e1) {           // both rows advance together: their loads overlap
            int c0 = 0, c1 = 0;
            float v0 = 0.f, v1 = 0.f;
            if (p0 < e0) { c0 = col[p0]; v0 = val[p0]; }
            if (p1 < e1) { c1 = col[p1]; v1 = val[p1]; }
            z0 += (ZT)v0 * (ZT)shared_at(w, c0, l1);
            z1 += (ZT)v1 * (ZT)shared_at(w, c1, l1);
            p0 += LPR; p1 += LPR;
        }
#pragma unroll
        for (int o = LPR / 2; o > 0; o >>= 1) { z0 += __shfl_xor(z0, o, 64); z1 += __shfl_xor(z1, o, 64); }
        kept.keep(sub == at, r0, z0);
        kept.keep(two && sub == at + 1, r1, z1);
        at += 2;
        if (at == LPR) {
            kept.template terms<LOSS>(ch.st, s_loss, s_conj);
            at = 0;
        }
    }
    kept.template terms<LOSS>(ch.st, s_loss, s_conj);
    gap_block_end<256>(s_loss, s_conj, part_loss + blockIdx.x, part_conj + blockIdx.x, part_loss, part_conj, E);
}

// The end of the row pass where the rows' dot products come in parts (column_dots).  Grid: see GapEnd; G threads per row, each with
// every G-th part, a wavefront's rows side by side.  Partial sums by workgroup, as above.
template <int LOSS, int G>
__global__ __launch_bounds__(256) void gap_rows_from_z(const ChunkDev *__restrict__ chunks, const double *__restrict__ z, int parts, int64_t n_total,
                                                       double l1, double *part_loss, double *part_conj, GapEnd E)
{
    if (gap_chunk(E) >= E.n_chunks) return gap_w_block<256>(l1, part_loss, part_conj, E);
    constexpr int ROWS = 256 / G;
    __shared__ double s_z[G][ROWS + 1];
    const ChunkDev &ch = chunks[gap_chunk(E)];
    const int t = threadIdx.x % ROWS, g = threadIdx.x / ROWS;
    double s_loss = 0.0, s_conj = 0.0;
    for (int r0 = gap_slot(E) * ROWS; r0 < ch.n_rows; r0 += E.per_chunk * ROWS) {
        const int r = r0 + t;
        const double *mine = z + (int64_t)ch.row_base + min(r, ch.n_rows - 1);
        double zi = 0.0;
        for (int k = g; k < parts; k += 8 * G) {     // (eight loads in flight)
            double x[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) x[q] = k + q * G < parts ? mine[(int64_t)(k + q * G) * n_total] : 0.0;
#pragma unroll
            for (int q = 0; q < 8; ++q) zi += x[q];
        }
        if (G > 1) {
            s_z[g][t] = zi;
            __syncthreads();
            if (g == 0)
#pragma unroll
                for (int q = 1; q < G; ++q) zi += s_z[q][t];
            __syncthreads();
        }
        if (g == 0 && r < ch.n_rows) gap_row_terms<LOSS, double>(ch.st + r, zi, s_loss, s_conj);
    }
    gap_block_end<256>(s_loss, s_conj, part_loss + blockIdx.x, part_conj + blockIdx.x, part_loss, part_conj, E);
}

// The same row pass where the columns are numbered by popularity: the first n_hot entries of w are
// copied into LDS once per workgroup and the frequent columns of every row are gathered from there;
// only the rare columns go to the cache hierarchy.  1024 threads; dynamic LDS = n_hot * sizeof(WT).
constexpr int GAP_HOT_THREADS = 1024;
constexpr int GAP_HOT_BYTES = 48 * 1024;
constexpr int GAP_HOT_MAX_LPR = 16;         // lanes per row at most; a lane takes 4 consecutive entries

template <int LOSS, int LPR, typename WT>
__global__ __launch_bounds__(GAP_HOT_THREADS) void gap_rows_csr_hot(const ChunkDev *__restrict__ chunks,
                                                                    const WT *__restrict__ w, double l1, int n_hot,
                                                                    double *part_loss, double *part_conj, GapEnd E)
{
    if (gap_chunk(E) >= E.n_chunks) return gap_w_block<GAP_HOT_THREADS>(l1, part_loss, part_conj, E);
    extern __shared__ __align__(16) unsigned char gap_hot_raw[];
    WT *hot = reinterpret_cast<WT *>(gap_hot_raw);
    // LPR lanes per row, as many whole rows per wavefront as fit (LPR need not divide 64: with rows of 40
    // entries ten lanes carry a row and six rows share a wavefront; the lanes left over idle)
    constexpr int ROWS_PER_WAVE = 64 / LPR;
    constexpr int GROUPS = (GAP_HOT_THREADS / 64) * ROWS_PER_WAVE;
    const int lane = threadIdx.x & 63;
    const int sub = lane % LPR;
    const bool idle = lane >= ROWS_PER_WAVE * LPR;
    const int grp = (threadIdx.x >> 6) * ROWS_PER_WAVE + lane / LPR;
    const ChunkDev &ch = chunks[gap_chunk(E)];
    const int n_rows = ch.n_rows;
    const int32_t *__restrict__ rp = ch.row_ptr;
    const int32_t *__restrict__ col = ch.col;
    const float *__restrict__ val = ch.val;
    const int stride = E.per_chunk * GROUPS;
    for (int i = threadIdx.x; i < n_hot; i += GAP_HOT_THREADS) hot[i] = shared_at(w, i, l1);
    __syncthreads();
    double s_loss = 0.0, s_conj = 0.0;
    KeptRow<WT> kept;
    int at = 0;                                  // the lane of the group that keeps the next row
    // (the trip count is the same for all lanes of a wavefront: the shuffles below need every lane)
    for (int rb = gap_slot(E) * GROUPS; rb < n_rows; rb += 2 * stride) {
        const int r0 = rb + grp;
        const int r1 = r0 + stride;
        const bool one = !idle && r0 < n_rows;
        const bool two = !idle && r1 < n_rows;
        const int b0 = one ? rp[r0] : 0, e0 = one ? rp[r0 + 1] : 0;
        const int b1 = two ? rp[r1] : 0, e1 = two ? rp[r1 + 1] : 0;
        WT z0 = 0, z1 = 0;
        // Each lane takes 4 consecutive entries of its row with one 16-byte load per array (the vector
        // memory pipeline is busy per instruction, not per byte, here); rows are at most 4 * LPR long where
        // this kernel is used, and every chunk's arrays are followed by readable slack.
        {
            const int p0 = b0 + 4 * sub, p1 = b1 + 4 * sub;
            int4_a4 c0 = {0, 0, 0, 0}, c1 = {0, 0, 0, 0};
            float4_a4 v0 = {0.f, 0.f, 0.f, 0.f}, v1 = {0.f, 0.f, 0.f, 0.f};
            if (p0 < e0) { c0 = gld4(col + p0); v0 = gld4(val + p0); }
            if (p1 < e1) { c1 = gld4(col + p1); v1 = gld4(val + p1); }
            WT w0[4], w1[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const bool in0 = p0 + k < e0, in1 = p1 + k < e1;
                const int a0 = in0 ? c0[k] : 0, a1 = in1 ? c1[k] : 0;
                w0[k] = a0 < n_hot ? hot[a0] : shared_at(w, a0, l1);
                w1[k] = a1 < n_hot ? hot[a1] : shared_at(w, a1, l1);
                if (!in0) v0[k] = 0.f;
                if (!in1) v1[k] = 0.f;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                z0 += (WT)v0[k] * w0[k];
                z1 += (WT)v1[k] * w1[k];
            }
        }
        // sum over the row's lanes into its first lane
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) {
            const WT y0 = __shfl_down(z0, o, 64), y1 = __shfl_down(z1, o, 64);
            if (sub < o && sub + o < LPR) { z0 += y0; z1 += y1; }
        }
        // ... and from there into the lane that keeps it
        z0 = __shfl(z0, lane - sub, 64);
        z1 = __shfl(z1, lane - sub, 64);
        kept.keep(one && sub == at, r0, z0);
        kept.keep(two && sub == at + 1, r1, z1);
        at += 2;
        if (at + 2 > LPR) {
            kept.template terms<LOSS>(ch.st, s_loss, s_conj);
            at = 0;
        }
    }
    kept.template terms<LOSS>(ch.st, s_loss, s_conj);
    gap_block_end<GAP_HOT_THREADS>(s_loss, s_conj, part_loss + blockIdx.x, part_conj + blockIdx.x, part_loss, part_conj, E);
}

// Dense rows (ld floats each, 16-byte aligned): LPR lanes per row, four columns at a time.  Same grid as the sparse kernel.
template <int LOSS, int LPR, typename WT>
__global__ __launch_bounds__(256) void gap_rows_dense(const ChunkDev *__restrict__ chunks, int d, int ld,
                                                      const WT *__restrict__ w, double l1,
                                                      double *part_loss, double *part_conj, GapEnd E)
{
    if (gap_chunk(E) >= E.n_chunks) return gap_w_block<256>(l1, part_loss, part_conj, E);
    constexpr int GROUPS = 256 / LPR;
    const int sub = threadIdx.x % LPR;
    const int grp = threadIdx.x / LPR;
    const ChunkDev &ch = chunks[gap_chunk(E)];
    double s_loss = 0.0, s_conj = 0.0;
    KeptRow<WT> kept;
    int at = 0;                                  // the lane of the group that keeps the next row
    for (int r = gap_slot(E) * GROUPS + grp; r < ch.n_rows; r += E.per_chunk * GROUPS) {
        const float *x = ch.val + (int64_t)r * ld;
        WT z = 0;
        for (int p = 4 * sub; p < d; p += 4 * LPR) {         // (w is readable up to a multiple of 64 columns, zero past d)
            const float4_v v = *reinterpret_cast<const float4_v *>(x + p);
#pragma unroll
            for (int e = 0; e < 4; ++e) z += (WT)v[e] * shared_at(w, p + e, l1);
        }
#pragma unroll
        for (int o = LPR / 2; o > 0; o >>= 1) z += __shfl_xor(z, o, 64);
        kept.keep(sub == at, r, z);
        if (++at == LPR) {
            kept.template terms<LOSS>(ch.st, s_loss, s_conj);
            at = 0;
        }
    }
    kept.template terms<LOSS>(ch.st, s_loss, s_conj);
    gap_block_end<256>(s_loss, s_conj, part_loss + blockIdx.x, part_conj + blockIdx.x, part_loss, part_conj, E);
}

}  // namespace chicle
