// Local solver for dense rows, blocks of 64 (or 32) coordinate steps at a time; the same sequence of steps as the
// row-wise solver (paper Section 2.2: L = 1, H = all local samples).
//
// Inside a block the steps obey the recurrence of sdca_batched.hpp over the block's Gram matrix, and that matrix
// depends on the data and the visiting order only.  The pass is therefore two kernels:
//   gram_dense   one workgroup per 64 rows, on the whole chip (and for announced orders a pass ahead): T, scaled as
//                the recurrence takes it, and the addresses of the block's rows;
//   sdca_dense   one workgroup per solver: dot products of the block's rows with the private vector, the
//                recurrence in one wavefront, update of the private vector.
// What is left in the second kernel is the chain of dependent blocks, and it is bound by the recurrence (a lane
// read, a multiply-add and a clamp that depend on each other per step) and by the compute unit's own arithmetic:
// four operations per entry of the row.  Every wavefront therefore keeps its rows of the block in registers from
// the dot products to the update, the next block's rows are loaded meanwhile into a second set, and the only
// traffic through LDS is one read of the private vector and one partial update vector per wavefront.
// Cycles per block, one wavefront's clock, K = 4 .. 16: 64 x 256 hinge 5.1e3 (recurrence 2.0e3, wait for the rows and dot
// products 1.9e3, update 0.8e3), 32 x 1001 hinge 5.9e3, 64 x 28 squared 3.2e3.  Jobs of ten rounds of 4096 x 256 with
// four solvers: 2.99 -> 0.72 ms (before: Gram matrix and rows of a block formed one after the other on the solver's
// compute unit); three rounds of 20011 x 1001, logistic, eight solvers: 52.4 -> 1.43 ms (before: one row at a time), 1.04 with
// series that are renewed where rows move;
// fifty rounds of 500000 x 28, squared, 16 solvers: 50.4 -> 37.2 ms, 28.1 with sdca_dense_squared, 10.8 with sdca_dense_affine.hpp (before: the solver for
// short sparse rows, whose lanes all add to the same 28 places of LDS); 1000 x 48: 103 -> 90 us.
// Precision: a tile's products and the sums of a wavefront's rows in the update are fp32, the sums over wavefronts and blocks
// double.  (The solver for short sparse rows, which rows of up to 48 columns had before, adds every product in double.  The
// updates' error against 64 bits is no larger: 81 jobs of 700 to 40000 rows of 2 to 48 columns, lambda n from 0.1 to 100,
// four rounds, geometric mean of now / before 0.87 hinge, 0.78 squared, 0.87 logistic loss; of w 0.96, 1.04, 0.96.)
#pragma once
#include <hip/hip_runtime.h>
#include <type_traits>
#include "device_types.hpp"
#include "mem.hpp"
#include "sdca_batched.hpp"
#include "sdca_rowwise.hpp"

namespace chicle {

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int DENSE_MAX_D = 1536;                // widest rows whose two register sets fit (sdca_dense<.., M = 6, ..>)
// Dense rows are stored with a length of a multiple of four columns, the last ones zero: every row is 16-byte aligned.
__host__ __device__ inline int dense_ld(int d) { return (d + 3) & ~3; }

// A dense tile: T (16 KB), then the 64 rows' addresses.  T[j][i] (step j's influence on step i, zero for j >= i)
// is stored as [j / 4][i][j % 4].
struct DenseRow {
    const float *x;      // always readable
    RowState *st;        // nullptr: a row that takes no step (past the end, empty, or a refused order entry)
};
constexpr int DENSE_TILE_FLOATS = BATCH * BATCH + BATCH * (int)(sizeof(DenseRow) / sizeof(float));

constexpr int GD_THREADS = 256;
constexpr int GD_COLS = 64;                      // columns of the block in LDS at a time
constexpr int GD_LD = GD_COLS + 4;               // 16-byte aligned rows, spread over the banks

// A row takes steps where its squared norm is neither zero nor beyond what a float holds (the row-wise solver's step is zero
// there).  The two quotients by it that a float may not hold either, for norms below 6e-20, are kept finite: a clamped step
// only needs them large, and infinity times a product of zero would be no number.
__device__ __forceinline__ bool takes_steps(float q) { return q != 0.f && q <= 3.4028235e38f; }
template <int LOSS>
__device__ __forceinline__ float tile_scale(float q, float c)
{
    return LOSS == 0 ? fmaxf(-1.f / q, -3.4028235e38f) : LOSS == 1 ? -1.f / (c + q) : -1.f / c;
}
__device__ __forceinline__ float hinge_scale(float q, float c) { return fminf(c / q, 3.4028235e38f); }

// One workgroup per tile.  The product is on the matrix cores (fp32 in and out): per 64 columns every wavefront
// takes 16 of them for the three 32 x 32 blocks that hold pairs j < i (the fourth is their mirror image).
template <int LOSS>
__global__ __launch_bounds__(GD_THREADS) void gram_dense(
    const ChunkDev *__restrict__ chunks, const SolverDev *__restrict__ solvers, const int32_t *__restrict__ row_chunk,
    const int32_t *__restrict__ chunk_first, const int32_t *__restrict__ perm, const int32_t *__restrict__ tile_solver,
    float *tiles, int ld, float c, bool solve, int *err)
{
    __shared__ __align__(16) float X[BATCH * GD_LD];
    __shared__ float G[BATCH * (BATCH + 1)];
    __shared__ const float *r_x[BATCH];
    __shared__ float r_sgn[BATCH], r_scale[BATCH];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const SolverDev S = solvers[tile_solver[blockIdx.x]];
    float *out = tiles + (int64_t)blockIdx.x * DENSE_TILE_FLOATS;
    if (tid < BATCH) {
        const int t = ((int)blockIdx.x - S.tile_begin) * BATCH + tid;
        DenseRow row = {chunks[0].val, nullptr};
        float sgn = 0.f, scale = 0.f;            // a row that takes no step: no part in T
        if (t < S.n_rows) {
            const int lr = perm[S.perm_off + t];
            if ((unsigned)lr >= (unsigned)S.n_rows) {
                atomicOr(err, ERR_PERM_RANGE);
            } else {
                const int ci = row_chunk[S.perm_off + lr];
                const ChunkDev &ch = chunks[ci];
                const int r = lr - chunk_first[ci];
                const float4_v st = gld_state(ch.st + r);
                row.x = ch.val + (int64_t)r * ld;
                const float q = st.z;
                if (takes_steps(q)) {
                    row.st = ch.st + r;
                    sgn = LOSS == 1 ? 1.f : st.x;
                    scale = tile_scale<LOSS>(q, c);
                }
            }
        }
        r_x[tid] = row.x; r_sgn[tid] = sgn; r_scale[tid] = scale;
        reinterpret_cast<DenseRow *>(out + BATCH * BATCH)[tid] = row;
    }
    __syncthreads();
    // 64 rows x 16 groups of 4 columns: 4 groups per thread
    const float *src[4];
    int dst[4];
    const int c4 = 4 * (tid & 15);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int row = (tid >> 4) + 16 * k;
        src[k] = r_x[row]; dst[k] = row * GD_LD + c4;
    }
    float4_v in[4];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            in[k] = {0.f, 0.f, 0.f, 0.f};
            if (k0 + c4 < ld) in[k] = *(const CHICLE_GLOBAL float4_v *)(src[k] + k0 + c4);
        }
    };
    floatx16 acc[3];
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[q][r] = 0.f;
    fetch(0);
    for (int k0 = 0; k0 < ld; k0 += GD_COLS) {
#pragma unroll
        for (int k = 0; k < 4; ++k) *reinterpret_cast<float4_v *>(X + dst[k]) = in[k];
        __syncthreads();
        if (k0 + GD_COLS < ld) fetch(k0 + GD_COLS);
        // A 32 x 2 by 2 x 32 product takes A[l % 32][l / 32] and B[l / 32][l % 32] from lane l; any pairing of the
        // columns works for a dot product, so a lane feeds four consecutive ones to four products
        if (k0 + 16 * wv < ld) {
            const float *p = X + (lane & 31) * GD_LD + 16 * wv + 4 * (lane >> 5);
#pragma unroll
            for (int kk = 0; kk < 16; kk += 8) {
                const float4_v a = *reinterpret_cast<const float4_v *>(p + kk);
                const float4_v b = *reinterpret_cast<const float4_v *>(p + 32 * GD_LD + kk);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], a[e], acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], acc[1], 0, 0, 0);
                    acc[2] = __builtin_amdgcn_mfma_f32_32x32x2f32(b[e], b[e], acc[2], 0, 0, 0);
                }
            }
        }
        __syncthreads();
    }
    // the wavefronts' shares are added one after the other (fixed order).  Result layout: register r of lane l is
    // row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32
    for (int w = 0; w < GD_THREADS / 64; ++w) {
        if (wv == w) {
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const int j0 = q == 2 ? 32 : 0, i0 = q == 0 ? 0 : 32;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    float *g = G + (j0 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * (BATCH + 1) + i0 + (lane & 31);
                    *g = w == 0 ? acc[q][r] : *g + acc[q][r];
                }
            }
        }
        __syncthreads();
    }
    const int i = lane;
    const float si = r_scale[i] * r_sgn[i];
    if (LOSS != 1 || !solve) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int jq = wv + 4 * k;
            float4_v v;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int j = 4 * jq + e;
                v[e] = j < i && si != 0.f && r_sgn[j] != 0.f ? G[j * (BATCH + 1) + i] * si * r_sgn[j] : 0.f;
            }
            *reinterpret_cast<float4_v *>(out + tile_at(4 * jq, i)) = v;
        }
        return;
    }
    // Squared loss (where it pays, see solve_tiles): the steps are not clamped, the recurrence delta_i = t_i + sum_{j < i} T_ji delta_j is a unit
    // triangular system and the tile holds its inverse, delta = N t: lane j follows the influence of t_j down the rows.
    // T goes to LDS by rows i (X is free), then one wavefront substitutes forward, 2016 multiply-adds.  (Shorter blocks
    // take diagonal blocks of the tile: N's are the inverses of T's.)
    float *Tt = X;                                       // [i][k], BATCH floats per row
    for (int k = wv; k < BATCH; k += GD_THREADS / 64) Tt[i * GD_LD + k] = k < i && si != 0.f && r_sgn[k] != 0.f ? G[k * (BATCH + 1) + i] * si : 0.f;
    __syncthreads();
    if (wv != 0) return;
    float x[BATCH];
#pragma unroll
    for (int r = 0; r < BATCH; ++r) {
        float s0 = lane == r ? 1.f : 0.f, s1 = 0.f;
#pragma unroll
        for (int k = 0; k < r; k += 4) {
            const float4_v tv = *reinterpret_cast<const float4_v *>(Tt + r * GD_LD + k);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (k + e < r) { if (e & 1) s1 = fmaf(tv[e], x[k + e], s1); else s0 = fmaf(tv[e], x[k + e], s0); }
        }
        x[r] = s0 + s1;
    }
    // lane = j, x[r] = N[j][r]: through LDS into the tile's layout (rows of G are padded by one: no conflicts)
#pragma unroll
    for (int r = 0; r < BATCH; ++r) G[lane * (BATCH + 1) + r] = x[r];
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int jq = 0; jq < BATCH / 4; ++jq) {
        float4_v v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = G[(4 * jq + e) * (BATCH + 1) + i];
        *reinterpret_cast<float4_v *>(out + tile_at(4 * jq, i)) = v;
    }
}

// All four words of a load count as used here.  (Squared losses do not look at the label: the register of a word that
// nobody uses is given to something else at once, which then waits for the load.)
__device__ __forceinline__ void keep_loaded(const float4_v &v) { asm volatile("" ::"v"(v)); }

// Sum over groups of L lanes, in the group's last lane.
template <int L>
__device__ __forceinline__ float group_sum_last(float v)
{
#define CHICLE_DPP_ADD(ctrl, rows) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, rows, 0xF, false))
    CHICLE_DPP_ADD(0x111, 0xF);                     // row_shr 1, 2, 4, 8
    CHICLE_DPP_ADD(0x112, 0xF);
    CHICLE_DPP_ADD(0x114, 0xF);
    if (L >= 16) CHICLE_DPP_ADD(0x118, 0xF);
    if (L >= 32) CHICLE_DPP_ADD(0x142, 0xA);        // row_bcast 15
    if (L >= 64) CHICLE_DPP_ADD(0x143, 0xC);        // row_bcast 31
#undef CHICLE_DPP_ADD
    return v;
}

// Sum over the lanes that share lane % L, in all of them.
template <int L>
__device__ __forceinline__ float sum_over_groups(float v)
{
    if (L <= 8) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xF, 0xF, false));   // row_ror 8
    // (a lane swap of a value with itself leaves the two halves side by side)
    if (L <= 16) {
        const auto h = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = __uint_as_float(h[0]) + __uint_as_float(h[1]);
    }
    if (L <= 32) {
        const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = __uint_as_float(h[0]) + __uint_as_float(h[1]);
    }
    return v;
}

// L lanes per row and M groups of 4 columns per lane (rows of at most 4 L M columns), NW wavefronts, blocks of BR
// rows.  Rows of up to 512 columns take blocks of 64; beyond, two register sets of 64 rows no longer fit, and blocks of
// 32 (from 1025 columns on, 16) take their place: the tile's diagonal blocks, with u brought up to date between them.
template <int L_, int NW_, int M_, int BR_>
struct DenseShape {
    static constexpr int L = L_, NW = NW_, M = M_, BR = BR_;
    static constexpr int THREADS = 64 * NW, G = 64 / L, R = BR / NW, I = R / G, UW = 4 * L * M;
    static constexpr int LDS_FLOATS = BR * BR + UW + NW * UW + 2 * BR;
    static constexpr size_t LDS_BYTES = sizeof(float) * LDS_FLOATS + sizeof(void *) * BR;
};

// The recurrence: lane i owns row i of the block; returns the row's step.  T: lane's coefficients, [j].
// SOLVED: T holds the inverse of the squared loss's recurrence (gram_dense) without its unit diagonal.
template <int LOSS, int BR, bool SOLVED>
__device__ __forceinline__ float dense_recurrence(const float *T_lds, float t, float lo, float hi, float a, float root, int lane, bool &rough)
{
    const int i = lane & (BR - 1);
    const float4_v *Tq = reinterpret_cast<const float4_v *>(T_lds) + i;
    if (LOSS == 2) {
        float none = 0.f;
        return logistic_block<BR, false>(t, a, hi, root, lane, [&](int jq) { return Tq[jq * BR]; }, [](int) { return float4_v{0.f, 0.f, 0.f, 0.f}; }, none, rough);
    }
    float4_v T4[BR / 4];
#pragma unroll
    for (int jq = 0; jq < BR / 4; ++jq) T4[jq] = Tq[jq * BR];
    if (LOSS == 1 && SOLVED) {       // no clamp: the tile holds the recurrence solved (gram_dense), a product is left
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j0 = 0; j0 < BR; j0 += 16) {      // (lane reads in groups: a product right behind its lane read stalls)
            float s[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) s[j] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), j0 + j));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[j & 3] = fmaf(s[j], T4[(j0 + j) >> 2][j & 3], acc[j & 3]);
        }
        return t + ((acc[0] + acc[1]) + (acc[2] + acc[3]));
    }
    if (LOSS == 1) {
        // The other steps' influence is summed apart from the row's own t: 63 small terms added to t one after the other
        // would each round it, three times the error of a row-wise step (2e-7 of alpha against 5e-8).  The step of row j is
        // t_j + s_j; its t_j part does not wait for s_j.
        float s = 0.f;
#pragma unroll
        for (int j = 0; j < BR; ++j) {
            const float tj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), j));
            const float sj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(s), j));
            s = fmaf(sj, T4[j >> 2][j & 3], fmaf(tj, T4[j >> 2][j & 3], s));
        }
        return t + s;
    }
#pragma unroll
    for (int j = 0; j < BR; ++j) {
        const float dj = clamp_step<LOSS>(t, lo, hi);
        const float s = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(dj), j));
        t = fmaf(s, T4[j >> 2][j & 3], t);
    }
    return clamp_step<LOSS>(t, lo, hi);
}

// SOLVED: see dense_recurrence.
template <int LOSS, bool SOLVED, typename SH>
__global__ __launch_bounds__(SH::THREADS) void sdca_dense(
    const ChunkDev *__restrict__ chunks, const SolverDev *__restrict__ solvers, const float *__restrict__ tiles, float *u_all,
    int64_t ld_v, int d, int ld, RoundScalars sc)
{
    constexpr int L = SH::L, NW = SH::NW, M = SH::M, BR = SH::BR, G = SH::G, R = SH::R, I = SH::I, UW = SH::UW;
    constexpr int T4 = BR * BR / 4, TPT = (T4 + SH::THREADS - 1) / SH::THREADS;      // 16-byte words of T, per thread
    extern __shared__ __align__(16) float dn_smem[];
    float *T = dn_smem, *u = T + BR * BR, *part = u + UW, *s_dot = part + NW * UW, *s_coef = s_dot + BR;
    const float **s_x = reinterpret_cast<const float **>(s_coef + BR);

    const SolverDev S = solvers[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    stamp_solver(sc, 0);
    float *u_glb = u_all + (int64_t)blockIdx.x * ld_v;
    // a thread's columns of the private vector are summed in double in its registers; LDS holds them in float for the
    // dot products
    constexpr int UPT = (UW + SH::THREADS - 1) / SH::THREADS;
    double mine[UPT];
#pragma unroll
    for (int c = 0; c < UPT; ++c) {
        const int k = tid + c * SH::THREADS;
        const float v = k < d ? u_glb[k] : 0.f;
        mine[c] = (double)v;
        if (k < UW) u[k] = v;
    }
    const int nb = (S.n_rows + BR - 1) / BR;
    const float *my_tiles = tiles + (int64_t)S.tile_begin * DENSE_TILE_FLOATS;

    // wavefront 0: state of the block's rows (lane = row), of the next block's, addresses of the one after
    const int li = lane & (BR - 1);
    auto row_of = [&](int b) __attribute__((always_inline)) -> DenseRow {
        b = min(b, nb - 1);            // (past the end: the last block again, so that every block requests the same)
        const float *tile = my_tiles + (int64_t)(b * BR / BATCH) * DENSE_TILE_FLOATS;
        return reinterpret_cast<const DenseRow *>(tile + BATCH * BATCH)[(b * BR & (BATCH - 1)) + li];
    };
    // wavefront 0 keeps the rows of blocks b + 1 and b + 2 in registers and requests those of b + 3 in block b
    DenseRow row1 = {nullptr, nullptr}, row2 = row1, row3 = row1;
    RowState *st_cur = nullptr;
    bool rough = true;               // see logistic_block
    float4_v cur = {0.f, 0.f, 0.f, 0.f}, nxt = {0.f, 0.f, 0.f, 0.f};
    const RowState *any = chunks[0].st;
    auto state_of = [&](const DenseRow &r) __attribute__((always_inline)) -> const RowState * { return r.st != nullptr ? r.st : any; };
    // all threads: their 16-byte words of the next block's T, and where these lie in a tile
    float4_v t_in[TPT];
    auto fetch_T = [&](int b) __attribute__((always_inline)) {
        b = min(b, nb - 1);
        const float *tile = my_tiles + (int64_t)(b * BR / BATCH) * DENSE_TILE_FLOATS;
        const int h = (b * BR & (BATCH - 1));
#pragma unroll
        for (int k = 0; k < TPT; ++k) {
            const int idx = tid + k * SH::THREADS;
            if (T4 % SH::THREADS == 0 || idx < T4)
                t_in[k] = *(const CHICLE_GLOBAL float4_v *)(tile + (((h >> 2) + idx / BR) * BATCH + h + (idx & (BR - 1))) * 4);
        }
    };
    auto store_T = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < TPT; ++k) {
            const int idx = tid + k * SH::THREADS;
            if (SOLVED) {                              // without the diagonal: t itself is added last (dense_recurrence)
                const int e = (idx & (BR - 1)) - 4 * (idx / BR);
#pragma unroll
                for (int q = 0; q < 4; ++q) t_in[k][q] = e == q ? 0.f : t_in[k][q];
            }
            if (T4 % SH::THREADS == 0 || idx < T4) reinterpret_cast<float4_v *>(T)[idx] = t_in[k];
        }
    };
    // a lane's columns of its rows; columns past the row's end are read from its start (u is zero there)
    int xo[M];
#pragma unroll
    for (int m = 0; m < M; ++m) { xo[m] = 4 * (lane & (L - 1)) + 4 * L * m; if (xo[m] >= ld) xo[m] = 0; }
    const int row0 = wv * R + lane / L;                // the lane's row in step it: row0 + it * G
    auto fetch_X = [&](float4_v (&X)[I][M]) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < I; ++it) {
            const float *x = s_x[row0 + it * G];
            if (L == 64) {                             // one row per wavefront: its address in scalar registers
                const unsigned long long a = (unsigned long long)x;
                x = (const float *)(((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(a >> 32)) << 32) |
                                    (unsigned)__builtin_amdgcn_readfirstlane((int)a));
            }
#pragma unroll
            for (int m = 0; m < M; ++m) X[it][m] = *(const CHICLE_GLOBAL float4_v *)(x + xo[m]);
        }
    };

    float4_v XA[I][M], XB[I][M];
    if (nb > 0) {
        if (wv == 0) {
            const DenseRow r0 = row_of(0);
            if (lane < BR) s_x[lane] = r0.x;
            st_cur = r0.st;
            cur = gld_state(state_of(r0));
            row1 = row_of(1); row2 = row_of(2);
        }
        fetch_T(0);
        store_T();
        __syncthreads();
        fetch_X(XA);
        __syncthreads();
        if (wv == 0 && lane < BR) s_x[lane] = row1.x;
        __syncthreads();
    }

    // One block: rows in X, the next block's are loaded into Y.  The compute unit's memory pipeline takes a block's rows
    // at 64 bytes a cycle, so the loads are issued while the recurrence runs (wavefront 0's own before it).  The loop is
    // compiled once for wavefront 0 and once for the others: the compiler counts the loads in flight, and where paths
    // join it assumes the smaller count and waits for loads that have just been issued.
    auto block = [&](auto chain, int b, float4_v (&X)[I][M], float4_v (&Y)[I][M]) __attribute__((always_inline)) {
        constexpr bool CHAIN = decltype(chain)::value;
        // 1. dot products with the private vector
        {
            float4_v uu[M];
#pragma unroll
            for (int m = 0; m < M; ++m) uu[m] = *reinterpret_cast<const float4_v *>(u + 4 * (lane & (L - 1)) + 4 * L * m);
#pragma unroll
            for (int it = 0; it < I; ++it) {
                float p = 0.f;
#pragma unroll
                for (int m = 0; m < M; ++m)
#pragma unroll
                    for (int e = 0; e < 4; ++e) p = fmaf(X[it][m][e], uu[m][e], p);
                p = group_sum_last<L>(p);
                if ((lane & (L - 1)) == L - 1) s_dot[row0 + it * G] = p;
            }
        }
        if (CHAIN) {
            fetch_T(b + 1);
            fetch_X(Y);
            nxt = gld_state(state_of(row1));
            row3 = row_of(b + 3);
        }
        __syncthreads();
        // 2. the recurrence
        if (!CHAIN) {
            fetch_T(b + 1);
            fetch_X(Y);
        } else {
            const float xu = s_dot[li], y = cur.x, a = cur.y, q = cur.z, rw = cur.w;
            float t = 0.f, lo = 0.f, hi = 0.f, root = 0.f;
            if (st_cur != nullptr) {
                if (LOSS == 0) {
                    t = hinge_scale(q, sc.c) * (rw - y * xu);
                    lo = -a; hi = 1.f - a;
                } else if (LOSS == 1) {
                    t = (sc.c / (sc.c + q)) * (rw - a - xu);
                } else {
                    t = rw - y * xu;
                    hi = q * sc.inv_c;
                    root = logistic_root(t, hi, a);
                }
            }
            const float dl = dense_recurrence<LOSS, BR, SOLVED>(T, t, lo, hi, a, root, lane, rough);
            if (lane < BR) {
                if (st_cur != nullptr) {
                    float an = a + dl;
                    if (LOSS != 1) an = fminf(fmaxf(an, 0.f), 1.f);
                    gst(&st_cur->alpha, an);
                }
                s_coef[lane] = dl * (LOSS == 1 ? 1.f : y) * sc.inv_c;      // the row's coefficient in the update
            }
            st_cur = b + 1 < nb ? row1.st : nullptr;
        }
        __syncthreads();
        // 3. the wavefront's part of the update; T of the next block
        {
            float4_v p[M];
#pragma unroll
            for (int m = 0; m < M; ++m) p[m] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int it = 0; it < I; ++it) {
                const float cf = s_coef[row0 + it * G];
#pragma unroll
                for (int m = 0; m < M; ++m)
#pragma unroll
                    for (int e = 0; e < 4; ++e) p[m][e] = fmaf(cf, X[it][m][e], p[m][e]);
            }
#pragma unroll
            for (int m = 0; m < M; ++m) {
#pragma unroll
                for (int e = 0; e < 4; ++e) p[m][e] = sum_over_groups<L>(p[m][e]);
                if (lane < L) *reinterpret_cast<float4_v *>(part + wv * UW + 4 * lane + 4 * L * m) = p[m];
            }
        }
        store_T();
        __syncthreads();
        // 4. update of the private vector (columns past the row's end stay zero)
#pragma unroll
        for (int c = 0; c < UPT; ++c) {
            const int k = tid + c * SH::THREADS;
            if (k < d) {
                double s = 0.0;
#pragma unroll
                for (int w = 0; w < NW; ++w) s += (double)part[w * UW + k];
                mine[c] += s;
                u[k] = (float)mine[c];
            }
        }
        if (CHAIN) {
            if (lane < BR) s_x[lane] = row2.x;               // (every wavefront has read the next block's)
            keep_loaded(nxt);
            cur = nxt; row1 = row2; row2 = row3;
        }
        __syncthreads();
    };
    auto pass = [&](auto chain) __attribute__((always_inline)) {
        for (int b = 0; b < nb; b += 2) {    // (an odd last block is followed by one that takes no step)
            block(chain, b, XA, XB);
            block(chain, b + 1, XB, XA);
        }
    };
    if (__builtin_amdgcn_readfirstlane(wv) == 0) pass(std::true_type());
    else pass(std::false_type());
#pragma unroll
    for (int c = 0; c < UPT; ++c)
        if (tid + c * SH::THREADS < d) u_glb[tid + c * SH::THREADS] = (float)mine[c];
    stamp_solver(sc, 1);
}

// Squared loss, rows of up to 64 columns.  With the recurrence solved in the tile nothing of a block is serial any more
// but block after block, and a block is so short (a few hundred multiply-adds per wavefront) that it is over before a load
// issued in the block before has returned: every load is issued three blocks ahead, into one of four register sets (the
// loop is unrolled over them), from row addresses that were loaded three blocks before that.  Every wavefront turns the
// dot products of its own 16 rows into their share of all 64 steps, so that the steps need no wavefront of their own and no
// tile in LDS; three workgroup barriers per block.  500000 x 28, 16 solvers: 64 rows in 3.1e3 cycles with sdca_dense,
// 2.2e3 here; fifty rounds 37.2 -> 28.1 ms.
template <typename SH>
__global__ __launch_bounds__(SH::THREADS) void sdca_dense_squared(
    const ChunkDev *__restrict__ chunks, const SolverDev *__restrict__ solvers, const float *__restrict__ tiles, float *u_all,
    int64_t ld_v, int d, int ld, RoundScalars sc)
{
    constexpr int L = SH::L, NW = SH::NW, G = SH::G, R = SH::R, I = SH::I, UW = SH::UW;
    static_assert(SH::BR == BATCH && SH::M == 1 && UW <= SH::THREADS, "whole tiles, four columns per lane");
    constexpr int SETS = 4, AHEAD = SETS - 1;
    __shared__ __align__(16) float u[UW], part[NW][UW], s_step[NW][BATCH];
    __shared__ __align__(16) float s_kb[2][BATCH][2];        // per row: c / (c + q) and residual - alpha (0, 0: no step)
    __shared__ float s_alpha[2][BATCH];
    __shared__ RowState *s_st[8][BATCH];
    const SolverDev S = solvers[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    stamp_solver(sc, 0);
    float *u_glb = u_all + (int64_t)blockIdx.x * ld_v;
    const int nb = (S.n_rows + BATCH - 1) / BATCH;
    const float *my_tiles = tiles + (int64_t)S.tile_begin * DENSE_TILE_FLOATS;
    double mine = tid < d ? (double)u_glb[tid] : 0.0;        // thread: column
    if (tid < UW) u[tid] = (float)mine;

    const int row0 = wv * R + lane / L;                      // the lane's row in step it: row0 + it * G
    const int col = 4 * (lane & (L - 1)), xo = col < ld ? col : 0;
    auto tile_of = [&](int b) __attribute__((always_inline)) { return my_tiles + (int64_t)min(b, nb - 1) * DENSE_TILE_FLOATS; };
    auto rows_of = [&](int b) __attribute__((always_inline)) { return reinterpret_cast<const DenseRow *>(tile_of(b) + BATCH * BATCH); };
    const float *xp[SETS][I];
    float4_v X[SETS][I], T[SETS][R / 4], st[SETS];
    RowState *rec[SETS];
    auto load_xp = [&](int b, const float *(&to)[I]) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < I; ++it) to[it] = rows_of(b)[row0 + it * G].x;
    };
    auto load_X = [&](const float *(&from)[I], float4_v (&to)[I]) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < I; ++it) to[it] = *(const CHICLE_GLOBAL float4_v *)(from[it] + xo);
    };
    auto load_T = [&](int b, float4_v (&to)[R / 4]) __attribute__((always_inline)) {
#pragma unroll
        for (int jq = 0; jq < R / 4; ++jq) to[jq] = *(const CHICLE_GLOBAL float4_v *)(tile_of(b) + tile_at(wv * R + 4 * jq, lane));
    };
    const RowState *any = chunks[0].st;
    auto load_state = [&](RowState *r) __attribute__((always_inline)) { return gld_state(r != nullptr ? r : any); };
    // what block b's steps need of its rows, from their state
    auto publish = [&](int b, const float4_v &s) __attribute__((always_inline)) {
        keep_loaded(s);
        const bool live = s_st[b & 7][lane] != nullptr;
        s_kb[b & 1][lane][0] = live ? sc.c / (sc.c + s.z) : 0.f;
        s_kb[b & 1][lane][1] = live ? s.w - s.y : 0.f;
        s_alpha[b & 1][lane] = s.y;
    };
    auto block = [&](auto first_wave, auto set, int b) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first_wave)::value;
        constexpr int s0 = decltype(set)::value, s1 = (s0 + 1) % SETS, s3 = (s0 + AHEAD) % SETS, s6 = (s0 + 2 * AHEAD) % SETS;
        // loads of block b + 3, addresses of block b + 6
        load_X(xp[s3], X[s3]);
        load_T(b + AHEAD, T[s3]);
        load_xp(b + 2 * AHEAD, xp[s6]);
        if (FIRST) {
            st[s3] = load_state(rec[s3]);
            s_st[(b + AHEAD) & 7][lane] = b + AHEAD < nb ? rec[s3] : nullptr;
            rec[s6] = rows_of(b + 2 * AHEAD)[lane].st;
        }
        // 1. dot products of the wavefront's rows, and what their unclipped steps add to all 64
        const float4_v uu = *reinterpret_cast<const float4_v *>(u + col);
        float p[I], acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int it = 0; it < I; ++it) {
            p[it] = X[s0][it][0] * uu[0];
#pragma unroll
            for (int e = 1; e < 4; ++e) p[it] = fmaf(X[s0][it][e], uu[e], p[it]);
            p[it] = group_sum_last<L>(p[it]);
        }
        float dot[R];
#pragma unroll
        for (int j = 0; j < R; ++j) dot[j] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(p[j / G]), (j % G) * L + L - 1));
        __builtin_amdgcn_sched_barrier(0);       // (a use right behind its lane read stalls)
#pragma unroll
        for (int j = 0; j < R; j += 2) {
            const float4_v kb = *reinterpret_cast<const float4_v *>(&s_kb[b & 1][wv * R + j][0]);
            acc[j & 3] = fmaf(kb[0] * (kb[1] - dot[j]), T[s0][j >> 2][j & 3], acc[j & 3]);
            acc[(j + 1) & 3] = fmaf(kb[2] * (kb[3] - dot[j + 1]), T[s0][j >> 2][(j + 1) & 3], acc[(j + 1) & 3]);
        }
        s_step[wv][lane] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
        __syncthreads();
        // 2. the wavefront's part of the update
        float4_v q = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int it = 0; it < I; ++it) {
            float dl = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) dl += s_step[w][row0 + it * G];
            const float cf = dl * sc.inv_c;
#pragma unroll
            for (int e = 0; e < 4; ++e) q[e] = fmaf(cf, X[s0][it][e], q[e]);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) q[e] = sum_over_groups<L>(q[e]);
        if (lane < L) *reinterpret_cast<float4_v *>(&part[wv][4 * lane]) = q;
        if (FIRST) {
            float dl = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) dl += s_step[w][lane];
            RowState *r = s_st[b & 7][lane];
            if (r != nullptr) gst(&r->alpha, s_alpha[b & 1][lane] + dl);
            publish(b + 1, st[s1]);
        }
        __syncthreads();
        // 3. update of the private vector
        if (tid < d) {
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < NW; ++w) s += (double)part[w][tid];
            mine += s;
            u[tid] = (float)mine;
        }
        __syncthreads();
    };
    auto pass = [&](auto first_wave) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first_wave)::value;
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) {
            load_xp(k, xp[k]);
            if (FIRST) rec[k] = rows_of(k)[lane].st;
        }
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) {    // (in the order of the loop)
            load_X(xp[k], X[k]);
            load_T(k, T[k]);
            load_xp(k + AHEAD, xp[(k + AHEAD) % SETS]);
            if (FIRST) {
                st[k] = load_state(rec[k]);
                s_st[k][lane] = k < nb ? rec[k] : nullptr;
                rec[(k + AHEAD) % SETS] = rows_of(k + AHEAD)[lane].st;
            }
        }
        if (FIRST) publish(0, st[0]);
        __syncthreads();
        // whole rounds of the register sets (blocks past the end take no step): a loop left in the middle has paths that
        // the compiler joins at its head, with the smaller counts of loads in flight
        for (int b = 0; b < nb; b += SETS) {
            block(first_wave, std::integral_constant<int, 0>(), b);
            block(first_wave, std::integral_constant<int, 1>(), b + 1);
            block(first_wave, std::integral_constant<int, 2>(), b + 2);
            block(first_wave, std::integral_constant<int, 3>(), b + 3);
        }
    };
    if (nb > 0) {
        if (wv == 0) pass(std::true_type());
        else pass(std::false_type());
    }
    if (tid < d) u_glb[tid] = (float)mine;
    stamp_solver(sc, 1);
}

// For inspection: the tiles in the layout of the sparse batched solver's ([128][64]).  This block's own pairs are what
// gram_dense has written; the pairs of the previous block against this one, which this solver does not need, are plain dot
// products.
template <int LOSS>
__global__ __launch_bounds__(256) void dense_tiles_out(const SolverDev *__restrict__ solvers, const int32_t *__restrict__ tile_solver,
                                                       const float *__restrict__ tiles, int first, int d, float c, float *out)
{
    const int64_t tile = first + (int)blockIdx.x;
    const int beta = (int)(tile - solvers[tile_solver[tile]].tile_begin);
    const float *T = tiles + tile * DENSE_TILE_FLOATS;
    const DenseRow *own = reinterpret_cast<const DenseRow *>(T + BATCH * BATCH);
    const DenseRow *prev = reinterpret_cast<const DenseRow *>(T - DENSE_TILE_FLOATS + BATCH * BATCH);
    for (int idx = threadIdx.x; idx < TILE_FLOATS; idx += 256) {
        const int jp = idx >> 6, i = idx & 63;
        float v = 0.f;
        if (jp >= BATCH) {
            v = T[tile_at(jp - BATCH, i)];
        } else if (beta > 0) {
            const DenseRow a = prev[jp], b = own[i];
            if (a.st != nullptr && b.st != nullptr) {
                double g = 0.0;
                for (int k = 0; k < d; ++k) g += (double)a.x[k] * (double)b.x[k];
                v = (float)g * tile_scale<LOSS>(b.st->q, c) * (LOSS == 1 ? 1.f : a.st->y * b.st->y);
            }
        }
        out[(int64_t)blockIdx.x * TILE_FLOATS + idx] = v;
    }
}

}  // namespace chicle
