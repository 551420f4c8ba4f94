// Local solver for long passes over narrow dense rows, squared loss (paper Section 2.2: L = 1, H = all local samples): the
// same steps as row by row, without a chain through the rows.
//
// A step of this loss is affine in the private vector v, v + s (k - x.v) x with s = 1 / (c + |x|^2), k = residual - alpha,
// and so is a run of them: P v + b.  For rows of up to 32 columns P (d x d) is smaller than the run's rows, so a pass is
//   affine_maps    P and b of every run of rows, on the whole chip: P' = P - s x (x'P), b' = b + s (k - x.b) x;
//   affine_starts  one wavefront per solver: the private vector before every run and after the last, a d x d product per run;
//   affine_steps   every run's steps one row after the other from its own start, on the whole chip: the new alphas.
// Only the second kernel is a chain, of some 440 cycles per run of 128 rows; blocks of 64 rows solved by their inverse took
// 2.2e3 (see sdca_dense_squared).  The first is bound by its multiply-adds (2 d^2 per row, of rank one updates that depend on
// each other), the third by the dozen dependent instructions of a row.  500000 x 28, 16 solvers, a pass: 57 + 50
// + 38 us (450 before); fifty rounds 28.2 -> 9.96 ms.
// Precision: dot products and P are fp32; b, the starts, the private vector inside a run and the diagonal of 1 - P are summed
// in double (P's own would round what a weak run does to its v relative to v).  The solver's update is the vector after the
// last run, not a sum over the runs: an error in the vector shrinks with every row after it, one in a run's share would stay.
// Errors against 64 bits, 80 jobs of 3500 to 60000 rows of 2 to 32 columns, lambda n from 0.1 to 100, three rounds, geometric
// mean of now / blocks solved by their inverse: updates 0.88, alpha 0.91, w 0.94.  (Updates as sums over runs, or 1 - P in place
// of P, came to 10 times as much; without the diagonal's sum in double 1.1.  Products P v in double changed nothing and took
// 20 us more.)
#pragma once
#include <hip/hip_runtime.h>
#include "device_types.hpp"
#include "mem.hpp"
#include "sdca_dense.hpp"

namespace chicle {

typedef float float2_v __attribute__((ext_vector_type(2)));

constexpr int AFFINE_MAX_D = 32;
constexpr int AFFINE_GROUP = 16;                 // rows in flight per run
constexpr int AFFINE_UNITS = 4;                  // runs per wavefront: 16 lanes each, two columns per lane
// Wavefronts per workgroup, each on its own: one per SIMD (workgroups of one wavefront: affine_maps 70 us for 55).
constexpr int AFFINE_WAVES = 4;
// A run's place is the first of the tiles its rows have (their addresses stay with their tiles): P[k][m], zero for k = m, at
// [m / 4][k][m % 4], then vectors of 32 doubles: b, the diagonal of 1 - P, the start; and words that nobody reads.
constexpr int AFFINE_B = AFFINE_MAX_D * AFFINE_MAX_D, AFFINE_DIAG = AFFINE_B + 64, AFFINE_START = AFFINE_DIAG + 64,
              AFFINE_SINK = AFFINE_START + 64;
static_assert(AFFINE_SINK + 64 <= BATCH * BATCH, "before the rows' addresses");
static_assert(DENSE_TILE_FLOATS % 4 == 0, "16-byte aligned places");
typedef double double2_v __attribute__((ext_vector_type(2)));

// Orders the LDS accesses of one wavefront (they are performed in order; the compiler has to keep them so).
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Sum over 16 lanes, in all of them.
__device__ __forceinline__ float sum16(float v)
{
#define CHICLE_DPP_ADD(ctrl) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xF, 0xF, true))
    CHICLE_DPP_ADD(0xB1);                        // lanes xor 1, xor 2, then mirrored halves and rows
    CHICLE_DPP_ADD(0x4E);
    CHICLE_DPP_ADD(0x141);
    CHICLE_DPP_ADD(0x140);
#undef CHICLE_DPP_ADD
    return v;
}
// The value of lane R of each 16.
template <int R>
__device__ __forceinline__ float of_lane16(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + R, 0xF, 0xF, true));
}

// Grid: (groups of 16 runs, solver), four runs per wavefront.  A lane holds two columns of its run's P in registers; rows come
// through LDS, where 16 lanes read the same words.  The lookups (order entry -> chunk -> row) are four groups deep, so that
// each group's loads have a group's arithmetic to return in.  DK: columns, rounded up to four.
template <int DK>
__global__ __launch_bounds__(64 * AFFINE_WAVES) void affine_maps(
    const ChunkDev *__restrict__ chunks, const SolverDev *__restrict__ solvers, const int32_t *__restrict__ row_chunk,
    const int32_t *__restrict__ chunk_first, const int32_t *__restrict__ perm, float *tiles, int run, float c, float inv_c, int *err)
{
    constexpr int Q = DK / 4, LDR = AFFINE_MAX_D + 4, LDU = AFFINE_GROUP * LDR + 4;      // (runs and rows on other banks)
    __shared__ __align__(16) float sh_x[AFFINE_WAVES][AFFINE_UNITS * LDU];
    __shared__ __align__(16) float sh_sk[AFFINE_WAVES][AFFINE_UNITS][AFFINE_GROUP][2];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), first = ((int)blockIdx.x * AFFINE_WAVES + wv) * AFFINE_UNITS;
    float *s_x = sh_x[wv];
    auto &s_sk = sh_sk[wv];
    const SolverDev S = solvers[blockIdx.y];
    const int units = (S.n_rows + run - 1) / run;
    if (first >= units) return;
    const int lane = threadIdx.x & 63, m = lane & 15, un = lane >> 4, unit = first + un;
    const int t0 = unit * run + m, groups = run / AFFINE_GROUP, tile_rows = (S.n_rows + BATCH - 1) / BATCH * BATCH;
    const int my_rows = unit < units ? S.n_rows : 0;
    float *tile0 = tiles + (int64_t)S.tile_begin * DENSE_TILE_FLOATS;
    float *out = tile0 + (int64_t)min(unit, units - 1) * (run / BATCH) * DENSE_TILE_FLOATS;
    // No load or store stands behind a condition (the compiler would wait for all that are in flight), and what a load
    // returns is first looked at a group later: rows that do not exist look up a row that does.
    struct Order { int lr; bool ok; };
    struct Chunk { int ci, lr; bool ok; };
    struct Place { const float *val; RowState *st; int first, lr; bool ok; };
    bool refused = false;
    auto order = [&](int g) __attribute__((always_inline)) {
        const int t = t0 + g * AFFINE_GROUP;
        return Order{perm[S.perm_off + min(t, S.n_rows - 1)], (bool)((g < groups) & (t < my_rows))};
    };
    auto chunk_of = [&](Order o) __attribute__((always_inline)) {
        const bool in = (unsigned)o.lr < (unsigned)S.n_rows;
        refused |= o.ok & !in;
        const int lr = in ? o.lr : 0;
        return Chunk{row_chunk[S.perm_off + lr], lr, (bool)(o.ok & in)};
    };
    auto place_of = [&](Chunk w) __attribute__((always_inline)) {
        return Place{chunks[w.ci].val, chunks[w.ci].st, chunk_first[w.ci], w.lr, w.ok};
    };
    float4_v x_in[Q], st_in;
    DenseRow row;
    bool row_ok;
    auto fetch = [&](const Place &w) __attribute__((always_inline)) {
        row = DenseRow{w.val + (int64_t)(w.lr - w.first) * DK, w.st + (w.lr - w.first)};
        row_ok = w.ok;
#pragma unroll
        for (int q = 0; q < Q; ++q) x_in[q] = *(const CHICLE_GLOBAL float4_v *)(row.x + 4 * q);
        st_in = gld_state(row.st);
    };
    for (int i = lane; i < AFFINE_UNITS * LDU; i += 64) s_x[i] = 0.f;       // (columns past the row's end stay zero)
    fetch(place_of(chunk_of(order(0))));
    Place next = place_of(chunk_of(order(1)));
    Chunk far = chunk_of(order(2));
    Order farther = order(3);
    float P0[DK], P1[DK];                        // P[k][2m], P[k][2m + 1]
#pragma unroll
    for (int k = 0; k < DK; ++k) { P0[k] = k == 2 * m ? 1.f : 0.f; P1[k] = k == 2 * m + 1 ? 1.f : 0.f; }
    double b0 = 0.0, b1 = 0.0, a0 = 0.0, a1 = 0.0;      // a: the diagonal of 1 - P
    float *mine = s_x + un * LDU;
    wave_lds_fence();
    for (int g = 0; g < groups; ++g) {
        {
            const bool live = row_ok & takes_steps(st_in.z);
#pragma unroll
            for (int q = 0; q < Q; ++q) *reinterpret_cast<float4_v *>(mine + m * LDR + 4 * q) = live ? x_in[q] : float4_v{0.f, 0.f, 0.f, 0.f};
            const float s = (c / (c + st_in.z)) * inv_c;
            s_sk[un][m][0] = live ? s : 0.f;
            s_sk[un][m][1] = live ? st_in.w - st_in.y : 0.f;
            const int t = t0 + g * AFFINE_GROUP;
            // (a tile's rows past the end too: they take no step)
            float *tile = unit * run + g * AFFINE_GROUP < tile_rows ? tile0 + (int64_t)(t / BATCH) * DENSE_TILE_FLOATS + BATCH * BATCH + 4 * (t % BATCH)
                                                                    : out + AFFINE_SINK + 4 * m;
            const DenseRow kept = {row.x, live ? row.st : nullptr};
            *(CHICLE_GLOBAL float4_v *)tile = __builtin_bit_cast(float4_v, kept);
        }
        fetch(next);
        next = place_of(far);
        far = chunk_of(farther);
        farther = order(g + 4);
        wave_lds_fence();
        // (a row's words are read during the arithmetic of the row before it)
        struct Words { float4_v x[Q]; float2_v xm, sk; };
        auto read = [&](int r) __attribute__((always_inline)) {
            Words w;
#pragma unroll
            for (int q = 0; q < Q; ++q) w.x[q] = *reinterpret_cast<const float4_v *>(mine + r * LDR + 4 * q);
            w.xm = *reinterpret_cast<const float2_v *>(mine + r * LDR + 2 * m);
            w.sk = *reinterpret_cast<const float2_v *>(&s_sk[un][r][0]);
            return w;
        };
        auto add_row = [&](const Words &w) __attribute__((always_inline)) {
            const float4_v (&x)[Q] = w.x;
            const float2_v xm = w.xm, sk = w.sk;
            float d0[2] = {0.f, 0.f}, d1[2] = {0.f, 0.f};
#pragma unroll
            for (int k = 0; k < DK; ++k) {
                d0[k & 1] = fmaf(x[k >> 2][k & 3], P0[k], d0[k & 1]);
                d1[k & 1] = fmaf(x[k >> 2][k & 3], P1[k], d1[k & 1]);
            }
            const float n0 = -sk.x * (d0[0] + d0[1]), n1 = -sk.x * (d1[0] + d1[1]);
            const float p = sk.x * (sk.y - sum16(fmaf(xm.x, (float)b0, xm.y * (float)b1)));
#pragma unroll
            for (int k = 0; k < DK; ++k) {
                P0[k] = fmaf(x[k >> 2][k & 3], n0, P0[k]);
                P1[k] = fmaf(x[k >> 2][k & 3], n1, P1[k]);
            }
            a0 = fma((double)xm.x, (double)-n0, a0);
            a1 = fma((double)xm.y, (double)-n1, a1);
            b0 = fma((double)xm.x, (double)p, b0);
            b1 = fma((double)xm.y, (double)p, b1);
        };
        Words even = read(0);
        for (int r = 0; r < AFFINE_GROUP; r += 2) {
            const Words odd = read(r + 1);
            __builtin_amdgcn_sched_barrier(0);   // (or all reads are put first, and waited for)
            add_row(even);
            __builtin_amdgcn_sched_barrier(0);
            even = read(min(r + 2, AFFINE_GROUP - 1));
            __builtin_amdgcn_sched_barrier(0);
            add_row(odd);
            __builtin_amdgcn_sched_barrier(0);
        }
        // the diagonal anew from its sum in double: beside the ones of a weak run, every row's rounding stays in it
        const float p0 = (float)(1.0 - a0), p1 = (float)(1.0 - a1);
#pragma unroll
        for (int k = 0; k < DK; ++k) { P0[k] = k == 2 * m ? p0 : P0[k]; P1[k] = k == 2 * m + 1 ? p1 : P1[k]; }
        wave_lds_fence();
    }
    if (refused) atomicOr(err, ERR_PERM_RANGE);
    if (unit >= units) return;
#pragma unroll
    for (int k = 0; k < DK; ++k)
        *(CHICLE_GLOBAL float2_v *)(out + ((m >> 1) * AFFINE_MAX_D + k) * 4 + (m & 1) * 2) = float2_v{k == 2 * m ? 0.f : P0[k], k == 2 * m + 1 ? 0.f : P1[k]};
    *(CHICLE_GLOBAL double2_v *)(out + AFFINE_B + 4 * m) = double2_v{b0, b1};
    *(CHICLE_GLOBAL double2_v *)(out + AFFINE_DIAG + 4 * m) = double2_v{a0, a1};
}

// Grid: one wavefront per solver.  Lane: row of P, and half of the columns (four Q of them).  The maps of eight runs are in
// flight.
template <int Q>
__global__ __launch_bounds__(64) void affine_starts(const SolverDev *__restrict__ solvers, float *tiles, float *u_all,
                                                    int64_t ld_v, int d, int run, RoundScalars sc)
{
    constexpr int SETS = 8;
    __shared__ __align__(16) float s_v[AFFINE_MAX_D];
    const SolverDev S = solvers[blockIdx.x];
    stamp_solver(sc, 0);
    const int units = (S.n_rows + run - 1) / run;
    const int lane = threadIdx.x, i = lane & 31, h = lane >> 5;
    const int64_t stride = (int64_t)(run / BATCH) * DENSE_TILE_FLOATS;
    float *place = tiles + (int64_t)S.tile_begin * DENSE_TILE_FLOATS;
    double v = i < d ? (double)u_all[(int64_t)blockIdx.x * ld_v + i] : 0.0;
    float4_v P[SETS][Q];
    double b[SETS], a[SETS];
    auto load = [&](int s, int at) __attribute__((always_inline)) {
        const float *p = place + min(at, units - 1) * stride;
#pragma unroll
        for (int e = 0; e < Q; ++e) P[s][e] = *(const CHICLE_GLOBAL float4_v *)(p + ((h * Q + e) * AFFINE_MAX_D + i) * 4);
        b[s] = *(const CHICLE_GLOBAL double *)(p + AFFINE_B + 2 * i);
        a[s] = *(const CHICLE_GLOBAL double *)(p + AFFINE_DIAG + 2 * i);
    };
    if (units > 0) {
        s_v[i] = (float)v;
        wave_lds_fence();
#pragma unroll
        for (int s = 0; s < SETS; ++s) load(s, s);
        for (int u0 = 0; u0 < units; u0 += SETS) {
#pragma unroll
            for (int s = 0; s < SETS; ++s) {     // (runs past the end change nothing)
                const int at = u0 + s;
                *(CHICLE_GLOBAL double *)(place + min(at, units - 1) * stride + (at < units ? AFFINE_START : AFFINE_SINK) + 2 * i) = v;
                float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int e = 0; e < Q; ++e) {
                    const float4_v w = *reinterpret_cast<const float4_v *>(s_v + 4 * (h * Q + e));
#pragma unroll
                    for (int k = 0; k < 4; ++k) part[k] = fmaf(P[s][e][k], w[k], part[k]);
                }
                const float sum = (part[0] + part[1]) + (part[2] + part[3]);
                const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(sum), __float_as_uint(sum), false, false);
                const float Pv = __uint_as_float(both[0]) + __uint_as_float(both[1]);
                const double dv = fma(-a[s], v, b[s]) + (double)Pv;
                v += ((i < d) & (at < units)) ? dv : 0.0;
                wave_lds_fence();
                s_v[i] = (float)v;
                wave_lds_fence();
                load(s, at + SETS);
            }
        }
    }
    if (lane < d) u_all[(int64_t)blockIdx.x * ld_v + i] = (float)v;
    stamp_solver(sc, 1);
}

// Grid: (groups of 16 runs, solver), four runs per wavefront; lanes as in affine_maps.  The next 16 rows are loaded during the steps
// of these.
__global__ __launch_bounds__(64 * AFFINE_WAVES) void affine_steps(const ChunkDev *__restrict__ chunks, const SolverDev *__restrict__ solvers,
                                                   float *tiles, int run, int ld, RoundScalars sc)
{
    const SolverDev S = solvers[blockIdx.y];
    const int units = (S.n_rows + run - 1) / run;
    const int first = ((int)blockIdx.x * AFFINE_WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * AFFINE_UNITS;
    if (first >= units) return;
    const int lane = threadIdx.x & 63, m = lane & 15, unit = first + (lane >> 4);
    const int groups = run / AFFINE_GROUP, tiles_end = (S.n_rows + BATCH - 1) / BATCH;
    const bool has = 2 * m < ld;
    const int xo = has ? 2 * m : 0;
    float *tile0 = tiles + (int64_t)S.tile_begin * DENSE_TILE_FLOATS;
    float *place = tile0 + (int64_t)min(unit, units - 1) * (run / BATCH) * DENSE_TILE_FLOATS;
    auto rows_of = [&](int g) __attribute__((always_inline)) {       // of the group; past the end: any
        const int t = unit * run + g * AFFINE_GROUP;
        return reinterpret_cast<const DenseRow *>(tile0 + (int64_t)min(t / BATCH, tiles_end - 1) * DENSE_TILE_FLOATS + BATCH * BATCH) + t % BATCH;
    };
    const RowState *any = chunks[0].st;
    const float *xp[AFFINE_GROUP];
    RowState *rec_next, *rec;
    float2_v X[2][AFFINE_GROUP];
    float4_v st;
    auto load_rows = [&](int g) __attribute__((always_inline)) {
        const DenseRow *r = rows_of(g);
#pragma unroll
        for (int j = 0; j < AFFINE_GROUP; ++j) xp[j] = r[j].x;
        rec_next = r[m].st;
    };
    auto load_x = [&](float2_v (&to)[AFFINE_GROUP]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < AFFINE_GROUP; ++j) to[j] = *(const CHICLE_GLOBAL float2_v *)(xp[j] + xo);
        st = gld_state(rec_next != nullptr ? rec_next : any);
        rec = rec_next;
    };
    const double2_v start = *(const CHICLE_GLOBAL double2_v *)(place + AFFINE_START + 4 * m);
    double q0 = has ? start.x : 0.0, q1 = has ? start.y : 0.0;
    load_rows(0);
    load_x(X[0]);
    load_rows(1);
    auto group = [&](int g, float2_v (&now)[AFFINE_GROUP], float2_v (&then)[AFFINE_GROUP]) __attribute__((always_inline)) {
        // (groups past the solver's tiles read its last tile's rows: they take no step)
        const bool live = (rec != nullptr) & (unit * run + g * AFFINE_GROUP < tiles_end * BATCH);
        const float s0 = sc.c / (sc.c + st.z), scale = live ? s0 : 0.f, kk = live ? st.w - st.y : 0.f, alpha = st.y;
        float *alpha_out = live ? &rec->alpha : place + AFFINE_SINK + m;
        load_x(then);
        load_rows(g + 2);
        float delta = 0.f;
        auto step = [&](auto J) __attribute__((always_inline)) {
            constexpr int j = decltype(J)::value;
            const float s = of_lane16<j>(scale), k = of_lane16<j>(kk);
            const bool on = has && s != 0.f;     // (a row that takes no step may hold what is no number)
            const float x0 = on ? now[j].x : 0.f, x1 = on ? now[j].y : 0.f;
            const float left = k - sum16(fmaf(x0, (float)q0, x1 * (float)q1)), dl = s * left;
            const double cf = (double)(s * sc.inv_c * left);
            q0 = fma(cf, (double)x0, q0);
            q1 = fma(cf, (double)x1, q1);
            delta = m == j ? dl : delta;
        };
#define CHICLE_STEP(j) step(std::integral_constant<int, j>())
        CHICLE_STEP(0); CHICLE_STEP(1); CHICLE_STEP(2); CHICLE_STEP(3); CHICLE_STEP(4); CHICLE_STEP(5); CHICLE_STEP(6); CHICLE_STEP(7);
        CHICLE_STEP(8); CHICLE_STEP(9); CHICLE_STEP(10); CHICLE_STEP(11); CHICLE_STEP(12); CHICLE_STEP(13); CHICLE_STEP(14); CHICLE_STEP(15);
#undef CHICLE_STEP
        gst(alpha_out, alpha + delta);
    };
    for (int g = 0; g < groups; g += 2) {
        group(g, X[0], X[1]);
        group(g + 1, X[1], X[0]);
    }
}

}  // namespace chicle
