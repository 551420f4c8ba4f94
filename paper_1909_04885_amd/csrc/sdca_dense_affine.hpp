// Local solver for long passes over narrow dense rows, squared loss (paper Section 2.2: L = 1, H = all local samples): the
// same steps as row by row, without a chain through the rows.
//
// A step of this loss is affine in the private vector v, v + s (k - x.v) x with s = 1 / (c + |x|^2), k = residual - alpha,
// and so is a run of them: P v + b.  For rows of up to 32 columns P (d x d) is smaller than the run's rows, so a pass is
//   affine_maps    P and b of every run of rows, on the whole chip: P' = P - s x (x'P), b' = b + s (k - x.b) x;
//   affine_starts  one wavefront per solver: the private vector before every run and after the last, a d x d product per run;
//   affine_steps   every run's steps one row after the other from its own start, on the whole chip: the new alphas.
// Only the second kernel is a chain, of some 600 cycles per run; blocks of 64 rows solved by their inverse took 2.2e3 each (see
// sdca_dense_squared).  The first is bound by its multiply-adds (2 d^2 per row in double, of rank one updates that depend on
// each other), the third by the dozen dependent instructions of a row.  500000 x 28, 16 solvers, a pass in runs of 256 rows:
// 79 + 33 + 47 us (450 in blocks); fifty rounds 28.2 -> 9.8 ms.
// Precision: all is in double but what is stored (alpha, the solver's update, the rows and their state).  The update is the
// vector after the last run, not a sum over the runs: an error in the vector shrinks with every row after it, one in a run's
// share would stay.  It is not formed from the stored alphas, so that whatever either is off by parts w from the sum of the
// alphas' rows: with P and the dot products in float (57 + 50 + 38 us in runs of 128 rows, 9.9 ms) by 6e-7 of w after one
// round, here by 4e-8, the rounding of what is stored (blocks: 7e-8).
// Errors against 64 bits over those of blocks solved by their inverse, updates and alpha, geometric means of eight jobs each of
// 3500 to 40000 rows, three rounds (with P and the dot products in float up to 1.33 and 1.06, for lambda n from 10 on):
//   columns  lambda n: 0.1        1            10           50           100
//    2             0.21 0.15    0.24 0.18    0.57 0.30    0.48 0.37    0.72 0.41
//    8             0.20 0.16    0.38 0.17    0.45 0.23    0.56 0.30    0.60 0.33
//   17             0.27 0.17    0.35 0.18    0.42 0.22    0.53 0.27    0.56 0.30
//   24             0.33 0.18    0.34 0.19    0.47 0.24    0.57 0.27    0.59 0.31
//   28             0.28 0.18    0.35 0.19    0.48 0.23    0.55 0.28    0.62 0.31
//   32             0.29 0.19    0.35 0.20    0.45 0.25    0.53 0.28    0.64 0.31
#pragma once
#include <hip/hip_runtime.h>
#include "device_types.hpp"
#include "mem.hpp"
#include "sdca_dense.hpp"

namespace chicle {

typedef float float2_v __attribute__((ext_vector_type(2)));

constexpr int AFFINE_MAX_D = 32;
constexpr int AFFINE_GROUP = 16;                 // affine_steps: lanes per run, two columns each, and rows in flight per run
constexpr int AFFINE_UNITS = 64 / AFFINE_GROUP;  // ... and runs per wavefront
// Wavefronts per workgroup, each on its own: one per SIMD (workgroups of one wavefront: affine_maps with P in float 70 us for 55).
constexpr int AFFINE_WAVES = 4;
// A run's place is the first of the tiles its rows have (their addresses stay with their tiles), in doubles: P - 1 at
// [m / 2][k][m % 2] for row k and column m, then vectors of 32: b, the start; then words that nobody reads.
constexpr int AFFINE_B = AFFINE_MAX_D * AFFINE_MAX_D, AFFINE_START = AFFINE_B + AFFINE_MAX_D, AFFINE_SINK = AFFINE_START + AFFINE_MAX_D;
static_assert(2 * (AFFINE_SINK + 64) <= BATCH * BATCH, "before the rows' addresses");
static_assert(DENSE_TILE_FLOATS % 4 == 0, "16-byte aligned places");
typedef double double2_v __attribute__((ext_vector_type(2)));

// Orders the LDS accesses of one wavefront (they are performed in order; the compiler has to keep them so).
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The value of another lane, by a data-parallel-primitive move.
template <int CTRL>
__device__ __forceinline__ double of_lane(double v)
{
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, true),
                            __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, true));
}
constexpr int DPP_LANE_OF_16 = 0x150;            // + r: lane r of each 16
// Sum over 16 lanes, in all of them: lanes xor 1, xor 2, then mirrored halves and rows.
__device__ __forceinline__ double sum16(double v)
{
    v += of_lane<0xB1>(v);
    v += of_lane<0x4E>(v);
    v += of_lane<0x141>(v);
    v += of_lane<0x140>(v);
    return v;
}
// ... over 32 lanes: the other 16 by a swap.
__device__ __forceinline__ double sum32(double v)
{
    v = sum16(v);
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false), h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}
// What a row's step is scaled with: c / (c + q), in double (in float it would err by as much as the rounded result).
__device__ __forceinline__ double affine_scale(float q, float c) { return (double)c / ((double)c + (double)q); }

// Grid: (groups of runs, solver), LANES lanes per run.  A lane holds one column of its run's P in registers; rows come through
// LDS, where a run's lanes read the same words.  The lookups (order entry -> chunk -> row) are four groups of LANES rows deep,
// so that each group's loads have a group's arithmetic to return in.  DK: columns, rounded up to four.
// SPARE: a run has more lanes than a row has columns, and the one after the last holds b as a column of its own (a row without
// a column there leaves P's as it is), so that no sum over lanes stands in the chain from row to row.
// ALONE: the wavefronts are no more than the SIMDs, so that nothing hides a wavefront's reads of a row's words but its own
// arithmetic on the row before (rows of more than 24 columns: the shorter ones' words are here soon enough, see launch_affine).
template <int DK, int LANES, bool SPARE, bool ALONE>
__global__ __launch_bounds__(64 * AFFINE_WAVES) void affine_maps(
    const ChunkDev *__restrict__ chunks, const SolverDev *__restrict__ solvers, const int32_t *__restrict__ row_chunk,
    const int32_t *__restrict__ chunk_first, const int32_t *__restrict__ perm, float *tiles, int d, int run, float c, float inv_c, int *err)
{
    constexpr int Q = DK / 4, LDR = AFFINE_MAX_D + 2, LDU = LANES * LDR + 2, UNITS = 64 / LANES;      // (runs and rows on other banks)
    __shared__ __align__(16) double sh_x[AFFINE_WAVES][UNITS * LDU];
    __shared__ __align__(16) double sh_sk[AFFINE_WAVES][UNITS][LANES][2];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), first = ((int)blockIdx.x * AFFINE_WAVES + wv) * UNITS;
    double *s_x = sh_x[wv];
    auto &s_sk = sh_sk[wv];
    const SolverDev S = solvers[blockIdx.y];
    const int units = (S.n_rows + run - 1) / run;
    if (first >= units) return;
    const int lane = threadIdx.x & 63, m = lane & (LANES - 1), un = lane / LANES, unit = first + un;
    const int t0 = unit * run + m, groups = run / LANES, tile_rows = (S.n_rows + BATCH - 1) / BATCH * BATCH;
    const int my_rows = unit < units ? S.n_rows : 0;
    float *tile0 = tiles + (int64_t)S.tile_begin * DENSE_TILE_FLOATS;
    double *out = reinterpret_cast<double *>(tile0 + (int64_t)min(unit, units - 1) * (run / BATCH) * DENSE_TILE_FLOATS);
    // No load or store stands behind a condition (the compiler would wait for all that are in flight), and what a load
    // returns is first looked at a group later: rows that do not exist look up a row that does.
    struct Order { int lr; bool ok; };
    struct Chunk { int ci, lr; bool ok; };
    struct Place { const float *val; RowState *st; int first, lr; bool ok; };
    bool refused = false;
    auto order = [&](int g) __attribute__((always_inline)) {
        const int t = t0 + g * LANES;
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
    for (int i = lane; i < UNITS * LDU; i += 64) s_x[i] = 0.0;       // (columns past the row's end stay zero)
    fetch(place_of(chunk_of(order(0))));
    Place next = place_of(chunk_of(order(1)));
    Chunk far = chunk_of(order(2));
    Order farther = order(3);
    const bool holds_b = SPARE && m == d;
    double P[DK], b = 0.0;                       // P[k][m], b[m] (SPARE: b[k] in P[k] of lane d)
#pragma unroll
    for (int k = 0; k < DK; ++k) P[k] = k == m && !holds_b ? 1.0 : 0.0;
    double *mine = s_x + un * LDU;
    wave_lds_fence();
    for (int g = 0; g < groups; ++g) {
        {
            const bool live = row_ok & takes_steps(st_in.z);
#pragma unroll
            for (int q = 0; q < Q; ++q)
#pragma unroll
                for (int e = 0; e < 4; e += 2)
                    *reinterpret_cast<double2_v *>(mine + m * LDR + 4 * q + e) = double2_v{live ? x_in[q][e] : 0.f, live ? x_in[q][e + 1] : 0.f};
            const double s = affine_scale(st_in.z, c) * (double)inv_c, k = (double)st_in.w - (double)st_in.y;
            *reinterpret_cast<double2_v *>(&s_sk[un][m][0]) = live ? double2_v{s, k} : double2_v{0.0, 0.0};
            const int t = t0 + g * LANES;
            // (a tile's rows past the end too: they take no step)
            float *tile = unit * run + g * LANES < tile_rows ? tile0 + (int64_t)(t / BATCH) * DENSE_TILE_FLOATS + BATCH * BATCH + 4 * (t % BATCH)
                                                                    : reinterpret_cast<float *>(out + AFFINE_SINK + 2 * m);
            const DenseRow kept = {row.x, live ? row.st : nullptr};
            *(CHICLE_GLOBAL float4_v *)tile = __builtin_bit_cast(float4_v, kept);
        }
        fetch(next);
        next = place_of(far);
        far = chunk_of(farther);
        farther = order(g + 4);
        wave_lds_fence();
        struct Words { double2_v x[DK / 2], sk; double xm; };
        auto read = [&](int r) __attribute__((always_inline)) {
            Words w;
#pragma unroll
            for (int q = 0; q < DK / 2; ++q) w.x[q] = *reinterpret_cast<const double2_v *>(mine + r * LDR + 2 * q);
            w.xm = SPARE ? 0.0 : mine[r * LDR + m];
            w.sk = *reinterpret_cast<const double2_v *>(&s_sk[un][r][0]);
            return w;
        };
        auto add_row = [&](const Words &w) __attribute__((always_inline)) {
            double t[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int k = 0; k < DK; ++k) t[k & 3] = fma(w.x[k >> 1][k & 1], P[k], t[k & 3]);
            const double n = w.sk.x * ((holds_b ? w.sk.y : 0.0) - ((t[0] + t[1]) + (t[2] + t[3])));
            if (!SPARE) b = fma(w.xm, w.sk.x * (w.sk.y - sum32(w.xm * b)), b);
#pragma unroll
            for (int k = 0; k < DK; ++k) P[k] = fma(w.x[k >> 1][k & 1], n, P[k]);
        };
        // One wavefront per SIMD reads a row's words during the arithmetic of the row before it (500000 x 28 in runs of 256 rows, 977
        // wavefronts: 86 us without, 79 with); two of them hide each other's
        // reads, and a second set of words would take the registers that the second one needs.
        if (LANES == 16 || ALONE) {
            Words even = read(0);
            for (int r = 0; r < LANES; r += 2) {
                const Words odd = read(r + 1);
                __builtin_amdgcn_sched_barrier(0);   // (or all reads are put first, and waited for)
                add_row(even);
                __builtin_amdgcn_sched_barrier(0);
                even = read(min(r + 2, LANES - 1));
                __builtin_amdgcn_sched_barrier(0);
                add_row(odd);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            for (int r = 0; r < LANES; ++r) add_row(read(r));
        }
        wave_lds_fence();
    }
    if (refused) atomicOr(err, ERR_PERM_RANGE);
    if (unit >= units) return;
#pragma unroll
    for (int k = 0; k < DK; ++k) {
        *(CHICLE_GLOBAL double *)(out + ((m >> 1) * AFFINE_MAX_D + k) * 2 + (m & 1)) = holds_b ? 0.0 : k == m ? P[k] - 1.0 : P[k];
        if (holds_b) *(CHICLE_GLOBAL double *)(out + AFFINE_B + k) = P[k];
    }
    if (!SPARE) *(CHICLE_GLOBAL double *)(out + AFFINE_B + m) = b;
}

// Grid: one wavefront per solver.  Lane: row of P, and half of the columns (four Q of them).  The maps of SETS runs are in
// flight.
template <int Q>
__global__ __launch_bounds__(64) void affine_starts(const SolverDev *__restrict__ solvers, float *tiles, float *u_all,
                                                    int64_t ld_v, int d, int run, RoundScalars sc)
{
    constexpr int SETS = 6;
    __shared__ __align__(16) double s_v[AFFINE_MAX_D];
    const SolverDev S = solvers[blockIdx.x];
    stamp_solver(sc, 0);
    const int units = (S.n_rows + run - 1) / run;
    const int lane = threadIdx.x, i = lane & 31, h = lane >> 5;
    const int64_t stride = (int64_t)(run / BATCH) * DENSE_TILE_FLOATS;
    float *place = tiles + (int64_t)S.tile_begin * DENSE_TILE_FLOATS;
    auto place_of = [&](int at) __attribute__((always_inline)) { return reinterpret_cast<double *>(place + min(at, units - 1) * stride); };
    const bool has = i < d;
    double v = has ? (double)u_all[(int64_t)blockIdx.x * ld_v + i] : 0.0;
    double2_v P[SETS][2 * Q];
    double b[SETS];
    auto load = [&](int s, int at) __attribute__((always_inline)) {
        const double *p = place_of(at);
#pragma unroll
        for (int e = 0; e < 2 * Q; ++e) P[s][e] = *(const CHICLE_GLOBAL double2_v *)(p + ((h * 2 * Q + e) * AFFINE_MAX_D + i) * 2);
        b[s] = *(const CHICLE_GLOBAL double *)(p + AFFINE_B + i);
    };
    if (units > 0) {
        s_v[i] = v;
        wave_lds_fence();
#pragma unroll
        for (int s = 0; s < SETS; ++s) load(s, s);
        for (int u0 = 0; u0 < units; u0 += SETS) {
#pragma unroll
            for (int s = 0; s < SETS; ++s) {
                const int at = u0 + s;
                if (at >= units) break;          // (so that the solver's clock ends with its last run)
                *(CHICLE_GLOBAL double *)(place_of(at) + AFFINE_START + i) = v;
                double part[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int e = 0; e < 2 * Q; ++e) {
                    const double2_v w = *reinterpret_cast<const double2_v *>(s_v + 2 * (h * 2 * Q + e));
                    part[2 * (e & 1)] = fma(P[s][e][0], w[0], part[2 * (e & 1)]);
                    part[2 * (e & 1) + 1] = fma(P[s][e][1], w[1], part[2 * (e & 1) + 1]);
                }
                const double sum = (part[0] + part[1]) + (part[2] + part[3]);
                const unsigned lo = (unsigned)__double2loint(sum), hi = (unsigned)__double2hiint(sum);
                const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false), u = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
                const double dv = b[s] + (__hiloint2double((int)u[0], (int)l[0]) + __hiloint2double((int)u[1], (int)l[1]));
                v += has ? dv : 0.0;             // (the places' rows past the last column are not written)
                wave_lds_fence();
                s_v[i] = v;
                wave_lds_fence();
                load(s, at + SETS);
            }
        }
    }
    if (lane < d) u_all[(int64_t)blockIdx.x * ld_v + i] = (float)v;
    stamp_solver(sc, 1);
}

// Grid: (groups of 16 runs, solver), four runs per wavefront, two columns per lane.  The next 16 rows are loaded during the
// steps of these.
__global__ __launch_bounds__(64 * AFFINE_WAVES) void affine_steps(const ChunkDev *__restrict__ chunks, const SolverDev *__restrict__ solvers,
                                                   float *tiles, int run, int ld, RoundScalars sc)
{
    constexpr int GROUP = AFFINE_GROUP;
    const SolverDev S = solvers[blockIdx.y];
    const int units = (S.n_rows + run - 1) / run;
    const int first = ((int)blockIdx.x * AFFINE_WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * AFFINE_UNITS;
    if (first >= units) return;
    const int lane = threadIdx.x & 63, m = lane & (GROUP - 1), unit = first + lane / GROUP;
    const int groups = run / GROUP, tiles_end = (S.n_rows + BATCH - 1) / BATCH;
    const bool has = 2 * m < ld;
    const int xo = has ? 2 * m : 0;
    float *tile0 = tiles + (int64_t)S.tile_begin * DENSE_TILE_FLOATS;
    double *place = reinterpret_cast<double *>(tile0 + (int64_t)min(unit, units - 1) * (run / BATCH) * DENSE_TILE_FLOATS);
    auto rows_of = [&](int g) __attribute__((always_inline)) {       // of the group; past the end: any
        const int t = unit * run + g * GROUP;
        return reinterpret_cast<const DenseRow *>(tile0 + (int64_t)min(t / BATCH, tiles_end - 1) * DENSE_TILE_FLOATS + BATCH * BATCH) + t % BATCH;
    };
    const RowState *any = chunks[0].st;
    const float *xp[GROUP];
    RowState *rec_next, *rec;
    float2_v X[2][GROUP];
    float4_v st;
    auto load_rows = [&](int g) __attribute__((always_inline)) {
        const DenseRow *r = rows_of(g);
#pragma unroll
        for (int j = 0; j < GROUP; ++j) xp[j] = r[j].x;
        rec_next = r[m].st;
    };
    auto load_x = [&](float2_v (&to)[GROUP]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < GROUP; ++j) to[j] = *(const CHICLE_GLOBAL float2_v *)(xp[j] + xo);
        st = gld_state(rec_next != nullptr ? rec_next : any);
        rec = rec_next;
    };
    const double2_v start = *(const CHICLE_GLOBAL double2_v *)(place + AFFINE_START + 2 * m);
    double q0 = has ? start.x : 0.0, q1 = has ? start.y : 0.0;
    load_rows(0);
    load_x(X[0]);
    load_rows(1);
    auto group = [&](int g, float2_v (&now)[GROUP], float2_v (&then)[GROUP]) __attribute__((always_inline)) {
        // (groups past the solver's tiles read its last tile's rows: they take no step)
        const bool live = (rec != nullptr) & (unit * run + g * GROUP < tiles_end * BATCH);
        const double s0 = affine_scale(st.z, sc.c), alpha = (double)st.y;
        const double scale = live ? s0 : 0.0, kk = live ? (double)st.w - alpha : 0.0;
        float *alpha_out = live ? &rec->alpha : reinterpret_cast<float *>(place + AFFINE_SINK + m);
        load_x(then);
        load_rows(g + 2);
        double delta = 0.0;
        auto step = [&](auto J) __attribute__((always_inline)) {
            constexpr int j = decltype(J)::value;
            const double s = of_lane<DPP_LANE_OF_16 + j>(scale), k = of_lane<DPP_LANE_OF_16 + j>(kk);
            const bool on = has && s != 0.0;     // (a row that takes no step may hold what is no number)
            const double x0 = (double)(on ? now[j].x : 0.f), x1 = (double)(on ? now[j].y : 0.f);
            const double dl = s * (k - sum16(fma(x0, q0, x1 * q1))), cf = dl * (double)sc.inv_c;
            q0 = fma(cf, x0, q0);
            q1 = fma(cf, x1, q1);
            delta = m == j ? dl : delta;
        };
#define CHICLE_STEP(j) step(std::integral_constant<int, j>())
        CHICLE_STEP(0); CHICLE_STEP(1); CHICLE_STEP(2); CHICLE_STEP(3); CHICLE_STEP(4); CHICLE_STEP(5); CHICLE_STEP(6); CHICLE_STEP(7);
        CHICLE_STEP(8); CHICLE_STEP(9); CHICLE_STEP(10); CHICLE_STEP(11); CHICLE_STEP(12); CHICLE_STEP(13); CHICLE_STEP(14); CHICLE_STEP(15);
#undef CHICLE_STEP
        gst(alpha_out, (float)(alpha + delta));
    };
    for (int g = 0; g < groups; g += 2) {
        group(g, X[0], X[1]);
        group(g + 1, X[1], X[0]);
    }
}

}  // namespace chicle
