// Local solver, one coordinate step at a time (paper Section 2.2: L = 1, H = all local samples).
//
// One workgroup per solver.  Every step is: row dot product against the solver's private vector
// (workgroup reduction), closed-form dual step, alpha update inside the chunk, scatter of the row
// into the private vector.  With v_k = w + sigma * Delta w_k the CoCoA subproblem step is a plain
// coordinate step against v_k:
//     hinge   : a' = clip(a + c (1 - y z) / q, 0, 1),  c = lambda n / sigma,  z = x_i . v_k
//     squared : delta = (y - z - a) / (1 + q / c)
//     v_k += (delta s / c) x_i,  s = y (hinge) or 1 (squared).
// The private vector is stored as its difference u_k = v_k - w (zero when the pass starts).  The part
// of a step that depends on w alone is the per-row residual rw that the gap pass left in the chunk
// (hinge: 1 - y x_i.w, squared: y - x_i.w, formed in double from the double-precision w), so a step
// needs only x_i . u_k on top of it.  Keeping the small quantities apart from the O(1) ones keeps fp32
// rounding relative to the update: near convergence y - z - a is a difference of nearly equal numbers.
#pragma once
#include <hip/hip_runtime.h>
#include "device_types.hpp"
#include "mem.hpp"

namespace chicle {

// Logistic loss: a' = 1 / (1 + exp(-s)) with s the root of f(s) = m - s - r (a'(s) - a), where m = -y z and r = q / c.
// Returns the root to within about a hundredth (the series of logistic_block take it from there), one row per lane.  f
// decreases strictly (slope in [-1 - r/4, -1]) and, a' lying in (0, 1), its root lies in [m - r (1 - a), m + r a].
// Newton steps inside that bracket from the previous a's own s, where the root is late in a run; a bisection step
// whenever Newton would leave the bracket or fails to halve the last step (r can be in the hundreds, where plain
// Newton cycles between the two flat ends of the sigmoid).
__device__ __forceinline__ float logistic_root(float m, float r, float a)
{
    float lo = m - r * (1.0f - a), hi = m + r * a;
    const float s0 = a > 1e-6f && a < 1.0f - 1e-6f ? __logf(a * __builtin_amdgcn_rcpf(1.0f - a)) : m + r * (a - 0.5f);
    float s = fminf(fmaxf(s0, lo), hi), dx = hi - lo;
    for (int it = 0; it < 48; ++it) {
        const float e = __expf(-fabsf(s));
        const float t = __builtin_amdgcn_rcpf(1.0f + e);
        const float f = (m - s) - r * ((s >= 0.f ? t : e * t) - a);
        if (f > 0.f) lo = s; else hi = s;
        float step = f * __builtin_amdgcn_rcpf(fmaf(r, e * t * t, 1.0f)), to = s + step;
        if (!(to >= lo && to <= hi) || fabsf(2.0f * step) > fabsf(dx)) { to = 0.5f * (lo + hi); step = to - s; }
        s = to;
        dx = step;
        if (fabsf(dx) <= 1e-2f) break;
    }
    return s;
}

// One dual step of the logistic loss computed by a whole wavefront from uniform arguments (see
// logistic_root for the equation).  f decreases strictly, so the 64 lanes evaluate it at 64 evenly spaced
// points of the bracket and the first lane with f <= 0 narrows the bracket 63-fold; when the bracket is so
// narrow that a chord of f misses the root by less than fp32 resolution (|f''| <= 0.0963 r, |f'| >= 1:
// error <= 0.012 h^2 r), the root and a' are read off the chord.  [lo, lo + w] is a bracket of the root:
// the general one, [m - r (1 - a), m + r a], costs two evaluations for r of order one and four for r in
// the hundreds; no derivative, no iteration that could cycle.
__device__ __forceinline__ float logistic_step_wave(float m, float r, float a, float lo, float w, int lane)
{
    const float frac = (float)lane * (1.0f / 63.0f);
    float s = 0.f, ap = 0.f, f = 0.f;
    int k = 1;
    for (int it = 0; it < 8; ++it) {
        s = fmaf(frac, w, lo);
        const float e = __expf(-fabsf(s));
        const float t = __builtin_amdgcn_rcpf(1.0f + e);
        ap = s >= 0.f ? t : e * t;
        f = (m - s) - r * (ap - a);
        const unsigned long long pos = __ballot(f > 0.f);
        k = ~pos ? __builtin_ctzll(~pos) : 64;
        k = min(max(k, 1), 63);
        const float h = w * (1.0f / 63.0f);
        if (h * h * r <= 4e-6f || h <= 1e-7f * (1.0f + fabsf(lo))) break;
        lo = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(s), k - 1));
        w = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(s), k)) - lo;
    }
    const float f0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(f), k - 1));
    const float f1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(f), k));
    const float a0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ap), k - 1));
    const float a1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ap), k));
    const float den = f0 - f1;
    const float th = den > 0.f ? fminf(fmaxf(f0 * __builtin_amdgcn_rcpf(den), 0.f), 1.f) : 0.5f;
    return fmaf(th, a1 - a0, a0) - a;
}

// The same equation followed through a block.  A lane keeps its row's m, and s, the root for an earlier m, with what the
// sigmoid does there: p = a'(s) and its derivatives, from which the step for the current m follows as a series in
//     d = x g,   x = (m - s) - r (p - a),   g = 1 / (1 + r p').
// The root is s + ds with ds = d + c2 d^2 + c3 d^3 + c4 d^4 + ... (the inverse of f's own series: c2 = -A, c3 = 2 A^2 - B,
// c4 = -(5 A^3 - 5 A B + C) with A, B, C = r g times p'' / 2, p''' / 6, p'''' / 24, bounded for every r because
// r p' g < 1), and a' follows by inserting ds into the sigmoid's series: a' - a = q0 + q1 d + q2 d^2 + q3 d^3 + q4 d^4.
// Nothing of this but d depends on the current m: what a step waits for is one multiply-add for d, three for the
// polynomial and the lane read, where a search of the row's bracket evaluates the sigmoid at least once per step.
struct LogisticTrack {
    float s, g, h, c2, c3, c4, q0, q1, q2, q3, q4;      // h: d = m g + h
    __device__ __forceinline__ void at(float root, float a, float r, bool live)
    {
        s = root;
        const float e = __expf(-fabsf(s));
        const float t = __builtin_amdgcn_rcpf(1.0f + e);
        const float p = s >= 0.f ? t : e * t;
        const float p1 = e * t * t;                                        // p' = p (1 - p) without cancellation
        const float k = s >= 0.f ? (e - 1.0f) * t : (1.0f - e) * t;        // 1 - 2 p
        const float p2 = 0.5f * p1 * k;
        const float p3 = p1 * fmaf(-6.0f, p1, 1.0f) * (1.0f / 6.0f);
        const float p4 = p1 * k * fmaf(-12.0f, p1, 1.0f) * (1.0f / 24.0f);
        g = live ? __builtin_amdgcn_rcpf(fmaf(r, p1, 1.0f)) : 0.f;         // a row that takes no step: d = 0, a' - a = 0
        const float rg = r * g, A = rg * p2, B = rg * p3;
        c2 = -A;
        c3 = fmaf(2.0f * A, A, -B);
        c4 = -fmaf(5.0f * A, fmaf(A, A, -B), rg * p4);
        q0 = live ? p - a : 0.f;
        h = -fmaf(r, q0, s) * g;
        q1 = p1;
        q2 = fmaf(p1, c2, p2);
        q3 = fmaf(p1, c3, fmaf(2.0f * p2, c2, p3));
        q4 = fmaf(p1, c4, fmaf(p2, fmaf(c2, c2, 2.0f * c3), fmaf(3.0f * p3, c2, p4)));
    }
};
// Largest |d| for which the series is used: its error in a' there is at most 1.7e-8 (r from 1e-3 to 3e3, all s; half a
// unit in the last place of a' is 3e-8).
constexpr float LOGISTIC_SERIES = 0.07f;

// Rows further than this from where their series were expanded have them renewed before their group's steps.
constexpr float LOGISTIC_NEAR = 0.05f;
constexpr int LOGISTIC_CALM = 16, LOGISTIC_ROUGH = 4;     // steps taken before their rows' |d| are looked at

// The BR steps of a block with the logistic loss: lane i owns row i; m = -y z against the private vector at the start
// of the block, root: the root for it, r = q / c (0: a row that takes no step); coef4(jq) returns the lane's T of steps
// 4 jq .. 4 jq + 3 (zero from the lane's own step on); CROSS: cross4(jq) returns their influence on the block after this one,
// and x takes up what the steps add there.  GROUP steps at a
// time: they are taken from the series, and then the rows' |d| are looked at; from the first one that was too large on, the
// group's steps are taken again one by one, with the expansions renewed where that is needed, or the row's bracket searched.
// Returns whether that happened in `rough`.
// Bound by the chain of a step (series, lane read, multiply-add: some 45 cycles) and by what a group costs around its steps (two
// comparisons with the scalar unit's answer, branches: 200 cycles).  Expansions renewed before every four steps, some 300 cycles
// whether rows had moved or not: 300000 rows of 40 entries, 32 solvers, five rounds 6.47 ms on a run that continues and 10.8 from
// alpha = 0; in groups of 16 3.68 and 12.5, of 8 4.02 and 10.9, of 4 4.65 and 9.4, and with 16 where nothing moves and 4 where it
// does 3.80 and 9.4.  Three rounds of 20011 x 1001, eight solvers: 1.44 ms before, 1.08 so.  The updates' errors against 64 bits
// are the same on average (160 jobs of dense and ragged rows, geometric mean 1.00, alpha 1.01); the largest of the dense jobs went from
// 7.9e-8 to 9.3e-8 of alpha and from 1.10e-7 to 1.22e-7 of w.
template <int BR, int GROUP, bool CROSS, typename COEF, typename ALSO>
__device__ __forceinline__ float logistic_steps(float m, float a, float r, float root, int lane, COEF coef4, ALSO cross4, float &x_sum, bool &rough)
{
    static_assert(BR % GROUP == 0 && GROUP % 4 == 0, "whole groups of coefficients");
#define CHICLE_LANE(x, j) __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), j))
    const bool live = r > 0.f;
    LogisticTrack k;
    // the row's m is the m at the start of the block and `moved`, the sum of the steps' influence, apart: added to m one by
    // one, each of them would round it
    float mine = 0.f, moved = 0.f, h = 0.f;          // d = moved g + h
    int from = 0;                                    // rows before this one have their steps in `mine`
    k.s = root;
    float d = 0.f;
    rough = false;
    auto renew = [&]() __attribute__((always_inline)) {
        const float dc = fminf(fmaxf(d, -0.5f), 0.5f);
        const float ds = fabsf(d) <= LOGISTIC_SERIES ? d * fmaf(d, fmaf(d, fmaf(d, k.c4, k.c3), k.c2), 1.0f) : dc;
        k.at(k.s + ds, a, r, live);
        h = fmaf(m, k.g, k.h);
        d = fmaf(moved, k.g, h);
    };
    auto step = [&]() __attribute__((always_inline)) {
        const float d2 = d * d;
        return fmaf(d, fmaf(d2, fmaf(d, k.q4, k.q3), fmaf(d, k.q2, k.q1)), k.q0);
    };
    // (a row's m does not move any more after its own step, so that its step can be read from its series later on)
    auto keep = [&](int end) __attribute__((always_inline)) {
        const float x = step();
        mine = lane >= from && lane < end ? x : mine;
        from = end;
    };
    // the group's rows that are further than `most` from their expansions (or no number)
    auto beyond = [&](float most, int j0) __attribute__((always_inline)) {
        return (unsigned)(__ballot(!(fabsf(d) <= most)) >> j0) & ((1u << GROUP) - 1u);
    };
    k.at(root, a, r, live);
    d = h = fmaf(m, k.g, k.h);
    float4_v next[GROUP / 4], next_x[GROUP / 4];
    auto request = [&](int jq) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < GROUP / 4; ++q) next[q] = coef4(jq + q);
        if (CROSS)
#pragma unroll
            for (int q = 0; q < GROUP / 4; ++q) next_x[q] = cross4(jq + q);
    };
    request(0);
#pragma unroll 1
    for (int j0 = 0; j0 < BR; j0 += GROUP) {
        float4_v T[GROUP / 4], X[GROUP / 4];
#pragma unroll
        for (int q = 0; q < GROUP / 4; ++q) { T[q] = next[q]; if (CROSS) X[q] = next_x[q]; }
        request(min(j0 + GROUP, BR - GROUP) / 4);
        if (beyond(LOGISTIC_NEAR, j0)) {
            keep(j0);
            renew();
        }
        const float moved_before = moved, x_before = x_sum;
        float dj[GROUP];
#pragma unroll
        for (int e = 0; e < GROUP; ++e) {
            const float own = step();
            if (CROSS && e > 0) {                    // (in one of the slots that the lane read waits for)
                __builtin_amdgcn_sched_barrier(0);
                x_sum = fmaf(dj[e - 1], X[(e - 1) >> 2][(e - 1) & 3], x_sum);
                asm volatile("" : "+v"(x_sum));
                __builtin_amdgcn_sched_barrier(0);
            }
            dj[e] = CHICLE_LANE(own, j0 + e);
            moved = fmaf(dj[e], T[e >> 2][e & 3], moved);
            d = fmaf(moved, k.g, h);
        }
        if (CROSS) x_sum = fmaf(dj[GROUP - 1], X[GROUP / 4 - 1][3], x_sum);
        const unsigned out = beyond(LOGISTIC_SERIES, j0);
        if (out) {                                   // the first such row's step and those after it again, one by one
            const int first = __builtin_ctz(out);
            rough = true;
            moved = moved_before;
#pragma unroll
            for (int e = 0; e < GROUP - 1; ++e)
                if (e < first) moved = fmaf(dj[e], T[e >> 2][e & 3], moved);
            d = fmaf(moved, k.g, h);
            keep(j0 + first);
            float4_v Tj = coef4((j0 + first) >> 2);
#pragma unroll 1
            for (int j = j0 + first; j < j0 + GROUP; ++j) {
                const float Te = (j & 2) ? ((j & 1) ? Tj[3] : Tj[2]) : ((j & 1) ? Tj[1] : Tj[0]);
                Tj = coef4(min(j + 1, BR - 1) >> 2);
                for (int it = 0; it < 3 && fabsf(CHICLE_LANE(d, j)) > LOGISTIC_SERIES; ++it) renew();
                float x = CHICLE_LANE(step(), j);
                if (fabsf(CHICLE_LANE(d, j)) > LOGISTIC_SERIES) {
                    // f falls at least as fast as s grows: the root lies between s and s + f(s), f(s) = d / g
                    const float sj = CHICLE_LANE(k.s, j), xj = CHICLE_LANE(d, j) / CHICLE_LANE(k.g, j);
                    x = logistic_step_wave(CHICLE_LANE(m + moved, j), CHICLE_LANE(r, j), CHICLE_LANE(a, j), sj + fminf(xj, 0.f), fabsf(xj), lane);
                }
                moved = fmaf(x, Te, moved);
                d = fmaf(moved, k.g, h);
                mine = lane == j ? x : mine;
            }
            from = j0 + GROUP;
            if (CROSS) {
                x_sum = x_before;
#pragma unroll
                for (int e = 0; e < GROUP; ++e) x_sum = fmaf(e >= first ? CHICLE_LANE(mine, j0 + e) : dj[e], X[e >> 2][e & 3], x_sum);
            }
        }
    }
    keep(BR);
#undef CHICLE_LANE
    return mine;
}

// rough: whether the solver's block before had rows that moved out of their series' range (first block: true), and then
// whether this one has.
template <int BR, bool CROSS, typename COEF, typename ALSO>
__device__ __forceinline__ float logistic_block(float m, float a, float r, float root, int lane, COEF coef4, ALSO cross4, float &x_sum, bool &rough)
{
    if (rough) return logistic_steps<BR, LOGISTIC_ROUGH, CROSS>(m, a, r, root, lane, coef4, cross4, x_sum, rough);
    return logistic_steps<BR, LOGISTIC_CALM, CROSS>(m, a, r, root, lane, coef4, cross4, x_sum, rough);
}

// rw: residual at w (see above; logistic: -y x_i.w); xu = x_i . u_k.  The arguments are the same in every
// lane of a wavefront (the logistic step is computed by the wavefront as a whole).
template <int LOSS>
__device__ __forceinline__ float dual_step(float a, float y, float rw, float xu, float q, float c)
{
    if (LOSS == 0) {
        float an = a + c * (rw - y * xu) / q;
        an = fminf(fmaxf(an, 0.0f), 1.0f);
        return an - a;
    }
    if (LOSS == 2) {
        // (taken from the first lane so that the compiler knows them to be uniform)
        const float m = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(rw - y * xu)));
        const float r = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(q / c)));
        const float a1 = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(a)));
        return logistic_step_wave(m, r, a1, m - r * (1.0f - a1), r, threadIdx.x & 63);
    }
    return (rw - xu - a) / (1.0f + q / c);
}

__device__ __forceinline__ float wave_sum(float x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

// Sum over the workgroup; every thread gets the result.  red: BLOCK/64 floats of LDS.
template <int BLOCK>
__device__ __forceinline__ float block_sum(float x, float *red)
{
    x = wave_sum(x);
    if (BLOCK == 64) return x;
    const int wave = threadIdx.x >> 6;
    __syncthreads();                       // red may still be read from the previous use
    if ((threadIdx.x & 63) == 0) red[wave] = x;
    __syncthreads();
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < BLOCK / 64; ++i) s += red[i];
    return s;
}

// Largest j in [0, n) with prefix[j] <= lr (prefix ascending, prefix[0] = 0).
__device__ __forceinline__ int find_chunk(const int *prefix, int n, int lr)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (prefix[mid] <= lr) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// What a step needs to know about its row; len = 0 marks a row to skip.
struct RowMeta {
    const int32_t *col;
    const float *val;
    RowState *st;
    int len;
    float y, alpha, q, rw;
};

// Sparse rows of any length.  The step itself is gather - reduce - step - scatter; everything that does
// not depend on the private vector is fetched ahead by a small software pipeline so that a step costs
// one trip to memory (the gather) instead of five dependent ones:
//     step t issues   the order entry of row t+4, the chunk lookup and state loads of row t+3,
//     publishes       the resolved row t+2 in LDS (thread 0 does these three),
//     loads           the first EPT * BLOCK entries of row t+1 into registers (all threads),
//     computes        row t.
// The scatter uses atomic adds that are not waited for: accesses of one compute unit to one address
// are served in order, and the gathers read past the vector cache (ld_l2).
// Dynamic LDS: max_list chunk descriptors, then max_list local-row prefixes.
template <int LOSS, int BLOCK, int EPT>
__global__ __launch_bounds__(BLOCK) void sdca_rowwise_csr(
    const ChunkDev *__restrict__ chunks, const SolverDev *__restrict__ solvers,
    const int32_t *__restrict__ solver_chunks, const int32_t *__restrict__ solver_prefix,
    const int32_t *__restrict__ perm, float *u_all, int64_t ld_v, int max_list, RoundScalars sc, int *err,
    const int64_t *__restrict__ u_off)
{
    // u_off != nullptr: private vectors are stored compactly, solver k's at u_all + u_off[k], and every
    // entry's index into it is found in the array behind the chunk's column ids
    extern __shared__ __align__(16) unsigned char rw_smem[];
    __shared__ float red[BLOCK / 64];
    __shared__ RowMeta ring[4];
    const SolverDev S = solvers[blockIdx.x];
    ChunkDev *l_desc = reinterpret_cast<ChunkDev *>(rw_smem);
    int *l_prefix = reinterpret_cast<int *>(l_desc + max_list);
    const int tid = threadIdx.x;
    stamp_solver(sc, 0);
    for (int i = tid; i < S.n_chunks; i += BLOCK) {
        l_desc[i] = chunks[solver_chunks[S.list_begin + i]];
        l_prefix[i] = solver_prefix[S.list_begin + i];
    }
    __syncthreads();
    float *u = u_off ? u_all + u_off[blockIdx.x] : u_all + (int64_t)blockIdx.x * ld_v;
    const int32_t *pk = perm + S.perm_off;
    const int n = S.n_rows;

    // thread 0: rows being resolved
    int p_val = -1;                       // order entry of the row resolved next step
    int m_ci = -1, m_r = 0;               // row whose state loads are in flight
    int2_a4 m_rp = {0, 0};
    float4_v m_st = {0.f, 0.f, 0.f, 0.f};
    // all threads: entries of the current and of the next row
    int c_c[EPT], n_c[EPT];
    float c_v[EPT], n_v[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) { c_c[e] = n_c[e] = 0; c_v[e] = n_v[e] = 0.f; }

    for (int t = -4; t < n; ++t) {
        if (tid == 0) {
            // publish row t + 2 (state loads issued last step)
            if (t + 2 >= 0 && t + 2 < n) {
                RowMeta m;
                m.col = nullptr; m.val = nullptr; m.st = nullptr; m.len = 0;
                m.y = m_st.x; m.alpha = m_st.y; m.q = m_st.z; m.rw = m_st.w;
                const int len = m_rp.y - m_rp.x;
                if (m_ci >= 0 && m.q != 0.f && len > 0) {
                    const ChunkDev &ch = l_desc[m_ci];
                    m.col = (u_off ? chunk_compact_ids(ch) : ch.col) + m_rp.x;
                    m.val = ch.val + m_rp.x; m.st = ch.st + m_r; m.len = len;
                }
                ring[(t + 2) & 3] = m;
            }
            // state loads of row t + 3
            m_ci = -1;
            if (t + 3 >= 0 && t + 3 < n) {
                if ((unsigned)p_val >= (unsigned)n) {
                    atomicOr(err, ERR_PERM_RANGE);
                } else {
                    m_ci = find_chunk(l_prefix, S.n_chunks, p_val);
                    m_r = p_val - l_prefix[m_ci];
                    const ChunkDev &ch = l_desc[m_ci];
                    m_rp = gld2(ch.row_ptr + m_r);
                    m_st = gld_state(ch.st + m_r);
                }
            }
            // order entry of row t + 4
            p_val = (t + 4 >= 0 && t + 4 < n) ? pk[t + 4] : -1;
        }
        // The gather of row t is requested first and the entries of row t + 1 (published last step) after it:
        // loads return in the order they were issued, so the step does not wait for the next row's entries,
        // which come from memory.
        const RowMeta m = ring[t & 3];                            // (t < 0: an unused slot)
        const bool step = t >= 0 && m.len > 0;                    // uniform over the workgroup
        float got[EPT];
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            got[e] = 0.f;
            if (step && tid + e * BLOCK < m.len) got[e] = gather_entry(u, c_c[e]);
        }
        if (t + 1 >= 0 && t + 1 < n) {
            const RowMeta &mn = ring[(t + 1) & 3];
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                const int p = tid + e * BLOCK;
                n_c[e] = 0; n_v[e] = 0.f;
                if (p < mn.len) { n_c[e] = gld(mn.col + p); n_v[e] = gld(mn.val + p); }
            }
        }
        {
            if (step) {
                float part = 0.f;
#pragma unroll
                for (int e = 0; e < EPT; ++e) part += c_v[e] * got[e];
                for (int p = tid + EPT * BLOCK; p < m.len; p += BLOCK) part += gld(m.val + p) * gather_entry(u, gld(m.col + p));
                const float xu = block_sum<BLOCK>(part, red);
                const float delta = dual_step<LOSS>(m.alpha, m.y, m.rw, xu, m.q, sc.c);
                if (tid == 0) {
                    float an = m.alpha + delta;                      // a + (clip(..) - a) can leave [0, 1] by an ulp
                    if (LOSS != 1) an = fminf(fmaxf(an, 0.f), 1.f);
                    gst(&m.st->alpha, an);
                }
                const float coef = delta * (LOSS == 1 ? 1.0f : m.y) * sc.inv_c;
                if (coef != 0.0f) {
#pragma unroll
                    for (int e = 0; e < EPT; ++e)
                        if (tid + e * BLOCK < m.len) add_entry(u, c_c[e], coef * c_v[e]);
                    for (int p = tid + EPT * BLOCK; p < m.len; p += BLOCK)
                        add_entry(u, gld(m.col + p), coef * gld(m.val + p));
                }
            }
        }
#pragma unroll
        for (int e = 0; e < EPT; ++e) { c_c[e] = n_c[e]; c_v[e] = n_v[e]; }
        __syncthreads();   // ring slots written this step are read next step; orders scatter before gather
    }
    stamp_solver(sc, 1);
}

// Dense rows.  The private vector is staged in LDS when it fits (V_LDS), else it stays in HBM.
// Dynamic LDS: 2 * max_list ints, then d floats when V_LDS.
template <int LOSS, int BLOCK, bool V_LDS>
__global__ __launch_bounds__(BLOCK) void sdca_rowwise_dense(
    const ChunkDev *__restrict__ chunks, const SolverDev *__restrict__ solvers,
    const int32_t *__restrict__ solver_chunks, const int32_t *__restrict__ solver_prefix,
    const int32_t *__restrict__ perm, float *u_all, int64_t ld_v, int d, int ld, int max_list,
    RoundScalars sc, int *err)
{
    extern __shared__ int lists[];
    __shared__ float red[BLOCK / 64];
    const SolverDev S = solvers[blockIdx.x];
    int *l_chunk = lists;
    int *l_prefix = lists + max_list;
    float *v_lds = reinterpret_cast<float *>(lists + 2 * max_list);
    float *v_glb = u_all + (int64_t)blockIdx.x * ld_v;
    const int tid = threadIdx.x;
    stamp_solver(sc, 0);
    for (int i = tid; i < S.n_chunks; i += BLOCK) {
        l_chunk[i] = solver_chunks[S.list_begin + i];
        l_prefix[i] = solver_prefix[S.list_begin + i];
    }
    if (V_LDS)
        for (int i = tid; i < d; i += BLOCK) v_lds[i] = v_glb[i];
    __syncthreads();
    float *v = V_LDS ? v_lds : v_glb;
    const int32_t *pk = perm + S.perm_off;

    for (int t = 0; t < S.n_rows; ++t) {
        const int lr = pk[t];
        if ((unsigned)lr >= (unsigned)S.n_rows) {
            if (tid == 0) atomicOr(err, ERR_PERM_RANGE);
            continue;
        }
        const int j = find_chunk(l_prefix, S.n_chunks, lr);
        const ChunkDev &ch = chunks[l_chunk[j]];
        const int r = lr - l_prefix[j];
        const RowState st = ch.st[r];
        const float q = st.q;
        if (q == 0.0f) continue;
        const float *x = ch.val + (int64_t)r * ld;
        const float y = st.y;
        const float a = st.alpha;
        const float rw = st.rw;
        float part = 0.0f;
        for (int p = tid; p < d; p += BLOCK) part += x[p] * v[p];
        const float xu = block_sum<BLOCK>(part, red);
        const float delta = dual_step<LOSS>(a, y, rw, xu, q, sc.c);
        if (tid == 0) {
            float an = a + delta;
            if (LOSS != 1) an = fminf(fmaxf(an, 0.f), 1.f);
            ch.st[r].alpha = an;
        }
        const float coef = delta * (LOSS == 1 ? 1.0f : y) * sc.inv_c;
        if (coef != 0.0f)
            for (int p = tid; p < d; p += BLOCK) v[p] += coef * x[p];
        __syncthreads();
    }
    if (V_LDS)
        for (int i = tid; i < d; i += BLOCK) v_glb[i] = v_lds[i];
    stamp_solver(sc, 1);
}

}  // namespace chicle
