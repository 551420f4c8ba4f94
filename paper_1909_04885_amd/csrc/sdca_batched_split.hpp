// Batched local solver with every solver spread over three compute units (paper Section 4.2: a
// solver may use all the processors of its node; Section 2.2: L = 1, the coordinate steps keep their order).
//
// One compute unit gets a memory request served every few cycles, whatever its size.  Per block of 64 steps
// the single-workgroup solver (sdca_batched.hpp) asks for the block's entries, its tile of T, and for some
// five hundred lonely 4-byte reads and as many atomic adds in the unpopular part of the private vector; the
// last two take about half of its requests and it waits for both inside every block.  Here the columns of
// the private vector are divided:
//   - the head workgroup keeps the popular columns [0, n_hot) in LDS, runs the recurrence, stages the tiles;
//     its gathers and scatters touch LDS only (where that is all columns, it is all there is: sdca_batched_heads);
//   - two tail workgroups on the same L2 partition own the other columns, half of them each, in memory.
// For every block each tail hands the head 64 partial dot products and the head hands the tails the 64 steps,
// through rings of 64-bit words in memory.  A word carries its value together with the number of the block
// it belongs to, so no fence is needed; every wait is bounded: a workgroup that waits too long raises the
// error flag, stops waiting for the rest of the pass and finishes.
//
// Block b's dot products see the private vector with blocks <= b - 2 applied in the popular columns, and with blocks
// <= b - 4 in the others, where blocks b - 2 and b - 3 enter through pairs of rows; block b - 1 enters through the cross part of T.
#pragma once
#include <hip/hip_runtime.h>
#include "device_types.hpp"
#include "mem.hpp"
#include "sdca_batched.hpp"
#include "split_pairs.hpp"

namespace chicle {

constexpr int SPLIT_RING = 8;                  // blocks a ring holds
constexpr int SPLIT_TAILS = 2;
constexpr int LAG = 4;                         // unpopular columns: blocks <= b - LAG are in what block b gathers
constexpr int SPLIT_WORDS = (1 + SPLIT_TAILS) * SPLIT_RING * BATCH;      // 64-bit words per solver
constexpr int SPLIT_SPIN_LIMIT = 1 << 22;      // polls before a wait for the partner gives up
constexpr int HEAD_THREADS = BATCHED_THREADS + 64;    // the single-workgroup solver's wavefronts, and one that resolves rows
constexpr int SPLIT_THREADS = HEAD_THREADS + 128;     // with tails, one each that polls the rings and adds up pairs

__device__ __forceinline__ void ring_put(unsigned long long *p, float v, int tag)
{
    const unsigned long long w = ((unsigned long long)(unsigned)tag << 32) | (unsigned long long)__float_as_uint(v);
    __hip_atomic_store(p, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The wait of a polling wavefront: every lane for N ring words, `stride` apart, until all of them carry `tag`; the sum of
// their values.  Bounded: after SPLIT_SPIN_LIMIT polls the wait
// gives up, raises the error flag and sets *dead (LDS), which makes every later wait of the workgroup return
// at once, so a lost partner costs one time-out, not one per block.
template <int N>
__device__ __forceinline__ float ring_wait(const unsigned long long *word, int stride, int tag, int *dead, int *err)
{
    for (int spins = 0;; ++spins) {
        unsigned long long v[N];
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = __hip_atomic_load(word + k * stride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        bool ok = true;
        float sum = 0.f;
#pragma unroll
        for (int k = 0; k < N; ++k) {
            ok = ok && (int)(v[k] >> 32) == tag;
            sum += __uint_as_float((unsigned)v[k]);
        }
        if (__builtin_amdgcn_ballot_w64(!ok) == 0ull) return sum;              // every lane's words are here
        __builtin_amdgcn_s_sleep(1);
        if (spins > SPLIT_SPIN_LIMIT || __hip_atomic_load(dead, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) {
            if (spins > SPLIT_SPIN_LIMIT) {
                __hip_atomic_store(dead, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                atomicOr(err, ERR_PARTNER_TIMEOUT);
            }
            return 0.f;
        }
    }
}

// Barrier among the helper wavefronts that orders their LDS traffic only (it does not wait for loads from
// memory that are still in flight).
// In two parts: work that neither side of it depends on goes between arrival and wait.
__device__ __forceinline__ void helper_arrive_lds(int *cnt)
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if ((threadIdx.x & 63) == 0) atomicAdd(cnt, 1);
}
__device__ __forceinline__ void helper_wait_lds(const int *cnt, int target)
{
    while (__hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < target)
        __builtin_amdgcn_s_sleep(1);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

__device__ __forceinline__ void helper_barrier_lds(int *cnt, int target)
{
    helper_arrive_lds(cnt);
    helper_wait_lds(cnt, target);
}

// Sum over the LPR = 8 lanes that share a row, in every one of them, by data-parallel-primitive moves (the
// neighbour inside pairs, the other pair of the quad, then the mirrored half of the eight): register to
// register, where a shuffle goes through the LDS crossbar and costs a trip's latency each time.
__device__ __forceinline__ float sum_over_row_lanes(float v)
{
    static_assert(LPR == 8, "the moves below cover groups of eight lanes");
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, false));    // quad_perm [1,0,3,2]
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, false));    // quad_perm [2,3,0,1]
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xF, 0xF, false));   // row_half_mirror
    return v;
}

// The same over the four lanes of a quad.
__device__ __forceinline__ float sum_over_quad(float v)
{
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, false));
    return v;
}

// Wait until an LDS word that only grows has reached `target`.
__device__ __forceinline__ void wait_flag(const int *flag, int target)
{
    while (__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < target)
        __builtin_amdgcn_s_sleep(1);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// Everything this wavefront did in LDS before, then the word.
__device__ __forceinline__ void raise_flag(int *flag, int v)
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if ((threadIdx.x & 63) == 0) __hip_atomic_store(flag, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The row resolver both kinds of workgroup run in one wavefront (one lane per row of a block).  A workgroup
// works through the blocks first, first + stride, ...; call x publishes the rows of its (x+3)-th block,
// requests row extents and state of the (x+4)-th and reads the order entries of the (x+5)-th.  Its registers
// live across iterations.
struct RowResolver {
    int p_cur = -1, m_ci = -1, m_r = 0;
    int2_a4 m_rp = {0, 0};
    float4_v m_st = {0.f, 0.f, 0.f, 0.f};

    __device__ __forceinline__ void step(RowSlot (*rows)[BATCH], int ring_mask, const ChunkDev *l_desc,
                                         const int *l_prefix, const SolverDev &S, const int32_t *pk, int x, int first,
                                         int stride, int n_own, int lane, int *err, bool report)
    {
        if (x + 3 >= 0 && x + 3 < n_own) {
            RowSlot s;
            s.col = l_desc[0].col; s.val = l_desc[0].val; s.st = nullptr; s.len = 0;
            s.y = m_st.x; s.alpha = m_st.y; s.q = m_st.z; s.rw = m_st.w;
            const int len = m_rp.y - m_rp.x;
            if (m_ci >= 0 && s.q != 0.f && len > 0 && len <= GRAM_MAX_ROW) {
                const ChunkDev &ch = l_desc[m_ci];
                s.col = ch.col + m_rp.x; s.val = ch.val + m_rp.x; s.st = ch.st + m_r;
                s.len = len;
            }
            rows[(x + 3) & ring_mask][lane] = s;
        }
        m_ci = -1;
        if (x + 4 >= 0 && x + 4 < n_own && (first + stride * (x + 4)) * BATCH + lane < S.n_rows) {
            if (p_cur < 0 || p_cur >= S.n_rows) {
                if (report) atomicOr(err, ERR_PERM_RANGE);
            } else {
                m_ci = find_chunk(l_prefix, S.n_chunks, p_cur);
                m_r = p_cur - l_prefix[m_ci];
                const ChunkDev &ch = l_desc[m_ci];
                m_rp = gld2(ch.row_ptr + m_r);
                m_st = gld_state(ch.st + m_r);
            }
        }
        // always some valid position: the value is only looked at next iteration, under the range test above
        p_cur = gld(pk + min(max((first + stride * (x + 5)) * BATCH + lane, 0), S.n_rows - 1));
    }
};

struct SplitArgs {
    const ChunkDev *chunks;
    const SolverDev *solvers;
    const int32_t *solver_chunks, *solver_prefix, *perm;
    const float *tiles;
    float *u_all;
    int64_t ld_v;
    const int64_t *u_off;       // compact private vectors: where each solver's starts (else nullptr)
    int max_list, n_hot, hot_off;
    RoundScalars sc;
    int *err;
    unsigned long long *xchg_all;
    int lag;                    // LAG, or 2: no pairs were listed
    const unsigned long long *pair_list;     // beside the tiles (split_pairs)
    const int32_t *pair_count;
};

// Common start of both kinds of workgroup: the solver's chunk list into LDS.
template <int THREADS>
__device__ __forceinline__ void split_stage_lists(unsigned char *smem, const SplitArgs &A, const SolverDev &S,
                                                  ChunkDev *l_desc, int *l_prefix)
{
    for (int i = threadIdx.x; i < S.n_chunks; i += THREADS) {
        l_desc[i] = A.chunks[A.solver_chunks[S.list_begin + i]];
        if (A.u_off) l_desc[i].col = chunk_compact_ids(l_desc[i]);     // compact private vector: its indices, not column ids
        l_prefix[i] = A.solver_prefix[S.list_begin + i];
    }
}

// How many blocks before a block are not in what its gather sees of the unpopular columns: all workgroups of a solver
// look through the same counts.
__device__ __forceinline__ int split_lag(const SplitArgs &A, const SolverDev &S, int nb, int *flag)
{
    if (threadIdx.x == 0) *flag = 0;
    __syncthreads();
    if (A.lag < LAG) return A.lag;
    for (int t = threadIdx.x; t < nb; t += SPLIT_THREADS)
        if (A.pair_count[S.tile_begin + t] > PAIR_CAP) __hip_atomic_store(flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __syncthreads();
    return __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) ? 2 : LAG;
}

// ---- the head workgroup: recurrence, tiles, the popular columns in LDS -------------------------------------
// Wavefront 0 runs the chain, 1..8 gather and scatter (LDS only), 9..10 stage the tiles, one more (APART) or 9 resolves rows, and
// where there are tails two more fetch their partial sums and add up what comes through pairs.  12 is the one that shares a SIMD with the
// chain, whose issue slots polls would take; which of the three is which was measured (polls, rows, pairs): six solvers of 5000
// rows, hinge loss, 129 us a pass as 11, 13, 12, 130 as 11, 12, 13, 132 as 13, 11, 12 and 135 as 12, 11, 13; 32 of 9400 rows,
// logistic loss, 1104, 1103, 1093 and 1088.  One loop per role, all with the same number of iterations and one workgroup barrier
// per iteration, so that the registers of one role are not kept alive through the code of the others.
// TAILS: there are tails.  Else all columns are in the head and nothing is waited for but its own LDS: no wavefront takes issue
// slots that has nothing to do, a row's entries are asked for before the adds, and they go to its lanes in turn, so that short
// rows take as many adds and reads as they have entries to a lane (sixteen bytes at a time, a lane's entries lie together, and
// all six of its adds are issued whatever the row's length).  Five solvers of 40000 rows of 12 entries in 466 columns, squared
// loss: 1.44 us a block with the wavefronts and loads that tails need, 1.21 so; six of 30700 rows of 29 1.52 and 1.29; hinge
// loss, 40 of 5000 rows of 12 1.53 and 1.33, two of 30000 rows of 40 in 5000 columns 1.29 and 1.23.
// APART: rows are resolved by a wavefront of their own (heads_resolve_apart).
template <int LOSS, bool TAILS, bool APART>
__device__ __forceinline__ void split_head(unsigned char *smem, const SplitArgs &A, int sid)
{
    BatchedShared &sh = *reinterpret_cast<BatchedShared *>(smem);
    ChunkDev *l_desc = reinterpret_cast<ChunkDev *>(smem + sizeof(BatchedShared));
    int *l_prefix = reinterpret_cast<int *>(l_desc + A.max_list);
    const SolverDev S = A.solvers[sid];
    const RoundScalars &sc = A.sc;
    const int tid = threadIdx.x, n_hot = A.n_hot;
    stamp_solver(sc, sid, 0);
    static_assert(APART || !TAILS, "with tails, rows are resolved apart");
    constexpr int THREADS = TAILS ? SPLIT_THREADS : APART ? HEAD_THREADS : BATCHED_THREADS;
    constexpr int POLLER = LOSS == 2 ? 13 : 11, RESOLVER = LOSS == 2 || !TAILS ? 11 : 13, PAIRS = 12;
    split_stage_lists<THREADS>(smem, A, S, l_desc, l_prefix);
    double *hot = reinterpret_cast<double *>(smem + A.hot_off);
    for (int i = tid; i < n_hot; i += THREADS) hot[i] = 0.0;
    if (tid == 0) { sh.hb = 0; sh.dead = 0; sh.xflag = 0; sh.cflag = 0; }
    const int nb = (S.n_rows + BATCH - 1) / BATCH;
    const bool pairs = TAILS && split_lag(A, S, nb, &sh.over) == LAG;
    __syncthreads();
    float *u = A.u_off ? A.u_all + A.u_off[sid] : A.u_all + (int64_t)sid * A.ld_v;
    const int32_t *pk = A.perm + S.perm_off;
    const float *my_tiles = A.tiles + (int64_t)S.tile_begin * TILE_FLOATS;
    unsigned long long *x_steps = A.xchg_all + (int64_t)sid * SPLIT_WORDS;
    unsigned long long *x_parts = x_steps + SPLIT_RING * BATCH;
    const int lane = tid & 63, wave = tid >> 6;
    const int hl = tid - 64, rho = hl / LPR, sub = hl & (LPR - 1);     // helper coordinates
    if (nb == 0) {                                   // a solver without rows (uniform for its workgroups)
        stamp_solver(sc, sid, 1);
        return;
    }
#define HEAD_ITERATIONS for (int i = -6; i <= nb; ++i)
    if (wave == 0) {
        float x_carry = 0.f;
        bool rough = true;
        HEAD_ITERATIONS {
            if (i >= 0 && i < nb) {
                chain_block<LOSS>(sh, i, lane, x_carry, rough, sc.inv_c, sh.steps[i & 3]);
                // the tails add these steps into their columns
                if (TAILS) ring_put(x_steps + (i & (SPLIT_RING - 1)) * BATCH + lane, sh.steps[i & 3][lane], i + 1);
            }
            __syncthreads();
        }
    } else if (TAILS && wave == POLLER) {
        // What the tails send for this iteration, fetched by a wavefront that has no other loads in flight
        // (loads return in the order they were issued) and handed on through LDS.
        HEAD_ITERATIONS {
            if (i + 1 >= 0 && i + 1 < nb) {
                float part = ring_wait<SPLIT_TAILS>(x_parts + ((i + 1) & (SPLIT_RING - 1)) * BATCH + lane, SPLIT_RING * BATCH, i + 2, &sh.dead, A.err);
                if (pairs) {
                    wait_flag(&sh.cflag, i + 2);
                    part += (float)sh.xc[lane];
                }
                sh.xv[lane] = part;
                raise_flag(&sh.xflag, i + 2);
            }
            __syncthreads();
        }
    } else if (TAILS && wave == PAIRS) {
        // What blocks i - 1 and i - 2, whose steps are at hand, add to block i + 1's dot products through pairs.  The pairs were
        // asked for an iteration ago, their number two.  (In the polling wavefront this kept the polls waiting: 5.0e3
        // cycles an iteration, 4.7e3 now; 32 solvers of 62500 rows 2.15 and 2.02 ms.)
        const int32_t *counts = A.pair_count + S.tile_begin;
        const unsigned long long *lists = A.pair_list + (int64_t)S.tile_begin * PAIR_CAP + lane;
        int n_now = 0, n_next = 0, far = 0;              // pairs of blocks i + 1 and i + 2; of block i + 3 in lane 0, in flight
        unsigned long long w[PAIR_CAP / 64];
#pragma unroll
        for (int s = 0; s < PAIR_CAP / 64; ++s) w[s] = 0ull;
        HEAD_ITERATIONS {
            n_next = __builtin_amdgcn_readfirstlane(far);
            if (pairs && i + 1 >= 0 && i + 1 < nb) {
                sh.xc[lane] = 0.0;
                asm volatile("" ::: "memory");
#pragma unroll
                for (int s = 0; s < PAIR_CAP / 64; ++s)
                    if (64 * s + lane < n_now) {
                        const unsigned at = (unsigned)(w[s] >> 32);
                        const int j = at & 63, b = i - 1 - (int)(at >> 12);
                        const float coef = sh.steps[b & 3][j] * (LOSS == 1 ? 1.f : sh.rows[b & (RING - 1)][j].y) * sc.inv_c;
                        atomicAdd(&sh.xc[at >> 6 & 63], (double)(coef * __uint_as_float((unsigned)w[s])));
                    }
                raise_flag(&sh.cflag, i + 2);
            }
            n_now = 0;
            if (pairs && i + 2 >= 0 && i + 2 < nb) {
                n_now = n_next;
#pragma unroll
                for (int s = 0; s < PAIR_CAP / 64; ++s)
                    if (64 * s < n_now) w[s] = lists[(int64_t)(i + 2) * PAIR_CAP + 64 * s];
            }
            // (a scalar load would be waited for at the barrier)
            if (pairs && i + 3 >= 0 && i + 3 < nb) far = gld(counts + min(i + 3 + lane, nb - 1));
            __syncthreads();
        }
    } else if (APART && wave == RESOLVER) {
        // (one block further ahead than the tails' resolvers: the helpers ask for a block's entries three
        // iterations before they gather it)
        RowResolver resolver;
        HEAD_ITERATIONS {
            resolver.step(sh.rows, RING - 1, l_desc, l_prefix, S, pk, i + 1, 0, 1, nb, lane, A.err, true);
            __syncthreads();
        }
    } else if (wave >= 9) {
        const int sw = wave - 9;
        float4 stage[16];                                // tile part fetched ahead
        bool staged = false;
        RowResolver resolver;
        HEAD_ITERATIONS {
            // tiles for iteration i + 1 (wavefront 9: own part of T(i+1), wavefront 10: cross part of T(i+2),
            // 16 KB each) were fetched into registers during the last iteration
            const int buf = (i + 1) & 1;
            float4 *dst = reinterpret_cast<float4 *>(sw == 0 ? &sh.Tw[buf][0][0] : &sh.Tx[buf][0][0]);
#pragma unroll
            for (int j = 0; j < 16; ++j) dst[lane + 64 * j] = staged ? stage[j] : make_float4(0.f, 0.f, 0.f, 0.f);
            if (!APART && sw == 0) resolver.step(sh.rows, RING - 1, l_desc, l_prefix, S, pk, i + 1, 0, 1, nb, lane, A.err, true);
            const int tb = sw == 0 ? i + 2 : i + 3;
            staged = tb >= 0 && tb < nb;
            if (staged) {
                const float4 *src = reinterpret_cast<const float4 *>(
                    my_tiles + (int64_t)tb * TILE_FLOATS + (sw == 0 ? BATCH * BATCH : 0));
#pragma unroll
                for (int j = 0; j < 16; ++j) stage[j] = src[lane + 64 * j];
            }
            __syncthreads();
        }
    } else {
        // Entries of a row (ENT per helper lane) travel through five stages:
        // ld (loads in flight) -> ar (arrived: asked for one iteration ago) -> g (gathered this iteration) ->
        // c (its block is in the chain) -> s (scattered).  Loads get a whole iteration before anything looks at
        // them; ld and ar swap register sets from one iteration to the next (nothing moves a register that a
        // load is still due to write).  Only entries in the head's columns are kept; the others are masked when
        // the set leaves ar.
        int a_c[ENT], b_c[ENT], g_c[ENT], c_c[ENT], s_c[ENT];
        float a_v[ENT], b_v[ENT], g_v[ENT], c_v[ENT], s_v[ENT];
#pragma unroll
        for (int e = 0; e < ENT; ++e) {
            a_c[e] = b_c[e] = g_c[e] = c_c[e] = s_c[e] = 0;
            a_v[e] = b_v[e] = g_v[e] = c_v[e] = s_v[e] = 0.f;
        }
        int a_len = 0, b_len = 0, hb_target = 0;
        auto iteration = [&](const int i, int (&ld_c)[ENT], float (&ld_v)[ENT], int &ld_len,
                             const int (&ar_c)[ENT], const float (&ar_v)[ENT], const int ar_len) {
            // 0. what this iteration needs of the rows of blocks i + 3, i - 1 and i + 1 (published at least one
            //    iteration ago) and the steps of block i - 1, read together: one trip to LDS instead of one per use
            const bool has_in = i + 3 >= 0 && i + 3 < nb, has_s = i - 1 >= 0 && i - 1 < nb, has_g = i + 1 >= 0 && i + 1 < nb;
            const RowSlot r_in = sh.rows[(i + 3) & (RING - 1)][rho];
            const RowSlot r_s = sh.rows[(i - 1) & (RING - 1)][rho];
            const RowSlot r_g = sh.rows[(i + 1) & (RING - 1)][rho];
            const float dl = sh.steps[(i - 1) & 3][rho];
            ld_len = has_in ? r_in.len : 0;
            if (!TAILS && has_in) {                      // this lane's entries of the row of block i + 3
                const int32_t *cp = r_in.col + sub;
                const float *vp = r_in.val + sub;
#pragma unroll
                for (int e = 0; e < ENT; ++e) { ld_c[e] = gld(cp + e * LPR); ld_v[e] = gld(vp + e * LPR); }
            }
            // 1. block i - 1 is added to the head of the private vector
            if (has_s && r_s.len > 0 && dl != 0.f) {
                const float coef = dl * (LOSS == 1 ? 1.f : r_s.y) * sc.inv_c;
#pragma unroll
                for (int e = 0; e < ENT; ++e)
                    if (s_v[e] != 0.f) atomicAdd(&hot[s_c[e]], (double)(coef * s_v[e]));
                if (sub == 0) {
                    float an = r_s.alpha + dl;
                    if (LOSS != 1) an = fminf(fmaxf(an, 0.f), 1.f);
                    gst(&r_s.st->alpha, an);
                }
            }
            // 2. ... completely, before block i + 1 is gathered (LDS traffic only); meanwhile, with tails, this lane's segment
            //    of the row of block i + 3 is asked for
            helper_arrive_lds(&sh.hb);
            if (TAILS && has_in) {
                const int32_t *cp = r_in.col + sub * ENT;
                const float *vp = r_in.val + sub * ENT;
                static_assert(ENT == 6, "a lane's entries are loaded four and two at a time");
                const int4_a4 c4 = gld4(cp);
                const int2_a4 c2 = gld2(cp + 4);
                const float4_a4 v4 = gld4(vp);
                const float2_a4 v2 = gld2(vp + 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) { ld_c[e] = c4[e]; ld_v[e] = v4[e]; }
#pragma unroll
                for (int e = 0; e < 2; ++e) { ld_c[4 + e] = c2[e]; ld_v[4 + e] = v2[e]; }
            }
            hb_target += HELPER_WAVES;
            helper_wait_lds(&sh.hb, hb_target);
            // 3. gather block i + 1 (blocks <= i - 1 applied)
            if (has_g) {
                float got[ENT];
#pragma unroll
                for (int e = 0; e < ENT; ++e) got[e] = (float)hot[g_c[e]];   // (masked entries: column 0 times 0)
                float part = 0.f;
#pragma unroll
                for (int e = 0; e < ENT; ++e) part += g_v[e] * got[e];
                part = sum_over_row_lanes(part);
                if (sub == 0) {
                    // everything that does not need the tails' share is done before it is waited for: what follows
                    // the wait is on the path between the workgroups
                    const int buf = (i + 1) & 1;
                    const bool live = r_g.len > 0;
                    float scale = 0.f, lo = 0.f, hi = 0.f;
                    if (live && LOSS == 0) { scale = sc.c / r_g.q; lo = -r_g.alpha; hi = 1.f - r_g.alpha; }
                    if (live && LOSS == 1) scale = sc.c / (sc.c + r_g.q);
                    if (LOSS != 2) { sh.lo[buf][rho] = lo; sh.hi[buf][rho] = hi; }
                    if (TAILS) {
                        wait_flag(&sh.xflag, i + 2);
                        part += sh.xv[rho];                               // the tails' share of x_i . u
                        asm volatile("" : "+v"(part));       // (read at once, not behind the condition below)
                    }
                    float t0 = 0.f;
                    if (live) {
                        if (LOSS == 0) {
                            t0 = scale * (r_g.rw - r_g.y * part);
                        } else if (LOSS == 1) {
                            t0 = scale * (r_g.rw - r_g.alpha - part);
                        } else {
                            t0 = r_g.rw - r_g.y * part;
                            const float rr = r_g.q * sc.inv_c;
                            lo = logistic_root(t0, rr, r_g.alpha);
                        }
                    }
                    sh.t0[buf][rho] = t0;
                    if (LOSS == 2) { sh.lo[buf][rho] = lo; sh.hi[buf][rho] = hi; }
                }
            }
            // 4. move the entry sets one stage on; the set that arrived (block i + 2) is masked to the row's
            //    length and to the head's columns
#pragma unroll
            for (int e = 0; e < ENT; ++e) {
                s_c[e] = c_c[e]; s_v[e] = c_v[e];
                c_c[e] = g_c[e]; c_v[e] = g_v[e];
                const bool live = (TAILS ? sub * ENT + e : sub + e * LPR) < ar_len && ar_c[e] < n_hot;
                g_c[e] = live ? ar_c[e] : 0;
                g_v[e] = live ? ar_v[e] : 0.f;
            }
            __syncthreads();
        };
        for (int i = -6; i <= nb; i += 2) {          // HEAD_ITERATIONS, two at a time
            iteration(i, a_c, a_v, a_len, b_c, b_v, b_len);
            if (i + 1 <= nb) iteration(i + 1, b_c, b_v, b_len, a_c, a_v, a_len);
        }
    }
#undef HEAD_ITERATIONS
    for (int i = tid; i < n_hot; i += THREADS) u[i] = (float)hot[i];
    stamp_solver(sc, sid, 1);
}

// ---- a tail workgroup: the unpopular columns, in memory -----------------------------------------------------
// The unpopular columns are divided over the solver's two tails (lines of 128 bytes of the private vector in turn), so that what
// a tail adds and what it gathers meet in one compute unit, whose accesses to one address are served in the order in which
// they are issued: nothing waits for memory but the partial sums themselves.  (Tails that took the blocks in turn and all
// columns had to wait for each other's gathers: a trip to memory, its adds and its gather per block, which bounded the solver.)
// Block b's gather sees blocks <= b - 4.  Block b - 1 enters through the cross part of T, and of blocks b - 2 and b - 3 only the
// rows matter that share an unpopular column with one of block b: a handful of pairs, which depend on the data and the orders
// only and are listed beside the tiles (split_pairs); the head adds what they give when it has the steps at hand.  So the way
// from the steps to a tail, through its adds and its gather, and back may take as long as the chains of four blocks.  A solver
// one of whose blocks has more pairs than its list holds (PAIR_CAP) gathers with blocks <= b - 2 added, and no pairs; so do
// all solvers where listing pairs would cost more than it saves (lists_pairs).
// Two groups of four wavefronts take the blocks in turn.  In its turn, which begins when the other group has issued its
// gathers, a group adds block b - 4, whose steps have arrived, and issues block b's gathers; while they are on their way
// the other group has its turn.  A block's entries are asked for a turn ahead; between gather and add they wait in LDS.  Two
// wavefronts resolve rows, one for each group, one waits for the steps; the wavefronts hand on through words in LDS that only
// grow, there is no workgroup barrier.
// TE: entries per lane (TAIL_LPR lanes a row), taken from the end of the row, where its unpopular columns are (rows are sorted
// by popularity): TE * TAIL_LPR must cover the largest number of entries a row has in the tails' columns (checked on the host).
// 32 solvers of 62500 rows of 40 entries, 1M columns: 6.9e3 cycles per block of 64 steps with blocks in turn and look-back two
// (2.84 ms a pass), 7.7e3 with blocks in turn and look-back three, 4.7e3 now (2.02 ms); six of 5000 rows, 20k columns: 169 us
// a pass, 127 now.  A tail waits for steps 3.9e3 of its 1.04e4 cycles per two blocks; the head's tile loads, which miss the
// cache, take as long as an iteration.
constexpr int TAIL_LPR = 4, TAIL_GROUPS = 2, TAIL_WAVES = BATCH * TAIL_LPR / 64;
constexpr int TAIL_RING = 4;                        // resolved rows of a group's blocks
constexpr int TAIL_LINE_LOG2 = 5;                   // columns of a tail's share of the private vector that lie side by side

struct TailShared {
    RowSlot rows[TAIL_GROUPS][TAIL_RING][BATCH];
    float xv[LAG][BATCH];                           // steps of the latest blocks
    int steps_ready, issued, dead, over;                  // blocks whose steps are in xv; wavefronts that have issued a block's gathers
    int rows_ready[TAIL_GROUPS], loaded[TAIL_GROUPS], bar[TAIL_GROUPS];
};
struct __align__(8) TailEntry { int col; float val; };          // val: with the row's label, as its step is added
__host__ __device__ constexpr size_t tail_lists_at(int te)
{
    return sizeof(TailShared) + sizeof(TailEntry) * (size_t)(LAG * te * BATCH * TAIL_LPR);
}

template <int LOSS, int TE>
__device__ __forceinline__ void split_tail(unsigned char *smem, const SplitArgs &A, int sid, int tail)
{
    TailShared &sh = *reinterpret_cast<TailShared *>(smem);
    TailEntry *kept = reinterpret_cast<TailEntry *>(smem + sizeof(TailShared));        // [block & (LAG - 1)][entry][lane of the group]
    ChunkDev *l_desc = reinterpret_cast<ChunkDev *>(smem + tail_lists_at(TE));
    int *l_prefix = reinterpret_cast<int *>(l_desc + A.max_list);
    const SolverDev S = A.solvers[sid];
    const RoundScalars &sc = A.sc;
    const int tid = threadIdx.x, n_hot = A.n_hot;
    split_stage_lists<SPLIT_THREADS>(smem, A, S, l_desc, l_prefix);
    if (tid == 0) {
        sh.steps_ready = sh.issued = sh.dead = 0;
        for (int g = 0; g < TAIL_GROUPS; ++g) sh.rows_ready[g] = sh.loaded[g] = sh.bar[g] = 0;
    }
    const int nb = (S.n_rows + BATCH - 1) / BATCH;
    const int lag = split_lag(A, S, nb, &sh.over);      // (a workgroup barrier)
    if (nb == 0) return;
    float *u = A.u_off ? A.u_all + A.u_off[sid] : A.u_all + (int64_t)sid * A.ld_v;
    const int32_t *pk = A.perm + S.perm_off;
    unsigned long long *x_steps = A.xchg_all + (int64_t)sid * SPLIT_WORDS;
    unsigned long long *x_parts = x_steps + (1 + tail) * SPLIT_RING * BATCH;
    const int lane = tid & 63, wave = tid >> 6;
    constexpr int POLLER = TAIL_GROUPS * TAIL_WAVES, RESOLVER = POLLER + 1;
    if (wave == POLLER) {
        for (int a = 0; a < nb; ++a) {
            // (block a + LAG's partial sums, without which there are no steps of its own, leave after a's steps were read)
            sh.xv[a & (LAG - 1)][lane] = ring_wait<1>(x_steps + (a & (SPLIT_RING - 1)) * BATCH + lane, 0, a + 1, &sh.dead, A.err);
            raise_flag(&sh.steps_ready, a + 1);
        }
    } else if (wave >= RESOLVER) {
        const int grp = wave - RESOLVER;
        if (grp >= TAIL_GROUPS) return;
        const int n_own = (nb - grp + TAIL_GROUPS - 1) / TAIL_GROUPS;
        RowResolver resolver;
        for (int x = -5; x + 3 < n_own; ++x) {
            if (x + 3 >= TAIL_RING) wait_flag(&sh.loaded[grp], TAIL_WAVES * (x + 3 - TAIL_RING + 1));      // the slot is free
            resolver.step(sh.rows[grp], TAIL_RING - 1, l_desc, l_prefix, S, pk, x, grp, TAIL_GROUPS, n_own, lane, A.err, false);
            if (x + 3 >= 0) raise_flag(&sh.rows_ready[grp], x + 4);
        }
    } else {
        const int grp = wave / TAIL_WAVES, gl = tid & (TAIL_WAVES * 64 - 1), rho = gl / TAIL_LPR, sub = gl & (TAIL_LPR - 1);
        static_assert(TE % 6 == 0, "entries are loaded four and two at a time");
        int in_c[TE];
        float in_v[TE], in_y = 0.f;
        int in_n = 0;                                // entries of this lane's that are inside the row
        auto request = [&](int b) __attribute__((always_inline)) {
            wait_flag(&sh.rows_ready[grp], b / TAIL_GROUPS + 1);
            const RowSlot &r = sh.rows[grp][b / TAIL_GROUPS & (TAIL_RING - 1)][rho];
            const int at = max(r.len - TE * TAIL_LPR, 0) + sub * TE;
            const int32_t *cp = r.col + at;
            const float *vp = r.val + at;
            in_n = r.len - at;
            in_y = LOSS == 1 ? 1.f : r.y;
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (lane == 0) atomicAdd(&sh.loaded[grp], 1);
#pragma unroll
            for (int e = 0; e < TE; e += 6) {
                const int4_a4 c4 = gld4(cp + e);
                const int2_a4 c2 = gld2(cp + e + 4);
                const float4_a4 v4 = gld4(vp + e);
                const float2_a4 v2 = gld2(vp + e + 4);
#pragma unroll
                for (int q = 0; q < 4; ++q) { in_c[e + q] = c4[q]; in_v[e + q] = v4[q]; }
#pragma unroll
                for (int q = 0; q < 2; ++q) { in_c[e + 4 + q] = c2[q]; in_v[e + 4 + q] = v2[q]; }
            }
        };
        if (grp < nb) request(grp);
        int bar_target = 0;
        for (int b = grp; b < nb + lag; b += TAIL_GROUPS) {
            // 1. block b's entries, as far as they are inside the row and in this tail's columns; those of b + 2 are asked for
            int g_c[TE];
            float g_v[TE];
            const float y = in_y;
#pragma unroll
            for (int e = 0; e < TE; ++e) {
                const bool live = b < nb && e < in_n && in_c[e] >= n_hot && (in_c[e] >> TAIL_LINE_LOG2 & 1) == tail;
                g_c[e] = live ? in_c[e] : 0;
                g_v[e] = live ? in_v[e] : 0.f;
            }
            if (b + TAIL_GROUPS < nb) request(b + TAIL_GROUPS);
            // 2. this group's turn: block b - lag is added
            const int a = b - lag;
            TailEntry *slot = kept + (size_t)(b & (LAG - 1)) * TE * (BATCH * TAIL_LPR) + gl;
            TailEntry add[TE];
            float coef = 0.f;
            if (a >= 0 && a < nb) {
                const TailEntry *from = kept + (size_t)(a & (LAG - 1)) * TE * (BATCH * TAIL_LPR) + gl;
#pragma unroll
                for (int e = 0; e < TE; ++e) add[e] = from[e * (BATCH * TAIL_LPR)];
                wait_flag(&sh.steps_ready, a + 1);
                coef = sh.xv[a & (LAG - 1)][rho] * sc.inv_c;
            }
            wait_flag(&sh.issued, TAIL_WAVES * b);
            if (coef != 0.f) {
#pragma unroll
                for (int e = 0; e < TE; ++e)
                    if (add[e].val != 0.f) unsafeAtomicAdd(&u[add[e].col], coef * add[e].val);
            }
            // 3. ... by every wavefront of the group, before block b is gathered
            asm volatile("" ::: "memory");
            bar_target += TAIL_WAVES;
            helper_barrier_lds(&sh.bar[grp], bar_target);
            float got[TE];
#pragma unroll
            for (int e = 0; e < TE; ++e) {
                got[e] = 0.f;
                if (g_v[e] != 0.f) got[e] = ld_l2(u + g_c[e]);
            }
            asm volatile("" ::: "memory");
            if (lane == 0) atomicAdd(&sh.issued, 1);
            // 4. the other group's turn; the partial sums are handed over when they are here
            if (b < nb) {
#pragma unroll
                for (int e = 0; e < TE; ++e) slot[e * (BATCH * TAIL_LPR)] = TailEntry{g_c[e], g_v[e] * y};
                float part = 0.f;
#pragma unroll
                for (int e = 0; e < TE; ++e) part += g_v[e] * got[e];
                part = sum_over_quad(part);
                if (sub == 0) ring_put(x_parts + (b & (SPLIT_RING - 1)) * BATCH + rho, part, b + 1);
            }
        }
    }
}

// Workgroup role * k_pad + k: role 0 is the head of solver k, roles 1 .. n_tails are its tails (k_pad is a
// multiple of the number of L2 partitions workgroups are dealt over, so all of them share one).
// xchg_all: SPLIT_WORDS zeroed 64-bit words per solver: the ring of steps, one ring of partial dot products
// per tail.
// Dynamic LDS: in the head BatchedShared, then max_list chunk descriptors, max_list local-row prefixes, then (at byte
// offset hot_off) n_hot doubles; in a tail TailShared, the kept entries, then the same lists.
template <int LOSS, int TE>
__global__ __launch_bounds__(SPLIT_THREADS) void sdca_batched_split(SplitArgs A, int k_pad)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int role = (int)blockIdx.x / k_pad, sid = (int)blockIdx.x % k_pad;
    if (sid >= A.sc.K) return;
    if (role == 0) split_head<LOSS, true, true>(smem, A, sid);
    else split_tail<LOSS, TE>(smem, A, sid, role - 1);
}

// Solvers all of whose columns are in the head: workgroup k is solver k.
template <int LOSS, bool APART>
__global__ __launch_bounds__(APART ? HEAD_THREADS : BATCHED_THREADS) void sdca_batched_heads(SplitArgs A, int)
{
    extern __shared__ __align__(16) unsigned char smem[];
    if ((int)blockIdx.x < A.sc.K) split_head<LOSS, false, APART>(smem, A, (int)blockIdx.x);
}

}  // namespace chicle
