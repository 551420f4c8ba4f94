// Pairs of rows that the split batched solver's tails leave out of their gathers (see sdca_batched_split.hpp).
#pragma once
#include <hip/hip_runtime.h>
#include "device_types.hpp"
#include "mem.hpp"
#include "sdca_batched.hpp"

namespace chicle {

// ---- pairs of rows two and three blocks apart that share an unpopular column ---------------------------------
// list[tile * PAIR_CAP ..]: the pairs of the tile's block b with blocks b - 2 and b - 3 of the same solver (a value
// x_ic x_jc below; i, j and which block above), count[tile]: how many there are, of which the list holds PAIR_CAP at most.
// A workgroup takes `run` tiles (PAIR_RUN at most) and, to begin with, the three blocks before them; it resolves all their rows side by side
// (a chain of dependent loads), then takes block after block: its unpopular entries follow the chains of the hash tables of the
// blocks two and three before, and are put into one of their own (a slot holds the entry put there last and the number of its
// block, an entry the one before it; nothing is cleared).  A block's entries are asked for one block ahead.  LDS leaves room for two
// workgroups on a compute unit.  Entries in random order are what it waits for: 31250 tiles in 354 us beside a pass, on 160
// compute units (0.64 GB of entries looked through, 1.8 TB/s), 480 tiles in 10 us (23 in runs of twelve, which leave most of
// the chip idle).
constexpr int PAIR_CAP = 512;                       // rows of 40 entries in uniform columns, 8704 of them in the head: 376 on average
                                                    // at most, whatever the number of columns (2 * 64 * 64 (d - 8704) (40 / d)^2).  Longer
                                                    // chunk lists leave the head fewer, 6144 at least: up to 533, and no list where
                                                    // that is foreseen or one overflows
constexpr int PAIR_RUN = 12;                        // at most
constexpr int PAIR_THREADS = 512;
constexpr int PAIR_ROWS = (PAIR_RUN + 3) * BATCH;

__device__ __forceinline__ unsigned long long pair_word(float v, int i, int j, int back)
{
    return (unsigned long long)(unsigned)(back << 12 | i << 6 | j) << 32 | (unsigned long long)__float_as_uint(v);
}

template <int TE>
struct PairShared {
    static constexpr int POS_BITS = TE <= 3 ? 11 : 12, HASH_LOG2 = POS_BITS - 1, REST_BITS = 31 - HASH_LOG2;
    static constexpr int ENTRIES = PAIR_THREADS * TE;
    static constexpr unsigned END = (1u << POS_BITS) - 1u;
    static_assert(REST_BITS + POS_BITS <= 32 && ENTRIES <= (int)END, "an entry is two words");
    struct __align__(8) Entry { unsigned rest_next; float val; };
    struct Row { const int32_t *col; int val_at, n; };              // where its last entries begin, their values 64 val_at places on, how many there are
    Row rows[PAIR_ROWS];
    Entry entry[4][ENTRIES];                        // by tile & 3; position PAIR_THREADS * k + thread
    unsigned head[4][1 << HASH_LOG2];
    int found[2];
};

template <int TE>
__global__ __launch_bounds__(PAIR_THREADS) void split_pairs(const ChunkDev *__restrict__ chunks, const SolverDev *__restrict__ solvers,
                                                            const int32_t *__restrict__ row_chunk, const int32_t *__restrict__ chunk_first,
                                                            const int32_t *__restrict__ perm, const int32_t *__restrict__ tile_solver,
                                                            int n_tiles, int run, int n_hot, unsigned long long *list,
                                                            int32_t *count)
{
    using SH = PairShared<TE>;
    extern __shared__ __align__(16) unsigned char psm[];
    SH &sh = *reinterpret_cast<SH *>(psm);
    const int tid = threadIdx.x, t0 = (int)blockIdx.x * run, t1 = min(n_tiles, t0 + run);
    const int32_t *dummy = chunks[0].col;            // readable for GRAM_MAX_ROW entries
    for (int q = tid; q < (run + 3) * BATCH; q += PAIR_THREADS) {
        const int tile = t0 - 3 + q / BATCH;
        typename SH::Row row = {dummy, 0, 0};
        if (tile >= 0 && tile < t1) {
            const SolverDev S = solvers[tile_solver[tile]];
            const int t = (tile - S.tile_begin) * BATCH + q % BATCH;
            const int lr = t < S.n_rows ? perm[S.perm_off + t] : -1;
            if ((unsigned)lr < (unsigned)S.n_rows) {                // (the tiles' kernel reports entries out of range)
                const int ci = row_chunk[S.perm_off + lr];
                const ChunkDev ch = chunks[ci];
                const int r = lr - chunk_first[ci];
                const int2_a4 rp = gld2(ch.row_ptr + r);
                const int len = rp.y - rp.x, skip = max(len - TE * LPR, 0);
                if (len > 0 && len <= GRAM_MAX_ROW) row = {ch.col + rp.x + skip, (int)((ch.val - reinterpret_cast<const float *>(ch.col)) / 64), len - skip};
            }
        }
        sh.rows[q] = row;
    }
    for (int i = tid; i < 4 << SH::HASH_LOG2; i += PAIR_THREADS) (&sh.head[0][0])[i] = 0u;
    if (tid < 2) sh.found[tid] = 0;
    __syncthreads();
    const int rho = tid / LPR, sub = tid & (LPR - 1);
    int in_c[TE], in_n = 0;
    float in_v[TE];
    auto request = [&](int q) __attribute__((always_inline)) {       // block q of the run
        const typename SH::Row r = sh.rows[q * BATCH + rho];
        in_n = r.n;
        const int32_t *cp = r.col + sub;
        const float *vp = reinterpret_cast<const float *>(r.col) + 64 * (int64_t)r.val_at + sub;
#pragma unroll
        for (int e = 0; e < TE; ++e) { in_c[e] = gld(cp + e * LPR); in_v[e] = gld(vp + e * LPR); }
    };
    request(0);
    constexpr unsigned REST = (1u << SH::REST_BITS) - 1u;
    for (int q = 0; q < t1 - t0 + 3; ++q) {
        const int tile = t0 - 3 + q;
        unsigned key[TE];
        float val[TE];
#pragma unroll
        for (int e = 0; e < TE; ++e) {
            val[e] = sub + e * LPR < in_n && in_c[e] >= n_hot ? in_v[e] : 0.f;
            key[e] = ((unsigned)in_c[e] * 2654435761u) & 0x7fffffffu;
        }
        if (q + 1 < run + 3) request(q + 1);
        if (q >= 3) {
            const int behind = tile - solvers[tile_solver[tile]].tile_begin;      // blocks of the same solver before this one
            unsigned at[2 * TE];
#pragma unroll
            for (int e = 0; e < 2 * TE; ++e) {       // all lookups in flight together: blocks b - 2, then b - 3
                const int back = 2 + e / TE;
                const unsigned slot = val[e % TE] != 0.f && back <= behind ? sh.head[(q - back) & 3][key[e % TE] >> SH::REST_BITS] : 0u;
                at[e] = slot >> SH::POS_BITS == (unsigned)(q - back + 1) ? slot & SH::END : SH::END;
            }
#pragma unroll
            for (int e = 0; e < 2 * TE; ++e)
                while (at[e] != SH::END) {
                    const typename SH::Entry p = sh.entry[(q - 2 - e / TE) & 3][at[e]];
                    // (a product beyond a float's range is of a row whose squared norm is too: it takes no step, and infinity
                    // times a step of zero would be no number)
                    if (p.rest_next >> SH::POS_BITS == (key[e % TE] & REST) && fabsf(val[e % TE] * p.val) <= 3.4028235e38f) {
                        const int k = atomicAdd(&sh.found[q & 1], 1);
                        if (k < PAIR_CAP)
                            list[(int64_t)tile * PAIR_CAP + k] = pair_word(val[e % TE] * p.val, rho, (int)(at[e] & (PAIR_THREADS - 1)) / LPR, e / TE);
                    }
                    at[e] = p.rest_next & SH::END;
                }
        }
#pragma unroll
        for (int e = 0; e < TE; ++e) {
            if (val[e] == 0.f) continue;
            const unsigned pos = (unsigned)(tid + e * PAIR_THREADS);
            const unsigned was = atomicExch(&sh.head[q & 3][key[e] >> SH::REST_BITS], (unsigned)(q + 1) << SH::POS_BITS | pos);
            const unsigned next = was >> SH::POS_BITS == (unsigned)(q + 1) ? was & SH::END : SH::END;
            sh.entry[q & 3][pos] = typename SH::Entry{(key[e] & REST) << SH::POS_BITS | next, val[e]};
        }
        __syncthreads();
        if (tid == 0 && q >= 3) { count[tile] = sh.found[q & 1]; sh.found[q & 1] = 0; }
    }
}

}  // namespace chicle
