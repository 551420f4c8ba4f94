// Gram blocks of the batched solver.
//
// A tile couples the 64 rows of one block (i) with the 64 rows of the previous block and the earlier
// rows of the same block (jp): T[jp][i] = scale_i s_i s_j (x_i . x_j).  Columns are stored as popularity
// ranks, so a row's entries split by a range test:
//   - popular columns (rank < GRAM_DENSE): the values go into a small dense matrix in LDS and their contribution
//     is a dense product on the matrix cores, fp32 in and out (the rows share so many of these columns that the
//     join's lists would be long);
//   - all other columns: a hash join in LDS by chains.  A slot holds the entry that was put there last, every entry
//     the one that was there before it, so that putting an entry in is one exchange, and an entry meets the earlier
//     members of its column by following its chain, adding its products with atomics in LDS.
// Each workgroup owns a contiguous range of tiles and works through it.  The two latest blocks are kept, each with a
// table of its own (by the parity of its number): a block is put in once, for the tile of its own and as the previous
// block of the next.  Slots hold the block's number beside the entry's position, so the tables are never cleared: a slot
// of an older block is an empty one.  A thread follows the chains of its three entries through both tables side by side,
// six trips to LDS in flight; an entry is one 64-bit word (its column is told by what its slot leaves open of the hash, which
// permutes the column numbers), because the number of LDS reads is what a chain's step costs.
// The dense product stays in the registers of the wavefronts that write the tile out; half of them multiply while the other
// half follows chains.
// Three workgroup barriers per tile; the row lookups of the tiles to come (visiting order -> chunk -> row offsets, a
// chain of dependent loads) are spread over the phases of the current one, entries are requested a tile ahead.
// What bounds it is the longest chain among a wavefront's lanes: per tile of rows of 40 Zipf-distributed entries 18.5e3
// cycles, of which 9e3 go into chains, 3e3 into the dense product, 1.7e3 into putting the block in and 1.5e3 into writing the
// tile.  4688 such tiles on 256 compute units: 298 us with a table per tile that was cleared, counted, scanned and laid out
// as lists; 251 with chains of both blocks' entries kept, 212 with one word per entry and the dense product in registers,
// 199 with the chains of one entry at a time, 187 with slots of their own for the more frequent columns, 173 in longer runs.
// The summation order of the join is not fixed, so tiles can differ in the last bits between runs.
#pragma once
#include <hip/hip_runtime.h>
#include "device_types.hpp"
#include "sdca_batched.hpp"

namespace chicle {

constexpr int GRAM_DENSE = 64;                        // columns handled by the dense product
constexpr int GRAM_THREADS = 1024;
constexpr int GRAM_DIRECT = 1024;                     // the columns that follow have a slot each,
constexpr int GRAM_HASH_LOG2 = 11;                    // all others share these (chains, not probing: fewer than entries is fine)
constexpr int GRAM_SLOTS = GRAM_DIRECT + (1 << GRAM_HASH_LOG2);
constexpr int GRAM_ENTRIES = BATCH * GRAM_MAX_ROW;    // entry positions of a block
constexpr int GRAM_EPT = GRAM_ENTRIES / GRAM_THREADS; // entry positions per thread
constexpr int GRAM_LPR = GRAM_THREADS / BATCH;        // threads per row: thread 16 s + l takes entries l, l + 16, l + 32 of row s
                                                      // (rows are sorted by popularity: a wavefront's k-th entries have chains of like length)
constexpr int GRAM_POS_BITS = 12;                     // a slot: the block's number above, the entry's position below
constexpr int GRAM_REST_BITS = 31 - GRAM_HASH_LOG2;  // of a column's hash, beside its slot
static_assert(GRAM_ENTRIES < 1 << GRAM_POS_BITS && GRAM_EPT * GRAM_THREADS == GRAM_ENTRIES && GRAM_EPT * GRAM_LPR == GRAM_MAX_ROW, "positions");
static_assert(GRAM_REST_BITS + GRAM_POS_BITS <= 32 && (unsigned)GRAM_SLOTS < 0xffffffffu >> GRAM_REST_BITS, "an entry is two words");
constexpr int G_LD = BATCH + 1;                       // padded row of the accumulator tile
constexpr int A_LD = TILE_W + 2;                      // padded row of the dense part

typedef float floatx4 __attribute__((ext_vector_type(4)));
struct GramRows {                                     // the 64 rows of a block
    const int32_t *col[BATCH];
    const float *val[BATCH];
    int len[BATCH];
    float sgn[BATCH], scale[BATCH];
};

// The accumulators are doubles: the join adds into them with LDS atomics, and on this hardware those run
// at the rate of the LDS pipeline for doubles while they are serialised lane by lane for floats.
// next: position of the entry that was in the slot before it, or CHAIN_END.
struct __align__(8) GramEntry { unsigned rest_next; float val; };
constexpr unsigned CHAIN_END = (1u << GRAM_POS_BITS) - 1u;
struct GramShared {
    double Gx[BATCH][G_LD];                // accumulators: previous block [jp][i] ...
    double Go[BATCH * (BATCH - 1) / 2];    // ... and the block's own pairs j < i, at own_at(j, i)
    float A[GRAM_DENSE][A_LD];             // dense part, [column][64 * (block & 1) + row]
    unsigned head[2][GRAM_SLOTS];          // by block & 1: the slot's latest entry (block number 0: none yet)
    GramEntry entry[2][GRAM_ENTRIES];      // of the two latest blocks, by block & 1; position GRAM_THREADS * k + thread
    GramRows rows[4];                      // previous block, current one and the two after it
};
static_assert(sizeof(GramShared) <= LDS_BYTES, "fits a compute unit");

__device__ __forceinline__ int own_at(int j, int i) { return i * (i - 1) / 2 + j; }
// A column's slot (above GRAM_REST_BITS) and what tells it from the slot's other columns: multiplication by an odd number
// permutes the 31-bit column numbers, the upper bits choose the slot and the lower ones are left.
__device__ __forceinline__ unsigned gram_key(int col)
{
    const unsigned h = ((unsigned)col * 2654435761u) & 0x7fffffffu;
    return col < GRAM_DENSE + GRAM_DIRECT ? (unsigned)(col - GRAM_DENSE) << GRAM_REST_BITS : h + ((unsigned)GRAM_DIRECT << GRAM_REST_BITS);
}

// Row lookups of one block, one row per lane of a wavefront, as steps of dependent loads.
struct RowLookup {
    SolverDev S;
    int lr, ci, r;
    const int32_t *row_ptr, *colp;
    const float *valp;
    const RowState *stp;
    int2_a4 rp;
    float4_v st;
    bool live;
};

// row_chunk[perm_off + lr] = chunk of the solver's local row lr; chunk_first[c] = local index of the
// chunk's first row inside its solver.
template <int LOSS>
__global__ __launch_bounds__(GRAM_THREADS) void gram_tiles_join(
    const ChunkDev *__restrict__ chunks, const SolverDev *__restrict__ solvers,
    const int32_t *__restrict__ row_chunk, const int32_t *__restrict__ chunk_first,
    const int32_t *__restrict__ perm, const int32_t *__restrict__ tile_solver, float *tiles, int n_tiles,
    float c, int *err)
{
    extern __shared__ __align__(16) unsigned char gsm[];
    GramShared &sh = *reinterpret_cast<GramShared *>(gsm);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int per = (n_tiles + gridDim.x - 1) / gridDim.x;
    const int t_begin = blockIdx.x * per;
    const int t_end = min(n_tiles, t_begin + per);
    if (t_begin >= t_end) return;

    const int32_t *dummy_col = chunks[0].col;      // readable for at least GRAM_MAX_ROW entries
    const float *dummy_val = chunks[0].val;
    // step 1: visiting-order entry of the lane's row in tile `tile`
    auto lookup1 = [&](RowLookup &L, int tile, bool wanted) __attribute__((always_inline)) {
        L.live = false;
        if (!wanted) return;
        L.S = solvers[tile_solver[tile]];
        const int t = (tile - L.S.tile_begin) * BATCH + lane;
        if (t < L.S.n_rows) { L.lr = gld(perm + L.S.perm_off + t); L.live = true; }
    };
    auto lookup2 = [&](RowLookup &L) __attribute__((always_inline)) {       // -> chunk id
        if (!L.live) return;
        if ((unsigned)L.lr >= (unsigned)L.S.n_rows) { atomicOr(err, ERR_PERM_RANGE); L.live = false; return; }
        L.ci = gld(row_chunk + L.S.perm_off + L.lr);
    };
    auto lookup3 = [&](RowLookup &L) __attribute__((always_inline)) {       // -> chunk descriptor
        if (!L.live) return;
        const ChunkDev &ch = chunks[L.ci];
        L.r = L.lr - gld(chunk_first + L.ci);
        L.row_ptr = ch.row_ptr; L.colp = ch.col; L.valp = ch.val; L.stp = ch.st;
    };
    auto lookup4 = [&](RowLookup &L) __attribute__((always_inline)) {       // -> row offsets and state
        if (!L.live) return;
        L.rp = gld2(L.row_ptr + L.r);
        L.st = gld_state(L.stp + L.r);
    };
    auto publish = [&](const RowLookup &L, GramRows &R) __attribute__((always_inline)) {
        int len = 0;
        float sgn = 1.f, scale = 0.f;
        const int32_t *cp = dummy_col;
        const float *vp = dummy_val;
        if (L.live) {
            const int n = L.rp.y - L.rp.x;
            const float q = L.st.z;
            if (q != 0.f && n > 0 && n <= GRAM_MAX_ROW) {
                len = n; cp = L.colp + L.rp.x; vp = L.valp + L.rp.x;
                sgn = LOSS == 1 ? 1.f : L.st.x;
                scale = LOSS == 0 ? -1.f / q : LOSS == 1 ? -1.f / (c + q) : -1.f / c;
            }
        }
        R.col[lane] = cp; R.val[lane] = vp; R.len[lane] = len; R.sgn[lane] = sgn; R.scale[lane] = scale;
    };
    // a thread's entry positions are the same in every block; loads are unconditional (a row without entries points at
    // readable dummy data and the store keeps slack behind every chunk)
    int e_col[GRAM_EPT], n_col[GRAM_EPT];
    float e_val[GRAM_EPT], n_val[GRAM_EPT];
    const int e_row = tid / GRAM_LPR, e_p = tid % GRAM_LPR;
    auto request = [&](const GramRows &R, int (&to_c)[GRAM_EPT], float (&to_v)[GRAM_EPT]) __attribute__((always_inline)) {
        const int32_t *cp = R.col[e_row] + e_p;
        const float *vp = R.val[e_row] + e_p;
#pragma unroll
        for (int k = 0; k < GRAM_EPT; ++k) { to_c[k] = gld(cp + k * GRAM_LPR); to_v[k] = gld(vp + k * GRAM_LPR); }
    };
    auto clear_half = [&](int half) __attribute__((always_inline)) {        // of the dense part
        for (int i = tid; i < GRAM_DENSE * BATCH; i += GRAM_THREADS) sh.A[i / BATCH][half * BATCH + (i & (BATCH - 1))] = 0.f;
    };
    // Block number `seq` (its rows in R, its entries in e_col, e_val) is put in.  key[k]: of the thread's k-th entry
    // (NO_KEY: it is in no slot); at[k]: where its chain in its own block goes on.
    constexpr unsigned NO_KEY = 0xffffffffu, REST = (1u << GRAM_REST_BITS) - 1u;
    unsigned key[GRAM_EPT], at[2 * GRAM_EPT];
    auto position = [&](unsigned slot, int seq) __attribute__((always_inline)) {       // of the entry in a slot of block seq's
        return (int)(slot >> GRAM_POS_BITS) == seq ? slot & CHAIN_END : CHAIN_END;
    };
    auto insert = [&](const GramRows &R, int seq) __attribute__((always_inline)) {
        unsigned was[GRAM_EPT];
        const int len = R.len[e_row];
#pragma unroll
        for (int k = 0; k < GRAM_EPT; ++k) {       // all exchanges in flight together
            was[k] = 0u; key[k] = NO_KEY;
            if (e_p + k * GRAM_LPR >= len) continue;
            if (e_col[k] < GRAM_DENSE) {
                sh.A[e_col[k]][(seq & 1) * BATCH + e_row] = e_val[k];
            } else {
                key[k] = gram_key(e_col[k]);
                was[k] = atomicExch(&sh.head[seq & 1][key[k] >> GRAM_REST_BITS], (unsigned)seq << GRAM_POS_BITS | (unsigned)(tid + k * GRAM_THREADS));
            }
        }
#pragma unroll
        for (int k = 0; k < GRAM_EPT; ++k) {
            at[k] = key[k] == NO_KEY ? CHAIN_END : position(was[k], seq);
            if (key[k] != NO_KEY) sh.entry[seq & 1][tid + k * GRAM_THREADS] = GramEntry{(key[k] & REST) << GRAM_POS_BITS | at[k], e_val[k]};
        }
    };

    // ---- start: rows of the previous block, the first, the second and the third tile's, looked up side by side by four
    // wavefronts.  The fourth goes on looking rows up: LA two and three tiles ahead; the loop expects the third tile's at its
    // last step.
    int solver = tile_solver[t_begin];
    const bool has_prev = t_begin > solvers[solver].tile_begin;
    constexpr int RESOLVER = 3;
    RowLookup LA;
    LA.live = false;
    if (wv <= RESOLVER) {
        const int tile = t_begin - 1 + wv;
        lookup1(LA, tile, wv == 0 ? has_prev : tile < t_end);
        lookup2(LA); lookup3(LA);
        if (wv < RESOLVER) { lookup4(LA); publish(LA, sh.rows[wv]); }
    }
    for (int i = tid; i < 2 * GRAM_SLOTS; i += GRAM_THREADS) (&sh.head[0][0])[i] = 0u;
    for (int i = tid; i < BATCH * G_LD; i += GRAM_THREADS) (&sh.Gx[0][0])[i] = 0.0;
    for (int i = tid; i < BATCH * (BATCH - 1) / 2; i += GRAM_THREADS) sh.Go[i] = 0.0;
    clear_half(0);
    clear_half(1);
    __syncthreads();
    int seq = 2;                                   // number of the block put in last
    request(sh.rows[0], e_col, e_val);
    request(sh.rows[1], n_col, n_val);
    insert(sh.rows[0], seq);
#pragma unroll
    for (int k = 0; k < GRAM_EPT; ++k) { e_col[k] = n_col[k]; e_val[k] = n_val[k]; }

    for (int tile = t_begin; tile < t_end; ++tile) {
        const int slot = tile - t_begin + 1;       // rows[slot & 3]: this tile's
        GramRows &R = sh.rows[slot & 3];
        const GramRows &P = sh.rows[(slot - 1) & 3];
        ++seq;
        if (tile > t_begin) {
            const int now = tile_solver[tile];
            if (now != solver) {                   // another solver: the block before is not this one's previous
                solver = now;
                clear_half((seq - 1) & 1);
                seq += 2;                          // (the parity of the next number, the number before it unused)
            }
        }
        // ---- 1. this block's entries; the next tile's are requested; lookups
        request(sh.rows[(slot + 1) & 3], n_col, n_val);
        RowLookup LB = LA;                         // two tiles ahead
        if (wv == RESOLVER) {
            lookup4(LB);
            lookup1(LA, tile + 3, tile + 3 < t_end);
        }
        insert(R, seq);
        __syncthreads();

        // ---- 2. the products: popular columns on the matrix cores, the others along the chains
        if (wv == RESOLVER) lookup2(LA);
        const int cur = seq & 1, old = cur ^ 1;
        // A 16 x 4 by 4 x 16 product takes A[l % 16][l / 16] and B[l / 16][l % 16] from lane l.  The tile is 8 x 4 blocks of
        // 16 x 16 (jp, i); of the lower half those above the diagonal are zero.  Wavefront w takes block (w / 4, w % 4) of the
        // upper half and the same of the lower.
        const int bj = wv >> 2, bi = wv & 3;
        floatx4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        auto multiply = [&]() __attribute__((always_inline)) {
            const float *pi = &sh.A[lane >> 4][cur * BATCH + 16 * bi + (lane & 15)];
            const float *po = &sh.A[lane >> 4][cur * BATCH + 16 * bj + (lane & 15)];
            const float *px = &sh.A[lane >> 4][old * BATCH + 16 * bj + (lane & 15)];
#pragma unroll
            for (int h = 0; h < GRAM_DENSE; h += 4) {
                acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(px[h * A_LD], pi[h * A_LD], acc[0], 0, 0, 0);
                if (bj <= bi) acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(po[h * A_LD], pi[h * A_LD], acc[1], 0, 0, 0);
            }
        };
        if (wv < GRAM_THREADS / 128) multiply();
        // chains k < GRAM_EPT are in the entry's own block, the others in the previous one
#pragma unroll
        for (int k = 0; k < GRAM_EPT; ++k) {
            const unsigned slot = key[k] != NO_KEY ? sh.head[old][key[k] >> GRAM_REST_BITS] : 0u;
            at[GRAM_EPT + k] = position(slot, seq - 1);
        }
#pragma unroll
        for (int k = GRAM_EPT - 1; k >= 0; --k) {
            unsigned own = at[k], prev = at[GRAM_EPT + k];
            const unsigned rest = key[k] & REST;
            while (own != CHAIN_END || prev != CHAIN_END) {
                GramEntry a = {CHAIN_END, 0.f}, b = a;
                if (own != CHAIN_END) a = sh.entry[cur][own];
                if (prev != CHAIN_END) b = sh.entry[old][prev];
                if (own != CHAIN_END && a.rest_next >> GRAM_POS_BITS == rest) {
                    const int j = (int)(own & (GRAM_THREADS - 1)) / GRAM_LPR;
                    if (j != e_row) atomicAdd(&sh.Go[own_at(min(j, e_row), max(j, e_row))], (double)(e_val[k] * a.val));
                }
                if (prev != CHAIN_END && b.rest_next >> GRAM_POS_BITS == rest)
                    atomicAdd(&sh.Gx[(int)(prev & (GRAM_THREADS - 1)) / GRAM_LPR][e_row], (double)(e_val[k] * b.val));
                own = a.rest_next & CHAIN_END;
                prev = b.rest_next & CHAIN_END;
            }
        }
        if (wv >= GRAM_THREADS / 128) multiply();
        __syncthreads();

        // ---- 3. summed, scaled and written out (result layout of a product: register r of lane l is row 4 (l / 16) + r, column
        // l % 16); what the next tile adds into starts from zero
        {
            float *out = tiles + (int64_t)tile * TILE_FLOATS;
            const int i = 16 * bi + (lane & 15), j0 = 16 * bj + 4 * (lane >> 4);
            const float si = R.scale[i] * R.sgn[i];
            float4_v x, o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x[e] = (float)(sh.Gx[j0 + e][i] + (double)acc[0][e]) * si * P.sgn[j0 + e];
                sh.Gx[j0 + e][i] = 0.0;
                if (j0 + e < i) {
                    o[e] = (float)(sh.Go[own_at(j0 + e, i)] + (double)acc[1][e]) * si * R.sgn[j0 + e];
                    sh.Go[own_at(j0 + e, i)] = 0.0;
                }
            }
            *reinterpret_cast<float4_v *>(out + tile_at(j0, i)) = x;
            *reinterpret_cast<float4_v *>(out + tile_at(BATCH + j0, i)) = o;
        }
        clear_half((seq + 1) & 1);
        if (wv == RESOLVER) {
            publish(LB, sh.rows[(slot + 2) & 3]);
            lookup3(LA);
        }
#pragma unroll
        for (int k = 0; k < GRAM_EPT; ++k) { e_col[k] = n_col[k]; e_val[k] = n_val[k]; }
        __syncthreads();
    }
}
static_assert(GRAM_THREADS == 64 * 16, "a wavefront per 16 x 16 block of either half of the tile");

// Fill row_chunk for one (solver, chunk) list entry per workgroup.
__global__ __launch_bounds__(256) void fill_row_chunk(const ChunkDev *__restrict__ chunks,
                                                      const int32_t *__restrict__ solver_chunks,
                                                      const int32_t *__restrict__ list_base, int32_t *row_chunk)
{
    const int ci = solver_chunks[blockIdx.x];
    const int n = chunks[ci].n_rows;
    int32_t *dst = row_chunk + list_base[blockIdx.x];
    for (int r = threadIdx.x; r < n; r += 256) dst[r] = ci;
}

}  // namespace chicle
