// Local solver for sparse rows of any length, blocks of 64 coordinate steps at a time; the same sequence of steps as the
// row-wise solver (paper Section 2.2: L = 1, H = all local samples).
//
// Of the entries of a solver's rows only those matter to the other steps whose column another row of the solver holds
// as well ("shared"; see mark_columns).  A column that a single row holds is zero in the private vector when its row's
// turn comes, and what the step adds there nobody reads before the merge.  The pass is therefore three kernels:
//   gram_blocks      one workgroup per 64 rows, on the whole chip: T of the block (the recurrence of sdca_batched.hpp)
//                    from the shared entries, by a hash join in LDS;
//   sdca_blocks      per solver a cluster of G workgroups, each with a part of the shared columns' private vector in
//                    LDS for the whole pass: gather, recurrence, scatter;
//   scatter_unique   on the whole chip: the entries of unshared columns, from the steps the second kernel leaves.
// A step of the row-wise solvers costs a trip to memory (1.7 us for rows of 36 entries, 2.9 us for rows of a thousand on
// four workgroups); here 64 steps cost one recurrence (2e3 cycles) and as much again for gather and scatter.
//
// Shared entries are laid out once per assignment, per row and cluster member, in segments of eight (eight indices, eight
// values: 64 bytes, the row's last segment filled up with zeros).  A thread takes a segment, so rows of 10 and of 1000
// entries load the wavefronts alike.  The shared columns of a solver are numbered 0, 1, ...; member g owns those with
// number mod G = g, at place number / G.
#pragma once
#include <hip/hip_runtime.h>
#include "device_types.hpp"
#include "mem.hpp"
#include "sdca_batched.hpp"
#include "sdca_batched_split.hpp"
#include "sdca_dense.hpp"

namespace chicle {

constexpr int SB_SEG = 8;                       // entries per segment
constexpr int SB_SEG_WORDS = 2 * SB_SEG;
constexpr int SB_MAX_G = 8;                     // cluster members per solver at most
constexpr int SB_THREADS = 1024;
constexpr int SB_WORKERS = SB_THREADS - 64;     // wavefront 0 runs the recurrence
constexpr int SB_RING = 4;                      // blocks a ring between members holds (they are at most one block apart)
constexpr int SB_RING_WORDS = SB_MAX_G * SB_RING * BATCH;   // 64-bit words per solver

struct SegRef { int32_t begin, n; };            // a row's segments in one member's columns
struct BlockRow {
    RowState *st;                               // nullptr: a row that takes no step
    int32_t row;                                // context-wide row index (readable tables also where st is nullptr)
    int32_t unused;
};
static_assert(sizeof(BlockRow) == sizeof(DenseRow), "a tile of this solver has the size of a dense one");

// ---- laid out once per assignment ---------------------------------------------------------------------------------

// number[k][c] of shared columns comes from prefix counts over the solver's `multi` bitmap; place[off[k] + number] = the
// column's index in the solver's compact private vector.  Grid: (blocks over words, solver).
__global__ __launch_bounds__(256) void shared_places(const unsigned *__restrict__ bits, const int32_t *__restrict__ pref,
                                                     const unsigned *__restrict__ multi, const int32_t *__restrict__ mpref,
                                                     int64_t words, const int64_t *__restrict__ off, int32_t *place)
{
    const int64_t base = (int64_t)blockIdx.y * words;
    for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < words; j += (int64_t)gridDim.x * 256) {
        unsigned m = multi[base + j];
        if (m == 0u) continue;
        const unsigned b = bits[base + j];
        const int p = pref[base + j];
        int32_t *out = place + off[blockIdx.y] + mpref[base + j];
        for (; m; m &= m - 1) {
            const unsigned below = (m & (0u - m)) - 1u;
            *out++ = p + __popc(b & below);
        }
    }
}

// The shared entries of every row, by member, in segments.  One wavefront per row, 4 rows per workgroup; segments are
// taken from *next, one addition per workgroup.  Grid: (blocks over rows, chunk).
__global__ __launch_bounds__(256) void build_segments(const ChunkDev *__restrict__ chunks, const int32_t *__restrict__ owner,
                                                      const unsigned *__restrict__ multi, const int32_t *__restrict__ mpref,
                                                      int64_t words, int G, int64_t n_total, SegRef *refs, int32_t *segs,
                                                      int *next, int capacity)
{
    __shared__ int cnt[4][SB_MAX_G], first[4][SB_MAX_G];
    const ChunkDev &ch = chunks[blockIdx.y];
    const int32_t *cid = chunk_compact_ids(ch);
    const int64_t base = (int64_t)owner[blockIdx.y] * words;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int r0 = blockIdx.x * 4; r0 < ch.n_rows; r0 += gridDim.x * 4) {
        const int r = r0 + wv;
        const int b = r < ch.n_rows ? ch.row_ptr[r] : 0, e = r < ch.n_rows ? ch.row_ptr[r + 1] : 0;
        auto number_of = [&](int p) -> int {     // -1: not shared
            if (p >= e || cid[p] < 0) return -1;
            const int c = ch.col[p];
            return mpref[base + (c >> 5)] + __popc(multi[base + (c >> 5)] & ((1u << (c & 31)) - 1u));
        };
        int mine = 0;                            // lane g < G: the row's entries of member g
        for (int p = b; p < e; p += 64) {
            const int s = number_of(p + lane);
            for (int g = 0; g < G; ++g) {
                const int n = __popcll(__ballot(s >= 0 && s % G == g));
                if (lane == g) mine += n;
            }
        }
        if (lane < G) cnt[wv][lane] = (mine + SB_SEG - 1) / SB_SEG;
        __syncthreads();
        if (threadIdx.x == 0) {
            int sum = 0;
            for (int w = 0; w < 4; ++w)
                for (int g = 0; g < G; ++g) { first[w][g] = sum; sum += cnt[w][g]; }
            const int at = sum ? atomicAdd(next, sum) : 0;
            for (int w = 0; w < 4; ++w)
                for (int g = 0; g < G; ++g) first[w][g] += at;
        }
        __syncthreads();
        if (r < ch.n_rows) {
            if (lane < G) refs[lane * n_total + ch.row_base + r] = SegRef{first[wv][lane], cnt[wv][lane]};
            int done[SB_MAX_G];
#pragma unroll
            for (int g = 0; g < SB_MAX_G; ++g) done[g] = 0;
            for (int p = b; p < e; p += 64) {
                const int s = number_of(p + lane);
                const float v = s >= 0 ? ch.val[p + lane] : 0.f;
#pragma unroll
                for (int g = 0; g < SB_MAX_G; ++g) {
                    if (g >= G) break;
                    const bool is = s >= 0 && s % G == g;
                    const unsigned long long m = __ballot(is);
                    if (is) {
                        const int q = done[g] + __popcll(m & ((1ull << lane) - 1ull));
                        const int seg = first[wv][g] + q / SB_SEG;
                        if (seg < capacity) {
                            int32_t *w = segs + (int64_t)seg * SB_SEG_WORDS + q % SB_SEG;
                            w[0] = s / G;
                            w[SB_SEG] = __float_as_int(v);
                        }
                    }
                    done[g] += __popcll(m);
                }
            }
#pragma unroll
            for (int g = 0; g < SB_MAX_G; ++g) {
                if (g >= G) break;
                const int q = done[g] + lane, seg = first[wv][g] + q / SB_SEG;       // the rest of the last segment
                if (q < cnt[wv][g] * SB_SEG && seg < capacity) {
                    int32_t *w = segs + (int64_t)seg * SB_SEG_WORDS + q % SB_SEG;
                    w[0] = 0;
                    w[SB_SEG] = 0;
                }
            }
        }
        __syncthreads();
    }
}

// ---- tiles ----------------------------------------------------------------------------------------------------------

constexpr int GB_SLOTS = 8192;                  // hash slots
constexpr int GB_POST = 6144;                   // entries joined at a time
constexpr int GB_LD = BATCH + 1;

struct GramBlocksShared {
    double G[BATCH][GB_LD];                     // accumulators [j][i] (doubles: see GramShared)
    int keys[GB_SLOTS];
    int cursor[GB_SLOTS];                       // entries per slot, then where the slot's list goes on; at the end: where it ends
    float post_val[GB_POST];
    unsigned char post_row[GB_POST];
    SegRef refs[SB_MAX_G][BATCH];
    float sgn[BATCH], scale[BATCH];
    int row[BATCH];
    int scan[SB_THREADS / 64];
    int total, in_part;
};

// One workgroup per tile.  Entries are inserted into an open-addressing table keyed by column, counted per slot, laid
// out as lists of (row, value) by a scan, and every entry adds its products with the earlier rows of its column's list.
// Where the 64 rows hold more entries than the lists do, the columns are taken in parts, by the leading bits of the hash
// (a part that is still too large halves the parts: different columns differ in the hash, so this ends).
template <int LOSS>
__global__ __launch_bounds__(SB_THREADS) void gram_blocks(
    const ChunkDev *__restrict__ chunks, const SolverDev *__restrict__ solvers, const int32_t *__restrict__ row_chunk,
    const int32_t *__restrict__ chunk_first, const int32_t *__restrict__ perm, const int32_t *__restrict__ tile_solver,
    float *tiles, int G, int64_t n_total, const SegRef *__restrict__ refs, const int32_t *__restrict__ segs, float c, int *err)
{
    extern __shared__ __align__(16) unsigned char gb_smem[];
    GramBlocksShared &sh = *reinterpret_cast<GramBlocksShared *>(gb_smem);
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const SolverDev S = solvers[tile_solver[blockIdx.x]];
    float *out = tiles + (int64_t)blockIdx.x * DENSE_TILE_FLOATS;
    if (tid == 0) sh.total = 0;
    for (int i = tid; i < BATCH * GB_LD; i += SB_THREADS) (&sh.G[0][0])[i] = 0.0;
    if (tid < BATCH) {
        const int t = ((int)blockIdx.x - S.tile_begin) * BATCH + tid;
        BlockRow row = {nullptr, 0, 0};
        float sgn = 1.f, scale = 0.f;
        if (t < S.n_rows) {
            const int lr = perm[S.perm_off + t];
            if ((unsigned)lr >= (unsigned)S.n_rows) {
                atomicOr(err, ERR_PERM_RANGE);
            } else {
                const int ci = row_chunk[S.perm_off + lr];
                const ChunkDev &ch = chunks[ci];
                const int r = lr - chunk_first[ci];
                const float4_v st = gld_state(ch.st + r);
                const float q = st.z;
                if (q != 0.f) {
                    row.st = ch.st + r;
                    row.row = ch.row_base + r;
                    sgn = LOSS == 1 ? 1.f : st.x;
                    scale = LOSS == 0 ? -1.f / q : LOSS == 1 ? -1.f / (c + q) : -1.f / c;
                }
            }
        }
        sh.sgn[tid] = sgn; sh.scale[tid] = scale; sh.row[tid] = row.st != nullptr ? row.row : -1;
        reinterpret_cast<BlockRow *>(out + BATCH * BATCH)[tid] = row;
    }
    __syncthreads();
    for (int i = tid; i < G * BATCH; i += SB_THREADS) {
        const int r = sh.row[i & 63];
        const SegRef ref = r >= 0 ? refs[(i >> 6) * n_total + r] : SegRef{0, 0};
        sh.refs[i >> 6][i & 63] = ref;
        if (ref.n) atomicAdd(&sh.total, ref.n * SB_SEG);
    }
    __syncthreads();
    // a wavefront takes every 16th row, a lane every 64th entry of it
    auto each_entry = [&](auto f) __attribute__((always_inline)) {
        for (int i = wv; i < BATCH; i += SB_THREADS / 64)
            for (int g = 0; g < G; ++g) {
                const SegRef ref = sh.refs[g][i];
                for (int q = lane; q < ref.n * SB_SEG; q += 64) {
                    const int32_t *w = segs + (int64_t)(ref.begin + q / SB_SEG) * SB_SEG_WORDS + q % SB_SEG;
                    const float v = __int_as_float(w[SB_SEG]);
                    if (v != 0.f) f(i, (unsigned)(w[0] * G + g), v);
                }
            }
    };
    int lp = 0;                                  // 2^lp parts
    while (((int64_t)GB_POST << lp) < (int64_t)sh.total && lp < 16) ++lp;
    for (unsigned part = 0; part < (1u << lp); ++part) {
        auto mine = [&](unsigned h) { return lp == 0 || (h >> (32 - lp)) == part; };
        auto slot0 = [&](unsigned h) { return (int)((h << lp) >> 19); };          // the 13 bits that follow the part's
        if (lp > 0) {
            __syncthreads();
            if (tid == 0) sh.in_part = 0;
            __syncthreads();
            int n = 0;
            each_entry([&](int, unsigned key, float) { n += mine(key * 2654435761u); });
            if (n) atomicAdd(&sh.in_part, n);
            __syncthreads();
            if (sh.in_part > GB_POST) {
                if (lp == 16) {                  // (cannot be: more entries than 64 rows have of 2^16 columns)
                    if (tid == 0) atomicOr(err, ERR_PARTNER_TIMEOUT);
                    continue;
                }
                // finer parts; what the parts before this one have added stays
                part = 2u * part - 1u;
                ++lp;
                continue;
            }
        }
        for (int i = tid; i < GB_SLOTS; i += SB_THREADS) { sh.keys[i] = -1; sh.cursor[i] = 0; }
        __syncthreads();
        each_entry([&](int, unsigned key, float) {
            const unsigned hash = key * 2654435761u;
            if (!mine(hash)) return;
            int h = slot0(hash);
            for (;;) {                           // ends: fewer entries than slots
                const int prev = atomicCAS(&sh.keys[h], -1, (int)key);
                if (prev == -1 || prev == (int)key) break;
                h = (h + 1) & (GB_SLOTS - 1);
            }
            atomicAdd(&sh.cursor[h], 1);
        });
        __syncthreads();
        {                                        // exclusive scan, 8 slots per thread
            int v[GB_SLOTS / SB_THREADS], sum = 0;
#pragma unroll
            for (int k = 0; k < GB_SLOTS / SB_THREADS; ++k) { v[k] = sh.cursor[tid * (GB_SLOTS / SB_THREADS) + k]; sum += v[k]; }
            int incl = sum;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(incl, o, 64);
                if (lane >= o) incl += y;
            }
            if (lane == 63) sh.scan[wv] = incl;
            __syncthreads();
            int off = incl - sum;
            for (int w = 0; w < wv; ++w) off += sh.scan[w];
#pragma unroll
            for (int k = 0; k < GB_SLOTS / SB_THREADS; ++k) { sh.cursor[tid * (GB_SLOTS / SB_THREADS) + k] = off; off += v[k]; }
        }
        __syncthreads();
        auto find = [&](unsigned key, unsigned hash) {
            int h = slot0(hash);
            while (sh.keys[h] != (int)key) h = (h + 1) & (GB_SLOTS - 1);          // (it is there)
            return h;
        };
        each_entry([&](int i, unsigned key, float v) {
            const unsigned hash = key * 2654435761u;
            if (!mine(hash)) return;
            const int pos = atomicAdd(&sh.cursor[find(key, hash)], 1);
            sh.post_val[pos] = v;
            sh.post_row[pos] = (unsigned char)i;
        });
        __syncthreads();
        each_entry([&](int i, unsigned key, float v) {
            const unsigned hash = key * 2654435761u;
            if (!mine(hash)) return;
            const int h = find(key, hash);
            const int pb = h ? sh.cursor[h - 1] : 0, pe = sh.cursor[h];
            if (pe - pb < 2) return;
            for (int p = pb; p < pe; p += 4) {   // four list members per round of LDS latency
                int j[4];
                float x[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) { const int pk = min(p + k, pe - 1); j[k] = sh.post_row[pk]; x[k] = sh.post_val[pk]; }
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (p + k < pe && j[k] < i) atomicAdd(&sh.G[j[k]][i], (double)(v * x[k]));
            }
        });
        __syncthreads();
    }
    const int i = lane, jq = wv;
    const float si = sh.scale[i] * sh.sgn[i];
    float4_v v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int j = 4 * jq + e;
        v[e] = j < i ? (float)sh.G[j][i] * si * sh.sgn[j] : 0.f;
    }
    *reinterpret_cast<float4_v *>(out + tile_at(4 * jq, i)) = v;
}
static_assert(SB_THREADS / 64 * 4 == BATCH, "every wavefront writes four steps of the tile");

// ---- the pass -------------------------------------------------------------------------------------------------------

struct BlocksShared {
    float4_v T[BATCH / 4][BATCH];
    double dot[2][BATCH];
    int pref[4][BATCH + 1];                     // segments of the block's rows before each row, four blocks in turn
    int begin[4][BATCH];
    float coef[BATCH];
    int dead;
};
// Shared columns per member.  UT: double where the members' LDS holds them (LDS additions run at the rate of its pipeline
// for doubles and lane by lane for floats), else float.
template <typename UT>
constexpr int SB_CAP = (int)((160 * 1024 - sizeof(BlocksShared)) / sizeof(UT)) & ~63;

struct BlocksArgs {
    const SolverDev *solvers;
    const ChunkDev *chunks;
    const float *tiles;
    float *u_all;
    const int64_t *u_off, *place_off;
    const int32_t *place, *count;               // where shared columns lie in the compact vector; how many there are
    const SegRef *refs;
    const int32_t *segs;
    float *coef_out;                            // per row of the context: its coefficient in the update, for scatter_unique
    int64_t n_total;
    int G, k_pad;
    RoundScalars sc;
    int *err;
    unsigned long long *rings;
};

// The members' partial dot products, summed in member order (one ring word per lane and member, all of them requested by
// each poll).  The wait is bounded as in ring_wait.
__device__ __forceinline__ float rings_sum(const unsigned long long *word, int g, int G, float own, int tag, int *dead, int *err)
{
    for (int spins = 0;; ++spins) {
        float v[SB_MAX_G];
        bool ok = true;
#pragma unroll
        for (int m = 0; m < SB_MAX_G; ++m) {
            v[m] = 0.f;
            if (m < G && m != g) {
                const unsigned long long x = __hip_atomic_load(word + m * SB_RING * BATCH, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ok = ok && (int)(x >> 32) == tag;
                v[m] = __uint_as_float((unsigned)x);
            } else if (m == g) {
                v[m] = own;
            }
        }
        float sum = 0.f;
#pragma unroll
        for (int m = 0; m < SB_MAX_G; ++m) sum += v[m];
        if (__builtin_amdgcn_ballot_w64(!ok) == 0ull) return sum;
        __builtin_amdgcn_s_sleep(1);
        if (*dead) return sum;                   // (only this wavefront uses it)
        if (spins > SPLIT_SPIN_LIMIT) {
            *dead = 1;
            atomicOr(err, ERR_PARTNER_TIMEOUT);
            return sum;
        }
    }
}

// Workgroup member * k_pad + k (k_pad: a multiple of the number of L2 partitions workgroups are dealt over, so a solver's
// members share one).  Members form their dot products, hand them to each other through rings of tagged 64-bit words and
// all take the same steps from the same sums, in member order.  Wavefront 0 runs the recurrence; meanwhile the others
// load the next block's segments and tile.  Three workgroup barriers per block.  Bounded waits: see ring_wait.
template <int LOSS, typename UT>
__global__ __launch_bounds__(SB_THREADS) void sdca_blocks(BlocksArgs A)
{
    extern __shared__ __align__(16) unsigned char sb_smem[];
    BlocksShared &sh = *reinterpret_cast<BlocksShared *>(sb_smem);
    UT *u = reinterpret_cast<UT *>(sb_smem + sizeof(BlocksShared));
    const int g = (int)blockIdx.x / A.k_pad, sid = (int)blockIdx.x % A.k_pad, G = A.G;
    if (sid >= A.sc.K) return;
    const SolverDev S = A.solvers[sid];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (g == 0) stamp_solver(A.sc, sid, 0);
    const int nb = (S.n_rows + BATCH - 1) / BATCH;
    const int n_shared = A.count[sid], n_loc = n_shared > g ? (n_shared - g + G - 1) / G : 0;
    for (int i = tid; i < n_loc; i += SB_THREADS) u[i] = (UT)0;
    if (tid < 2 * BATCH) (&sh.dot[0][0])[tid] = 0.0;
    if (tid == 0) sh.dead = 0;
    const float *my_tiles = A.tiles + (int64_t)S.tile_begin * DENSE_TILE_FLOATS;
    const SegRef *refs = A.refs + (int64_t)g * A.n_total;
    auto row_of = [&](int b) __attribute__((always_inline)) {
        return reinterpret_cast<const BlockRow *>(my_tiles + (int64_t)min(b, nb - 1) * DENSE_TILE_FLOATS + BATCH * BATCH)[lane];
    };
    // segments of block b's rows (lane = row) -> LDS, with the running count
    auto publish = [&](int b, SegRef ref) __attribute__((always_inline)) {
        int incl = ref.n;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        sh.begin[b & 3][lane] = ref.begin;
        sh.pref[b & 3][lane + 1] = incl;
        if (lane == 0) sh.pref[b & 3][0] = 0;
    };
    auto ref_of = [&](const BlockRow &r) __attribute__((always_inline)) {
        SegRef ref = refs[r.row];
        if (r.st == nullptr) ref.n = 0;
        return ref;
    };
    if (nb > 0) {
        if (wv == 0) {
            unsigned long long *ring = A.rings + (int64_t)sid * SB_RING_WORDS;
            BlockRow cur_row = row_of(0), next_row = row_of(1);
            const RowState *any = A.chunks[0].st;
            float4_v cur = gld_state(cur_row.st != nullptr ? cur_row.st : any);
            __syncthreads();                     // (the workers' first block is loaded)
            __syncthreads();
            for (int b = 0; b < nb; ++b) {
                const float4_v nxt = gld_state(next_row.st != nullptr ? next_row.st : any);
                const BlockRow far_row = row_of(b + 2);
                __syncthreads();                 // the dot products are in
                float xu = (float)sh.dot[b & 1][lane];
                if (G > 1) {
                    ring_put(ring + (g * SB_RING + (b & (SB_RING - 1))) * BATCH + lane, xu, b + 1);
                    xu = rings_sum(ring + (b & (SB_RING - 1)) * BATCH + lane, g, G, xu, b + 1, &sh.dead, A.err);
                }
                const float y = cur.x, a = cur.y, q = cur.z, rw = cur.w;
                float t = 0.f, lo = 0.f, hi = 0.f, root = 0.f;
                if (cur_row.st != nullptr) {
                    if (LOSS == 0) {
                        t = (A.sc.c / q) * (rw - y * xu);
                        lo = -a; hi = 1.f - a;
                    } else if (LOSS == 1) {
                        t = (A.sc.c / (A.sc.c + q)) * (rw - a - xu);
                    } else {
                        t = rw - y * xu;
                        hi = q * A.sc.inv_c;
                        root = logistic_root(t, hi, a);
                    }
                }
                const float dl = dense_recurrence<LOSS, BATCH, false>(reinterpret_cast<const float *>(&sh.T[0][0]), t, lo, hi, a, root, lane);
                const float coef = dl * (LOSS == 1 ? 1.f : y) * A.sc.inv_c;
                sh.coef[lane] = coef;
                if (g == 0 && cur_row.st != nullptr) {
                    float an = a + dl;
                    if (LOSS != 1) an = fminf(fmaxf(an, 0.f), 1.f);
                    gst(&cur_row.st->alpha, an);
                    gst(A.coef_out + cur_row.row, coef);
                }
                cur_row = next_row; next_row = far_row; cur = nxt;
                __syncthreads();                 // the steps are known
                __syncthreads();                 // ... and added
            }
        } else {
            const int t = tid - 64;              // worker
            const bool resolver = wv == 1;
            BlockRow rows_ahead = {nullptr, 0, 0};
            SegRef refs_ahead = {0, 0};
            if (resolver) {
                publish(0, ref_of(row_of(0)));
                publish(1, ref_of(row_of(1)));
                refs_ahead = ref_of(row_of(2));
                rows_ahead = row_of(3);
            }
            constexpr int TPT = (BATCH * BATCH / 4 + SB_WORKERS - 1) / SB_WORKERS;     // 16-byte words of T per worker
            float4_v t_in[TPT];
            auto fetch_T = [&](int b) __attribute__((always_inline)) {
                const float4_v *src = reinterpret_cast<const float4_v *>(my_tiles + (int64_t)min(b, nb - 1) * DENSE_TILE_FLOATS);
#pragma unroll
                for (int k = 0; k < TPT; ++k) t_in[k] = src[min(t + k * SB_WORKERS, BATCH * BATCH / 4 - 1)];
            };
            auto store_T = [&]() __attribute__((always_inline)) {
#pragma unroll
                for (int k = 0; k < TPT; ++k)
                    if (t + k * SB_WORKERS < BATCH * BATCH / 4) (&sh.T[0][0])[t + k * SB_WORKERS] = t_in[k];
            };
            // segment s of block b: its row (-1: there is no such segment) and place
            auto segment = [&](int b, int s, int &row) __attribute__((always_inline)) {
                const int *pref = sh.pref[b & 3];
                row = -1;
                if (s >= pref[BATCH]) return (const int32_t *)A.segs;
                int at = 0;                      // largest with pref[at] <= s (rows without segments are passed over)
#pragma unroll
                for (int o = 32; o > 0; o >>= 1)
                    if (pref[at + o] <= s) at += o;
                row = at;
                return (const int32_t *)(A.segs + (int64_t)(sh.begin[b & 3][at] + s - pref[at]) * SB_SEG_WORDS);
            };
            struct Seg { int4_a4 c0, c1; float4_a4 v0, v1; };
            auto load = [&](const int32_t *p) __attribute__((always_inline)) {
                return Seg{gld4(p), gld4(p + 4), gld4(reinterpret_cast<const float *>(p) + 8), gld4(reinterpret_cast<const float *>(p) + 12)};
            };
            auto gather = [&](const Seg &s, double *dot) __attribute__((always_inline)) {
                float p = 0.f;
#pragma unroll
                for (int e = 0; e < 4; ++e) p = fmaf(s.v0[e], (float)u[s.c0[e]], p);
#pragma unroll
                for (int e = 0; e < 4; ++e) p = fmaf(s.v1[e], (float)u[s.c1[e]], p);
                atomicAdd(dot, (double)p);
            };
            auto scatter = [&](const Seg &s, float cf) __attribute__((always_inline)) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (s.v0[e] != 0.f) atomicAdd(&u[s.c0[e]], (UT)(cf * s.v0[e]));
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (s.v1[e] != 0.f) atomicAdd(&u[s.c1[e]], (UT)(cf * s.v1[e]));
            };
            __syncthreads();                     // (wavefront 1 has published the first blocks)
            int row, next_row = -1;
            Seg seg = load(segment(0, t, row)), next_seg;
            fetch_T(0);
            store_T();
            __syncthreads();
            for (int b = 0; b < nb; ++b) {
                const int n_seg = sh.pref[b & 3][BATCH];
                if (row >= 0) gather(seg, &sh.dot[b & 1][row]);
                for (int s = t + SB_WORKERS; s < n_seg; s += SB_WORKERS) {      // beyond one segment per thread
                    int r;
                    const Seg more = load(segment(b, s, r));
                    gather(more, &sh.dot[b & 1][r]);
                }
                __syncthreads();
                // while the recurrence runs: the next block's segments and tile, the rows of those after it
                next_seg = load(segment(b + 1, t, next_row));
                fetch_T(b + 1);
                if (resolver) {
                    publish(b + 2, refs_ahead);
                    refs_ahead = ref_of(rows_ahead);
                    rows_ahead = row_of(b + 4);
                    sh.dot[(b + 1) & 1][lane] = 0.0;      // (last read in block b - 1)
                }
                __syncthreads();
                if (row >= 0) {
                    const float cf = sh.coef[row];
                    if (cf != 0.f) scatter(seg, cf);
                }
                for (int s = t + SB_WORKERS; s < n_seg; s += SB_WORKERS) {
                    int r;
                    const Seg more = load(segment(b, s, r));
                    const float cf = sh.coef[r];
                    if (cf != 0.f) scatter(more, cf);
                }
                store_T();
                seg = next_seg; row = next_row;
                __syncthreads();
            }
        }
    }
    __syncthreads();
    float *u_glb = A.u_all + A.u_off[sid];
    const int32_t *place = A.place + A.place_off[sid];
    for (int i = tid; i < n_loc; i += SB_THREADS) u_glb[place[i * G + g]] = (float)u[i];
    if (g == 0) stamp_solver(A.sc, sid, 1);
}

// The updates of columns that a single row of the solver holds.  One wavefront per row.  Grid: (blocks over rows, chunk).
__global__ __launch_bounds__(256) void scatter_unique(const ChunkDev *__restrict__ chunks, const int32_t *__restrict__ owner,
                                                      const float *__restrict__ coef, float *u_all, const int64_t *__restrict__ u_off)
{
    const ChunkDev &ch = chunks[blockIdx.y];
    const int32_t *cid = chunk_compact_ids(ch);
    float *u = u_all + u_off[owner[blockIdx.y]];
    const int lane = threadIdx.x & 63;
    for (int r = blockIdx.x * 4 + (threadIdx.x >> 6); r < ch.n_rows; r += gridDim.x * 4) {
        const float cf = coef[ch.row_base + r];
        if (cf == 0.f) continue;
        const int e = ch.row_ptr[r + 1];
        for (int p = ch.row_ptr[r] + lane; p < e; p += 256) {
            int c[4];
            float v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) { c[k] = p + 64 * k < e ? cid[p + 64 * k] : 0; v[k] = p + 64 * k < e ? ch.val[p + 64 * k] : 0.f; }
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (c[k] < 0) u[vec_index(c[k])] = cf * v[k];
        }
    }
}

}  // namespace chicle
