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
//   spread_unique    on the whole chip: the entries of unshared columns, from the steps the second kernel leaves.
// Where the merge takes the updates of long rows from the steps' coefficients (merge_pays), the third kernel runs only when a caller
// asks for a solver's update.
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
    int32_t row;                                // context-wide row index (a readable one also where st is nullptr)
    int32_t lr;                                 // ... and the solver's local one
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

// What the rows of a solver come to in segments: all of them, the row with the most, the sum of their squares.
struct SegStat { double squares; int32_t total, longest; };
// One workgroup per chunk; stat starts at zero.
__global__ __launch_bounds__(256) void segment_stats(const ChunkDev *__restrict__ chunks, const int32_t *__restrict__ owner,
                                                     const SegRef *__restrict__ refs, int G, int64_t n_total, SegStat *stat)
{
    __shared__ SegStat part[4];
    const ChunkDev &ch = chunks[blockIdx.x];
    SegStat s = {0.0, 0, 0};
    for (int r = threadIdx.x; r < ch.n_rows; r += 256) {
        int n = 0;
        for (int g = 0; g < G; ++g) n += refs[(int64_t)g * n_total + ch.row_base + r].n;
        s.squares += (double)n * (double)n;
        s.total += n;
        s.longest = max(s.longest, n);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        s.squares += __shfl_xor(s.squares, o, 64);
        s.total += __shfl_xor(s.total, o, 64);
        s.longest = max(s.longest, __shfl_xor(s.longest, o, 64));
    }
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x != 0) return;
    SegStat *out = stat + owner[blockIdx.x];
    atomicAdd(&out->squares, part[0].squares + part[1].squares + part[2].squares + part[3].squares);
    atomicAdd(&out->total, part[0].total + part[1].total + part[2].total + part[3].total);
    atomicMax(&out->longest, max(max(part[0].longest, part[1].longest), max(part[2].longest, part[3].longest)));
}

// ---- tiles ----------------------------------------------------------------------------------------------------------

constexpr int GB_SLOTS = 8192;                  // hash slots, columns in parts
constexpr int GB_POST = 6144;                   // entries joined at a time
constexpr int GB_EPT = 12;                      // entries per thread, all at once
constexpr int GB_ALL = GB_EPT * SB_THREADS;     // a block of no more entries is joined at once, from registers
constexpr int GB_ALL_SLOTS = 16384;
constexpr int GB_DENSE_MIN = 6;                 // columns that this many rows of the block hold go through a dense product,
constexpr int GB_DENSE = 96;                    // this many at a time (their values' place: [GB_DENSE][GB_LD])
constexpr int GB_MARK = 0x8000;                 // cursor of such a column's slot: this and its number
constexpr int GB_LD = BATCH + 1;

struct GramBlocksShared {
    union {
        struct {                                // columns in parts
            double G[BATCH][GB_LD];             // accumulators [j][i] (doubles: see GramShared)
            int keys[GB_SLOTS];
            int cursor[GB_SLOTS];               // entries per slot, then where the slot's list goes on; at the end: where it ends
            float post_val[GB_POST];
            unsigned char post_row[GB_POST];
            SegRef refs[SB_MAX_G][BATCH];
        } p;
        struct {                                // all entries at once
            union {
                int keys[GB_ALL_SLOTS];         // until every entry knows its slot
                struct {
                    double G[BATCH][GB_LD];     // from then on
                    float A[GB_DENSE][GB_LD];   // [column][row]
                };
            };
            unsigned short cursor[GB_ALL_SLOTS];
            float post_val[GB_ALL];
            union {
                unsigned char post_row[GB_ALL];
                struct { int pref[SB_MAX_G * BATCH + 1], begin[SB_MAX_G * BATCH]; };   // until the entries are loaded: segments
            };                                  // of (member, row), running count and place
        } a;
    };
    float sgn[BATCH], scale[BATCH];
    int row[BATCH];
    int scan[SB_THREADS / 64];
    int total, in_part;
};

// The block's entries joined at once.  A thread holds up to twelve entries of its own in registers (a segment's eight
// entries lie in eight neighbouring lanes), so that all their loads are in flight together and no entry is looked up
// twice.  Columns that one row of the block holds take no part in the lists.  G is left in sh.a.G.
__device__ __forceinline__ void join_all(GramBlocksShared &sh, int G, const int32_t *__restrict__ segs)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int n_seg = sh.a.pref[G * BATCH];
    // an entry: its value, and first its column, then where its column is: slot | row << 14 | entries of the column << 20
    int pk[GB_EPT];
    float val[GB_EPT];
    constexpr int SLOT = GB_ALL_SLOTS - 1;
    unsigned long long rows[2] = {0, 0};         // rows of the entries until then, six bits each
#pragma unroll
    for (int k = 0; k < GB_EPT; ++k) {
        const int s = (tid >> 3) + k * (SB_THREADS / 8);
        pk[k] = -1; val[k] = 0.f;
        if (s < n_seg) {
            int at = 0;                          // largest with pref[at] <= s
            for (int o = G * BATCH / 2; o > 0; o >>= 1)
                if (sh.a.pref[at + o] <= s) at += o;
            const int32_t *w = segs + (int64_t)(sh.a.begin[at] + s - sh.a.pref[at]) * SB_SEG_WORDS + (tid & 7);
            pk[k] = w[0] * G + (at >> 6);
            val[k] = __int_as_float(w[SB_SEG]);
            rows[k / 10] |= (unsigned long long)(at & 63) << (6 * (k % 10));
        }
    }
    {
        int4 *q = reinterpret_cast<int4 *>(sh.a.keys);
        for (int i = tid; i < GB_ALL_SLOTS / 4; i += SB_THREADS) q[i] = make_int4(-1, -1, -1, -1);
        int4 *c = reinterpret_cast<int4 *>(sh.a.cursor);
        for (int i = tid; i < GB_ALL_SLOTS / 8; i += SB_THREADS) c[i] = make_int4(0, 0, 0, 0);
    }
    __syncthreads();
    unsigned *packed = reinterpret_cast<unsigned *>(sh.a.cursor);      // two 16-bit counters share a word
#pragma unroll
    for (int k = 0; k < GB_EPT; ++k) {
        if (val[k] == 0.f) { pk[k] = -1; continue; }
        int h = (int)(((unsigned)pk[k] * 2654435761u) >> 18);
        for (;;) {                               // ends: three quarters as many entries as slots at most
            const int prev = atomicCAS(&sh.a.keys[h], -1, pk[k]);
            if (prev == -1 || prev == pk[k]) break;
            h = (h + 1) & SLOT;
        }
        pk[k] = h | (int)(rows[k / 10] >> (6 * (k % 10)) & 63) << 14;
        atomicAdd(packed + (h >> 1), (h & 1) ? 0x10000u : 1u);
    }
    __syncthreads();
    // lists of the slots with two entries or more: exclusive scan, 16 slots per thread; G takes the keys' place
    constexpr int SPT = GB_ALL_SLOTS / SB_THREADS;
    // (the scanned word: list entries in the lower 16 bits, columns for the dense product in the upper)
    auto weight = [](int n) { return n >= GB_DENSE_MIN ? 0x10000 : n > 1 ? n : 0; };
    unsigned cnt[SPT / 2];
    int sum = 0;
#pragma unroll
    for (int k = 0; k < SPT / 2; ++k) {
        cnt[k] = packed[tid * (SPT / 2) + k];
        sum += weight((int)(cnt[k] & 0xffff)) + weight((int)(cnt[k] >> 16));
    }
    int incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    if (lane == 63) sh.scan[wv] = incl;
    for (int i = tid; i < BATCH * GB_LD; i += SB_THREADS) (&sh.a.G[0][0])[i] = 0.0;
#pragma unroll
    for (int k = 0; k < GB_EPT; ++k)             // -1 from here on: takes no part
        if (pk[k] >= 0) {
            const int n = sh.a.cursor[pk[k] & SLOT];
            pk[k] = n < 2 ? -1 : pk[k] | n << 20;
        }
    __syncthreads();
    int off = incl - sum;
    for (int w = 0; w < wv; ++w) off += sh.scan[w];
    auto start = [&](int n) {
        const unsigned at = n >= GB_DENSE_MIN ? (unsigned)(GB_MARK | (off >> 16)) : (unsigned)(off & 0xffff);
        off += weight(n);
        return at;
    };
#pragma unroll
    for (int k = 0; k < SPT / 2; ++k) {
        const unsigned a = start((int)(cnt[k] & 0xffff)), b = start((int)(cnt[k] >> 16));
        packed[tid * (SPT / 2) + k] = a | (b << 16);
    }
    if (tid == SB_THREADS - 1) sh.in_part = off >> 16;
    __syncthreads();
    // columns many rows hold (the head of a Zipf distribution: every pair of rows shares some of them): a product of
    // dense columns on the matrix cores, 12 wavefronts for three 32 x 32 blocks times a quarter of the columns
    const int n_dense = sh.in_part;
    if (n_dense > 0) {
        floatx16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
        const int quad = wv % 3, j0 = quad == 2 ? 32 : 0, i0 = quad == 0 ? 0 : 32;
        for (int d0 = 0; d0 < n_dense; d0 += GB_DENSE) {
            __syncthreads();
            for (int i = tid; i < GB_DENSE * GB_LD; i += SB_THREADS) (&sh.a.A[0][0])[i] = 0.f;
            __syncthreads();
#pragma unroll
            for (int k = 0; k < GB_EPT; ++k)
                if (pk[k] >= GB_DENSE_MIN << 20) {
                    const int at = (sh.a.cursor[pk[k] & SLOT] & (GB_MARK - 1)) - d0;
                    if (at >= 0 && at < GB_DENSE) sh.a.A[at][pk[k] >> 14 & 63] = val[k];
                }
            __syncthreads();
            if (wv < 12) {
                const int c0 = wv / 3 * (GB_DENSE / 4) + (lane >> 5);
#pragma unroll 4
                for (int c = 0; c < GB_DENSE / 4; c += 2)
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(sh.a.A[c0 + c][j0 + (lane & 31)], sh.a.A[c0 + c][i0 + (lane & 31)], acc, 0, 0, 0);
            }
        }
        if (wv < 12) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                atomicAdd(&sh.a.G[j0 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)][i0 + (lane & 31)], (double)acc[r]);
        }
    }
#pragma unroll
    for (int k = 0; k < GB_EPT; ++k) {
        if (pk[k] < 0 || pk[k] >= GB_DENSE_MIN << 20) continue;
        const int slot = pk[k] & SLOT;
        const unsigned old = atomicAdd(packed + (slot >> 1), (slot & 1) ? 0x10000u : 1u);
        const int pos = (slot & 1) ? old >> 16 : old & 0xffff;
        sh.a.post_val[pos] = val[k];
        sh.a.post_row[pos] = (unsigned char)(pk[k] >> 14 & 63);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < GB_EPT; ++k) {
        if (pk[k] < 0 || pk[k] >= GB_DENSE_MIN << 20) continue;
        // (the slot's cursor has reached its list's end)
        const int i = pk[k] >> 14 & 63, pe = sh.a.cursor[pk[k] & SLOT], pb = pe - (pk[k] >> 20);
        for (int p = pb; p < pe; p += 4) {       // four list members per round of LDS latency
            int j[4];
            float x[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) { const int pm = min(p + m, pe - 1); j[m] = sh.a.post_row[pm]; x[m] = sh.a.post_val[pm]; }
#pragma unroll
            for (int m = 0; m < 4; ++m)
                if (p + m < pe && j[m] < i) atomicAdd(&sh.a.G[j[m]][i], (double)(val[k] * x[m]));
        }
    }
    __syncthreads();
}

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
                if (takes_steps(q)) {
                    row.st = ch.st + r;
                    row.row = ch.row_base + r;
                    row.lr = lr;
                    sgn = LOSS == 1 ? 1.f : st.x;
                    scale = tile_scale<LOSS>(q, c);
                }
            }
        }
        sh.sgn[tid] = sgn; sh.scale[tid] = scale; sh.row[tid] = row.st != nullptr ? row.row : -1;
        reinterpret_cast<BlockRow *>(out + BATCH * BATCH)[tid] = row;
    }
    __syncthreads();
    SegRef ref = {0, 0};                         // thread: (member, row)
    static_assert(SB_MAX_G * BATCH <= SB_THREADS, "one thread per member and row");
    if (tid < G * BATCH) {
        const int r = sh.row[lane];
        if (r >= 0) ref = refs[(int64_t)wv * n_total + r];
    }
    {
        int incl = ref.n;                        // running count over members, then rows
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        if (lane == 63) sh.scan[wv] = incl;
        __syncthreads();
        int before = 0;
        for (int w = 0; w < wv; ++w) before += sh.scan[w];
        if (tid < G * BATCH) {
            sh.a.pref[tid + 1] = before + incl;
            sh.a.begin[tid] = ref.begin;
        }
        if (tid == 0) sh.a.pref[0] = 0;
        if (tid == SB_THREADS - 1) sh.total = (before + incl) * SB_SEG;
    }
    __syncthreads();
    const int total = sh.total;
    const bool at_once = total <= GB_ALL;
    if (at_once) {
        join_all(sh, G, segs);
    } else {
    __syncthreads();
    if (tid < G * BATCH) sh.p.refs[wv][lane] = ref;
    for (int i = tid; i < BATCH * GB_LD; i += SB_THREADS) (&sh.p.G[0][0])[i] = 0.0;
    __syncthreads();
    // a wavefront takes every 16th row, a lane every 64th entry of it
    auto each_entry = [&](auto f) __attribute__((always_inline)) {
        for (int i = wv; i < BATCH; i += SB_THREADS / 64)
            for (int g = 0; g < G; ++g) {
                const SegRef ref = sh.p.refs[g][i];
                for (int q = lane; q < ref.n * SB_SEG; q += 64) {
                    const int32_t *w = segs + (int64_t)(ref.begin + q / SB_SEG) * SB_SEG_WORDS + q % SB_SEG;
                    const float v = __int_as_float(w[SB_SEG]);
                    if (v != 0.f) f(i, (unsigned)(w[0] * G + g), v);
                }
            }
    };
    int lp = 0;                                  // 2^lp parts
    while (((int64_t)GB_POST << lp) < (int64_t)total && lp < 16) ++lp;
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
        for (int i = tid; i < GB_SLOTS; i += SB_THREADS) { sh.p.keys[i] = -1; sh.p.cursor[i] = 0; }
        __syncthreads();
        each_entry([&](int, unsigned key, float) {
            const unsigned hash = key * 2654435761u;
            if (!mine(hash)) return;
            int h = slot0(hash);
            for (;;) {                           // ends: fewer entries than slots
                const int prev = atomicCAS(&sh.p.keys[h], -1, (int)key);
                if (prev == -1 || prev == (int)key) break;
                h = (h + 1) & (GB_SLOTS - 1);
            }
            atomicAdd(&sh.p.cursor[h], 1);
        });
        __syncthreads();
        {                                        // exclusive scan, 8 slots per thread
            int v[GB_SLOTS / SB_THREADS], sum = 0;
#pragma unroll
            for (int k = 0; k < GB_SLOTS / SB_THREADS; ++k) { v[k] = sh.p.cursor[tid * (GB_SLOTS / SB_THREADS) + k]; sum += v[k]; }
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
            for (int k = 0; k < GB_SLOTS / SB_THREADS; ++k) { sh.p.cursor[tid * (GB_SLOTS / SB_THREADS) + k] = off; off += v[k]; }
        }
        __syncthreads();
        auto find = [&](unsigned key, unsigned hash) {
            int h = slot0(hash);
            while (sh.p.keys[h] != (int)key) h = (h + 1) & (GB_SLOTS - 1);          // (it is there)
            return h;
        };
        each_entry([&](int i, unsigned key, float v) {
            const unsigned hash = key * 2654435761u;
            if (!mine(hash)) return;
            const int pos = atomicAdd(&sh.p.cursor[find(key, hash)], 1);
            sh.p.post_val[pos] = v;
            sh.p.post_row[pos] = (unsigned char)i;
        });
        __syncthreads();
        each_entry([&](int i, unsigned key, float v) {
            const unsigned hash = key * 2654435761u;
            if (!mine(hash)) return;
            const int h = find(key, hash);
            const int pb = h ? sh.p.cursor[h - 1] : 0, pe = sh.p.cursor[h];
            if (pe - pb < 2) return;
            for (int p = pb; p < pe; p += 4) {   // four list members per round of LDS latency
                int j[4];
                float x[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) { const int pk = min(p + k, pe - 1); j[k] = sh.p.post_row[pk]; x[k] = sh.p.post_val[pk]; }
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (p + k < pe && j[k] < i) atomicAdd(&sh.p.G[j[k]][i], (double)(v * x[k]));
            }
        });
        __syncthreads();
    }
    }
    const int i = lane, jq = wv;
    const float si = sh.scale[i] * sh.sgn[i];
    float4_v v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int j = 4 * jq + e;
        v[e] = j < i ? (float)(at_once ? sh.a.G[j][i] : sh.p.G[j][i]) * si * sh.sgn[j] : 0.f;
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
    float *coef_out;                            // per row (solver by solver): its coefficient in the update, for spread_unique
    float *coef_by_row;                         // the same by context-wide row (nullptr: not wanted)
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
        int incl = ref.n;                        // running sum over the lanes, register to register
#define CHICLE_DPP_SCAN(ctrl, rows) incl += __builtin_amdgcn_update_dpp(0, incl, ctrl, rows, 0xF, false)
        CHICLE_DPP_SCAN(0x111, 0xF);             // row_shr 1, 2, 4, 8, then row_bcast 15 and 31
        CHICLE_DPP_SCAN(0x112, 0xF);
        CHICLE_DPP_SCAN(0x114, 0xF);
        CHICLE_DPP_SCAN(0x118, 0xF);
        CHICLE_DPP_SCAN(0x142, 0xA);
        CHICLE_DPP_SCAN(0x143, 0xC);
#undef CHICLE_DPP_SCAN
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
            bool rough = true;                   // see logistic_block
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
                        t = hinge_scale(q, A.sc.c) * (rw - y * xu);
                        lo = -a; hi = 1.f - a;
                    } else if (LOSS == 1) {
                        t = (A.sc.c / (A.sc.c + q)) * (rw - a - xu);
                    } else {
                        t = rw - y * xu;
                        hi = q * A.sc.inv_c;
                        root = logistic_root(t, hi, a);
                    }
                }
                const float dl = dense_recurrence<LOSS, BATCH, false>(reinterpret_cast<const float *>(&sh.T[0][0]), t, lo, hi, a, root, lane, rough);
                const float coef = dl * (LOSS == 1 ? 1.f : y) * A.sc.inv_c;
                sh.coef[lane] = coef;
                if (g == 0 && cur_row.st != nullptr) {
                    float an = a + dl;
                    if (LOSS != 1) an = fminf(fmaxf(an, 0.f), 1.f);
                    gst(&cur_row.st->alpha, an);
                    gst(A.coef_out + S.perm_off + cur_row.lr, coef);
                    if (A.coef_by_row) gst(A.coef_by_row + cur_row.row, coef);
                }
                keep_loaded(nxt);
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
                // (wavefront 1's own loads first: it waits for last block's before it asks for anything new)
                if (resolver) {
                    publish(b + 2, refs_ahead);
                    refs_ahead = ref_of(rows_ahead);
                    rows_ahead = row_of(b + 4);
                    sh.dot[(b + 1) & 1][lane] = 0.0;      // (last read in block b - 1)
                }
                next_seg = load(segment(b + 1, t, next_row));
                fetch_T(b + 1);
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

// The updates of columns that a single row of the solver holds.  Where there is room, the assignment lays out for every
// place of a solver's compact vector which of its rows writes there and the row's value (lr = -1: a shared column); the
// update is then one stream over the vector, with the steps' coefficients in LDS.  (Row by row a scattered 4-byte store
// per entry is bound by the compute unit's address path, about seven cycles each whichever cache it hits: 1.8 ms for 92
// million of them, against 0.33 ms here.)
struct UniqueSource { int32_t lr; float val; };
constexpr int SPREAD_LDS_ROWS = 12288;           // coefficients of so many rows are staged in LDS
constexpr int SPREAD_PER = 4096;                 // places per workgroup

__global__ __launch_bounds__(256) void unique_sources(const ChunkDev *__restrict__ chunks, const int32_t *__restrict__ owner,
                                                      const int32_t *__restrict__ chunk_first, const int64_t *__restrict__ u_off,
                                                      UniqueSource *src)
{
    const ChunkDev &ch = chunks[blockIdx.y];
    const int32_t *cid = chunk_compact_ids(ch);
    UniqueSource *out = src + u_off[owner[blockIdx.y]];
    const int lane = threadIdx.x & 63, first = chunk_first[blockIdx.y];
    for (int r = blockIdx.x * 4 + (threadIdx.x >> 6); r < ch.n_rows; r += gridDim.x * 4)
        for (int p = ch.row_ptr[r] + lane; p < ch.row_ptr[r + 1]; p += 64) {
            const int c = cid[p];
            if (c < 0) out[vec_index(c)] = UniqueSource{first + r, ch.val[p]};
        }
}

// Grid: (workgroups over a solver's places, solver).
__global__ __launch_bounds__(256) void spread_unique(const SolverDev *__restrict__ solvers, const int32_t *__restrict__ columns,
                                                     const UniqueSource *__restrict__ src, const float *__restrict__ coef,
                                                     float *u_all, const int64_t *__restrict__ u_off, int lds_rows)
{
    extern __shared__ float sp_coef[];
    const int k = blockIdx.y, n = columns[k];
    const int64_t base = u_off[k];
    const SolverDev S = solvers[k];
    const float *cf = coef + S.perm_off;
    const int i0 = (int)blockIdx.x * SPREAD_PER, i1 = min(n, i0 + SPREAD_PER);
    if (i0 >= n) return;
    const bool staged = S.n_rows <= lds_rows;
    if (staged)
        for (int i = threadIdx.x; i < S.n_rows; i += 256) sp_coef[i] = cf[i];
    __syncthreads();
    const UniqueSource *s = src + base;
    float *u = u_all + base;
    for (int i = i0 + threadIdx.x; i < i1; i += 4 * 256) {
        UniqueSource q[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) q[j] = i + 256 * j < i1 ? s[i + 256 * j] : UniqueSource{-1, 0.f};
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (q[j].lr >= 0) u[i + 256 * j] = (staged ? sp_coef[q[j].lr] : cf[q[j].lr]) * q[j].val;
    }
}

// Without that room: one wavefront per row.  all: also of rows whose coefficient is zero (the vectors were not zero before).
// Grid: (blocks over rows, chunk).
__global__ __launch_bounds__(256) void scatter_unique(const ChunkDev *__restrict__ chunks, const int32_t *__restrict__ owner,
                                                      const SolverDev *__restrict__ solvers, const int32_t *__restrict__ chunk_first,
                                                      const float *__restrict__ coef, float *u_all, const int64_t *__restrict__ u_off, bool all)
{
    const ChunkDev &ch = chunks[blockIdx.y];
    const int32_t *cid = chunk_compact_ids(ch);
    const int k = owner[blockIdx.y];
    float *u = u_all + u_off[k];
    const float *of = coef + solvers[k].perm_off + chunk_first[blockIdx.y];
    const int lane = threadIdx.x & 63;
    for (int r = blockIdx.x * 4 + (threadIdx.x >> 6); r < ch.n_rows; r += gridDim.x * 4) {
        const float cf = of[r];
        if (cf == 0.f && !all) continue;
        const int e = ch.row_ptr[r + 1];
        for (int p = ch.row_ptr[r] + lane; p < e; p += 256) {
            int c[4];
            float v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) { c[j] = p + 64 * j < e ? cid[p + 64 * j] : 0; v[j] = p + 64 * j < e ? ch.val[p + 64 * j] : 0.f; }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (c[j] < 0) u[vec_index(c[j])] = cf * v[j];
        }
    }
}

}  // namespace chicle
