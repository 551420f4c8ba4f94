// C ABI of the CoCoA round (see include/chicle_round.h for the contract of every call).
// Host logic: chunk store carved from a caller-supplied arena, chunk -> solver tables, launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <numeric>
#include <string>
#include <thread>
#include <vector>

#include "../../include/chicle_round.h"
#include "aggregate_gap.hpp"
#include "column_order.hpp"
#include "device_types.hpp"
#include "gram_join.hpp"
#include "layout.hpp"
#include "policies.hpp"
#include "sdca_batched.hpp"
#include "sdca_batched_split.hpp"
#include "sdca_dense.hpp"
#include "sdca_dense_affine.hpp"
#include "sdca_rowwise.hpp"
#include "sdca_rowwise_cluster.hpp"
#include "sdca_sparse_blocks.hpp"
#include "split_pairs.hpp"

using namespace chicle;

namespace {

constexpr size_t ALIGN = 256;
constexpr int GAP_PARTS = 8192;        // workgroups (and partial sums) of the gap row kernels, at least
constexpr int WSQ_PARTS = 512;
constexpr int MAX_LIST_LDS = 768;      // chunks one solver may own (their descriptors are staged in LDS)
constexpr int DENSE_V_LDS_MAX_D = 8192;
constexpr int BATCHED_MAX_LIST = MAX_LIST_LDS;  // chunk descriptors of one solver the batched solver stages in LDS (they take
                                               // the place of columns of the private vector's LDS-resident head)
constexpr int RENUMBER_MAX_ROW = 64;   // rows are re-sorted by one thread each: short rows only
constexpr double LONG_ROW_AVG = 96.0;  // sparse rows longer than this on average: the row-wise solver uses whole workgroups per row

enum State { ST_LOADING = 0, ST_READY = 1, ST_EPOCH_DONE = 2 };

inline size_t align_up(size_t x) { return (x + ALIGN - 1) / ALIGN * ALIGN; }
inline int64_t pad_d(int64_t d) { return (d + 63) / 64 * 64; }
inline int64_t tiles_cap(int64_t n_total, int32_t max_solvers) { return n_total / BATCH + max_solvers + 1; }
inline size_t tile_bytes(bool dense) { return sizeof(float) * (size_t)(dense ? DENSE_TILE_FLOATS : TILE_FLOATS); }

// Vectors and visiting orders of at most so many bytes go through pinned memory that kernels write and read themselves: a copy and
// a wait less each.  One round of 1000 x 48 with orders from the host: 91.5 us and 54.0; four of 1500 long rows over 200k columns 448
// and 420.  Kernels read and write the link more slowly than copies do: rounds with orders of 262144 rows (1 MB) from the host 170 and 157, of
// 524288 230 and 229, of 1048576 394 and 431; read-outs of 1000 columns 37 and 14, of 65536 54 and 25, of 262144 99 and 67, of 1048576 250 and
// 237, of 2097152 389 and 457.  The line is below where they meet: what is pinned is held as long as the context.
constexpr size_t PINNED_HEAD = 256, PINNED_MOST = size_t(1) << 20;
constexpr int GAP_SPINS = 100000;                // reads of the word before the stream is waited for (a few milliseconds)
constexpr size_t READ_PIECE = size_t(2) << 20;   // bytes
constexpr int READ_THREADS = 6;

struct Seg {
    hipEvent_t start = nullptr, stop = nullptr;
    bool recorded = false;
};

// Partial sums of the gap kernels: one (loss, conjugate) pair per workgroup of the row pass, |w|^2 and |w|_1 partials.
struct GapScratch {
    double *loss = nullptr, *conj = nullptr, *wsq = nullptr, *wabs = nullptr;
    int parts = 0;            // length of loss[] and conj[]
    bool finish = false;      // the pass also forms the norms and the gap's sums
};

// Scratch of chicle_gap_noalloc: a fixed array in the code object, one copy per GPU, kept until the process
// ends.  Layout: GAP_PARTS loss partials, GAP_PARTS conjugate partials, WSQ_PARTS each for |w|^2 and |w|_1.
constexpr int STATIC_SCRATCH_DOUBLES = 2 * GAP_PARTS + 2 * WSQ_PARTS;
constexpr int MAX_DEVICES = 64;

}  // namespace

static __device__ __align__(256) double scratch[STATIC_SCRATCH_DOUBLES];

namespace {

// Device address of `scratch` on the current device (in host code the array's name is not one), looked
// up once per device.
double *scratch_ptr[MAX_DEVICES];
bool scratch_known[MAX_DEVICES];
std::mutex scratch_mutex;

hipError_t static_scratch_of_current_device(double **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_known[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        scratch_ptr[dev] = (double *)p;
        scratch_known[dev] = true;
    }
    *out = scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace

struct chicle_ctx {
    int loss = 0;
    int64_t n_total = 0;
    int32_t d = 0;
    int64_t ld_v = 0;
    double lambda = 0;
    double l1 = 0;             // elastic net: regulariser lambda (|w|^2 / 2 + l1 |w|_1); w64 then holds the dual image
    int32_t n_chunks = 0, max_solvers = 0;
    bool dense = false;        // chunks are dense row-major matrices, rows of dense_ld(d) floats
    int64_t total_entries = 0;
    char *arena = nullptr;
    size_t arena_bytes = 0, used = 0;
    hipStream_t stream = nullptr;
    State state = ST_LOADING;
    int solver_kind = CHICLE_SOLVER_AUTO;

    // fixed regions
    ChunkDev *chunks_dev = nullptr;
    SolverDev *solvers_dev = nullptr;
    int32_t *solver_chunks_dev = nullptr, *solver_prefix_dev = nullptr, *item_prefix_dev = nullptr;
    double *w64 = nullptr;     // shared vector (internal column order), double precision
    float *w = nullptr;        // its float mirror, gathered by the float kernels
    float *u = nullptr;        // private vectors as differences u_k = v_k - w, max_solvers x ld_v
    float *tmp_a = nullptr, *tmp_b = nullptr;   // d floats each: staging of host transfers
    int32_t *rank_of = nullptr, *col_of = nullptr;   // column renumbering tables (device)
    bool renumbered = false;
    int32_t max_row_len = 0;
    float *tiles[2] = {nullptr, nullptr};   // Gram tiles: one set in use by the chain, one being prepared
    int tile_buf = 0;                       // set the next chain kernel reads
    bool tiles_solved[2] = {false, false};  // dense rows, squared loss: the set holds the recurrence solved
    bool pairs_listed[2] = {false, false};  // short sparse rows: pairs were listed with the set (the solver kind may change
                                            // between forming a set and using it)
    hipStream_t side = nullptr;             // stream of Gram kernels prepared ahead
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    // Visiting orders announced for the next pass are copied here when they are announced (two buffers: the
    // running pass may itself read announced orders), so the caller's buffer is not referred to afterwards.
    int32_t *perm_ahead[2] = {nullptr, nullptr};
    int ahead_buf = 0;                      // buffer the next announcement goes to
    bool ahead_valid = false;               // perm_ahead[1 - ahead_buf] holds the orders of the next pass
    bool ahead_tiles = false;               // ... and their Gram tiles are in tiles[1 - tile_buf] (side stream)
    int32_t *tile_solver_dev = nullptr;
    int32_t *row_chunk_dev = nullptr, *chunk_first_dev = nullptr, *list_base_dev = nullptr;
    int64_t max_tiles = 0;
    int32_t n_tiles = 0;
    bool zw_valid = true;      // the rows' residuals match w (set at load time for w = 0)
    int32_t *perm_stage = nullptr;
    GapScratch gap_scratch;           // in the arena
    double *static_scratch = nullptr; // this device's copy of the fixed scratch array (chicle_gap_noalloc)
    // Pinned host memory: what the row pass's last workgroup writes (GapEnd; 6 doubles), then a word for the error flag, and from
    // PINNED_HEAD on a vector of up to PINNED_MOST bytes on its way out and visiting orders of as many on their way in.
    char *pinned = nullptr, *pinned_dev = nullptr;       // (as the host and as the device sees it)
    size_t pinned_vector = 0, pinned_orders = 0;         // where these two are; 0: there is none
    bool orders_in_flight = false;    // the orders there may not have been taken yet
    unsigned long long gap_seq = 0;
    int *err_dev = nullptr;
    unsigned *tickets_dev = nullptr;  // see n_tickets
    int *progress_dev = nullptr;      // per solver: block its batched pass has reached
    unsigned long long *split_ring_dev = nullptr;   // per solver: rings between the workgroups that share it
    unsigned long long *pair_list[2] = {nullptr, nullptr};   // per tile set: pairs of rows for the split solver, PAIR_CAP a tile,
    int32_t *pair_count[2] = {nullptr, nullptr};             // and how many there are (nullptr: no room, none are listed)
    std::vector<double> shares;       // [g]: over the columns of rank 64 g and on, sum of the squared shares of the rows that hold them
    bool split_allowed = true;        // the batched solver may spread a solver over several compute units
    int max_tail_entries = 0;         // most entries a row has outside the columns the batched solver keeps on chip
    // long sparse rows: several workgroups (a cluster) share every solver of the row-wise pass
    bool long_rows = false;           // average row longer than LONG_ROW_AVG
    int32_t *row_split_dev = nullptr; // per row: where the columns of cluster members 1.. begin
    unsigned long long *cluster_ring_dev = nullptr;
    int cluster = 1;                  // members per solver under the current assignment
    int split_built_for = 0;          // cluster size row_split_dev was built for
    // long rows: a copy of the entries by column (column_order.hpp), made at an assignment that has a use and room for it (copy_at)
    ColumnOrder columns{};            // blocks == 0: there is none
    long long *co_off_dev = nullptr;
    unsigned long long *co_count_dev = nullptr;
    double *co_z_dev = nullptr;       // co_parts x n_total shares of the rows' dot products
    float *co_coef_dev = nullptr;     // per row: its coefficient in the solvers' updates of the last pass
    bool dots_by_columns = false;     // the rows' dot products go over it (dots_pay)
    double fullest_bucket = 0.0;      // entries of the bucket that has most, over all blocks of rows
    bool merge_by_columns = false;    // ... is what the merge reads after a pass of the block solver (merge_pays)
    bool coef_pending = false;        // such a pass has left its updates there: private vectors lack the unshared columns
    bool updates_spread = false;      // ... until a caller asked for a solver's update
    bool private_stale = false;       // private vectors hold what has been merged from there, or what a failed pass has left
    bool cluster_allowed = true;
    // sparse rows longer than the batched solver takes: blocks over the columns that several rows of a solver hold
    bool blocks_ready = false;        // laid out for the current assignment
    int blocks_g = 1;                 // workgroups per solver
    bool blocks_double = true;        // its private vectors are kept in double
    int32_t *mpref_dev = nullptr;     // max_solvers x words: shared columns before each word
    int32_t *mcount_dev = nullptr;    // shared columns per solver; one more word: segments taken
    SegStat *seg_stat_dev = nullptr;  // per solver
    double crowding = -1.0;           // see column_crowding (< 0: not known yet)
    int64_t *place_off_dev = nullptr;
    float *coef_dev = nullptr;        // n_total
    unsigned long long *blocks_ring_dev = nullptr;
    char *layout_dev = nullptr;       // tiles, segment table, places and segments (in place of the batched solver's tile sets)
    size_t layout_bytes = 0;
    size_t layout_used = 0;           // ... of the current assignment's blocks
    SegRef *refs_dev = nullptr;
    UniqueSource *sources_dev = nullptr;   // u_used; nullptr: no room
    int most_columns = 0;             // most columns a solver's compact vector has
    int32_t *place_dev = nullptr, *segs_dev = nullptr;
    // Sparse chunks: private vectors are stored compactly (a solver touches a small part of the columns)
    bool compact = false;
    int64_t words = 0;                // 32-column words per bitmap
    unsigned *bits_dev = nullptr;     // max_solvers x words: columns a solver's chunks contain
    unsigned *multi_dev = nullptr;    // the same layout, columns that more than one row of the solver holds
    int32_t *pref_dev = nullptr;      // max_solvers x words: set bits before each word
    int32_t *count_dev = nullptr;     // max_solvers: columns per solver
    int64_t *u_off_dev = nullptr;     // max_solvers: start of each solver's compact vector in u
    int32_t *chunk_owner_dev = nullptr;
    int64_t u_capacity = 0;           // floats in u
    int64_t u_used = 0;               // floats of u in use under the current assignment (compact storage)
    int cu_count = 0;                 // compute units of the device
    long long *ticks_dev = nullptr;   // 2 per solver: clock at start / end of its last pass
    int wall_khz = 0;                 // rate of that clock
    bool epoch_ran = false;

    // host mirrors
    std::vector<ChunkDev> chunks;
    std::vector<char> loaded;
    int32_t n_loaded = 0;
    int64_t rows_loaded = 0, entries_loaded = 0;
    int32_t K = 0;
    std::vector<int32_t> chunk_to_solver;
    std::vector<SolverDev> solvers;
    int max_list = 0;
    int most_rows = 0;                // most rows a solver has
    int gap_lpr = 64, gap_items = 0, gap_hot_grid = 0;

    // read-out of large vectors: pinned pieces, one per copying thread (allocated by the first such read-out)
    int device = 0;
    char *read_pinned = nullptr;
    hipEvent_t read_ev[READ_THREADS] = {};

    bool profiling = false;
    Seg seg[CHICLE_SEG_COUNT];
    std::string err;
};

namespace {

int fail(chicle_ctx *c, int code, const char *fmt, ...)
{
    if (c) {
        char buf[512];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof buf, fmt, ap);
        va_end(ap);
        c->err = buf;
    }
    return code;
}

#define HIP_TRY(c, expr)                                                                         \
    do {                                                                                         \
        hipError_t e_ = (expr);                                                                  \
        if (e_ != hipSuccess)                                                                    \
            return fail((c), CHICLE_EDEVICE, "%s: %s", #expr, hipGetErrorString(e_));            \
    } while (0)

void *carve(chicle_ctx *c, size_t bytes)
{
    const size_t need = align_up(bytes);
    if (c->used + need > c->arena_bytes) return nullptr;
    void *p = c->arena + c->used;
    c->used += need;
    return p;
}

// Floats of private-vector storage: dense, one vector per solver; compact (long rows): a solver's vector
// holds only the columns its chunks contain, so all of them together hold at most one float per entry.
int64_t private_floats(int64_t total_entries, int64_t ld, int32_t max_solvers, bool long_rows)
{
    const int64_t dense = ld * (int64_t)max_solvers;
    return long_rows ? std::min(dense, total_entries + 64 * (int64_t)max_solvers) : dense;
}

// Room behind the tile sets for the shared entries of long rows: eight bytes per entry and four half-empty segments per row,
// and eight bytes per place of the private vectors, or per entry for the copy by column (copy_at).  Contexts of up to 96 entries a row on average have only the tile sets,
// of which the solver that takes rows of any length uses a quarter for its tiles: the rest holds about 89 shared entries a
// row where a solver has one workgroup, 84, 75 and 57 with two, four and eight.  Rows of more (60 to 96 entries, most of
// their columns shared) go row by row.
size_t long_row_layout_bytes(int64_t n_total, int64_t total_entries)
{
    return sizeof(int32_t) * (4 * (size_t)total_entries + 4 * (size_t)SB_SEG_WORDS * (size_t)n_total);
}

// The copy of long rows' entries by column (column_order.hpp): blocks of rows, columns of a bucket, buckets, and parts that a
// block's dot products are summed in.  Buckets are as wide as leaves the merge a thousand workgroups.
int co_blocks(int64_t n_total) { return (int)((n_total + CO_ROWS - 1) / CO_ROWS); }
int co_bucket_log2(int32_t d)
{
    int b = CO_MAX_BUCKET_LOG2;
    while (b > CO_MIN_BUCKET_LOG2 && (d >> b) < 1024) --b;
    return b;
}
int co_buckets(int32_t d) { return (int)(((int64_t)d + (1 << co_bucket_log2(d)) - 1) >> co_bucket_log2(d)); }
// As many parts as compute units have workgroups for, in whole multiples of the L2 partitions (column_part); from 33 blocks on, where
// that leaves fewer, the number up to CO_LEAST_PARTS that keeps the last round of workgroups fullest.
int co_parts(int64_t n_total)
{
    const int blocks = co_blocks(n_total), most = CO_PARTS / blocks;
    if (most >= L2_PARTITIONS) return most / L2_PARTITIONS * L2_PARTITIONS;
    auto rounds = [&](int parts) { return ((int64_t)blocks * parts + CO_PARTS - 1) / CO_PARTS; };
    int best = 1;
    for (int parts = 2; parts <= std::max(most, CO_LEAST_PARTS); ++parts)
        if (rounds(parts) * best < rounds(best) * parts) best = parts;
    return best;
}
// ... for so many entries: parts of some 4096 entries or more, and of two entries or more for each of the block's rows, whose sums a
// part writes out (16000 rows of 115, 256 parts 29 us, 128 25.6, 64 24.2; 4000 of 314, 256 19, 128 16.9, 64 19.4).
int dot_parts(int64_t n_total, int64_t entries)
{
    const int64_t most = std::min(entries / (4096 * (int64_t)co_blocks(n_total)), entries / (2 * n_total));
    const int parts = (int)std::max<int64_t>(1, std::min<int64_t>(co_parts(n_total), most));
    return parts < L2_PARTITIONS ? parts : parts / L2_PARTITIONS * L2_PARTITIONS;
}
// Where buckets begin, what counts them, the parts of the dot products and the coefficients.  In whole megabytes: what an arena grows by
// with the rows then does not depend, by the rounding of single arrays, on the columns, which the tests of its size rely on (for the
// times it makes no difference).  (The entries themselves lie in the room of the block solver's layout: copy_at.)
size_t co_offsets_bytes(int64_t n_total, int32_t d) { return align_up(sizeof(long long) * ((size_t)co_blocks(n_total) * (size_t)co_buckets(d) + 2)); }
size_t co_parts_bytes(int64_t n_total, int64_t entries) { return align_up(sizeof(double) * (size_t)dot_parts(n_total, entries) * (size_t)n_total); }
size_t co_scratch_bytes(int64_t n_total, int64_t entries, int32_t d)
{
    const size_t mb = size_t(1) << 20, bytes = 2 * co_offsets_bytes(n_total, d) + co_parts_bytes(n_total, entries) + align_up(sizeof(float) * ((size_t)n_total + 4));
    return (bytes + mb - 1) / mb * mb;
}

// Counters of workgroups that are done: the gap's, and one per workgroup's columns for the merge.  Zero between kernels.
size_t n_tickets(int32_t d) { return GAP_TICKETS + ((size_t)d + 32 * AGG_WORDS - 1) / (32 * AGG_WORDS); }

// Bytes of the split solver's two sets of pair lists, and of one.  They are reserved where that solver may have tails: the head
// keeps TAILS_MIN_HOT columns or more wherever there are tails, and rows longer than it takes are the rule in contexts of long
// rows.  (Where one of those is given short rows all the same, the lists take the place of the block solver's layout.)
constexpr int64_t TAILS_MIN_HOT = 2 * RING * BATCH * sizeof(RowSlot) / sizeof(double);
size_t pair_set_bytes(int64_t max_tiles) { return align_up(sizeof(unsigned long long) * PAIR_CAP * (size_t)max_tiles) + align_up(sizeof(int32_t) * (size_t)max_tiles); }
size_t pair_bytes(int64_t max_tiles, int32_t d, bool long_rows, bool compact)
{
    return compact && !long_rows && d > TAILS_MIN_HOT ? 2 * pair_set_bytes(max_tiles) : 0;
}

size_t fixed_bytes(int64_t n_total, int32_t d, int32_t n_chunks, int32_t max_solvers, bool long_rows, bool compact,
                   int64_t n_total_entries_hint)
{
    const int64_t ld = pad_d(d);
    size_t s = 0;
    s += align_up(sizeof(ChunkDev) * (size_t)n_chunks);
    s += align_up(sizeof(SolverDev) * (size_t)max_solvers);
    s += 2 * align_up(sizeof(int32_t) * (size_t)n_chunks);
    s += align_up(sizeof(int32_t) * ((size_t)n_chunks + 1));
    s += align_up(sizeof(float) * (size_t)ld) * 3;                       // w, tmp_a, tmp_b
    s += align_up(sizeof(double) * (size_t)ld);                          // w in double
    s += align_up(sizeof(float) * (size_t)private_floats(n_total_entries_hint, ld, max_solvers, long_rows));   // private vectors
    s += 2 * align_up(sizeof(int32_t) * (size_t)d);                      // renumbering tables
    s += 2 * align_up(tile_bytes(!compact) * (size_t)tiles_cap(n_total, max_solvers));
    if (long_rows) s += align_up(long_row_layout_bytes(n_total, n_total_entries_hint));
    s += align_up(sizeof(int32_t) * (size_t)tiles_cap(n_total, max_solvers));
    s += 4 * align_up(sizeof(int32_t) * (size_t)n_total);                // perm staging, announced orders (2), row -> chunk
    s += 2 * align_up(sizeof(int32_t) * (size_t)n_chunks);               // chunk_first, list_base
    s += 2 * align_up(sizeof(double) * (size_t)std::max(GAP_PARTS, 2 * n_chunks)) + 2 * align_up(sizeof(double) * WSQ_PARTS);
    s += align_up(sizeof(int));
    s += align_up(sizeof(unsigned) * n_tickets(d));
    s += align_up(sizeof(long long) * 2 * (size_t)max_solvers);
    s += align_up(sizeof(int) * (size_t)max_solvers);
    s += align_up(sizeof(unsigned long long) * (size_t)SPLIT_WORDS * (size_t)max_solvers);   // rings of the split batched solver
    if (long_rows) {
        s += align_up(co_scratch_bytes(n_total, n_total_entries_hint, d));
        s += align_up(sizeof(int32_t) * (size_t)SPLITS_PER_ROW * (size_t)n_total);
        s += align_up(sizeof(unsigned long long) * (size_t)CLUSTER_WORDS * (size_t)max_solvers);
    }
    if (compact) {
        const size_t words = ((size_t)d + 31) / 32;
        s += 2 * align_up(sizeof(int32_t) * words * (size_t)max_solvers);          // column bitmaps, prefix counts
        s += 2 * align_up(sizeof(int32_t) * words * (size_t)max_solvers);          // columns held by several rows, prefix counts
        s += align_up(sizeof(int32_t) * ((size_t)max_solvers + 1)) + align_up(sizeof(int64_t) * (size_t)max_solvers) + align_up(sizeof(SegStat) * (size_t)max_solvers);
        s += align_up(sizeof(float) * (size_t)n_total) + align_up(sizeof(unsigned long long) * (size_t)SB_RING_WORDS * (size_t)max_solvers);
        s += align_up(sizeof(int32_t) * (size_t)max_solvers) + align_up(sizeof(int64_t) * (size_t)max_solvers);
        s += align_up(sizeof(int32_t) * (size_t)n_chunks);
    }
    return s + pair_bytes(tiles_cap(n_total, max_solvers), d, long_rows, compact);
}

size_t chunk_bytes(bool dense, bool compact, int64_t n_rows, int64_t entries)
{
    size_t s = 0;
    if (!dense) {
        s += align_up(sizeof(int32_t) * (size_t)(n_rows + 1));
        s += align_up(sizeof(int32_t) * (size_t)(entries + ENTRY_SLACK)) * (compact ? 2 : 1);   // column ids (+ compact ids)
    }
    s += align_up(sizeof(float) * (size_t)(entries + ENTRY_SLACK));
    s += align_up(sizeof(RowState) * (size_t)n_rows);
    return s;
}

void seg_begin(chicle_ctx *c, int s)
{
    if (c->profiling) (void)hipEventRecord(c->seg[s].start, c->stream);
}
void seg_end(chicle_ctx *c, int s)
{
    if (c->profiling) {
        (void)hipEventRecord(c->seg[s].stop, c->stream);
        c->seg[s].recorded = true;
    }
}

// The kernels' error flag, which has been read out, as a status; it is cleared.
int flag_status(chicle_ctx *c, int flag)
{
    if (!flag) return CHICLE_OK;
    HIP_TRY(c, hipMemsetAsync(c->err_dev, 0, sizeof(int), c->stream));
    if (flag & ERR_PERM_RANGE)
        return fail(c, CHICLE_EDEVICE, "a visiting-order entry was outside [0, rows of its solver)");
    if (flag & ERR_PARTNER_TIMEOUT)
        return fail(c, CHICLE_EDEVICE, "the workgroups that share a solver lost each other; the pass is invalid");
    return fail(c, CHICLE_EDEVICE, "kernel error flag %d", flag);
}

int check_deferred(chicle_ctx *c)
{
    int flag = 0;
    HIP_TRY(c, hipMemcpyAsync(&flag, c->err_dev, sizeof(int), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    return flag_status(c, flag);
}

int grid_for(int64_t items, int per_block, int cap)
{
    int64_t g = (items + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

void clear_device_words(chicle_ctx *c, void *p, int64_t n_words)
{
    hipLaunchKernelGGL(clear_words, dim3(grid_for(n_words, 256, 256)), dim3(256), 0, c->stream, (unsigned *)p, n_words);
}

int clear_all_private(chicle_ctx *c)
{
    if (c->K <= 0) return CHICLE_OK;
    if (c->compact) {
        HIP_TRY(c, hipMemsetAsync(c->u, 0, sizeof(float) * (size_t)c->u_used, c->stream));
        return CHICLE_OK;
    }
    const int64_t d4 = c->ld_v / 4;
    hipLaunchKernelGGL(clear_private, dim3(grid_for(d4, 256, 4096)), dim3(256), 0, c->stream, c->u,
                       c->ld_v, d4, c->K);
    HIP_TRY(c, hipGetLastError());
    return CHICLE_OK;
}

RoundScalars scalars(const chicle_ctx *c)
{
    RoundScalars s;
    const double cc = c->lambda * (double)c->n_total / (double)c->K;
    s.c = (float)cc;
    s.inv_c = (float)(1.0 / cc);
    s.inv_sigma = (float)(1.0 / (double)c->K);
    s.K = c->K;
    s.ticks = c->ticks_dev;
    return s;
}

bool batched_eligible(const chicle_ctx *c)
{
    return !c->dense && c->max_row_len <= GRAM_MAX_ROW && c->max_list <= BATCHED_MAX_LIST;
}

// LDS layout of the batched solvers: BatchedShared, the solver's chunk descriptors and row prefixes, then
// the head of the private vector (the most popular columns, as many as fit), in double.
struct BatchedLayout { size_t hot_off, bytes; int n_hot; };
BatchedLayout batched_layout(const chicle_ctx *c)
{
    BatchedLayout L;
    const int ml = std::max(c->max_list, 1);
    L.hot_off = (sizeof(BatchedShared) + (sizeof(ChunkDev) + sizeof(int)) * (size_t)ml + 15) & ~(size_t)15;
    // (A context made for long rows holds its private vectors in as many floats as entries, and these columns take their place in
    // every solver's whether its rows hold them or not: 576 fewer there leave that much more for the columns the rows do hold.)
    const size_t room = LDS_BYTES - L.hot_off - (c->long_rows ? sizeof(double) * 576 : 0);
    L.n_hot = (int)std::min<int64_t>((int64_t)(room / sizeof(double)) & ~(int64_t)63, c->d);
    L.bytes = L.hot_off + sizeof(double) * (size_t)L.n_hot;
    return L;
}

// Dense rows narrow enough for two blocks of them to sit in registers.  (A caller that asks for the batched solver by name
// gets it up to DENSE_NAMED_MAX_D columns, the limit the interface states.)
constexpr int DENSE_NAMED_MAX_D = 320;
bool dense_eligible(const chicle_ctx *c, int32_t max_d) { return c->dense && c->d <= max_d; }

// Solvers of so few rows step through them one at a time faster than the tile kernel and the block kernel get under way.
// Whole rounds, row by row / in blocks.  Dense rows, four solvers of 4 rows: 64 columns 26 / 33 us, 1000 columns 42 / 56; of
// 8 rows 1000 columns equal; logistic loss, a run that continues (from alpha = 0), of 12 rows 64 columns 34 / 36 (36 / 38), 200 40 / 42
// (44 / 43), 400 46 / 47 (52 / 48), 1000 61 / 56 (75 / 59), 1500 73 / 65 (93 / 67), of 8 rows 50 / 56 (59 / 57) and 60 / 65 (74 / 66), of
// 16 rows 64 columns 38 / 36.  Sparse rows, 64 solvers: of 12 rows of 40 or 80
// entries 56 / 63 and 59 / 67, of 16 equal; of 8 rows of 120 (several workgroups share a solver, and a row takes longer)
// 59 / 66, of 12 equal.  Block kernels take a compute unit each, so more solvers than compute units queue up: 512 solvers of
// 10 rows of 400 columns 162 / 176, of 12 rows of 80 entries 84 / 92.
bool few_rows(const chicle_ctx *c)
{
    const int waves = (c->K + c->cu_count - 1) / c->cu_count;
    if (c->dense) return c->most_rows <= std::max(c->loss == CHICLE_LOSS_LOGISTIC && c->d <= 512 ? 12 : 8, 5 * waves);
    return c->most_rows <= (c->long_rows ? std::max(8, 4 * waves) : std::max(12, 6 * waves));
}

// The solver of the next pass.
enum Route { ROUTE_ROWWISE = 0, ROUTE_BATCHED = 1, ROUTE_DENSE = 2, ROUTE_BLOCKS = 3 };
Route route_of(const chicle_ctx *c)
{
    const bool by_name = c->solver_kind == CHICLE_SOLVER_BATCHED;
    if (!by_name && c->solver_kind != CHICLE_SOLVER_AUTO) return ROUTE_ROWWISE;
    if (c->dense) {
        if (by_name) return dense_eligible(c, DENSE_NAMED_MAX_D) ? ROUTE_DENSE : ROUTE_ROWWISE;
        // (rows of up to 48 columns stay with the solver that sums the private vector in double)
        return dense_eligible(c, DENSE_MAX_D) && (c->d <= GRAM_MAX_ROW || !few_rows(c)) ? ROUTE_DENSE : ROUTE_ROWWISE;
    }
    if (batched_eligible(c)) return ROUTE_BATCHED;
    return !by_name && c->blocks_ready ? ROUTE_BLOCKS : ROUTE_ROWWISE;
}

// Tail workgroups per solver of the batched solver, or -1: every solver on one compute unit.  Columns outside the
// LDS-resident head, and compute units to spare: every solver gets a head workgroup and SPLIT_TAILS tail workgroups (all of
// them must be resident together: they wait for each other).  Where every column is in the LDS-resident head there is
// nothing for tails to do: the head workgroups run alone, and their gathers and scatters never leave LDS.
int split_tails(const chicle_ctx *c)
{
    const int n_hot = batched_layout(c).n_hot, n_tails = n_hot < c->d ? SPLIT_TAILS : 0;
    const int k_pad = (c->K + L2_PARTITIONS - 1) / L2_PARTITIONS * L2_PARTITIONS;
    // (chunk lists that leave the head fewer popular columns than the tails' state has room for: the solver on one compute unit)
    return c->split_allowed && (1 + n_tails) * k_pad <= c->cu_count &&
           (n_tails == 0 || n_hot >= TAILS_MIN_HOT) ? n_tails : -1;
}

// Squared loss, dense rows: whether tiles are formed with the recurrence solved (gram_dense).  The inverse costs a tile 12 us
// more in latency and the chip 0.010 us per tile, and saves a solver 0.34 us per block.  One solver in 4 of 64 rows of 64
// columns: 36 us solved, 24 not; of 8192 rows 180 and 201; one in 64 of 8192 rows of 28 columns 307 and 269.  Tiles formed a
// pass ahead cost nothing while they hide behind the steps: one in 4 of 2048 rows of 28 columns 62 and 77, one in 64 96 and
// 97, of 8192 rows 252 and 264, one in 300 977 and 713.
bool solve_tiles(const chicle_ctx *c, bool ahead)
{
    if (c->loss != CHICLE_LOSS_SQUARED) return false;
    const int blocks = (c->most_rows + BATCH - 1) / BATCH;
    return ahead ? c->K <= 64 && blocks >= 16 + c->K : (int64_t)blocks * (34 - c->K) > 1200;
}

// Rows per run of the solver for long passes over narrow dense rows (sdca_dense_affine.hpp); 0: it does not take this pass.
// It saves 0.7 us per block of 64 rows of the longest solver and costs the pass a kernel more, one run's latency and, over all
// solvers' rows, 0.1 ns per row and column.  Whole rounds, solved blocks / runs of 64 rows, us: one solver of 1000 rows of 16
// columns 52 / 55, of 4096 of 10 101 / 60, one in four of 1024 rows of 32 53 / 69, of 2048 75 / 70, of 3075 92 / 76, of 8192
// 168 / 101, one in 64 of 3073 of 28 154 / 130, one in 256 of 3072 of 32 376 / 327, of 8 327 / 211.
// Longer runs shorten the chain, and fewer maps have to be stored, but each then takes its latency several times.  Runs of 64
// and of 128: one solver of 16384 rows of 28 columns 114 and 113, of 8192 of 32 93 and 104, one in eight of 16250 of 28 147 and
// 133, one in 16 of 6250 of 32 110 and 119, one in 64 of 6250 of 28 191 and 178.  Of 128 and of 256: one in 16 of 31250 of 28
// 224 and 210, one in four of 125000 394 and 294, one in two of 250000 623 and 410.
int affine_run(const chicle_ctx *c)
{
    if (!c->dense || c->loss != CHICLE_LOSS_SQUARED || c->d > AFFINE_MAX_D || c->K > 65535) return 0;      // (a grid's second dimension)
    const int blocks = (c->most_rows + BATCH - 1) / BATCH;
    return blocks < 48 ? 0 : blocks < 192 && c->n_tiles < 4096 ? BATCH : blocks < 400 ? 2 * BATCH : 4 * BATCH;
}

// Whether the tiles of announced orders are formed ahead for dense rows.  The second stream costs a round about 20 us of
// calls, which hide only behind a pass that is long enough: rounds of four solvers of 64 rows of 64 columns 33 us without, 56
// with; of 1024 rows 56 and 59, of 256 columns 68 and 64, of 1000 columns 129 and 111; 64 solvers of 512 rows of 64 columns
// 65 and 69, of 1024 rows 89 and 78.  A pass that could go in runs is solved in blocks from such tiles where they cost it
// less: one in 32 of 3075 rows of 28 columns 104 in runs, 97 in blocks, of 4700 of 32 128 and 119, one in 64 of 4688 of 32 174
// and 157, one in 128 of 3073 of 24 170 and 148; one in 16 of 3075 of 28 92 and 89, one in 64 of 4096 of 28 and one in 128 of
// 6250 of 32 equal, one in 64 of 6250 of 28 178 and 202, one in 64 of 3073 of 8 96 and 117.
bool dense_tiles_ahead(const chicle_ctx *c)
{
    if (affine_run(c)) return c->d > 20 && c->most_rows <= 80 * BATCH && c->n_tiles >= 1024;
    return c->most_rows / BATCH + c->d / 64 >= 16 || c->n_tiles >= 1024;
}

// LDS a dense solver asks for at least where it is to have a compute unit to itself: no other solver, and no workgroup of the
// next pass's tile kernel, which runs beside it, is placed there.  Where there are more solvers than compute units and no
// tiles ahead, solvers share them (512 solvers of 64 rows of 64 columns: 32 us alone, 28 sharing; 1024 of 20 rows 47 and 39).
constexpr int DENSE_ALONE_LDS = 130 * 1024;

template <int LOSS, typename SH>
int launch_dense_shape(chicle_ctx *c, bool alone)
{
    auto kern = LOSS == 1 && c->tiles_solved[c->tile_buf] ? sdca_dense<LOSS, true, SH> : sdca_dense<LOSS, false, SH>;
    const size_t sh = std::max<size_t>(SH::LDS_BYTES, alone ? DENSE_ALONE_LDS : 0);
    HIP_TRY(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh));
    hipLaunchKernelGGL(kern, dim3(c->K), dim3(SH::THREADS), sh, c->stream, c->chunks_dev, c->solvers_dev,
                       (const float *)c->tiles[c->tile_buf], c->u, c->ld_v, (int)c->d, dense_ld((int)c->d), scalars(c));
    HIP_TRY(c, hipGetLastError());
    return CHICLE_OK;
}

// The narrowest shape that holds a row: lanes per row, wavefronts, 4-column groups per lane, rows per block.
template <int LOSS>
int launch_dense(chicle_ctx *c, bool alone)
{
    const int d = (int)c->d;
    if (LOSS == 1 && d <= 64 && c->tiles_solved[c->tile_buf]) {
        const int sh = alone ? DENSE_ALONE_LDS : 0;
        auto kern = d <= 32 ? sdca_dense_squared<DenseShape<8, 4, 1, 64>> : sdca_dense_squared<DenseShape<16, 4, 1, 64>>;
        HIP_TRY(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, DENSE_ALONE_LDS));
        hipLaunchKernelGGL(kern, dim3(c->K), dim3(256), sh, c->stream, c->chunks_dev, c->solvers_dev,
                           (const float *)c->tiles[c->tile_buf], c->u, c->ld_v, d, dense_ld(d), scalars(c));
        HIP_TRY(c, hipGetLastError());
        return CHICLE_OK;
    }
    if (d <= 32) return launch_dense_shape<LOSS, DenseShape<8, 4, 1, 64>>(c, alone);
    if (d <= 64) return launch_dense_shape<LOSS, DenseShape<16, 4, 1, 64>>(c, alone);
    if (d <= 128) return launch_dense_shape<LOSS, DenseShape<32, 8, 1, 64>>(c, alone);
    if (d <= 256) return launch_dense_shape<LOSS, DenseShape<64, 8, 1, 64>>(c, alone);
    if (d <= 512) return launch_dense_shape<LOSS, DenseShape<64, 8, 2, 64>>(c, alone);
    if (d <= 768) return launch_dense_shape<LOSS, DenseShape<64, 8, 3, 32>>(c, alone);
    if (d <= 1024) return launch_dense_shape<LOSS, DenseShape<64, 8, 4, 32>>(c, alone);
    if (d <= 1280) return launch_dense_shape<LOSS, DenseShape<64, 8, 5, 16>>(c, alone);
    return launch_dense_shape<LOSS, DenseShape<64, 8, 6, 16>>(c, alone);
}

template <int LOSS>
int launch_rowwise(chicle_ctx *c, const int32_t *perm)
{
    const RoundScalars sc = scalars(c);
    const size_t list_bytes = 2 * sizeof(int) * (size_t)std::max(c->max_list, 1);
    if (c->dense) {
        const bool v_lds = c->d <= DENSE_V_LDS_MAX_D;
        const size_t sh = list_bytes + (v_lds ? sizeof(float) * (size_t)c->d : 0);
        if (v_lds)
            hipLaunchKernelGGL((sdca_rowwise_dense<LOSS, 64, true>), dim3(c->K), dim3(64), sh, c->stream,
                               c->chunks_dev, c->solvers_dev, c->solver_chunks_dev, c->solver_prefix_dev,
                               perm, c->u, c->ld_v, (int)c->d, dense_ld((int)c->d), std::max(c->max_list, 1), sc, c->err_dev);
        else
            hipLaunchKernelGGL((sdca_rowwise_dense<LOSS, 256, false>), dim3(c->K), dim3(256), sh, c->stream,
                               c->chunks_dev, c->solvers_dev, c->solver_chunks_dev, c->solver_prefix_dev,
                               perm, c->u, c->ld_v, (int)c->d, dense_ld((int)c->d), std::max(c->max_list, 1), sc, c->err_dev);
    } else {
        const double avg = c->n_total ? (double)c->total_entries / (double)c->n_total : 0.0;
        const int ml = std::max(c->max_list, 1);
        const size_t sh = (sizeof(ChunkDev) + sizeof(int)) * (size_t)ml;
        if (c->long_rows && c->cluster > 1 && c->cluster_allowed) {
            // every solver shared by a cluster of workgroups on one L2 partition, each owning a range of columns
            const int k_pad = (c->K + L2_PARTITIONS - 1) / L2_PARTITIONS * L2_PARTITIONS;
            clear_device_words(c, c->cluster_ring_dev, 2 * (int64_t)CLUSTER_WORDS * c->K);
            hipLaunchKernelGGL((sdca_rowwise_csr_cluster<LOSS, 512, 2>), dim3(k_pad * c->cluster), dim3(512), sh, c->stream,
                               c->chunks_dev, c->solvers_dev, c->solver_chunks_dev, c->solver_prefix_dev,
                               perm, c->u, c->ld_v, ml, sc, c->err_dev, k_pad, c->cluster, c->row_split_dev,
                               c->cluster_ring_dev, c->u_off_dev);
        } else if (avg <= LONG_ROW_AVG)
            hipLaunchKernelGGL((sdca_rowwise_csr<LOSS, 64, 2>), dim3(c->K), dim3(64), sh, c->stream,
                               c->chunks_dev, c->solvers_dev, c->solver_chunks_dev, c->solver_prefix_dev,
                               perm, c->u, c->ld_v, ml, sc, c->err_dev, (const int64_t *)(c->compact ? c->u_off_dev : nullptr));
        else
            hipLaunchKernelGGL((sdca_rowwise_csr<LOSS, 512, 4>), dim3(c->K), dim3(512), sh, c->stream,
                               c->chunks_dev, c->solvers_dev, c->solver_chunks_dev, c->solver_prefix_dev,
                               perm, c->u, c->ld_v, ml, sc, c->err_dev, (const int64_t *)c->u_off_dev);
    }
    HIP_TRY(c, hipGetLastError());
    return CHICLE_OK;
}

// The last 24 entries of a row cover every row's columns outside the LDS-resident head.
bool short_tails(const chicle_ctx *c) { return c->compact && c->max_tail_entries <= 3 * LPR; }

// Solvers without tails, hinge and squared loss: whether rows are resolved by a wavefront of their own.  It is faster while tiles
// and entries stay in the memory-side cache (256 MB); where they do not, the tiles' loads set the pace and lookups between them
// are better issued by the wavefront that stages a tile.  Apart / not, 2000 columns, 20 solvers: 64000 rows of 40 entries 79.5 /
// 83.8 us, 256000 285 / 300, of 12 248 / 252; 384000 of 12 (233 MB) 395 / 390, 300000 of 44 (260 MB) 394 / 387, 546000 of 44 770 /
// 741; four solvers of 64000 rows of 40 1218 / 1296, of 96000 2240 / 2230.  With the logistic loss, whose chain takes longer than
// either, the wavefront more only takes issue slots: 20 solvers of 3200 rows of 40 entries, a run that continues 214 / 213 us and from
// alpha = 0 815 / 799, of 27300 of 44 1413 / 1400 and 6142 / 6031, 16 of 56000 of 20 2514 / 2499 and 12041 / 11815, four of
// 16000 of 40 746 / 742 and 2579 / 2547.
bool heads_resolve_apart(const chicle_ctx *c)
{
    return (double)tile_bytes(false) * c->n_tiles + 8.0 * (double)c->entries_loaded <= 224e6;
}

// Whether pairs are listed beside the tiles (ahead: of the pass after this one), for the split solver's look-back of four blocks.
// It saves up to 0.9 us per block of the longest solver.  Lists formed ahead cost the chip what the pass leaves of it: where the
// last 24 entries of a row are enough, 0.008 us per tile, which 80 solvers do not reach; where not, 0.029: four rounds of 16
// solvers of 12500 rows of 40 entries in uniform columns 2.93 ms without and 2.56 with, 64 of 4688 rows of 44 2.99 and 3.40.  A
// few blocks save less than the kernel's launch: rounds of one solver of 512 rows 74.7 us without and 78.4 with, of 768 73.8 and
// 70.9; of 16 of 384 72.5 and 75.0, of 640 84.5 and 82.4, of 768 91.4 and 86.3.
// Lists formed before the pass that uses them add their kernel to it: 4.5 us and 0.005 per tile, where the last 24 entries are not
// enough 8 and 0.03, and up to 0.05 where blocks have hundreds of pairs; smaller jobs save 0.65 us per block, from the fifth or
// so on.  Passes without and with: one solver of 1024 rows 69 us and 68, of 2560 122 and 103; 16 of 640 rows 64 and 70, of 2560
// 152 and 159 (uniform columns: 166 and 189); 17 of 11000 rows of some 20 to 46 532 and 494, 71 of 2260 rows of 7 155 and 144.
// With the logistic loss the chain takes longer than the tails from alpha = 0, where nothing is saved, and about as long on a run that
// continues, where it is 0.15 to 0.3 us per block and lists formed ahead cost more of it.  Passes without and with, continuing (from
// alpha = 0): one of 2560 rows 193 and 195, 16 of 2560 217 and 220 (494 and 506), 17 of 11000 691 and 676 (1815 and 1832), 32 of 9375
// 745 and 721 (1902 and 1924), eight of 40000 2173 and 2008 (5120 and 5094), 71 of 2260 rows of 10 250 and 260; ahead 17 of 11000 628
// and 585, 32 of 9375 645 and 571, eight of 40000 2140 and 1875, 32 of 3000 of 10 217 and 210; 48 of 3000 of 10 or 40 240 and 241, 309
// and 310; 64 280 and 301, 381 and 393, 80 352 and 358, 441 and 453 (871 and 898).
// Nothing is saved where blocks have more pairs than a list holds, which the columns' shares of the rows tell for rows in random order
// (16 solvers of 12500 rows of 48 entries in 16400 columns, 3.12 and 3.27).
bool lists_pairs(const chicle_ctx *c, bool ahead)
{
    if (split_tails(c) <= 0 || !c->pair_list[0]) return false;
    const int blocks = (c->most_rows + BATCH - 1) / BATCH;
    const bool narrow = short_tails(c);
    if (blocks < 12 || (!narrow && 32 * (int64_t)blocks <= c->n_tiles)) return false;
    const size_t at = (size_t)batched_layout(c).n_hot / 64;
    const double pairs = at < c->shares.size() ? (LAG - 2) * (double)(BATCH * BATCH) * c->shares[at] : 0.0;       // of a block
    if (pairs > 0.85 * PAIR_CAP) return false;
    const double us = narrow ? 4.5 + 0.005 * c->n_tiles : 8.0 + (0.03 + 6e-5 * pairs) * c->n_tiles;
    if (c->loss == CHICLE_LOSS_LOGISTIC) return ahead ? 5 * (1 + SPLIT_TAILS) * c->K <= 3 * c->cu_count : 0.15 * (blocks - 4) > us;
    return ahead || 0.65 * (blocks - 4) > us;
}

template <int TE>
int launch_pairs(chicle_ctx *c, const int32_t *perm, int buf, hipStream_t stream)
{
    auto kern = split_pairs<TE>;
    const size_t sh = sizeof(PairShared<TE>);
    HIP_TRY(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh));
    // runs as long as two workgroups per compute unit make them: every run looks through three blocks more than it lists
    const int run = std::min(PAIR_RUN, (c->n_tiles + 2 * c->cu_count - 1) / (2 * c->cu_count));
    hipLaunchKernelGGL(kern, dim3((c->n_tiles + run - 1) / run), dim3(PAIR_THREADS), sh, stream, c->chunks_dev, c->solvers_dev,
                       c->row_chunk_dev, c->chunk_first_dev, perm, c->tile_solver_dev, c->n_tiles, run, batched_layout(c).n_hot,
                       c->pair_list[buf], c->pair_count[buf]);
    return CHICLE_OK;
}

// Gram tiles of the given visiting orders into tile set `buf`, on `stream` (ahead: beside the pass before theirs), and the pairs
// that the split solver's tails leave out.
constexpr int GRAM_RUN = 32;
template <int LOSS>
int launch_gram(chicle_ctx *c, const int32_t *perm, int buf, bool ahead, hipStream_t stream)
{
    const RoundScalars sc = scalars(c);
    if (c->dense) {
        c->tiles_solved[buf] = solve_tiles(c, ahead);
        if (c->n_tiles > 0)
            hipLaunchKernelGGL(gram_dense<LOSS>, dim3(c->n_tiles), dim3(GD_THREADS), 0, stream, c->chunks_dev, c->solvers_dev,
                               c->row_chunk_dev, c->chunk_first_dev, perm, c->tile_solver_dev, c->tiles[buf],
                               dense_ld((int)c->d), sc.c, c->tiles_solved[buf], c->err_dev);
    } else if (c->n_tiles > 0) {
        auto kern = gram_tiles_join<LOSS>;
        HIP_TRY(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)sizeof(GramShared)));
        // Each workgroup takes a contiguous run of tiles, no more of them than GRAM_RUN: the compute units that are free (beside
        // a pass: those its solvers leave) take their share of the tiles in as few runs as that allows.  A run begins with
        // some 16 us of dependent loads, which 3 tiles do not hide (4688 tiles: 187 us in runs of 10, 173 in runs of 19); runs
        // without a limit would keep the next pass's solvers off their compute units.  (Solvers on one compute unit each have
        // another that reads ahead of them; ten rounds with that one counted as taken too: 100 solvers of 4000 rows of 30 entries
        // 5.69 ms and 5.57, 120 of 6667 11.6 and 11.4, 90 of 8889 10.8 and 11.0, 200 of 2000 equal.)
        const int free = ahead ? std::max(c->cu_count / 4, c->cu_count - (1 + std::max(0, split_tails(c))) * c->K) : c->cu_count;
        const int runs = (c->n_tiles + GRAM_RUN * free - 1) / (GRAM_RUN * free);
        const int grid = std::min(c->n_tiles, runs * free);
        hipLaunchKernelGGL(kern, dim3(grid), dim3(GRAM_THREADS), sizeof(GramShared), stream,
                           c->chunks_dev, c->solvers_dev, c->row_chunk_dev, c->chunk_first_dev, perm,
                           c->tile_solver_dev, c->tiles[buf], c->n_tiles, sc.c, c->err_dev);
        c->pairs_listed[buf] = lists_pairs(c, ahead);
        if (c->pairs_listed[buf]) {
            const int rc = short_tails(c) ? launch_pairs<3>(c, perm, buf, stream) : launch_pairs<ENT>(c, perm, buf, stream);
            if (rc) return rc;
        }
    }
    HIP_TRY(c, hipGetLastError());
    return CHICLE_OK;
}

int launch_affine(chicle_ctx *c, const int32_t *perm, int run)
{
    const RoundScalars sc = scalars(c);
    float *tiles = c->tiles[c->tile_buf];
    const int units = (c->most_rows + run - 1) / run, d = (int)c->d;
    auto grid = [&](int lanes) {                       // lanes per run
        const int per = 64 / lanes * AFFINE_WAVES;
        return dim3((units + per - 1) / per, c->K);
    };
    seg_begin(c, CHICLE_SEG_EPOCH_GRAM);
    static_assert(AFFINE_MAX_D == 32, "all row lengths of affine_maps");
    const dim3 mg = grid(d < 16 ? 16 : 32);
    // A workgroup's wavefronts are on a SIMD each, and rows long enough (maps of 500000 rows, 16 solvers, and of 60000, one, with
    // a row's words read ahead / not, between events, which adds some 7 us: 16 columns 65 / 64 and 47.4 / 45.7 us, 20 72 / 72
    // and 52.7 / 51.8, 24 78 / 78 and 58.1 / 58.2, 28 86 / 91 and 64.3 / 70.2, 30 94 / 98 and 71.9 / 76.4, 32 102 / 107 and
    // 79.8 / 83.8).
    const bool alone = d > 24 && (int64_t)mg.x * mg.y <= c->cu_count;
    auto maps = d <= 4 ? affine_maps<4, 16, true, false> : d <= 8 ? affine_maps<8, 16, true, false> : d <= 12 ? affine_maps<12, 16, true, false>
                : d < 16 ? affine_maps<16, 16, true, false>
                : d <= 16 ? affine_maps<16, 32, true, false> : d <= 20 ? affine_maps<20, 32, true, false> : d <= 24 ? affine_maps<24, 32, true, false>
                : d <= 28 ? (alone ? affine_maps<28, 32, true, true> : affine_maps<28, 32, true, false>)
                : d < 32 ? (alone ? affine_maps<32, 32, true, true> : affine_maps<32, 32, true, false>)
                : (alone ? affine_maps<32, 32, false, true> : affine_maps<32, 32, false, false>);
    hipLaunchKernelGGL(maps, mg, dim3(64 * AFFINE_WAVES), 0, c->stream, c->chunks_dev, c->solvers_dev, c->row_chunk_dev, c->chunk_first_dev, perm,
                       tiles, d, run, sc.c, sc.inv_c, c->err_dev);
    seg_end(c, CHICLE_SEG_EPOCH_GRAM);
    seg_begin(c, CHICLE_SEG_EPOCH_CHAIN);
    auto starts = d <= 8 ? affine_starts<1> : d <= 16 ? affine_starts<2> : d <= 24 ? affine_starts<3> : affine_starts<4>;
    hipLaunchKernelGGL(starts, dim3(c->K), dim3(64), 0, c->stream, c->solvers_dev, tiles, c->u, c->ld_v, d, run, sc);
    hipLaunchKernelGGL(affine_steps, grid(AFFINE_GROUP), dim3(64 * AFFINE_WAVES), 0, c->stream, c->chunks_dev, c->solvers_dev, tiles, run, dense_ld(d), sc);
    seg_end(c, CHICLE_SEG_EPOCH_CHAIN);
    HIP_TRY(c, hipGetLastError());
    return CHICLE_OK;
}

// The batched local pass.  Tiles of `perm` come from the set prepared ahead when there is one (the main stream has
// waited for it), else they are computed first on the main stream.  With perm_next, the tiles of the next pass are started
// on the side stream so that they run beside this pass's chain kernel (which occupies K of the 256
// compute units); they depend on the data and the orders only.
template <int LOSS>
int launch_batched(chicle_ctx *c, const int32_t *perm, bool tiles_ready, const int32_t *perm_next)
{
    const RoundScalars sc = scalars(c);
    int rc;
    const int run = tiles_ready ? 0 : affine_run(c);
    if (tiles_ready) {
        c->tile_buf = 1 - c->tile_buf;
    } else if (!run) {
        seg_begin(c, CHICLE_SEG_EPOCH_GRAM);
        rc = launch_gram<LOSS>(c, perm, c->tile_buf, false, c->stream);
        seg_end(c, CHICLE_SEG_EPOCH_GRAM);
        if (rc) return rc;
    }
    if (perm_next) HIP_TRY(c, hipEventRecord(c->ev_fork, c->stream));   // everything enqueued so far
    const int ml = std::max(c->max_list, 1);
    const BatchedLayout lay = batched_layout(c);
    const size_t hot_off = lay.hot_off, sh = lay.bytes;
    const int n_hot = lay.n_hot;
    const int64_t *u_off = c->compact ? c->u_off_dev : nullptr;
    const int k_pad = (c->K + L2_PARTITIONS - 1) / L2_PARTITIONS * L2_PARTITIONS;
    const int n_tails = split_tails(c);
    if (run) {
        rc = launch_affine(c, perm, run);
        if (rc) return rc;
    } else if (c->dense) {
        seg_begin(c, CHICLE_SEG_EPOCH_CHAIN);
        rc = launch_dense<LOSS>(c, perm_next != nullptr || c->K <= c->cu_count);
        seg_end(c, CHICLE_SEG_EPOCH_CHAIN);
        if (rc) return rc;
    } else if (n_tails >= 0) {
        SplitArgs A;
        A.chunks = c->chunks_dev; A.solvers = c->solvers_dev; A.solver_chunks = c->solver_chunks_dev;
        A.solver_prefix = c->solver_prefix_dev; A.perm = perm; A.tiles = c->tiles[c->tile_buf]; A.u_all = c->u;
        A.ld_v = c->ld_v; A.u_off = u_off; A.max_list = ml; A.n_hot = n_hot; A.hot_off = (int)hot_off; A.sc = sc;
        A.err = c->err_dev; A.xchg_all = c->split_ring_dev;
        A.lag = c->pairs_listed[c->tile_buf] ? LAG : 2; A.pair_list = c->pair_list[c->tile_buf]; A.pair_count = c->pair_count[c->tile_buf];
        // a tail's lanes take the last 24 entries of a row where that covers every row's unpopular columns
        constexpr int TE_SHORT = 3 * LPR / TAIL_LPR, TE_ALL = GRAM_MAX_ROW / TAIL_LPR;
        auto kern = short_tails(c) ? sdca_batched_split<LOSS, TE_SHORT> : sdca_batched_split<LOSS, TE_ALL>;
        int threads = SPLIT_THREADS;
        if (n_tails == 0) {
            kern = sdca_batched_heads<LOSS, false>; threads = BATCHED_THREADS;
            if constexpr (LOSS != CHICLE_LOSS_LOGISTIC)
                if (heads_resolve_apart(c)) { kern = sdca_batched_heads<LOSS, true>; threads = HEAD_THREADS; }
        }
        static_assert(tail_lists_at(TE_ALL) <= sizeof(BatchedShared) + sizeof(double) * TAILS_MIN_HOT, "a tail fits the LDS of a head that has tails");
        HIP_TRY(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh));
        clear_device_words(c, c->split_ring_dev, 2 * (int64_t)SPLIT_WORDS * c->K);
        seg_begin(c, CHICLE_SEG_EPOCH_CHAIN);
        hipLaunchKernelGGL(kern, dim3((1 + n_tails) * k_pad), dim3(threads), sh, c->stream, A, k_pad);
        seg_end(c, CHICLE_SEG_EPOCH_CHAIN);
    } else {
        auto kern = sdca_batched_csr<LOSS>;
        HIP_TRY(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh));
        const int first_warmer = k_pad;
        clear_device_words(c, c->progress_dev, c->K);
        seg_begin(c, CHICLE_SEG_EPOCH_CHAIN);
        hipLaunchKernelGGL(kern, dim3(first_warmer + c->K), dim3(BATCHED_THREADS), sh, c->stream, c->chunks_dev,
                           c->solvers_dev, c->solver_chunks_dev, c->solver_prefix_dev, perm, c->tiles[c->tile_buf], c->u,
                           c->ld_v, u_off, ml, n_hot, (int)hot_off, sc, c->err_dev, c->progress_dev, first_warmer);
        seg_end(c, CHICLE_SEG_EPOCH_CHAIN);
    }
    HIP_TRY(c, hipGetLastError());
    if (perm_next) {
        // the other tile set was last read by the previous pass's chain kernel, which precedes ev_fork
        HIP_TRY(c, hipStreamWaitEvent(c->side, c->ev_fork, 0));
        if (c->profiling) (void)hipEventRecord(c->seg[CHICLE_SEG_EPOCH_GRAM].start, c->side);
        rc = launch_gram<LOSS>(c, perm_next, 1 - c->tile_buf, true, c->side);
        if (c->profiling) {
            (void)hipEventRecord(c->seg[CHICLE_SEG_EPOCH_GRAM].stop, c->side);
            c->seg[CHICLE_SEG_EPOCH_GRAM].recorded = true;
        }
        if (rc) return rc;
        HIP_TRY(c, hipEventRecord(c->ev_join, c->side));
        c->ahead_tiles = true;
    }
    return CHICLE_OK;
}

// The updates of the columns that one row of a solver holds, into its private vector.
void spread_updates(chicle_ctx *c)
{
    if (c->sources_dev) {
        int lds_rows = 1;
        for (const SolverDev &sol : c->solvers) lds_rows = std::max(lds_rows, std::min(sol.n_rows, SPREAD_LDS_ROWS));
        hipLaunchKernelGGL(spread_unique, dim3((c->most_columns + SPREAD_PER - 1) / SPREAD_PER, c->K), dim3(256), sizeof(float) * (size_t)lds_rows,
                           c->stream, c->solvers_dev, c->count_dev, (const UniqueSource *)c->sources_dev, c->coef_dev, c->u, c->u_off_dev, lds_rows);
    } else {
        int max_rows = 1;
        for (const ChunkDev &ch : c->chunks) max_rows = std::max(max_rows, ch.n_rows);
        hipLaunchKernelGGL(scatter_unique, dim3(grid_for(max_rows, 4, 1024), c->n_chunks), dim3(256), 0, c->stream, c->chunks_dev,
                           c->chunk_owner_dev, c->solvers_dev, c->chunk_first_dev, c->coef_dev, c->u, c->u_off_dev, c->private_stale);
    }
}

// Blocks over the shared columns (sparse rows of any length); the other columns' updates follow in a kernel of their own, unless
// the merge takes all updates from the steps' coefficients (column_merge): then only where a caller asks for a solver's update.
template <int LOSS>
int launch_blocks(chicle_ctx *c, const int32_t *perm)
{
    const RoundScalars sc = scalars(c);
    const int k_pad = (c->K + L2_PARTITIONS - 1) / L2_PARTITIONS * L2_PARTITIONS;
    float *tiles = (float *)c->layout_dev;
    seg_begin(c, CHICLE_SEG_EPOCH_GRAM);
    clear_device_words(c, c->coef_dev, c->n_total);
    if (c->merge_by_columns) clear_device_words(c, c->co_coef_dev, c->n_total);
    if (c->blocks_g > 1) clear_device_words(c, c->blocks_ring_dev, 2 * (int64_t)SB_RING_WORDS * c->K);
    if (c->n_tiles > 0) {
        auto kern = gram_blocks<LOSS>;
        HIP_TRY(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(GramBlocksShared)));
        hipLaunchKernelGGL(kern, dim3(c->n_tiles), dim3(SB_THREADS), sizeof(GramBlocksShared), c->stream, c->chunks_dev, c->solvers_dev,
                           c->row_chunk_dev, c->chunk_first_dev, perm, c->tile_solver_dev, tiles, c->blocks_g, c->n_total,
                           (const SegRef *)c->refs_dev, (const int32_t *)c->segs_dev, sc.c, c->err_dev);
    }
    seg_end(c, CHICLE_SEG_EPOCH_GRAM);
    BlocksArgs A;
    A.solvers = c->solvers_dev; A.chunks = c->chunks_dev; A.tiles = tiles; A.u_all = c->u; A.u_off = c->u_off_dev;
    A.place_off = c->place_off_dev; A.place = c->place_dev; A.count = c->mcount_dev; A.refs = c->refs_dev; A.segs = c->segs_dev;
    A.coef_out = c->coef_dev; A.coef_by_row = c->merge_by_columns ? c->co_coef_dev : nullptr; A.n_total = c->n_total; A.G = c->blocks_g; A.k_pad = k_pad; A.sc = sc; A.err = c->err_dev;
    A.rings = c->blocks_ring_dev;
    auto kern = c->blocks_double ? sdca_blocks<LOSS, double> : sdca_blocks<LOSS, float>;
    const size_t sh = sizeof(BlocksShared) + (c->blocks_double ? sizeof(double) * (size_t)SB_CAP<double> : sizeof(float) * (size_t)SB_CAP<float>);
    HIP_TRY(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh));
    seg_begin(c, CHICLE_SEG_EPOCH_CHAIN);
    hipLaunchKernelGGL(kern, dim3(c->blocks_g * k_pad), dim3(SB_THREADS), sh, c->stream, A);
    if (!c->merge_by_columns) spread_updates(c);
    seg_end(c, CHICLE_SEG_EPOCH_CHAIN);
    HIP_TRY(c, hipGetLastError());
    c->coef_pending = c->merge_by_columns;
    c->updates_spread = false;
    return CHICLE_OK;
}

// Work prepared ahead refers to the solver tables: finish it before they change.
int drop_ahead(chicle_ctx *c)
{
    if (c->side) HIP_TRY(c, hipStreamSynchronize(c->side));
    c->ahead_tiles = false;
    c->ahead_valid = false;
    return CHICLE_OK;
}

// What the workgroups of a row pass, `per_chunk` of `threads` for every chunk, do beside the rows, and the grid with those for
// the norms.
GapEnd gap_end(const chicle_ctx *c, const GapScratch &gs, int per_chunk, int threads, dim3 *grid)
{
    GapEnd E{};
    E.n_chunks = c->n_chunks; E.per_chunk = per_chunk;
    const unsigned rows = (unsigned)per_chunk * (unsigned)c->n_chunks;
    *grid = dim3(rows);
    if (!gs.finish) return E;
    E.tickets = c->tickets_dev;
    E.v = c->w64; E.d = (int64_t)c->d;
    E.part_wsq = gs.wsq; E.part_wabs = gs.wabs;
    E.n_w = grid_for(c->d, threads * 8, WSQ_PARTS * 256 / threads);
    E.err = c->err_dev; E.out = (double *)c->pinned_dev; E.seq = c->gap_seq;
    *grid = dim3(rows + (unsigned)E.n_w);
    return E;
}

template <int LOSS, int LPRG, typename WT>
void launch_gap_rows_t(chicle_ctx *c, int grid_x, const WT *w, const GapScratch &gs)
{
    dim3 grid;
    const GapEnd E = gap_end(c, gs, grid_x, c->gap_hot_grid > 0 ? GAP_HOT_THREADS : 256, &grid);
    if (c->gap_hot_grid > 0) {
        // lanes per row: the fewest that cover the longest row with 4 entries each
        const int n_hot = (int)std::min<int64_t>(c->d, GAP_HOT_BYTES / (int)sizeof(WT));
        const size_t sh = n_hot * sizeof(WT);
        const int need = (c->max_row_len + 3) / 4;
#define CHICLE_GAP_HOT(L)                                                                                   \
        hipLaunchKernelGGL((gap_rows_csr_hot<LOSS, L, WT>), grid, dim3(GAP_HOT_THREADS), sh, c->stream,      \
                           c->chunks_dev, w, c->l1, n_hot, gs.loss, gs.conj, E)
        if (need <= 4) CHICLE_GAP_HOT(4);
        else if (need <= 8) CHICLE_GAP_HOT(8);
        else if (need <= 10) CHICLE_GAP_HOT(10);
        else if (need <= 12) CHICLE_GAP_HOT(12);
        else CHICLE_GAP_HOT(16);
#undef CHICLE_GAP_HOT
    } else if (c->dense)
        hipLaunchKernelGGL((gap_rows_dense<LOSS, LPRG, WT>), grid, dim3(256), 0, c->stream, c->chunks_dev,
                           (int)c->d, dense_ld((int)c->d), w, c->l1, gs.loss, gs.conj, E);
    else if (LPRG == 64 && c->long_rows)             // (summed in double, as over the entries by column)
        hipLaunchKernelGGL((gap_rows_csr<LOSS, 64, WT, double>), grid, dim3(256), 0, c->stream, c->chunks_dev, w, c->l1,
                           gs.loss, gs.conj, E);
    else
        hipLaunchKernelGGL((gap_rows_csr<LOSS, LPRG, WT>), grid, dim3(256), 0, c->stream, c->chunks_dev, w, c->l1,
                           gs.loss, gs.conj, E);
}

// Squared loss: dot products in double against the double w (its steps cancel y - z - alpha down to the
// size of the update); logistic: in double as well (loss and conjugate nearly cancel in the gap close to
// the optimum); hinge: float against the float mirror.
template <int LOSS, int LPRG>
void launch_gap_rows(chicle_ctx *c, int grid, const GapScratch &gs)
{
    if (LOSS != 0) launch_gap_rows_t<LOSS, LPRG, double>(c, grid, c->w64, gs);
    else launch_gap_rows_t<LOSS, LPRG, float>(c, grid, c->w, gs);
}

template <int LOSS>
void launch_gap_lpr(chicle_ctx *c, int grid, const GapScratch &gs)
{
    switch (c->gap_lpr) {
        case 4: launch_gap_rows<LOSS, 4>(c, grid, gs); break;
        case 8: launch_gap_rows<LOSS, 8>(c, grid, gs); break;
        case 16: launch_gap_rows<LOSS, 16>(c, grid, gs); break;
        case 32: launch_gap_rows<LOSS, 32>(c, grid, gs); break;
        default: launch_gap_rows<LOSS, 64>(c, grid, gs); break;
    }
}

// The row pass of the gap: z_i = x_i . w into the chunks, loss and conjugate partial sums.
int run_row_pass(chicle_ctx *c, const GapScratch &gs)
{
    // Workgroups per chunk: enough to fill the chip several times over, within the partial-sum arrays.  (2048 in all; 8192, whose
    // counts and partial sums the last workgroup waits for: 500000 x 28 21.6 us and 29.0, in 512 chunks 21.4 and 29.8,
    // 200000 x 128 25.4 and 29.7, 20000 x 1000 22.4 and 23.0; 20000 sparse rows of 200 entries 32.3 and 30.0, 60000 x 1500 with
    // the logistic loss 108 and 103.  Between events.)
    int max_rows = 1;
    for (const ChunkDev &ch : c->chunks) max_rows = std::max(max_rows, ch.n_rows);
    const int rows_per_wg = 2 * (256 / c->gap_lpr);
    int gx = std::min((max_rows + rows_per_wg - 1) / rows_per_wg, std::max(1, 2048 / c->n_chunks));
    gx = std::max(1, std::min(gx, gs.parts / c->n_chunks));
    // popularity-numbered columns: frequent part of w from LDS, few large workgroups per chunk
    c->gap_hot_grid = 0;
    if (c->renumbered && !c->dense && c->max_row_len <= 4 * GAP_HOT_MAX_LPR) {
        const int lpr = std::max(4, (c->max_row_len + 3) / 4);
        const int rows_per_hot_wg = 2 * (GAP_HOT_THREADS / 64) * (64 / lpr);
        gx = std::max(1, std::min(std::min(2, (max_rows + rows_per_hot_wg - 1) / rows_per_hot_wg),
                                  gs.parts / c->n_chunks));
        c->gap_hot_grid = gx;
    }
    if (c->dots_by_columns) {
        const int parts = dot_parts(c->n_total, c->entries_loaded);
        const int per_row = parts <= 8 ? 1 : parts <= 64 ? 4 : 16;
        gx = std::max(1, std::min((max_rows * per_row + 255) / 256, std::min(gs.parts, 2048) / c->n_chunks));
        dim3 fg;
        const GapEnd E = gap_end(c, gs, gx, 256, &fg);
        const dim3 grid((unsigned)(parts * c->columns.blocks));
        const size_t sh = sizeof(double) * (size_t)std::min<int64_t>(CO_ROWS, c->n_total);
        if (c->loss == CHICLE_LOSS_HINGE) {
            HIP_TRY(c, hipFuncSetAttribute((const void *)column_dots<float>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh));
            hipLaunchKernelGGL(column_dots<float>, grid, dim3(CO_THREADS), sh, c->stream, c->columns, parts, (const float *)c->w, c->l1, c->co_z_dev);
        } else {
            HIP_TRY(c, hipFuncSetAttribute((const void *)column_dots<double>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh));
            hipLaunchKernelGGL(column_dots<double>, grid, dim3(CO_THREADS), sh, c->stream, c->columns, parts, (const double *)c->w64, c->l1, c->co_z_dev);
        }
        auto pick = [&](auto k1, auto k4, auto k16) { return per_row == 1 ? k1 : per_row == 4 ? k4 : k16; };
        auto kern = c->loss == CHICLE_LOSS_HINGE ? pick(gap_rows_from_z<0, 1>, gap_rows_from_z<0, 4>, gap_rows_from_z<0, 16>)
                    : c->loss == CHICLE_LOSS_SQUARED ? pick(gap_rows_from_z<1, 1>, gap_rows_from_z<1, 4>, gap_rows_from_z<1, 16>)
                                                     : pick(gap_rows_from_z<2, 1>, gap_rows_from_z<2, 4>, gap_rows_from_z<2, 16>);
        hipLaunchKernelGGL(kern, fg, dim3(256), 0, c->stream, c->chunks_dev, (const double *)c->co_z_dev, parts, c->n_total, c->l1, gs.loss, gs.conj, E);
    } else if (c->loss == CHICLE_LOSS_HINGE) launch_gap_lpr<0>(c, gx, gs);
    else if (c->loss == CHICLE_LOSS_SQUARED) launch_gap_lpr<1>(c, gx, gs);
    else launch_gap_lpr<2>(c, gx, gs);
    HIP_TRY(c, hipGetLastError());
    c->zw_valid = true;
    return CHICLE_OK;
}

int choose_lpr(double avg_row_len)
{
    if (avg_row_len <= 6) return 4;
    if (avg_row_len <= 12) return 8;
    if (avg_row_len <= 48) return 16;
    return 64;
}

// Greedy table of chicle_balance; integers only.
void greedy_table(const int64_t *load, int32_t n_chunks, int32_t K, const int32_t *speed, int32_t *out)
{
    std::vector<int32_t> order(n_chunks);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(),
                     [&](int32_t a, int32_t b) { return load[a] > load[b]; });
    std::vector<int64_t> L(K, 0);
    for (int32_t c : order) {
        int32_t best = 0;
        for (int32_t k = 1; k < K; ++k) {
            const __int128 fk = (__int128)(L[k] + load[c]) * (speed ? speed[best] : 1);
            const __int128 fb = (__int128)(L[best] + load[c]) * (speed ? speed[k] : 1);
            if (fk < fb) best = k;
        }
        out[c] = best;
        L[best] += load[c];
    }
}

// Once, when every chunk is in HBM: renumber the columns by popularity and re-sort the rows.
int renumber_columns(chicle_ctx *c)
{
    int32_t *count = c->rank_of;   // the table is built in place of the counts
    HIP_TRY(c, hipMemsetAsync(count, 0, sizeof(int32_t) * (size_t)c->d, c->stream));
    hipLaunchKernelGGL(count_columns, dim3(1, c->n_chunks), dim3(256), 0, c->stream, c->chunks_dev, count);
    HIP_TRY(c, hipGetLastError());
    std::vector<int32_t> cnt(c->d), order(c->d), rank(c->d);
    HIP_TRY(c, hipMemcpyAsync(cnt.data(), count, sizeof(int32_t) * (size_t)c->d, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return cnt[a] > cnt[b]; });
    for (int32_t r = 0; r < c->d; ++r) rank[order[r]] = r;
    c->shares.assign((size_t)c->d / 64 + 1, 0.0);
    double sum = 0.0;
    for (int32_t r = c->d - 1; r >= 0; --r) {
        const double share = (double)cnt[order[r]] / (double)c->n_total;
        sum += share * share;
        if (r % 64 == 0) c->shares[(size_t)r / 64] = sum;
    }
    HIP_TRY(c, hipMemcpyAsync(c->rank_of, rank.data(), sizeof(int32_t) * (size_t)c->d, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipMemcpyAsync(c->col_of, order.data(), sizeof(int32_t) * (size_t)c->d, hipMemcpyHostToDevice, c->stream));
    int max_rows = 1;
    for (const ChunkDev &ch : c->chunks) max_rows = std::max(max_rows, ch.n_rows);
    hipLaunchKernelGGL(renumber_rows, dim3(grid_for(max_rows, 256, 64), c->n_chunks), dim3(256), 0, c->stream,
                       c->chunks_dev, c->rank_of);
    HIP_TRY(c, hipGetLastError());
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    c->renumbered = true;
    return CHICLE_OK;
}

// Where that copy begins: it takes the end of the room for the block solver's layout, which is sized for data whose every entry is
// shared and for a table of all unshared ones beside.  Of these two few data sets need much of both.  (An arena without a place of
// its own for the copy is a fifth smaller.)
size_t copy_at(const chicle_ctx *c)
{
    return c->layout_bytes - align_up(sizeof(ColumnEntry) * (size_t)c->entries_loaded);      // (the room is twice the copy and more)
}

// What the solvers of the current assignment keep in front of it.
size_t layout_in_use(const chicle_ctx *c)
{
    if (batched_eligible(c))
        return (size_t)((char *)c->tiles[1] - c->layout_dev) + align_up(tile_bytes(false) * (size_t)c->max_tiles) +
               (c->pair_list[0] ? 2 * pair_set_bytes(c->max_tiles) : 0);
    return c->blocks_ready ? c->layout_used : 0;
}

// Makes that copy, when every chunk is in HBM and the columns have their numbers; it is of the data alone.
int order_by_column(chicle_ctx *c)
{
    ColumnEntry *entries = (ColumnEntry *)(c->layout_dev + copy_at(c));
    const int log2 = co_bucket_log2(c->d), buckets = co_buckets(c->d), blocks = co_blocks(c->n_total);
    const int64_t n = (int64_t)buckets * blocks;
    unsigned long long most = 0, *most_dev = c->co_count_dev + n + 1;
    int max_rows = 1;
    for (const ChunkDev &ch : c->chunks) max_rows = std::max(max_rows, ch.n_rows);
    const dim3 grid((max_rows + CO_GROUP_ROWS - 1) / CO_GROUP_ROWS, c->n_chunks);
    const size_t words = buckets <= CO_LDS_BUCKETS ? (size_t)buckets : 0;
    HIP_TRY(c, hipMemsetAsync(c->co_count_dev, 0, sizeof(unsigned long long) * (size_t)(n + 2), c->stream));
    HIP_TRY(c, hipFuncSetAttribute((const void *)co_count, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(sizeof(int) * words)));
    HIP_TRY(c, hipFuncSetAttribute((const void *)co_scatter, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(sizeof(unsigned long long) * words)));
    hipLaunchKernelGGL(co_count, grid, dim3(256), sizeof(int) * words, c->stream, c->chunks_dev, log2, buckets, c->co_count_dev);
    hipLaunchKernelGGL(co_scan, dim3(1), dim3(1024), 0, c->stream, c->co_count_dev, c->co_off_dev, n, buckets, most_dev);
    hipLaunchKernelGGL(co_scatter, grid, dim3(256), sizeof(unsigned long long) * words, c->stream, c->chunks_dev, log2, buckets, c->co_count_dev,
                       entries);
    hipLaunchKernelGGL(co_sort, dim3((unsigned)std::min<int64_t>(n, 65536)), dim3(1024), 0, c->stream, (const long long *)c->co_off_dev, n, log2, entries);
    HIP_TRY(c, hipGetLastError());
    HIP_TRY(c, hipMemcpyAsync(&most, most_dev, sizeof most, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    c->columns = ColumnOrder{entries, c->co_off_dev, buckets, log2, blocks, c->n_total};
    c->fullest_bucket = (double)most;
    return CHICLE_OK;
}

// Whether the merge takes the updates from the steps' coefficients, over the entries by column, and not from the private vectors,
// to which the unshared entries are then spread first.  By column a workgroup reads the coefficients of every block of rows for
// its bucket, whatever the bucket holds, and goes through its entries and columns: where there are few buckets, or most entries are in
// one, the chip waits for that one's workgroup.  Through the private vectors every solver's bitmaps are gone through, and every column
// that a solver holds is written once and read once.  What the former saves of a round, microseconds, fitted to 106 shapes of 1000 to
// 1.1M rows of 100 to 2500 entries, 5000 to 1000M columns and 2 to 64 solvers.  Measured, spread and merge, by column / through the
// vectors: 100000 rows of 1000 over 20M columns, 64 solvers 343 / 747, of 150 234 / 294, 300000 of 150 481 / 420, 1.1M of 100 1424 /
// 895; 2000 of 2500 over 200M, eight solvers 814 / 703, of 1000 over 1000M 2270 / 1436; 1000 of 150 over 2M, eight 48 / 43; 55134 of 261
// over 0.29M, ten (few of whose entries are in columns of their own) 75 / 22; 1500 of 370 over 0.2M, seven 8 / 24; of 16 solvers 4000
// of 314 over 20000 (20 buckets) 76 / 54, over 0.1M 42 / 55, 16000 over 20000 250 / 132.  Where there is no room for the table that the
// spread reads (sources_dev), spreading takes 9 us more per million entries.
bool merge_pays(const chicle_ctx *c)
{
    const double d = 1e-6 * (double)c->d, entries = 1e-6 * (double)c->entries_loaded, held = 1e-6 * (double)c->u_used;
    const double buckets = co_buckets(c->d), fullest = std::max(1e-6 * c->fullest_bucket, entries / buckets);    // (unknown before there is a copy)
    const double saved = 14.5 + 0.09 * d * c->K + 13.0 * held + (c->sources_dev ? 0.0 : 9.0 * entries);
    return saved > std::max(8.9 * entries, 930.0 * fullest) + 0.41 * d + buckets * (0.0026 + 0.0067 * co_blocks(c->n_total));
}

// Whether the rows' dot products go over the entries by column, and not row by row.  The former is two kernels, one of which writes
// and one of which reads a double per row and part; the latter is slower per entry the larger the shared vector is, most of all where
// an L2 partition does not hold it, or the matrix outgrows the L2s, and as slow as its longest rows.  Microseconds, fitted to 114 shapes
// of 1000 to 200000 rows of 115 to 1046 entries, 5000 to 20M columns, hinge and squared loss; the way that used to be is kept where
// the two are close.  By column / by row: 1000 rows of 115 over 20000 columns 15.1 / 10.1, 16000 24.2 / 17.7, 50000 30 / 36, over
// 2M 36 / 79; 1000 of 314 over 0.1M 14.8 / 14.0, over 2M 18.3 / 21.6; 16000 over 5000 31 / 23, over 0.1M 30 / 34, over 2M 35 / 58;
// 16000 of 1046 over 20M 115 / 327; 50000 of them over 5000 114 / 144, over 0.4M 121 / 389; logistic, 2500 of 490 over 30000 19 / 26,
// 60000 of 120 over 10000 34 / 50.
bool dots_pay(const chicle_ctx *c)
{
    const double n = (double)c->n_total, entries = 1e-6 * (double)c->entries_loaded, d = (double)c->d, blocks = co_blocks(c->n_total);
    const double parts = dot_parts(c->n_total, c->entries_loaded);
    const double per_entry = 2.5 + 0.6 * std::log2(std::max(1.0, d / 4096)) + 1.6 * std::log2(std::max(1.0, d / 524288));
    const double by_row = (c->loss == CHICLE_LOSS_LOGISTIC ? 12.0 : 9.0) + per_entry * (entries + 0.004 * (double)c->entries_loaded / n) +
                          (c->loss == CHICLE_LOSS_HINGE ? 1.5 : 3.0) * std::max(0.0, entries - 4.0);
    const double by_column = 18.0 + std::max(1.8 * entries, 97.0 * entries / (parts * blocks)) + 2e-6 * parts * n + 0.4e-6 * d;
    return by_column < 0.95 * by_row;
}

// For the average entry, the share of the other rows that hold its column: 64 times this is how many of a block's rows an
// entry meets in its column's list.  From about 4096 rows; of the data alone, and formed when it is first asked for.
int column_crowding(chicle_ctx *c, double *out)
{
    if (c->crowding < 0.0) {
        int32_t *count = (int32_t *)c->tmp_a;
        double *sums = c->gap_scratch.wabs, s[2] = {0.0, 0.0};
        const int stride = (int)std::max<int64_t>(1, c->n_total / 4096);
        int64_t rows = 0;
        int most = 1;
        for (const ChunkDev &ch : c->chunks) { rows += (ch.n_rows + stride - 1) / stride; most = std::max(most, ch.n_rows); }
        HIP_TRY(c, hipMemsetAsync(count, 0, sizeof(int32_t) * (size_t)c->d, c->stream));
        HIP_TRY(c, hipMemsetAsync(sums, 0, sizeof s, c->stream));
        hipLaunchKernelGGL(count_columns_of_some, dim3(grid_for(most, stride, 256), c->n_chunks), dim3(256), 0, c->stream, c->chunks_dev, stride, count);
        hipLaunchKernelGGL(sum_pairs, dim3(grid_for(c->d, 256, 1024)), dim3(256), 0, c->stream, count, (int64_t)c->d, sums);
        HIP_TRY(c, hipGetLastError());
        HIP_TRY(c, hipMemcpyAsync(s, sums, sizeof s, hipMemcpyDeviceToHost, c->stream));
        HIP_TRY(c, hipStreamSynchronize(c->stream));
        c->crowding = s[1] > 0.0 && rows > 1 ? s[0] / ((double)(rows - 1) * s[1]) : 0.0;
    }
    *out = c->crowding;
    return CHICLE_OK;
}

// Microseconds a tile of so many shared entries takes where they are joined in parts (nothing worth counting where they
// are joined at once, 26 to 51): its entries are read four times per part, and every entry walks its column's list.
// Measured, entries and share of the rows that hold a column: 12 800 and 1/16: 174 us, 1/4: 254, 1: 1166; 64 000: 2071,
// 3352, 9157; 256 000: 25 900, 36 600, 100 000.
double tile_in_parts_us(double entries, double crowding)
{
    if (entries <= GB_ALL) return 0.0;
    double parts = 1.0;
    while (parts * GB_POST < entries) parts *= 2.0;
    return 40.0 + (0.002 * parts + crowding * (0.075 + 0.9e-6 * entries)) * entries;
}

// Whether the block solver is the faster one for the entries laid out.  It is, unless tiles have to be joined in parts:
// then their cost (spread over the chip, but no less than one of them) stands against the steps of the row-wise solver,
// 1.7 us and more each, 2.4 and more on several workgroups per solver.  Both sides, 1024 rows that hold every column, four
// solvers: 300 columns 1.69 ms in blocks and 0.62 row by row, 1000 columns 9.4 and 0.64; 5000, eight solvers, 139 and 0.42;
// 256 rows of 200 out of 3200 columns, two solvers, 0.23 and 0.33.  A fifth is added for what the averages hide.
bool blocks_pay(const chicle_ctx *c, const std::vector<SegStat> &stat, int G, double crowding)
{
    double worst = 0.0, all = 0.0, chain = 0.0;
    for (int k = 0; k < c->K; ++k) {
        const double rows = c->solvers[k].n_rows, blocks = std::ceil(rows / BATCH);
        if (rows == 0) continue;
        const double per_row = stat[k].total / rows, mean = (double)SB_SEG * stat[k].total / blocks;
        // a tile's entries: spread of a sum of 64 rows, and the tile that holds the longest one
        const double spread = blocks > 1 ? SB_SEG * std::sqrt(BATCH * std::max(0.0, stat[k].squares / rows - per_row * per_row)) : 0.0;
        const double high = blocks > 1 ? mean + SB_SEG * (stat[k].longest - per_row) : mean;
        const double in_parts = 0.5 * std::erfc((GB_ALL - mean) / (1.5 * spread + 1.0));
        const double us = tile_in_parts_us(high, crowding);
        worst = std::max(worst, us);
        all += std::max(us, blocks * in_parts * tile_in_parts_us(std::max(mean, (double)GB_ALL) + spread, crowding));
        chain = std::max(chain, blocks * (4.0 + 0.8e-3 * mean / G));
    }
    if (worst == 0.0) return true;
    // (tiles on the whole chip at once take up to three times the time of a few: what they read again no longer fits the caches)
    const double waves = std::ceil((double)c->K * G / c->cu_count);
    return 1.2 * (std::max(worst, (c->n_tiles > c->cu_count ? 3.0 : 1.0) * all / c->cu_count) + chain * waves) <= c->most_rows * (c->cluster > 1 ? 2.4 : 1.7);
}

// The shared entries of the rows, for the solver that takes rows of any length in blocks: the fewest workgroups per solver
// whose LDS holds every solver's shared columns (more than one of them must be resident together: they wait for each
// other).  Where these or the room of so many bytes do not suffice (the latter: *too_small), or it would not be the faster one, the
// row-wise solver remains.
int lay_out_blocks(chicle_ctx *c, const std::vector<int32_t> &shared, const std::vector<int32_t> &columns, size_t layout_bytes, bool *too_small)
{
    *too_small = false;
    if (few_rows(c)) return CHICLE_OK;
    const int K = (int)shared.size();
    const int k_pad = (K + L2_PARTITIONS - 1) / L2_PARTITIONS * L2_PARTITIONS;
    const int64_t most = *std::max_element(shared.begin(), shared.end());
    auto members = [&](int cap) {          // 0: they do not fit
        int G = 1;
        while ((int64_t)G * cap < most) G *= 2;
        return G <= SB_MAX_G && (G == 1 || G * k_pad <= c->cu_count) ? G : 0;
    };
    c->blocks_double = members(SB_CAP<double>) > 0;
    const int G = c->blocks_double ? members(SB_CAP<double>) : members(SB_CAP<float>);
    if (G == 0) return CHICLE_OK;
    std::vector<int64_t> off(K);
    int64_t places = 0;
    for (int k = 0; k < K; ++k) { off[k] = places; places += shared[k]; }
    const size_t tiles = align_up(tile_bytes(true) * (size_t)c->n_tiles), refs = align_up(sizeof(SegRef) * (size_t)G * (size_t)c->n_total),
                 place = align_up(sizeof(int32_t) * (size_t)std::max<int64_t>(places, 1));
    *too_small = tiles + refs + place + SB_SEG_WORDS * sizeof(int32_t) > layout_bytes;
    if (*too_small) return CHICLE_OK;
    const size_t room = (layout_bytes - tiles - refs - place) / (SB_SEG_WORDS * sizeof(int32_t));
    const int capacity = (int)std::min<size_t>(room, (size_t)INT32_MAX);
    c->refs_dev = (SegRef *)(c->layout_dev + tiles);
    c->place_dev = (int32_t *)(c->layout_dev + tiles + refs);
    c->segs_dev = (int32_t *)(c->layout_dev + tiles + refs + place);
    int *taken = c->mcount_dev + c->max_solvers;
    HIP_TRY(c, hipMemcpyAsync(c->place_off_dev, off.data(), sizeof(int64_t) * (size_t)K, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipMemsetAsync(taken, 0, sizeof(int), c->stream));
    HIP_TRY(c, hipMemsetAsync(c->seg_stat_dev, 0, sizeof(SegStat) * (size_t)K, c->stream));
    hipLaunchKernelGGL(shared_places, dim3(grid_for(c->words, 256, 1024), K), dim3(256), 0, c->stream, c->bits_dev, c->pref_dev,
                       c->multi_dev, c->mpref_dev, c->words, c->place_off_dev, c->place_dev);
    int max_rows = 1;
    for (const ChunkDev &ch : c->chunks) max_rows = std::max(max_rows, ch.n_rows);
    hipLaunchKernelGGL(build_segments, dim3(grid_for(max_rows, 4, 1024), c->n_chunks), dim3(256), 0, c->stream, c->chunks_dev,
                       c->chunk_owner_dev, c->multi_dev, c->mpref_dev, c->words, G, c->n_total, c->refs_dev, c->segs_dev, taken, capacity);
    hipLaunchKernelGGL(segment_stats, dim3(c->n_chunks), dim3(256), 0, c->stream, c->chunks_dev, c->chunk_owner_dev, (const SegRef *)c->refs_dev, G,
                       c->n_total, c->seg_stat_dev);
    HIP_TRY(c, hipGetLastError());
    int n = 0;
    std::vector<SegStat> stat(K);
    HIP_TRY(c, hipMemcpyAsync(&n, taken, sizeof(int), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipMemcpyAsync(stat.data(), c->seg_stat_dev, sizeof(SegStat) * (size_t)K, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    *too_small = n < 0 || n > capacity;
    if (*too_small) return CHICLE_OK;
    double crowding = 1.0;
    if (!blocks_pay(c, stat, G, 0.0)) return CHICLE_OK;     // (not even with nothing shared twice)
    if (!blocks_pay(c, stat, G, crowding)) {
        const int rc = column_crowding(c, &crowding);
        if (rc) return rc;
        if (!blocks_pay(c, stat, G, crowding)) return CHICLE_OK;
    }
    c->blocks_g = G;
    c->blocks_ready = true;
    c->most_columns = *std::max_element(columns.begin(), columns.end());
    c->sources_dev = nullptr;
    c->layout_used = tiles + refs + place + align_up((size_t)SB_SEG_WORDS * sizeof(int32_t) * (size_t)std::max(n, 1));
    if (c->layout_used + sizeof(UniqueSource) * (size_t)c->u_used <= layout_bytes) {
        c->sources_dev = (UniqueSource *)(c->layout_dev + c->layout_used);
        c->layout_used += sizeof(UniqueSource) * (size_t)c->u_used;
        HIP_TRY(c, hipMemsetAsync(c->sources_dev, 0xff, sizeof(UniqueSource) * (size_t)c->u_used, c->stream));
        hipLaunchKernelGGL(unique_sources, dim3(grid_for(max_rows, 4, 1024), c->n_chunks), dim3(256), 0, c->stream, c->chunks_dev,
                           c->chunk_owner_dev, c->chunk_first_dev, c->u_off_dev, c->sources_dev);
        HIP_TRY(c, hipGetLastError());
    }
    return CHICLE_OK;
}

}  // namespace

extern "C" {

size_t chicle_arena_bytes(int64_t n_total, int64_t total_entries, int32_t d, int32_t n_chunks,
                          int32_t max_solvers, int32_t dense)
{
    if (n_total <= 0 || total_entries < 0 || d <= 0 || n_chunks <= 0 || max_solvers <= 0) return 0;
    const bool long_rows = !dense && (double)total_entries > LONG_ROW_AVG * (double)n_total;
    const bool compact = !dense;
    size_t s = fixed_bytes(n_total, d, n_chunks, max_solvers, long_rows, compact, total_entries);
    // chunk blocks: exact array bytes plus alignment slack per array and chunk
    const size_t per_chunk_slack = 8 * ALIGN + 2 * sizeof(float) * ENTRY_SLACK;
    if (dense)
        s += sizeof(float) * (size_t)(total_entries / d + n_chunks) * (size_t)dense_ld(d) + 4 * sizeof(float) * (size_t)n_total;
    else
        s += (sizeof(int32_t) * (compact ? 2 : 1) + sizeof(float)) * ((size_t)total_entries + (size_t)n_chunks) +
             sizeof(int32_t) * ((size_t)n_total + (size_t)n_chunks) + 4 * sizeof(float) * (size_t)n_total;
    s += (per_chunk_slack + (compact ? ALIGN + sizeof(int32_t) * ENTRY_SLACK : 0)) * (size_t)n_chunks;
    return s + ALIGN;
}

int chicle_create(chicle_ctx **out, int32_t loss, int64_t n_total, int32_t d, double lambda,
                  int32_t n_chunks, int32_t max_solvers, int32_t dense, int64_t total_entries,
                  void *device_arena, size_t arena_bytes, void *hip_stream)
{
    if (!out) return CHICLE_EINVAL;
    *out = nullptr;
    if ((loss != CHICLE_LOSS_HINGE && loss != CHICLE_LOSS_SQUARED && loss != CHICLE_LOSS_LOGISTIC) || n_total <= 0 ||
        n_total > INT32_MAX || d <= 0 || !(lambda > 0.0) || n_chunks <= 0 || max_solvers <= 0 ||
        total_entries < 0 || !device_arena || ((uintptr_t)device_arena % ALIGN) != 0)
        return CHICLE_EINVAL;
    const size_t need = chicle_arena_bytes(n_total, total_entries, d, n_chunks, max_solvers, dense);
    if (arena_bytes < need) return CHICLE_ENOMEM;
    chicle_ctx *c = new (std::nothrow) chicle_ctx();
    if (!c) return CHICLE_ENOMEM;
    c->loss = loss; c->n_total = n_total; c->d = d; c->ld_v = pad_d(d); c->lambda = lambda;
    c->n_chunks = n_chunks; c->max_solvers = max_solvers;
    c->dense = dense != 0;
    c->total_entries = total_entries;
    c->arena = (char *)device_arena; c->arena_bytes = arena_bytes;
    c->stream = (hipStream_t)hip_stream;
    c->max_tiles = tiles_cap(n_total, max_solvers);

    c->chunks_dev = (ChunkDev *)carve(c, sizeof(ChunkDev) * (size_t)n_chunks);
    c->solvers_dev = (SolverDev *)carve(c, sizeof(SolverDev) * (size_t)max_solvers);
    c->solver_chunks_dev = (int32_t *)carve(c, sizeof(int32_t) * (size_t)n_chunks);
    c->solver_prefix_dev = (int32_t *)carve(c, sizeof(int32_t) * (size_t)n_chunks);
    c->item_prefix_dev = (int32_t *)carve(c, sizeof(int32_t) * ((size_t)n_chunks + 1));
    c->w = (float *)carve(c, sizeof(float) * (size_t)c->ld_v);
    c->w64 = (double *)carve(c, sizeof(double) * (size_t)c->ld_v);
    c->tmp_a = (float *)carve(c, sizeof(float) * (size_t)c->ld_v);
    c->tmp_b = (float *)carve(c, sizeof(float) * (size_t)c->ld_v);
    c->long_rows = !c->dense && (double)total_entries > LONG_ROW_AVG * (double)n_total;
    c->compact = !c->dense;
    c->u_capacity = private_floats(total_entries, c->ld_v, max_solvers, c->long_rows);
    c->u = (float *)carve(c, sizeof(float) * (size_t)c->u_capacity);
    c->rank_of = (int32_t *)carve(c, sizeof(int32_t) * (size_t)d);
    c->col_of = (int32_t *)carve(c, sizeof(int32_t) * (size_t)d);
    c->tiles[0] = (float *)carve(c, tile_bytes(c->dense) * (size_t)c->max_tiles);
    c->tiles[1] = (float *)carve(c, tile_bytes(c->dense) * (size_t)c->max_tiles);
    char *pairs = c->long_rows ? (char *)carve(c, long_row_layout_bytes(n_total, total_entries)) : nullptr;
    if (pairs && (d <= TAILS_MIN_HOT || 2 * pair_set_bytes(c->max_tiles) > long_row_layout_bytes(n_total, total_entries))) pairs = nullptr;
    c->layout_dev = (char *)c->tiles[0];
    c->layout_bytes = c->layout_dev ? (size_t)(c->arena + c->used - c->layout_dev) : 0;
    c->tile_solver_dev = (int32_t *)carve(c, sizeof(int32_t) * (size_t)c->max_tiles);
    c->perm_stage = (int32_t *)carve(c, sizeof(int32_t) * (size_t)n_total);
    c->perm_ahead[0] = (int32_t *)carve(c, sizeof(int32_t) * (size_t)n_total);
    c->perm_ahead[1] = (int32_t *)carve(c, sizeof(int32_t) * (size_t)n_total);
    c->row_chunk_dev = (int32_t *)carve(c, sizeof(int32_t) * (size_t)n_total);
    c->chunk_first_dev = (int32_t *)carve(c, sizeof(int32_t) * (size_t)n_chunks);
    c->list_base_dev = (int32_t *)carve(c, sizeof(int32_t) * (size_t)n_chunks);
    c->gap_scratch.parts = std::max(GAP_PARTS, 2 * n_chunks);
    c->gap_scratch.loss = (double *)carve(c, sizeof(double) * (size_t)c->gap_scratch.parts);
    c->gap_scratch.conj = (double *)carve(c, sizeof(double) * (size_t)c->gap_scratch.parts);
    c->gap_scratch.wsq = (double *)carve(c, sizeof(double) * WSQ_PARTS);
    c->gap_scratch.wabs = (double *)carve(c, sizeof(double) * WSQ_PARTS);
    c->err_dev = (int *)carve(c, sizeof(int));
    c->tickets_dev = (unsigned *)carve(c, sizeof(unsigned) * n_tickets(d));
    c->ticks_dev = (long long *)carve(c, sizeof(long long) * 2 * (size_t)max_solvers);
    c->progress_dev = (int *)carve(c, sizeof(int) * (size_t)max_solvers);
    c->split_ring_dev = (unsigned long long *)carve(c, sizeof(unsigned long long) * (size_t)SPLIT_WORDS * (size_t)max_solvers);
    if (c->long_rows) {
        if (char *at = (char *)carve(c, co_scratch_bytes(n_total, total_entries, d))) {
            c->co_off_dev = (long long *)at;
            c->co_count_dev = (unsigned long long *)(at += co_offsets_bytes(n_total, d));
            c->co_z_dev = (double *)(at += co_offsets_bytes(n_total, d));
            c->co_coef_dev = (float *)(at += co_parts_bytes(n_total, total_entries));
        }
        c->row_split_dev = (int32_t *)carve(c, sizeof(int32_t) * (size_t)SPLITS_PER_ROW * (size_t)n_total);
        c->cluster_ring_dev = (unsigned long long *)carve(c, sizeof(unsigned long long) * (size_t)CLUSTER_WORDS * (size_t)max_solvers);
    }
    if (c->compact) {
        c->words = ((int64_t)d + 31) / 32;
        c->bits_dev = (unsigned *)carve(c, sizeof(unsigned) * (size_t)c->words * (size_t)max_solvers);
        c->pref_dev = (int32_t *)carve(c, sizeof(int32_t) * (size_t)c->words * (size_t)max_solvers);
        c->multi_dev = (unsigned *)carve(c, sizeof(unsigned) * (size_t)c->words * (size_t)max_solvers);
        c->mpref_dev = (int32_t *)carve(c, sizeof(int32_t) * (size_t)c->words * (size_t)max_solvers);
        c->mcount_dev = (int32_t *)carve(c, sizeof(int32_t) * ((size_t)max_solvers + 1));
        c->place_off_dev = (int64_t *)carve(c, sizeof(int64_t) * (size_t)max_solvers);
        c->seg_stat_dev = (SegStat *)carve(c, sizeof(SegStat) * (size_t)max_solvers);
        c->coef_dev = (float *)carve(c, sizeof(float) * (size_t)n_total);
        c->blocks_ring_dev = (unsigned long long *)carve(c, sizeof(unsigned long long) * (size_t)SB_RING_WORDS * (size_t)max_solvers);
        c->count_dev = (int32_t *)carve(c, sizeof(int32_t) * (size_t)max_solvers);
        c->u_off_dev = (int64_t *)carve(c, sizeof(int64_t) * (size_t)max_solvers);
        c->chunk_owner_dev = (int32_t *)carve(c, sizeof(int32_t) * (size_t)n_chunks);
    }
    const size_t own_pairs = pair_bytes(c->max_tiles, d, c->long_rows, c->compact);
    if (own_pairs) pairs = (char *)carve(c, own_pairs);
    for (int buf = 0; pairs && buf < 2; ++buf) {
        c->pair_list[buf] = (unsigned long long *)(pairs + pair_set_bytes(c->max_tiles) * (size_t)buf);
        c->pair_count[buf] = (int32_t *)(c->pair_list[buf] + (size_t)PAIR_CAP * (size_t)c->max_tiles);
    }
    if (!c->err_dev || !c->tickets_dev || !c->ticks_dev || !c->progress_dev || !c->split_ring_dev || (c->long_rows && (!c->cluster_ring_dev || !c->co_coef_dev)) || (c->compact && (!c->chunk_owner_dev || !c->blocks_ring_dev)) || (own_pairs && !pairs)) { delete c; return CHICLE_ENOMEM; }

    c->chunks.assign(n_chunks, ChunkDev{});
    c->loaded.assign(n_chunks, 0);
    bool ok = hipMemsetAsync(c->w, 0, sizeof(float) * (size_t)c->ld_v, c->stream) == hipSuccess &&
              hipMemsetAsync(c->w64, 0, sizeof(double) * (size_t)c->ld_v, c->stream) == hipSuccess &&
              hipMemsetAsync(c->tmp_a, 0, sizeof(float) * (size_t)c->ld_v, c->stream) == hipSuccess &&
              hipMemsetAsync(c->tmp_b, 0, sizeof(float) * (size_t)c->ld_v, c->stream) == hipSuccess &&
              hipMemsetAsync(c->u, 0, sizeof(float) * (size_t)c->u_capacity, c->stream) == hipSuccess &&
              hipMemsetAsync(c->err_dev, 0, sizeof(int), c->stream) == hipSuccess &&
              hipMemsetAsync(c->tickets_dev, 0, sizeof(unsigned) * n_tickets(d), c->stream) == hipSuccess &&
              (!c->long_rows || hipMemsetAsync(c->co_coef_dev, 0, sizeof(float) * ((size_t)n_total + 4), c->stream) == hipSuccess) &&
              hipMemsetAsync(c->ticks_dev, 0, sizeof(long long) * 2 * (size_t)max_solvers, c->stream) == hipSuccess;
    {
        int dev = 0;
        ok = ok && hipGetDevice(&dev) == hipSuccess && (c->device = dev, true) &&
             hipDeviceGetAttribute(&c->wall_khz, hipDeviceAttributeWallClockRate, dev) == hipSuccess && c->wall_khz > 0 &&
             hipDeviceGetAttribute(&c->cu_count, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && c->cu_count > 0;
    }
    for (int s = 0; ok && s < CHICLE_SEG_COUNT; ++s)
        ok = hipEventCreate(&c->seg[s].start) == hipSuccess && hipEventCreate(&c->seg[s].stop) == hipSuccess;
    {
        size_t bytes = PINNED_HEAD;
        if (sizeof(float) * (size_t)d <= PINNED_MOST) { c->pinned_vector = bytes; bytes += align_up(sizeof(float) * (size_t)d); }
        if (sizeof(int32_t) * (size_t)n_total <= PINNED_MOST) { c->pinned_orders = bytes; bytes += align_up(sizeof(int32_t) * (size_t)n_total); }
        ok = ok && hipHostMalloc((void **)&c->pinned, bytes, hipHostMallocMapped) == hipSuccess &&
             hipHostGetDevicePointer((void **)&c->pinned_dev, c->pinned, 0) == hipSuccess;
        if (ok) std::memset(c->pinned, 0, PINNED_HEAD);
    }
    ok = ok && static_scratch_of_current_device(&c->static_scratch) == hipSuccess;
    ok = ok && hipStreamCreateWithFlags(&c->side, hipStreamNonBlocking) == hipSuccess &&
         hipEventCreateWithFlags(&c->ev_fork, hipEventDisableTiming) == hipSuccess &&
         hipEventCreateWithFlags(&c->ev_join, hipEventDisableTiming) == hipSuccess;
    if (!ok) { chicle_destroy(c); return CHICLE_EDEVICE; }
    *out = c;
    return CHICLE_OK;
}

static int load_common(chicle_ctx *c, int32_t chunk_id, int32_t n_rows, int64_t entries)
{
    if (c->state != ST_LOADING) return fail(c, CHICLE_ESTATE, "chunks can only be loaded before the first assign");
    if (chunk_id < 0 || chunk_id >= c->n_chunks) return fail(c, CHICLE_EINVAL, "chunk id %d out of range", chunk_id);
    if (c->loaded[chunk_id]) return fail(c, CHICLE_EINVAL, "chunk %d already loaded", chunk_id);
    if (n_rows <= 0) return fail(c, CHICLE_EINVAL, "chunk %d: n_rows must be positive", chunk_id);
    if (c->rows_loaded + n_rows > c->n_total) return fail(c, CHICLE_EINVAL, "more rows than n_total");
    if (c->entries_loaded + entries > c->total_entries)
        return fail(c, CHICLE_EINVAL, "more stored entries than total_entries");
    if (c->used + chunk_bytes(c->dense, c->compact, n_rows, c->dense ? (int64_t)n_rows * dense_ld((int)c->d) : entries) > c->arena_bytes)
        return fail(c, CHICLE_ENOMEM, "chunk store full");
    return CHICLE_OK;
}

static int check_state_arrays(chicle_ctx *c, int32_t chunk_id, int32_t n_rows, const float *y,
                              const float *alpha0)
{
    if (!y) return fail(c, CHICLE_EINVAL, "chunk %d: y is NULL", chunk_id);
    for (int32_t r = 0; r < n_rows; ++r) {
        if (!std::isfinite(y[r])) return fail(c, CHICLE_EINVAL, "chunk %d row %d: label not finite", chunk_id, r);
        if (c->loss != CHICLE_LOSS_SQUARED && y[r] != 1.0f && y[r] != -1.0f)
            return fail(c, CHICLE_EINVAL, "chunk %d row %d: hinge label must be +1 or -1", chunk_id, r);
        if (alpha0) {
            if (!std::isfinite(alpha0[r])) return fail(c, CHICLE_EINVAL, "chunk %d row %d: alpha not finite", chunk_id, r);
            if (c->loss != CHICLE_LOSS_SQUARED && (alpha0[r] < 0.0f || alpha0[r] > 1.0f))
                return fail(c, CHICLE_EINVAL, "chunk %d row %d: hinge alpha outside [0,1]", chunk_id, r);
        }
    }
    return CHICLE_OK;
}

static int finish_load(chicle_ctx *c, int32_t chunk_id, ChunkDev &ch, const float *y, const float *alpha0,
                       const std::vector<float> &q)
{
    const size_t nb = sizeof(RowState) * (size_t)ch.n_rows;
    RowState *sd = (RowState *)carve(c, nb);
    if (!sd) return fail(c, CHICLE_ENOMEM, "chunk store full");
    ch.st = sd;
    std::vector<RowState> st(ch.n_rows);
    for (int32_t r = 0; r < ch.n_rows; ++r) {
        st[r].y = y[r]; st[r].alpha = alpha0 ? alpha0[r] : 0.f; st[r].q = q[r];
        st[r].rw = c->loss == CHICLE_LOSS_HINGE ? 1.f : c->loss == CHICLE_LOSS_SQUARED ? y[r] : 0.f;   // residual at w = 0
    }
    HIP_TRY(c, hipMemcpyAsync(sd, st.data(), nb, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));   // host arrays are the caller's again on return
    c->chunks[chunk_id] = ch;
    c->loaded[chunk_id] = 1;
    c->n_loaded += 1;
    c->rows_loaded += ch.n_rows;
    c->entries_loaded += ch.nnz;
    return CHICLE_OK;
}

static int load_csr(chicle_ctx *c, int32_t chunk_id, int32_t n_rows, const int32_t *row_ptr,
                    const int32_t *col, const float *val, const float *y, const float *alpha0);

int chicle_load_chunk_csr(chicle_ctx *c, int32_t chunk_id, int32_t n_rows, const int32_t *row_ptr,
                          const int32_t *col, const float *val, const float *y, const float *alpha0)
{
    if (!c) return CHICLE_EINVAL;
    if (c->dense) return fail(c, CHICLE_EINVAL, "context holds dense chunks");
    return load_csr(c, chunk_id, n_rows, row_ptr, col, val, y, alpha0);
}

static int load_csr(chicle_ctx *c, int32_t chunk_id, int32_t n_rows, const int32_t *row_ptr,
                    const int32_t *col, const float *val, const float *y, const float *alpha0)
{
    if (!row_ptr || n_rows <= 0) return fail(c, CHICLE_EINVAL, "chunk %d: row_ptr NULL or no rows", chunk_id);
    if (row_ptr[0] != 0) return fail(c, CHICLE_EINVAL, "chunk %d: row_ptr[0] must be 0", chunk_id);
    for (int32_t r = 0; r < n_rows; ++r)
        if (row_ptr[r + 1] < row_ptr[r]) return fail(c, CHICLE_EINVAL, "chunk %d: row_ptr decreases at row %d", chunk_id, r);
    const int64_t nnz = row_ptr[n_rows];
    int rc = load_common(c, chunk_id, n_rows, nnz);
    if (rc) return rc;
    if (nnz > 0 && (!col || !val)) return fail(c, CHICLE_EINVAL, "chunk %d: col/val NULL", chunk_id);
    rc = check_state_arrays(c, chunk_id, n_rows, y, alpha0);
    if (rc) return rc;
    std::vector<float> q(n_rows);
    int32_t longest = 0;
    for (int32_t r = 0; r < n_rows; ++r) {
        double s = 0.0;
        for (int32_t p = row_ptr[r]; p < row_ptr[r + 1]; ++p) {
            if (col[p] < 0 || col[p] >= c->d) return fail(c, CHICLE_EINVAL, "chunk %d row %d: column %d outside [0,d)", chunk_id, r, col[p]);
            if (p > row_ptr[r] && col[p] <= col[p - 1]) return fail(c, CHICLE_EINVAL, "chunk %d row %d: columns not strictly ascending", chunk_id, r);
            if (!std::isfinite(val[p])) return fail(c, CHICLE_EINVAL, "chunk %d row %d: value not finite", chunk_id, r);
            s += (double)val[p] * (double)val[p];
        }
        q[r] = (float)s;
        longest = std::max(longest, row_ptr[r + 1] - row_ptr[r]);
    }
    ChunkDev ch{};
    ch.n_rows = n_rows; ch.nnz = nnz; ch.row_base = (int32_t)c->rows_loaded;
    int32_t *rp = (int32_t *)carve(c, sizeof(int32_t) * (size_t)(n_rows + 1));
    // a few entries of slack: kernels read short rows with fixed-width vector loads
    int32_t *cd = (int32_t *)carve(c, sizeof(int32_t) * (size_t)(nnz + ENTRY_SLACK));
    if (c->compact) {      // compact ids, filled at every assign; must lie where chunk_compact_ids() looks
        int32_t *ci = (int32_t *)carve(c, sizeof(int32_t) * (size_t)(nnz + ENTRY_SLACK));
        if (!ci || ci != cd + padded_entries(nnz)) return fail(c, CHICLE_ENOMEM, "chunk store full");
    }
    float *vd = (float *)carve(c, sizeof(float) * (size_t)(nnz + ENTRY_SLACK));
    if (!vd) return fail(c, CHICLE_ENOMEM, "chunk store full");
    ch.row_ptr = rp; ch.col = cd; ch.val = vd;
    HIP_TRY(c, hipMemcpyAsync(rp, row_ptr, sizeof(int32_t) * (size_t)(n_rows + 1), hipMemcpyHostToDevice, c->stream));
    if (nnz > 0) {
        HIP_TRY(c, hipMemcpyAsync(cd, col, sizeof(int32_t) * (size_t)nnz, hipMemcpyHostToDevice, c->stream));
        HIP_TRY(c, hipMemcpyAsync(vd, val, sizeof(float) * (size_t)nnz, hipMemcpyHostToDevice, c->stream));
    }
    rc = finish_load(c, chunk_id, ch, y, alpha0, q);
    if (rc == CHICLE_OK) c->max_row_len = std::max(c->max_row_len, longest);
    return rc;
}

int chicle_load_chunk_dense(chicle_ctx *c, int32_t chunk_id, int32_t n_rows, const float *X,
                            const float *y, const float *alpha0)
{
    if (!c) return CHICLE_EINVAL;
    if (!c->dense) return fail(c, CHICLE_EINVAL, "context holds CSR chunks");
    if (!X || n_rows <= 0) return fail(c, CHICLE_EINVAL, "chunk %d: X NULL or no rows", chunk_id);
    const int64_t entries = (int64_t)n_rows * c->d;
    int rc = load_common(c, chunk_id, n_rows, entries);
    if (rc) return rc;
    rc = check_state_arrays(c, chunk_id, n_rows, y, alpha0);
    if (rc) return rc;
    std::vector<float> q(n_rows);
    for (int32_t r = 0; r < n_rows; ++r) {
        double s = 0.0;
        const float *x = X + (int64_t)r * c->d;
        for (int32_t j = 0; j < c->d; ++j) {
            if (!std::isfinite(x[j])) return fail(c, CHICLE_EINVAL, "chunk %d row %d: value not finite", chunk_id, r);
            s += (double)x[j] * (double)x[j];
        }
        q[r] = (float)s;
    }
    ChunkDev ch{};
    ch.n_rows = n_rows; ch.nnz = entries; ch.row_base = (int32_t)c->rows_loaded;
    const int ld = dense_ld((int)c->d);
    float *xd = (float *)carve(c, sizeof(float) * (size_t)n_rows * (size_t)ld);
    if (!xd) return fail(c, CHICLE_ENOMEM, "chunk store full");
    ch.val = xd;
    if (ld == c->d) {
        HIP_TRY(c, hipMemcpyAsync(xd, X, sizeof(float) * (size_t)entries, hipMemcpyHostToDevice, c->stream));
    } else {
        // Rows end in zero columns up to a multiple of four.  The caller's rows go as they are into device memory that is
        // free until the first assign (the private vectors or the tile sets), a part at a time, and from there into place:
        // the link is as fast as for rows that need no padding, and the host holds no second copy.
        char *part = c->layout_dev;
        size_t bytes = c->layout_bytes;
        if (sizeof(float) * (size_t)c->u_capacity > bytes) { part = (char *)c->u; bytes = sizeof(float) * (size_t)c->u_capacity; }
        const int64_t room = (int64_t)(bytes / sizeof(float));
        for (int64_t at = 0; at < entries; at += room) {
            const int64_t m = std::min(room, entries - at);
            HIP_TRY(c, hipMemcpyAsync(part, X + at, sizeof(float) * (size_t)m, hipMemcpyHostToDevice, c->stream));
            hipLaunchKernelGGL(pad_rows, dim3(grid_for(m, 256, 8192)), dim3(256), 0, c->stream, (const float *)part, at, m, (int)c->d, ld, xd);
            HIP_TRY(c, hipGetLastError());
        }
    }
    rc = finish_load(c, chunk_id, ch, y, alpha0, q);
    if (rc == CHICLE_OK) c->max_row_len = c->d;
    return rc;
}

int chicle_balance(const int64_t *chunk_load, int32_t n_chunks, int32_t K, const int32_t *speed_q,
                   int32_t *chunk_to_solver_out)
{
    if (!chunk_load || !chunk_to_solver_out || n_chunks < 0 || K <= 0) return CHICLE_EINVAL;
    for (int32_t i = 0; i < n_chunks; ++i)
        if (chunk_load[i] < 0) return CHICLE_EINVAL;
    if (speed_q)
        for (int32_t k = 0; k < K; ++k)
            if (speed_q[k] <= 0) return CHICLE_EINVAL;
    greedy_table(chunk_load, n_chunks, K, speed_q, chunk_to_solver_out);
    return CHICLE_OK;
}

int chicle_assign(chicle_ctx *c, int32_t K, const int32_t *chunk_to_solver)
{
    if (!c) return CHICLE_EINVAL;
    if (c->state == ST_EPOCH_DONE)
        return fail(c, CHICLE_ESTATE, "solvers own the chunks until their updates are aggregated");
    if (K <= 0 || K > c->max_solvers) return fail(c, CHICLE_EINVAL, "K=%d outside [1, max_solvers=%d]", K, c->max_solvers);
    if (!chunk_to_solver) return fail(c, CHICLE_EINVAL, "table is NULL");
    if (c->n_loaded != c->n_chunks) return fail(c, CHICLE_EINVAL, "%d of %d chunks loaded", c->n_loaded, c->n_chunks);
    if (c->rows_loaded != c->n_total) return fail(c, CHICLE_EINVAL, "chunks hold %lld rows, n_total is %lld", (long long)c->rows_loaded, (long long)c->n_total);
    { const int rc0 = drop_ahead(c); if (rc0) return rc0; }
    std::vector<int32_t> count(K, 0);
    for (int32_t i = 0; i < c->n_chunks; ++i) {
        if (chunk_to_solver[i] < 0 || chunk_to_solver[i] >= K)
            return fail(c, CHICLE_EINVAL, "chunk %d assigned to solver %d, K=%d", i, chunk_to_solver[i], K);
        count[chunk_to_solver[i]] += 1;
    }
    int max_list = 0;
    for (int32_t k = 0; k < K; ++k) max_list = std::max(max_list, count[k]);
    if (max_list > MAX_LIST_LDS) return fail(c, CHICLE_EINVAL, "a solver owns %d chunks, limit %d", max_list, MAX_LIST_LDS);

    std::vector<SolverDev> sol(K);
    std::vector<int32_t> list(c->n_chunks), prefix(c->n_chunks), chunk_first(c->n_chunks), list_base(c->n_chunks);
    int32_t pos = 0, tile = 0;
    int64_t perm_off = 0;
    for (int32_t k = 0; k < K; ++k) {
        sol[k].list_begin = pos; sol[k].n_chunks = count[k]; sol[k].perm_off = perm_off;
        int32_t rows = 0;
        for (int32_t i = 0; i < c->n_chunks; ++i) {        // ascending chunk id
            if (chunk_to_solver[i] != k) continue;
            list[pos] = i; prefix[pos] = rows; chunk_first[i] = rows; list_base[pos] = (int32_t)(perm_off + rows);
            rows += c->chunks[i].n_rows; ++pos;
        }
        sol[k].n_rows = rows;
        sol[k].tile_begin = tile;
        tile += (rows + BATCH - 1) / BATCH;
        perm_off += rows;
    }
    if (tile > c->max_tiles) return fail(c, CHICLE_ENOMEM, "tile scratch too small");
    std::vector<int32_t> tile_solver(std::max(tile, 1));
    for (int32_t k = 0; k < K; ++k)
        for (int32_t t = sol[k].tile_begin; t < sol[k].tile_begin + (sol[k].n_rows + BATCH - 1) / BATCH; ++t)
            tile_solver[t] = k;
    // work items of the gap kernels: blocks of 256/LPR rows inside a chunk
    const double avg = c->dense ? (double)c->d : (double)c->total_entries / (double)c->n_total;
    c->gap_lpr = choose_lpr(c->dense ? avg / 4 : avg);
    const int rows_per_item = 256 / c->gap_lpr;
    std::vector<int32_t> items(c->n_chunks + 1, 0);
    for (int32_t i = 0; i < c->n_chunks; ++i)
        items[i + 1] = items[i] + (c->chunks[i].n_rows + rows_per_item - 1) / rows_per_item;

    // Stream order keeps earlier kernels ahead of these copies; wait before the host vectors go away.
    HIP_TRY(c, hipMemcpyAsync(c->chunks_dev, c->chunks.data(), sizeof(ChunkDev) * (size_t)c->n_chunks, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipMemcpyAsync(c->solvers_dev, sol.data(), sizeof(SolverDev) * (size_t)K, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipMemcpyAsync(c->solver_chunks_dev, list.data(), sizeof(int32_t) * (size_t)c->n_chunks, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipMemcpyAsync(c->solver_prefix_dev, prefix.data(), sizeof(int32_t) * (size_t)c->n_chunks, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipMemcpyAsync(c->item_prefix_dev, items.data(), sizeof(int32_t) * ((size_t)c->n_chunks + 1), hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipMemcpyAsync(c->tile_solver_dev, tile_solver.data(), sizeof(int32_t) * (size_t)tile, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipMemcpyAsync(c->chunk_first_dev, chunk_first.data(), sizeof(int32_t) * (size_t)c->n_chunks, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipMemcpyAsync(c->list_base_dev, list_base.data(), sizeof(int32_t) * (size_t)c->n_chunks, hipMemcpyHostToDevice, c->stream));
    hipLaunchKernelGGL(fill_row_chunk, dim3(c->n_chunks), dim3(256), 0, c->stream, c->chunks_dev,
                       c->solver_chunks_dev, c->list_base_dev, c->row_chunk_dev);
    HIP_TRY(c, hipGetLastError());
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    if (c->state == ST_LOADING && !c->dense && c->max_row_len <= RENUMBER_MAX_ROW) {
        const int rc = renumber_columns(c);
        if (rc) return rc;
    }
    c->K = K;
    c->chunk_to_solver.assign(chunk_to_solver, chunk_to_solver + c->n_chunks);
    c->solvers = sol;
    c->max_list = max_list;
    c->most_rows = 0;
    for (const SolverDev &k : sol) c->most_rows = std::max(c->most_rows, k.n_rows);
    c->n_tiles = tile;
    c->gap_items = items[c->n_chunks];
    c->state = ST_READY;
    // long rows: as many workgroups per solver as the chip has compute units for, each owning a range of columns
    c->cluster = c->long_rows ? std::max(1, std::min(CLUSTER_MAX, c->cu_count / ((K + L2_PARTITIONS - 1) / L2_PARTITIONS * L2_PARTITIONS))) : 1;
    c->blocks_ready = false;
    if (c->compact) {
        // Compact private vectors: which columns each solver's chunks contain, where each of them lives in
        // the solver's vector, and that index for every stored entry.  The columns the batched solver keeps
        // on chip are present in every solver's vector, at their own index.
        int64_t max_nnz = 1;
        for (const ChunkDev &ch : c->chunks) max_nnz = std::max(max_nnz, padded_entries(ch.nnz));
        const dim3 egrid(grid_for(max_nnz, 256, 1024), c->n_chunks);
        HIP_TRY(c, hipMemcpyAsync(c->chunk_owner_dev, chunk_to_solver, sizeof(int32_t) * (size_t)c->n_chunks, hipMemcpyHostToDevice, c->stream));
        HIP_TRY(c, hipMemsetAsync(c->bits_dev, 0, sizeof(unsigned) * (size_t)c->words * (size_t)K, c->stream));
        // columns that several rows of a solver hold: for the solvers that take rows longer than the batched one does
        unsigned *multi = batched_eligible(c) ? nullptr : c->multi_dev;
        if (multi) HIP_TRY(c, hipMemsetAsync(c->multi_dev, 0, sizeof(unsigned) * (size_t)c->words * (size_t)K, c->stream));
        // (few workgroups per chunk: each of them adds a bitmap of its own to the solver's at the end)
        const dim3 mgrid(grid_for(max_nnz, 256 * 64, std::max(1, 4096 / c->n_chunks)), c->n_chunks);
        hipLaunchKernelGGL(mark_columns, mgrid, dim3(256), 0, c->stream, c->chunks_dev, c->chunk_owner_dev, c->bits_dev, c->words, multi);
        const int forced = batched_eligible(c) ? batched_layout(c).n_hot : 0;
        if (forced > 0)
            hipLaunchKernelGGL(force_columns, dim3(K), dim3(256), 0, c->stream, c->bits_dev, c->words, forced);
        hipLaunchKernelGGL(prefix_columns, dim3(K), dim3(1024), 0, c->stream, c->bits_dev, c->pref_dev, c->words, c->count_dev);
        if (multi)
            hipLaunchKernelGGL(prefix_columns, dim3(K), dim3(1024), 0, c->stream, multi, c->mpref_dev, c->words, c->mcount_dev);
        HIP_TRY(c, hipGetLastError());
        std::vector<int32_t> cnt(K), shared(K, 0);
        if (multi) HIP_TRY(c, hipMemcpyAsync(shared.data(), c->mcount_dev, sizeof(int32_t) * (size_t)K, hipMemcpyDeviceToHost, c->stream));
        HIP_TRY(c, hipMemcpyAsync(cnt.data(), c->count_dev, sizeof(int32_t) * (size_t)K, hipMemcpyDeviceToHost, c->stream));
        HIP_TRY(c, hipStreamSynchronize(c->stream));
        std::vector<int64_t> off(K);
        int64_t used = 0;
        for (int32_t k = 0; k < K; ++k) { off[k] = used; used += ((int64_t)cnt[k] + 63) / 64 * 64; }
        if (used > c->u_capacity) return fail(c, CHICLE_ENOMEM, "private vectors need %lld floats, %lld reserved", (long long)used, (long long)c->u_capacity);
        c->u_used = used;
        HIP_TRY(c, hipMemcpyAsync(c->u_off_dev, off.data(), sizeof(int64_t) * (size_t)K, hipMemcpyHostToDevice, c->stream));
        hipLaunchKernelGGL(compact_indices, egrid, dim3(256), 0, c->stream, c->chunks_dev, c->chunk_owner_dev, c->bits_dev,
                           c->pref_dev, c->words, (const unsigned *)multi);
        HIP_TRY(c, hipGetLastError());
        if (multi) {
            // Long rows: in front of the copy of the entries by column.  Where that leaves too little (rows of some 350 entries and
            // more, nearly all of them in columns that two rows of the solver hold), there is no copy under this assignment: the
            // gap goes over the rows, the merge through the private vectors.
            bool too_small;
            int rc = lay_out_blocks(c, shared, cnt, c->long_rows ? copy_at(c) : c->layout_bytes, &too_small);
            if (rc) return rc;
            if (too_small && c->long_rows) {
                c->columns.blocks = 0;
                rc = lay_out_blocks(c, shared, cnt, c->layout_bytes, &too_small);
                if (rc) return rc;
            }
        }
        if (forced > 0) {
            int max_rows = 1;
            for (const ChunkDev &ch : c->chunks) max_rows = std::max(max_rows, ch.n_rows);
            HIP_TRY(c, hipMemsetAsync(c->count_dev, 0, sizeof(int32_t), c->stream));
            hipLaunchKernelGGL(max_entries_beyond, dim3(grid_for(max_rows, 256, 64), c->n_chunks), dim3(256), 0, c->stream,
                               c->chunks_dev, forced, c->count_dev);
            HIP_TRY(c, hipGetLastError());
            HIP_TRY(c, hipMemcpyAsync(&c->max_tail_entries, c->count_dev, sizeof(int32_t), hipMemcpyDeviceToHost, c->stream));
        }
        HIP_TRY(c, hipStreamSynchronize(c->stream));      // cnt, off and the caller's table go out of scope
    }
    if (c->long_rows) {
        if (c->cluster > 1 && c->split_built_for != c->cluster) {
            int max_rows = 1;
            for (const ChunkDev &ch : c->chunks) max_rows = std::max(max_rows, ch.n_rows);
            hipLaunchKernelGGL(row_split_offsets, dim3(grid_for(max_rows, 256, 64), c->n_chunks), dim3(256), 0, c->stream,
                               c->chunks_dev, (int)c->d, c->cluster, c->row_split_dev);
            HIP_TRY(c, hipGetLastError());
            c->split_built_for = c->cluster;
        }
        if (layout_in_use(c) > copy_at(c)) c->columns.blocks = 0;
        else if (c->columns.blocks == 0 && (dots_pay(c) || (c->blocks_ready && merge_pays(c)))) {
            const int rc = order_by_column(c);
            if (rc) return rc;
        }
    }
    c->dots_by_columns = c->columns.blocks > 0 && dots_pay(c);
    c->merge_by_columns = c->columns.blocks > 0 && c->blocks_ready && merge_pays(c);
    c->coef_pending = c->private_stale = false;
    return clear_all_private(c);
}

int chicle_solver_rows(chicle_ctx *c, int64_t *rows_out)
{
    if (!c || !rows_out) return CHICLE_EINVAL;
    if (c->state == ST_LOADING) return fail(c, CHICLE_ESTATE, "no assignment yet");
    for (int32_t k = 0; k < c->K; ++k) rows_out[k] = c->solvers[k].n_rows;
    return CHICLE_OK;
}

int chicle_set_solver(chicle_ctx *c, int32_t kind)
{
    if (!c) return CHICLE_EINVAL;
    if (kind != CHICLE_SOLVER_AUTO && kind != CHICLE_SOLVER_ROWWISE && kind != CHICLE_SOLVER_BATCHED &&
        kind != CHICLE_SOLVER_ROWWISE_ONE_CU && kind != CHICLE_SOLVER_BATCHED_ONE_CU)
        return fail(c, CHICLE_EINVAL, "unknown solver kind %d", kind);
    c->cluster_allowed = kind != CHICLE_SOLVER_ROWWISE_ONE_CU;
    c->split_allowed = kind != CHICLE_SOLVER_BATCHED_ONE_CU;
    c->solver_kind = kind == CHICLE_SOLVER_ROWWISE_ONE_CU ? CHICLE_SOLVER_ROWWISE : kind == CHICLE_SOLVER_BATCHED_ONE_CU ? CHICLE_SOLVER_BATCHED : kind;
    return CHICLE_OK;
}

int chicle_set_l1(chicle_ctx *c, double l1)
{
    if (!c) return CHICLE_EINVAL;
    if (!(l1 >= 0.0) || !std::isfinite(l1)) return fail(c, CHICLE_EINVAL, "l1 must be finite and >= 0");
    if (c->state == ST_EPOCH_DONE) return fail(c, CHICLE_ESTATE, "aggregate first");
    c->l1 = l1;
    if (c->state != ST_LOADING) {      // the shared vector is the threshold's image of what the solvers have summed so far
        hipLaunchKernelGGL(mirror_from_double, dim3(grid_for(c->d, 256, 2048)), dim3(256), 0, c->stream, c->w64, c->w,
                           (int64_t)c->d, c->l1);
        HIP_TRY(c, hipGetLastError());
        c->zw_valid = false;
    }
    return CHICLE_OK;
}

int chicle_local_epoch(chicle_ctx *c, const int32_t *perm_device)
{
    if (!c) return CHICLE_EINVAL;
    if (!perm_device) return fail(c, CHICLE_EINVAL, "perm is NULL");
    return chicle_local_epoch_ahead(c, perm_device, nullptr);
}

int chicle_local_epoch_ahead(chicle_ctx *c, const int32_t *perm_device, const int32_t *perm_next_device)
{
    if (!c) return CHICLE_EINVAL;
    if (c->state != ST_READY) return fail(c, CHICLE_ESTATE, c->state == ST_LOADING ? "assign first" : "aggregate before the next local epoch");
    if (!perm_device && !c->ahead_valid)
        return fail(c, CHICLE_EINVAL, "perm is NULL and the previous pass announced no orders (or an assign dropped them)");
    const Route route = route_of(c);
    if (c->solver_kind == CHICLE_SOLVER_BATCHED && route == ROUTE_ROWWISE)      // (nothing announced is touched by a refused call)
        return fail(c, CHICLE_EINVAL, "batched solver needs sparse rows of at most %d entries and at most %d chunks per solver, or dense rows of at most %d columns", GRAM_MAX_ROW, BATCHED_MAX_LIST, DENSE_NAMED_MAX_D);
    const bool batched = route == ROUTE_BATCHED || route == ROUTE_DENSE;
    // NULL: the orders the previous call announced, from the library's own copy of them
    const bool announced = perm_device == nullptr;
    const bool tiles_ready = announced && batched && c->ahead_tiles;
    if (announced) perm_device = c->perm_ahead[1 - c->ahead_buf];
    c->ahead_valid = false;
    // Tiles prepared ahead are of the orders that the previous pass announced: this pass uses them or they are dropped,
    // whichever solver it runs.  Either way everything from here on follows the kernel that forms them (it reads its copy
    // of the orders, which the announcement after this one overwrites).
    if (c->ahead_tiles) HIP_TRY(c, hipStreamWaitEvent(c->stream, c->ev_join, 0));
    c->ahead_tiles = false;
    if (perm_next_device) {
        // Copied on the context's stream, so the caller's buffer is an ordinary stream-ordered input.
        HIP_TRY(c, hipMemcpyAsync(c->perm_ahead[c->ahead_buf], perm_next_device, sizeof(int32_t) * (size_t)c->n_total,
                                  hipMemcpyDeviceToDevice, c->stream));
        perm_next_device = c->perm_ahead[c->ahead_buf];
        c->ahead_buf = 1 - c->ahead_buf;
        c->ahead_valid = true;
    }
    if (route == ROUTE_DENSE && !dense_tiles_ahead(c)) perm_next_device = nullptr;      // (they are kept all the same)
    seg_begin(c, CHICLE_SEG_LOCAL_EPOCH);
    int rc = CHICLE_OK;
    c->coef_pending = false;
    if (c->private_stale && route != ROUTE_BLOCKS) {            // (all others start from zero)
        if (c->compact) clear_device_words(c, c->u, c->u_used);
        else rc = clear_all_private(c);
        if (rc) return rc;
        c->private_stale = false;
    }
    if (!c->zw_valid) rc = run_row_pass(c, c->gap_scratch);     // x_i . w for the current w
    if (rc == CHICLE_OK) {
        if (batched) {
            rc = c->loss == CHICLE_LOSS_HINGE ? launch_batched<0>(c, perm_device, tiles_ready, perm_next_device)
                 : c->loss == CHICLE_LOSS_SQUARED ? launch_batched<1>(c, perm_device, tiles_ready, perm_next_device)
                                                  : launch_batched<2>(c, perm_device, tiles_ready, perm_next_device);
        } else if (route == ROUTE_BLOCKS) {
            rc = c->loss == CHICLE_LOSS_HINGE ? launch_blocks<0>(c, perm_device)
                 : c->loss == CHICLE_LOSS_SQUARED ? launch_blocks<1>(c, perm_device)
                                                  : launch_blocks<2>(c, perm_device);
        } else {
            seg_begin(c, CHICLE_SEG_EPOCH_CHAIN);
            rc = c->loss == CHICLE_LOSS_HINGE ? launch_rowwise<0>(c, perm_device)
                 : c->loss == CHICLE_LOSS_SQUARED ? launch_rowwise<1>(c, perm_device)
                                                  : launch_rowwise<2>(c, perm_device);
            seg_end(c, CHICLE_SEG_EPOCH_CHAIN);
        }
    }
    seg_end(c, CHICLE_SEG_LOCAL_EPOCH);
    if (rc) {
        c->private_stale = true;
        return rc;
    }
    c->state = ST_EPOCH_DONE;
    c->epoch_ran = true;
    return CHICLE_OK;
}

int chicle_local_epoch_host_perm(chicle_ctx *c, const int32_t *perm_host)
{
    if (!c) return CHICLE_EINVAL;
    if (c->state != ST_READY) return fail(c, CHICLE_ESTATE, c->state == ST_LOADING ? "assign first" : "aggregate before the next local epoch");
    if (!perm_host) return fail(c, CHICLE_EINVAL, "perm is NULL");
    if (c->pinned_orders) {
        if (c->orders_in_flight) HIP_TRY(c, hipStreamSynchronize(c->stream));
        std::memcpy(c->pinned + c->pinned_orders, perm_host, sizeof(int32_t) * (size_t)c->n_total);
        c->orders_in_flight = true;
        hipLaunchKernelGGL(copy_words, dim3(grid_for(c->n_total, 256, 1024)), dim3(256), 0, c->stream,
                           (const int32_t *)(c->pinned_dev + c->pinned_orders), c->n_total, c->perm_stage);
        HIP_TRY(c, hipGetLastError());
    } else {
        HIP_TRY(c, hipMemcpyAsync(c->perm_stage, perm_host, sizeof(int32_t) * (size_t)c->n_total, hipMemcpyHostToDevice, c->stream));
        HIP_TRY(c, hipStreamSynchronize(c->stream));
    }
    return chicle_local_epoch(c, c->perm_stage);
}

int chicle_aggregate(chicle_ctx *c)
{
    if (!c) return CHICLE_EINVAL;
    if (c->state != ST_EPOCH_DONE) return fail(c, CHICLE_ESTATE, "no local epoch pending");
    seg_begin(c, CHICLE_SEG_AGGREGATE);
    const int64_t d4 = c->ld_v / 4;
    if (c->coef_pending) {
        const size_t sh = (sizeof(double) << c->columns.bucket_log2) + sizeof(float) * CO_ROWS;
        HIP_TRY(c, hipFuncSetAttribute((const void *)column_merge, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh));
        hipLaunchKernelGGL(column_merge, dim3((unsigned)c->columns.buckets), dim3(CO_THREADS), sh, c->stream, c->columns, (const float *)c->co_coef_dev, c->w64,
                           c->w, (int64_t)c->d, (float)(1.0 / (double)c->K), c->l1);
    } else if (c->compact) {
        // few words: the solvers are divided over slices too, so that the chip is filled.  Thinly occupied vectors (under an
        // eighth of the columns per solver on average): entries are picked straight from memory
        const bool thin = c->u_used * 8 < (int64_t)c->K * (int64_t)c->d;
        const int wg_words = thin ? AGG_THIN_WORDS : AGG_WORDS;
        const unsigned gx = (unsigned)((c->words + wg_words - 1) / wg_words);
        const unsigned gy = (unsigned)std::max(1, std::min(c->K, (int)(1024 / gx)));
        const float inv_sigma = (float)(1.0 / (double)c->K);
        if (thin) {
            hipLaunchKernelGGL(aggregate_compact_thin, dim3(gx, gy), dim3(AGG_THIN_WORDS), 0, c->stream, c->w64, c->w, c->u, c->u_off_dev, c->bits_dev,
                               c->pref_dev, c->words, (int64_t)c->d, c->K, inv_sigma, c->l1);
            if (gy > 1)
                hipLaunchKernelGGL(mirror_from_double, dim3(grid_for(c->d, 256, 2048)), dim3(256), 0, c->stream, c->w64, c->w, (int64_t)c->d, c->l1);
        } else
            hipLaunchKernelGGL(aggregate_compact, dim3(gx, gy), dim3(AGG_THREADS), 0, c->stream, c->w64, c->w, c->u, c->u_off_dev, c->bits_dev,
                               c->pref_dev, c->words, (int64_t)c->d, c->K, inv_sigma, c->l1, c->tickets_dev + GAP_TICKETS);
    } else
        hipLaunchKernelGGL(aggregate_broadcast, dim3(grid_for(d4, 256, 4096)), dim3(256), 0, c->stream, c->w64, c->w,
                           c->u, c->ld_v, d4, c->K, (float)(1.0 / (double)c->K), c->l1);
    seg_end(c, CHICLE_SEG_AGGREGATE);
    HIP_TRY(c, hipGetLastError());
    c->private_stale = c->coef_pending;      // (the other merges clear the private vectors)
    c->coef_pending = false;
    c->zw_valid = false;
    c->state = ST_READY;
    return CHICLE_OK;
}

static int gap_with(chicle_ctx *c, GapScratch gs, double *primal, double *dual, double *gap)
{
    if (c->state != ST_READY) return fail(c, CHICLE_ESTATE, "gap is defined on the aggregated state");
    seg_begin(c, CHICLE_SEG_GAP);
    gs.finish = true;
    c->gap_seq += 1;
    const int rc = run_row_pass(c, gs);
    seg_end(c, CHICLE_SEG_GAP);
    if (rc) return rc;
    // The sums and the error flag arrive in pinned host memory, and behind them the gap's number: what is waited for is that word
    // (waiting for the stream takes some 5 us more: ten rounds of 4096 x 256 706 us and 686).  Should it be long in coming, the stream is waited for.
    const double *h = (const double *)c->pinned;
    const unsigned long long *arrived = (const unsigned long long *)(h + 5);
    for (int spins = 0; __atomic_load_n(arrived, __ATOMIC_ACQUIRE) != c->gap_seq; ++spins) {
        if (spins == GAP_SPINS) {
            HIP_TRY(c, hipStreamSynchronize(c->stream));
            break;
        }
        __builtin_ia32_pause();
    }
    c->orders_in_flight = false;
    if (h[3] != 0.0) return flag_status(c, (int)h[3]);
    const double n = (double)c->n_total;
    const double P = c->lambda * (0.5 * h[2] + c->l1 * h[4]) + h[0] / n;     // (the regulariser's conjugate at the dual image is |w|^2 / 2)
    const double D = -0.5 * c->lambda * h[2] - h[1] / n;
    if (primal) *primal = P;
    if (dual) *dual = D;
    if (gap) *gap = P - D;
    return CHICLE_OK;
}

int chicle_gap(chicle_ctx *c, double *primal, double *dual, double *gap)
{
    if (!c) return CHICLE_EINVAL;
    return gap_with(c, c->gap_scratch, primal, dual, gap);
}

int chicle_gap_noalloc(chicle_ctx *c, double *primal, double *dual, double *gap)
{
    if (!c) return CHICLE_EINVAL;
    if (2 * (int64_t)c->n_chunks > GAP_PARTS)
        return fail(c, CHICLE_EINVAL, "%d chunks: the fixed scratch holds partial sums for at most %d", c->n_chunks, GAP_PARTS / 2);
    if (!c->static_scratch) return fail(c, CHICLE_EDEVICE, "the fixed scratch array was not found on this device");
    GapScratch gs;
    gs.loss = c->static_scratch;
    gs.conj = gs.loss + GAP_PARTS;
    gs.wsq = gs.conj + GAP_PARTS;
    gs.wabs = gs.wsq + WSQ_PARTS;
    gs.parts = GAP_PARTS;
    return gap_with(c, gs, primal, dual, gap);
}

// Device -> pageable host memory.  A copy straight to pageable memory of this size runs at a fifth of the link's rate (80 MB:
// 8 ms; to pinned memory 1.4 ms), and half of it is the pages of a fresh array being touched for the first time.  Pieces
// therefore go through pinned memory, and several threads copy them on, each with a piece and an event of its own.
// Vectors of less than two pieces take the plain copy, and so does everything on hipStreamPerThread: that handle means a
// stream of its own in every thread, and the helpers' copies would not follow the caller's kernels.
// The stream is idle up to the copy on return.
static int read_to_host(chicle_ctx *c, void *dst, const void *src, size_t bytes)
{
    const bool in_pieces = bytes >= 2 * READ_PIECE && c->stream != hipStreamPerThread;
    int before = 0;
    if (in_pieces) {                       // the events must be of the stream's device, whichever the caller has selected
        HIP_TRY(c, hipGetDevice(&before));
        HIP_TRY(c, hipSetDevice(c->device));
    }
    if (in_pieces && !c->read_pinned) {
        bool ok = hipHostMalloc((void **)&c->read_pinned, READ_PIECE * READ_THREADS, hipHostMallocDefault) == hipSuccess;
        for (int t = 0; ok && t < READ_THREADS; ++t)
            ok = c->read_ev[t] != nullptr || hipEventCreateWithFlags(&c->read_ev[t], hipEventDisableTiming) == hipSuccess;
        if (!ok) {
            if (c->read_pinned) (void)hipHostFree(c->read_pinned);
            c->read_pinned = nullptr;
            (void)hipGetLastError();
        }
    }
    if (!in_pieces || !c->read_pinned) {
        if (in_pieces) (void)hipSetDevice(before);
        HIP_TRY(c, hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, c->stream));
        return CHICLE_OK;
    }
    const size_t pieces = (bytes + READ_PIECE - 1) / READ_PIECE;
    std::atomic<size_t> next{0};
    std::atomic<int> failed{0};
    auto work = [&](int t) {
        hipError_t e = hipSetDevice(c->device);
        char *piece = c->read_pinned + READ_PIECE * (size_t)t;
        for (size_t p; e == hipSuccess && (p = next.fetch_add(1)) < pieces;) {
            const size_t at = p * READ_PIECE, n = std::min(READ_PIECE, bytes - at);
            e = hipMemcpyAsync(piece, (const char *)src + at, n, hipMemcpyDeviceToHost, c->stream);
            if (e == hipSuccess) e = hipEventRecord(c->read_ev[t], c->stream);
            if (e == hipSuccess) e = hipEventSynchronize(c->read_ev[t]);
            if (e == hipSuccess) std::memcpy((char *)dst + at, piece, n);
        }
        if (e != hipSuccess) failed.store((int)e);
    };
    std::thread others[READ_THREADS - 1];
    int started = 0;
    try {
        for (; started < READ_THREADS - 1; ++started) others[started] = std::thread(work, started + 1);
    } catch (...) {                        // no more threads to be had: those that run do it all
    }
    work(0);
    (void)hipSetDevice(before);
    for (int t = 0; t < started; ++t) others[t].join();
    if (failed.load()) return fail(c, CHICLE_EDEVICE, "read-out: %s", hipGetErrorString((hipError_t)failed.load()));
    return CHICLE_OK;
}

// d floats in internal order on the device -> caller's order on the host.
static int read_vector(chicle_ctx *c, const float *src_internal, float scale, float *host_out)
{
    if (c->pinned_vector) {
        int *flag = (int *)(c->pinned + PINNED_HEAD / 2);
        hipLaunchKernelGGL(to_host_in_caller_order, dim3(grid_for(c->d, 256, 1024)), dim3(256), 0, c->stream, src_internal,
                           c->renumbered ? c->rank_of : (const int32_t *)nullptr, (int64_t)c->d, scale,
                           (float *)(c->pinned_dev + c->pinned_vector), (const int *)c->err_dev, (int *)(c->pinned_dev + PINNED_HEAD / 2));
        HIP_TRY(c, hipGetLastError());
        HIP_TRY(c, hipStreamSynchronize(c->stream));
        c->orders_in_flight = false;
        std::memcpy(host_out, c->pinned + c->pinned_vector, sizeof(float) * (size_t)c->d);
        return flag_status(c, *flag);
    }
    hipLaunchKernelGGL(to_caller_order<float>, dim3(grid_for(c->d, 256, 4096)), dim3(256), 0, c->stream,
                       src_internal, c->renumbered ? c->col_of : (const int32_t *)nullptr, (int64_t)c->d,
                       scale, c->tmp_b);
    HIP_TRY(c, hipGetLastError());
    const int rc = read_to_host(c, host_out, c->tmp_b, sizeof(float) * (size_t)c->d);
    if (rc) return rc;
    return check_deferred(c);
}

int chicle_get_w(chicle_ctx *c, float *w_out)
{
    if (!c || !w_out) return CHICLE_EINVAL;
    return read_vector(c, c->w, 1.0f, w_out);
}

int chicle_set_w(chicle_ctx *c, const float *w_in)
{
    if (!c || !w_in) return CHICLE_EINVAL;
    if (c->state == ST_EPOCH_DONE) return fail(c, CHICLE_ESTATE, "aggregate first");
    if (c->state == ST_LOADING) return fail(c, CHICLE_ESTATE, "assign first (the column order is fixed at the first assign)");
    if (c->l1 > 0.0) return fail(c, CHICLE_ESTATE, "with l1 > 0 the state is the dual image, which w does not determine");
    for (int32_t j = 0; j < c->d; ++j)
        if (!std::isfinite(w_in[j])) return fail(c, CHICLE_EINVAL, "w not finite at %d", j);
    HIP_TRY(c, hipMemcpyAsync(c->tmp_b, w_in, sizeof(float) * (size_t)c->d, hipMemcpyHostToDevice, c->stream));
    hipLaunchKernelGGL(from_caller_order, dim3(grid_for(c->d, 256, 4096)), dim3(256), 0, c->stream, c->tmp_b,
                       c->renumbered ? c->col_of : (const int32_t *)nullptr, (int64_t)c->d, c->w64, c->w);
    HIP_TRY(c, hipGetLastError());
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    c->zw_valid = false;
    return CHICLE_OK;
}

int chicle_get_delta_w(chicle_ctx *c, int32_t solver, float *dw_out)
{
    if (!c || !dw_out) return CHICLE_EINVAL;
    if (c->state != ST_EPOCH_DONE) return fail(c, CHICLE_ESTATE, "updates exist only between local_epoch and aggregate");
    if (solver < -1 || solver >= c->K) return fail(c, CHICLE_EINVAL, "solver %d, K=%d", solver, c->K);
    if (c->coef_pending && !c->updates_spread) {
        spread_updates(c);
        HIP_TRY(c, hipGetLastError());
        c->updates_spread = true;
    }
    if (c->compact)
        hipLaunchKernelGGL(delta_w_out_compact, dim3(grid_for(c->d, 256, 4096)), dim3(256), 0, c->stream, c->u, c->u_off_dev,
                           c->bits_dev, c->pref_dev, c->words, (int64_t)c->d, c->K, solver, (float)(1.0 / (double)c->K), c->tmp_a);
    else
        hipLaunchKernelGGL(delta_w_out, dim3(grid_for(c->d, 256, 4096)), dim3(256), 0, c->stream, c->u, c->ld_v,
                           (int64_t)c->d, c->K, solver, (float)(1.0 / (double)c->K), c->tmp_a);
    HIP_TRY(c, hipGetLastError());
    return read_vector(c, c->tmp_a, 1.0f, dw_out);
}

int chicle_get_alpha(chicle_ctx *c, int32_t chunk_id, float *alpha_out)
{
    if (!c || !alpha_out) return CHICLE_EINVAL;
    if (chunk_id < 0 || chunk_id >= c->n_chunks || !c->loaded[chunk_id]) return fail(c, CHICLE_EINVAL, "chunk %d not loaded", chunk_id);
    const ChunkDev &ch = c->chunks[chunk_id];
    HIP_TRY(c, hipMemcpy2DAsync(alpha_out, sizeof(float), &ch.st->alpha, sizeof(RowState), sizeof(float),
                                (size_t)ch.n_rows, hipMemcpyDeviceToHost, c->stream));
    return check_deferred(c);
}

int chicle_set_alpha(chicle_ctx *c, int32_t chunk_id, const float *alpha_in)
{
    if (!c || !alpha_in) return CHICLE_EINVAL;
    if (c->state == ST_EPOCH_DONE) return fail(c, CHICLE_ESTATE, "solvers own the chunks until their updates are aggregated");
    if (chunk_id < 0 || chunk_id >= c->n_chunks || !c->loaded[chunk_id]) return fail(c, CHICLE_EINVAL, "chunk %d not loaded", chunk_id);
    const ChunkDev &ch = c->chunks[chunk_id];
    for (int32_t r = 0; r < ch.n_rows; ++r) {
        if (!std::isfinite(alpha_in[r])) return fail(c, CHICLE_EINVAL, "alpha not finite at row %d", r);
        if (c->loss != CHICLE_LOSS_SQUARED && (alpha_in[r] < 0.f || alpha_in[r] > 1.f))
            return fail(c, CHICLE_EINVAL, "hinge alpha outside [0,1] at row %d", r);
    }
    HIP_TRY(c, hipMemcpy2DAsync(&ch.st->alpha, sizeof(RowState), alpha_in, sizeof(float), sizeof(float),
                                (size_t)ch.n_rows, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    return CHICLE_OK;
}

int chicle_get_assignment(chicle_ctx *c, int32_t *chunk_to_solver_out, int32_t *K_out)
{
    if (!c) return CHICLE_EINVAL;
    if (c->state == ST_LOADING) return fail(c, CHICLE_ESTATE, "no assignment yet");
    if (chunk_to_solver_out) std::memcpy(chunk_to_solver_out, c->chunk_to_solver.data(), sizeof(int32_t) * (size_t)c->n_chunks);
    if (K_out) *K_out = c->K;
    return CHICLE_OK;
}

int chicle_solver_ms(chicle_ctx *c, float *ms_out)
{
    if (!c) return CHICLE_EINVAL;
    if (!ms_out) return fail(c, CHICLE_EINVAL, "output is NULL");
    if (!c->epoch_ran) return fail(c, CHICLE_ESTATE, "no local epoch has run");
    std::vector<long long> t(2 * (size_t)c->K);
    HIP_TRY(c, hipMemcpyAsync(t.data(), c->ticks_dev, sizeof(long long) * t.size(), hipMemcpyDeviceToHost, c->stream));
    const int rc = check_deferred(c);
    if (rc) return rc;
    for (int k = 0; k < c->K; ++k) ms_out[k] = (float)((double)(t[2 * k + 1] - t[2 * k]) / (double)c->wall_khz);
    return CHICLE_OK;
}

double chicle_projected_iteration_time(int32_t K_tasks, int32_t nodes, int32_t n_slow, double slow_factor,
                                       int32_t base_nodes)
{
    if (K_tasks < 0 || nodes <= 0 || n_slow < 0 || n_slow > nodes || base_nodes <= 0 ||
        (n_slow > 0 && !(slow_factor > 0.0)))
        return -1.0;
    return projected_iteration_time(K_tasks, nodes, n_slow, slow_factor, base_nodes);
}

int32_t chicle_next_solver_count(const double *gap, int32_t n_gaps, int32_t K, int32_t K_min,
                                 double stall_ratio, int32_t patience, int32_t since_change)
{
    if (!gap || n_gaps < 1 || K < 1 || K_min < 1 || !(stall_ratio > 0.0 && stall_ratio <= 1.0) ||
        patience < 1 || since_change < 0)
        return -1;
    return next_solver_count(gap, n_gaps, K, K_min, stall_ratio, patience, since_change);
}

static bool table_ok(const int32_t *t, int32_t n_chunks, int32_t K)
{
    if (!t || n_chunks < 0 || K <= 0) return false;
    for (int32_t i = 0; i < n_chunks; ++i)
        if (t[i] < 0 || t[i] >= K) return false;
    return true;
}

int chicle_scale_out(const int32_t *chunk_to_solver, int32_t n_chunks, int32_t K_old, int32_t K_new,
                     const uint32_t *draw, int32_t *chunk_to_solver_out)
{
    if (!table_ok(chunk_to_solver, n_chunks, K_old) || K_new <= K_old || !draw || !chunk_to_solver_out)
        return CHICLE_EINVAL;
    scale_out_table(n_chunks, chunk_to_solver, K_old, K_new, draw, chunk_to_solver_out);
    return CHICLE_OK;
}

int chicle_scale_in(const int32_t *chunk_to_solver, int32_t n_chunks, int32_t K_old, int32_t K_new,
                    int32_t *chunk_to_solver_out)
{
    if (!table_ok(chunk_to_solver, n_chunks, K_old) || K_new <= 0 || K_new >= K_old || !chunk_to_solver_out)
        return CHICLE_EINVAL;
    scale_in_table(n_chunks, chunk_to_solver, K_old, K_new, chunk_to_solver_out);
    return CHICLE_OK;
}

int chicle_rebalance(const int64_t *chunk_load, int32_t n_chunks, int32_t K, const double *unit_time,
                     int32_t n_iterations, int32_t max_moves, int32_t *chunk_to_solver, int32_t *n_moved_out)
{
    if (!chunk_load || !table_ok(chunk_to_solver, n_chunks, K) || !unit_time || n_iterations <= 0 || max_moves < 0)
        return CHICLE_EINVAL;
    for (int32_t i = 0; i < n_chunks; ++i)
        if (chunk_load[i] < 0) return CHICLE_EINVAL;
    for (int64_t i = 0; i < (int64_t)n_iterations * K; ++i)
        if (!(unit_time[i] > 0.0) || !std::isfinite(unit_time[i])) return CHICLE_EINVAL;
    const int moved = rebalance_table(chunk_load, n_chunks, K, unit_time, n_iterations, max_moves, chunk_to_solver);
    if (n_moved_out) *n_moved_out = moved;
    return CHICLE_OK;
}

int chicle_sync(chicle_ctx *c)
{
    if (!c) return CHICLE_EINVAL;
    return check_deferred(c);
}

int chicle_set_profiling(chicle_ctx *c, int32_t on)
{
    if (!c) return CHICLE_EINVAL;
    c->profiling = on != 0;
    return CHICLE_OK;
}

int chicle_last_kernel_ms(chicle_ctx *c, int32_t segment, float *ms_out)
{
    if (!c || !ms_out || segment < 0 || segment >= CHICLE_SEG_COUNT) return CHICLE_EINVAL;
    if (!c->seg[segment].recorded) return fail(c, CHICLE_ESTATE, "segment %d was not recorded (profiling off, or not run)", segment);
    HIP_TRY(c, hipEventSynchronize(c->seg[segment].stop));
    HIP_TRY(c, hipEventElapsedTime(ms_out, c->seg[segment].start, c->seg[segment].stop));
    return CHICLE_OK;
}

int chicle_debug_solver(chicle_ctx *c, int32_t *out)
{
    if (!c || !out) return CHICLE_EINVAL;
    if (c->state == ST_LOADING) return fail(c, CHICLE_ESTATE, "no assignment yet");
    const Route route = route_of(c);
    const bool clustered = c->long_rows && c->cluster > 1 && c->cluster_allowed;
    out[0] = route;
    out[1] = route == ROUTE_BLOCKS ? c->blocks_g : route == ROUTE_BATCHED ? 1 + std::max(0, split_tails(c)) : route == ROUTE_ROWWISE && clustered ? c->cluster : 1;
    out[2] = route == ROUTE_BLOCKS && !c->blocks_double;
    out[3] = route == ROUTE_BLOCKS && c->sources_dev == nullptr;
    return CHICLE_OK;
}

int chicle_debug_passes(chicle_ctx *c, int32_t *out)
{
    if (!c || !out) return CHICLE_EINVAL;
    if (c->state == ST_LOADING) return fail(c, CHICLE_ESTATE, "no assignment yet");
    const bool by_column = c->dots_by_columns;
    out[0] = by_column;
    out[1] = c->merge_by_columns;
    out[2] = by_column ? dot_parts(c->n_total, c->entries_loaded) : 0;
    out[3] = 0;
    if (by_column) {
        unsigned with_work = 0;
        for (int g = 0; g < out[2] * c->columns.blocks; ++g)
            if (column_part(g, c->columns.blocks, out[2]).part < out[2]) with_work |= 1u << (g % L2_PARTITIONS);
        out[3] = __builtin_popcount(with_work);
    }
    return CHICLE_OK;
}

// A tile that holds the recurrence solved, N[j][i] with N = (1 - T)^-1, back to T = 1 - N^-1 in place.
static void unsolve_tile(float *tile)
{
    static_assert(BATCH == 64, "64 x 64");
    double M[BATCH][BATCH];                       // M = N^-1, both unit triangular: M N = 1, column by column
    for (int i = 0; i < BATCH; ++i)
        for (int j = i; j >= 0; --j) {
            double sum = 0.0;
            for (int k = j + 1; k <= i; ++k) sum += (double)tile[j * BATCH + k] * M[k][i];
            M[j][i] = (j == i ? 1.0 : 0.0) - sum;
        }
    for (int j = 0; j < BATCH; ++j)
        for (int i = 0; i < BATCH; ++i) tile[j * BATCH + i] = j < i ? (float)-M[j][i] : 0.f;
}

int chicle_debug_gram(chicle_ctx *c, const int32_t *perm_device, float *tiles_out, int64_t capacity_floats,
                      int32_t *n_tiles_out)
{
    if (!c || !perm_device) return CHICLE_EINVAL;
    if (c->state != ST_READY) return fail(c, CHICLE_ESTATE, "needs an assignment and no pending epoch");
    if (!batched_eligible(c) && !dense_eligible(c, GRAM_MAX_ROW)) return fail(c, CHICLE_EINVAL, "batched solver not available for this data");
    if (n_tiles_out) *n_tiles_out = c->n_tiles;
    int rc = drop_ahead(c);
    if (rc) return rc;
    rc = c->loss == CHICLE_LOSS_HINGE ? launch_gram<0>(c, perm_device, c->tile_buf, false, c->stream)
         : c->loss == CHICLE_LOSS_SQUARED ? launch_gram<1>(c, perm_device, c->tile_buf, false, c->stream)
                                          : launch_gram<2>(c, perm_device, c->tile_buf, false, c->stream);
    if (rc) return rc;
    if (tiles_out) {
        const int64_t want = (int64_t)c->n_tiles * TILE_FLOATS;
        if (capacity_floats < want) return fail(c, CHICLE_EINVAL, "need room for %lld floats", (long long)want);
        if (c->dense) {        // in the sparse solver's layout, put together in the other tile set a few tiles at a time
            float *out = c->tiles[1 - c->tile_buf];
            const int at_once = (int)(c->max_tiles * DENSE_TILE_FLOATS / TILE_FLOATS);
            for (int32_t t0 = 0; t0 < c->n_tiles; t0 += at_once) {
                const int n = std::min(at_once, c->n_tiles - t0);
                auto kern = c->loss == CHICLE_LOSS_HINGE ? dense_tiles_out<0> : c->loss == CHICLE_LOSS_SQUARED ? dense_tiles_out<1> : dense_tiles_out<2>;
                hipLaunchKernelGGL(kern, dim3(n), dim3(256), 0, c->stream, c->solvers_dev, c->tile_solver_dev,
                                   (const float *)c->tiles[c->tile_buf], t0, (int)c->d, scalars(c).c, out);
                HIP_TRY(c, hipGetLastError());
                HIP_TRY(c, hipMemcpyAsync(tiles_out + (int64_t)t0 * TILE_FLOATS, out, sizeof(float) * (size_t)n * TILE_FLOATS, hipMemcpyDeviceToHost, c->stream));
                HIP_TRY(c, hipStreamSynchronize(c->stream));
            }
            if (c->tiles_solved[c->tile_buf])
                for (int64_t t = 0; t < want; t += TILE_FLOATS) unsolve_tile(tiles_out + t + BATCH * BATCH);
        } else {
            HIP_TRY(c, hipMemcpyAsync(tiles_out, c->tiles[c->tile_buf], sizeof(float) * (size_t)want, hipMemcpyDeviceToHost, c->stream));
            HIP_TRY(c, hipStreamSynchronize(c->stream));
            float raw[TILE_FLOATS];
            for (int64_t t = 0; t < want; t += TILE_FLOATS) {
                std::memcpy(raw, tiles_out + t, sizeof raw);
                for (int jp = 0; jp < TILE_W; ++jp)
                    for (int i = 0; i < BATCH; ++i) tiles_out[t + jp * BATCH + i] = raw[tile_at(jp, i)];
            }
        }
    }
    return check_deferred(c);
}

const char *chicle_last_error(chicle_ctx *c) { return c ? c->err.c_str() : "null context"; }

void chicle_destroy(chicle_ctx *c)
{
    if (!c) return;
    if (c->side) (void)hipStreamSynchronize(c->side);
    (void)hipStreamSynchronize(c->stream);
    if (c->pinned) (void)hipHostFree(c->pinned);
    if (c->read_pinned) (void)hipHostFree(c->read_pinned);
    for (hipEvent_t ev : c->read_ev)
        if (ev) (void)hipEventDestroy(ev);
    if (c->side) (void)hipStreamDestroy(c->side);
    if (c->ev_fork) (void)hipEventDestroy(c->ev_fork);
    if (c->ev_join) (void)hipEventDestroy(c->ev_join);
    for (int s = 0; s < CHICLE_SEG_COUNT; ++s) {
        if (c->seg[s].start) (void)hipEventDestroy(c->seg[s].start);
        if (c->seg[s].stop) (void)hipEventDestroy(c->seg[s].stop);
    }
    delete c;
}

}  // extern "C"
