// Internal host interface between the ABI layer (mdx_abi.cpp) and the kernel
// files (partition.hip, join.hip).  Not installed; not part of the ABI.
#pragma once

#include <algorithm>
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "mdx_device.hpp"

namespace mdx {

constexpr size_t kAlign = 256;
constexpr size_t kMaxLdsBytes = 160 * 1024;  // LDS of one gfx950 CU

__host__ __device__ inline size_t align_up(size_t x, size_t a = kAlign)
{
    return (x + a - 1) / a * a;
}

inline int ceil_log2(int64_t x)
{
    int b = 0;
    while (b < 62 && ((int64_t)1 << b) < x)
        ++b;
    return b;
}

// Rows<K> of n rows in one buffer: 16-byte rows, or int32 keys and then the
// payloads.
__host__ __device__ inline size_t row_keys_bytes(int64_t n)
{
    return align_up((size_t)n * 4);
}

inline size_t rows_bytes(int64_t n, int key_bytes)
{
    return key_bytes == 8 ? (size_t)n * 16 : row_keys_bytes(n) + (size_t)n * 8;
}

template <typename K>
__host__ __device__ inline Rows<K> make_rows(const void *buf, int64_t n)
{
    char *b = (char *)buf;
    if constexpr (sizeof(K) == 8)
        return Rows<K>{(i64x2 *)b, nullptr};
    else
        return Rows<K>{(K *)b, (int64_t *)(b + row_keys_bytes(n))};
}

inline Dest make_dest(int32_t P, int sbits = 0)
{
    Dest d;
    d.P = (uint64_t)P;
    d.pow2 = (P & (P - 1)) == 0;
    d.mask = d.pow2 ? (uint64_t)(P - 1) : 0;
    d.inv = d.pow2 ? 0 : ~0ull / (uint64_t)P;
    d.sbits = sbits;
    d.ndest = P << sbits;
    d.nbits = ceil_log2(d.ndest);
    return d;
}

// ---- partition ------------------------------------------------------------
// Rows per tile of the partition kernels: kBlock threads x R rows, R = 8, 4 or
// 2.  A tile's rows and its destinations' counts are staged in LDS: the
// largest of 8 and 4 that fits half a CU's, so that two workgroups share a CU
// (6E7 int64 rows, 1024 destinations: 4 rows 1.11 ms, 8 alone on a CU 1.18).
// Where neither does (from 1607 destinations, int32 from 1900), the largest
// that fits the whole: one workgroup per CU then costs less than the
// table of counts, 8 bytes per tile and destination, which smaller tiles write
// and scan (6E7 int64 rows: 2048 destinations, 2 rows 3.03 ms, 8 rows 1.66; 4096,
// 2 rows 7.6 ms, 4 rows 4.13; int32 alike).
constexpr int kPartRowsSmall = 8;      // fused batches, D <= kPartSmallMaxP
constexpr int kPartRowsLarge = 2;      // fused batches beyond
constexpr int kPartSmallMaxP = 256;

// LDS carve-up of part_scatter (bytes, 16-byte aligned pieces).
struct ScatterLds {
    size_t stage_v, stage_k, stage_p, stage_d, whist, tstart, gbase, scratch, total;
};

__host__ __device__ constexpr size_t al16(size_t x)
{
    return (x + 15) & ~(size_t)15;
}

// dig: the tile also stages every row's next-pass digit byte.
__host__ __device__ constexpr ScatterLds scatter_lds(int T, int P, int key_bytes, bool dig)
{
    ScatterLds L = {};
    size_t o = 0;
    L.stage_v = o;
    o = al16(o + (size_t)T * 8);
    L.stage_k = o;
    o = al16(o + (size_t)T * key_bytes);
    L.stage_p = o;
    o = al16(o + (size_t)T * 2);
    L.stage_d = o;  // next-pass digit bytes (when they are written)
    o = al16(o + (dig ? (size_t)T : 0));
    L.whist = o;  // 16-bit counts: a tile holds at most 4096 rows
    o = al16(o + (size_t)kWavesPerBlock * P * 2);
    L.tstart = o;
    o = al16(o + (size_t)P * 4);
    L.gbase = o;
    o = al16(o + (size_t)P * 8);
    L.scratch = o;
    o = al16(o + (size_t)kWavesPerBlock * 8);
    L.total = o;
    return L;
}

// Few rows take smaller tiles too, so that there are two workgroups for
// every CU (1E5 x 1E5, P = 4: 50 tiles of 4096 rows leave most CUs idle).
constexpr int64_t kFillTiles = 512;

inline int part_rows_per_thread(int64_t rows, int32_t ndest, int key_bytes)
{
    for (int R : {8, 4})
        if (rows >= kFillTiles * kBlock * R &&
            scatter_lds(kBlock * R, ndest, key_bytes, false).total <= kMaxLdsBytes / 2)
            return R;
    for (int R : {8, 4})
        if (rows >= kFillTiles / 2 * kBlock * R &&
            scatter_lds(kBlock * 4, ndest, key_bytes, false).total > kMaxLdsBytes / 2 &&
            scatter_lds(kBlock * R, ndest, key_bytes, true).total <= kMaxLdsBytes)
            return R;
    return 2;
}

struct PartLayout {
    int64_t ntiles;
    int rows_per_thread;
    size_t cnt_off, totals_off, bytes;
};

// Tiles of R rows per thread.
inline PartLayout part_layout(int64_t n, int32_t ndest, int R)
{
    PartLayout L;
    L.rows_per_thread = R;
    const int64_t tile = (int64_t)kBlock * L.rows_per_thread;
    L.ntiles = (n + tile - 1) / tile;
    size_t o = 0;
    L.cnt_off = o;
    o += align_up((size_t)ndest * (size_t)L.ntiles * sizeof(int64_t));
    L.totals_off = o;
    o += align_up((size_t)ndest * sizeof(int64_t));
    L.bytes = o;
    return L;
}

// Bytes for any layout that a table of at most n rows takes, alone or with
// another: smaller tables take smaller tiles, whose counts can need more, and
// what is sized for n rows serves fewer too.
inline size_t part_reserve_bytes(int64_t n, int32_t ndest, int key_bytes)
{
    const int top = part_rows_per_thread((int64_t)1 << 40, ndest, key_bytes);
    size_t most = 0;
    for (int R = 2; R <= top; R *= 2) {
        // rows from which larger tiles are taken
        const int64_t below = kFillTiles * kBlock * 2 * R;
        const int64_t rows = R < top && n > below ? below : n;
        most = std::max(most, part_layout(rows, ndest, R).bytes);
    }
    return most;
}

// The least a partition's workspace may hold: the counts of 4096-row tiles to
// 256 destinations and of 1024-row ones beyond.
inline int part_least_rows(int32_t ndest)
{
    return ndest <= 256 ? 8 : 2;
}

inline size_t part_least_bytes(int64_t n, int32_t P)
{
    return part_layout(n, P, part_least_rows(P)).bytes;
}

// What a partition asks of its caller.  With less, down to part_least_bytes, few
// rows take the larger tiles that it holds.
inline size_t part_workspace_bytes(int64_t n, int32_t P, int key_bytes)
{
    return std::max(part_least_bytes(n, P), part_reserve_bytes(n, P, key_bytes));
}

// One table of a partition launch: stable partition into
// make_dest(P, sbits).ndest destinations; off has ndest + 1 entries; ws holds
// part_layout(n, ndest, R).bytes, R = part_rows_per_thread of all the tables'
// rows.  The output is two columns, or with `rows_out` Rows<K> at keys_out
// (pay_out is null).  With dig (n bytes, rows only), every output row's
// digit_of(h, dshift, dbits) is written beside it, for the histogram of a
// following segmented pass.
struct PartArgs {
    const void *keys;
    const int64_t *pay;
    int64_t n;
    void *keys_out;
    int64_t *pay_out;
    int64_t *off;
    uint8_t *dig;
    void *ws;
};

// Partition 1 or 2 tables (same key width and destinations) with one set of
// launches.
hipError_t launch_partition(const PartArgs *tables, int ntables, int key_bytes, int32_t P,
                            int sbits, bool rows_out, int dshift, int dbits, hipStream_t s,
                            size_t ws_bytes = SIZE_MAX);

// ---- segmented partition (second split of the join) -------------------------
// Segment a (rows [segoff[a], segoff[a+1]) of an already partitioned table of
// Rows<K>) is split stably into 2^bits destinations by digit_of(h, shift, bits);
// destination (a, q) lands at [outoff[a 2^bits + q], outoff[a 2^bits + q + 1]).
#ifndef MDX_SEG_ROWS
#define MDX_SEG_ROWS 8
#endif
constexpr int kSegRows = MDX_SEG_ROWS;          // rows per thread
constexpr int kSegTile = kBlock * kSegRows;     // 4096 rows per tile
constexpr int kSegChunkTiles = 8;               // tiles per scan chunk
constexpr int kSegMaxDest = 256;

struct SegLayout {
    int64_t max_tiles, max_chunks;
    size_t tile_start_off, chunk_start_off, cnt_off, csum_off, tile_seg_off, chunk_seg_off, bytes;
};

inline SegLayout seg_layout(int64_t n, int64_t nseg, int bits)
{
    SegLayout L;
    const int64_t D = (int64_t)1 << bits;
    L.max_tiles = (n + kSegTile - 1) / kSegTile + nseg;
    L.max_chunks = L.max_tiles / kSegChunkTiles + nseg + 1;
    size_t o = 0;
    L.tile_start_off = o;
    o += align_up((size_t)(nseg + 1) * sizeof(int64_t));
    L.chunk_start_off = o;
    o += align_up((size_t)(nseg + 1) * sizeof(int64_t));
    L.cnt_off = o;
    o += align_up((size_t)L.max_tiles * D * sizeof(uint32_t));
    L.csum_off = o;
    o += align_up((size_t)L.max_chunks * D * sizeof(int64_t));
    L.tile_seg_off = o;
    o += align_up((size_t)L.max_tiles * sizeof(uint32_t));
    L.chunk_seg_off = o;
    o += align_up((size_t)L.max_chunks * sizeof(uint32_t));
    L.bytes = o;
    return L;
}

// One table of a segmented launch (rows and rows_out: Rows<K>): dig holds every row's
// digit_of(h, shift, bits), one byte per row (bits <= 8), 4-byte aligned and
// readable 4 bytes past its end (it is read as words); segoff has nseg + 1
// entries, outoff nseg 2^bits + 1; ws holds seg_layout(n, nseg, bits).bytes.
struct SegArgs {
    const void *rows;
    const uint8_t *dig;
    int64_t n;
    const int64_t *segoff;
    void *rows_out;
    int64_t *outoff;
    void *ws;
};

// Split 1 or 2 tables (same key width, segment count and digits) with one
// set of launches.
hipError_t launch_seg_partition(const SegArgs *tables, int ntables, int key_bytes, int64_t nseg,
                                int shift, int bits, hipStream_t s);

// ---- batch launches -------------------------------------------------------------
// One launch of a step covers many merges: merge m owns blocks
// [pre[m], pre[m+1]) of the grid (pre in device memory, M + 1 entries,
// pre[M] = blocks) and reads its arguments from record m of a device array
// of records written on the host by the *_rec functions.
struct BatchStage {
    const uint32_t *pre;
    uint32_t blocks;
};

// Record of a merge's first pass over its two tables (tables[0] build,
// tables[1] probe) into rows, with tiles of kBlock R rows, as
// launch_partition would run it; part_rec_bytes() bytes.
size_t part_rec_bytes();
void part_rec(const PartArgs *tables, int key_bytes, int32_t P, int sbits, int R, int dshift,
              int dbits, void *dst);
// Record of a merge's segmented pass, as launch_seg_partition would run it.
size_t seg_rec_bytes();
void seg_rec(const SegArgs *tables, int key_bytes, int64_t nseg, int shift, int bits, void *dst);

// First pass of M merges of one key width and rows per thread R: `tiles`
// (both tables' tiles per merge), `scan` (ceil(2 D / kWavesPerBlock) per
// merge: a wave per table and destination), `offs` (2 per merge).  maxD: the largest destination count; dig: some merge writes
// digit bytes.
hipError_t launch_partition_batch(const void *recs, int M, int key_bytes, int R, int maxD, bool dig,
                                  BatchStage tiles, BatchStage scan, BatchStage offs, hipStream_t s);
// Segmented pass of the merges that have one (others own no blocks): `plan`
// (2 per merge), `hist` (max_chunks of both tables), `scan` (2 nseg),
// `tiles` (max_tiles of both tables); maxbits: the largest digit width.
hipError_t launch_seg_batch(const void *recs, int M, int key_bytes, int maxbits, BatchStage plan,
                            BatchStage hist, BatchStage scan, BatchStage tiles, hipStream_t s);

// ---- radix join (LDS tables per sub-bucket) ---------------------------------
// Sub-bucket s of S = P 2^qbits holds build rows [subL[s], subL[s+1]) and
// probe rows [subR[s], subR[s+1]); partition p owns sub-buckets
// [p 2^qbits, (p+1) 2^qbits).
// Two 512-thread workgroups per CU, each with a 77 KB table in LDS: the time
// of a sub-bucket is mostly the latency of its dependent steps (ticket,
// offsets, row loads, chained scan), and a second workgroup on the CU runs
// while the first waits.  (One workgroup with a 152 KB table for twice the
// rows, and so half the sub-buckets, was 10% slower at 1E8 x 1E8.)  A
// merge's table holds 3456 rows under 4096 chain heads: sub-buckets average
// 0.9 of it (so 1E8 rows in 32 partitions still make 32768 sub-buckets), and
// chains average under 0.8 rows (3840 rows under 2048 heads was 7% slower),
// so a thread walks the chains of two probe rows at a time (four: 2%
// slower).  The fused batch's join keeps 3840 rows under 2048 heads and
// walks four chains at a time: its mid-size merges (1E4 to 1E6 rows) gain
// more from 10% larger sub-buckets (fewer of them) than from shorter chains.
#ifndef MDX_JOIN_PER_CU
#define MDX_JOIN_PER_CU 2
#endif
#ifndef MDX_JOIN_CAP
#define MDX_JOIN_CAP 3456
#endif
#ifndef MDX_JOIN_HEADS
#define MDX_JOIN_HEADS 4096
#endif
#ifndef MDX_BATCH_JOIN_CAP
#define MDX_BATCH_JOIN_CAP 3840
#endif
#ifndef MDX_BATCH_JOIN_HEADS
#define MDX_BATCH_JOIN_HEADS 2048
#endif
#ifndef MDX_JOIN_ROWS
#define MDX_JOIN_ROWS 8
#endif
constexpr int kJoinPerCu = MDX_JOIN_PER_CU;
constexpr int kJoinThreads = 512;
// Geometry of a join workgroup's LDS table: build rows, chain heads, and
// the probe rows of a thread whose chains are walked together.
template <int CAP, int HEADS, int WALK>
struct JoinGeo {
    static constexpr int cap = CAP;
    static constexpr int heads = HEADS;
    static constexpr int walk = WALK;
};
using MergeJoin = JoinGeo<MDX_JOIN_CAP, MDX_JOIN_HEADS, 2>;             // rj_join
using BatchJoin = JoinGeo<MDX_BATCH_JOIN_CAP, MDX_BATCH_JOIN_HEADS, 4>;  // rj_join_batch
constexpr int kJoinCap = MergeJoin::cap;       // build rows per table of a merge
constexpr int kBatchJoinCap = BatchJoin::cap;  // ... of the fused batch
constexpr int kJoinRows = MDX_JOIN_ROWS;    // probe rows per thread per batch
constexpr int kJoinBatch = kJoinThreads * kJoinRows;
// Sub-buckets are sized for this fraction of a table on average (the larger
// side's rows): the largest of thousands stays below the cap (at ~3100 rows
// the cap is six standard deviations of a sub-bucket's size away).
#ifndef MDX_JOIN_FILL
#define MDX_JOIN_FILL 0.9
#endif
constexpr double kJoinFill = MDX_JOIN_FILL;

// A join item: a sub-bucket, or one probe batch of a sub-bucket that holds
// several (a probe key repeated very often: each of its items builds the
// table again, which costs a fraction of a batch's count and emit, and runs
// on a workgroup of its own).  Items are numbered sub-bucket by sub-bucket,
// batch by batch, and are the tiles of the chained scan.
struct RJoinLayout {
    int64_t S, max_items;
    size_t status_off, cursor_off, istart_off, isub_off, plan_off, misc_off, bytes;
};

// Counters of the global-table join's one launch, each on a cache line of its
// own.
constexpr int kSyncStride = 32;
constexpr int kJoinSync = 3;

constexpr int64_t kPlanChunk = 1024;  // sub-buckets planned per workgroup of rj_plan

inline RJoinLayout rjoin_layout(int32_t P, int qbits, int64_t n_probe)
{
    RJoinLayout L;
    L.S = (int64_t)P << qbits;
    L.max_items = L.S + n_probe / kJoinBatch;
    size_t o = 0;
    L.status_off = o;
    o += align_up((size_t)L.max_items * sizeof(uint64_t));
    L.cursor_off = o;
    o += align_up((size_t)P * sizeof(uint64_t));
    L.istart_off = o;
    o += align_up((size_t)(L.S + 1) * sizeof(uint32_t));
    L.isub_off = o;
    o += align_up((size_t)L.max_items * sizeof(uint32_t));
    L.plan_off = o;
    o += align_up((size_t)((L.S + kPlanChunk - 1) / kPlanChunk) * sizeof(uint64_t));
    L.misc_off = o;  // ticket, plan ticket, the plan's results; then join_sync
    o += align_up(256 + kJoinSync * kSyncStride * sizeof(uint32_t));
    L.bytes = o;
    return L;
}

struct RJoinWs {
    uint64_t *status;       // [max_items] chained scan (the first P of them by partition)
    uint64_t *cursor;       // [P] output cursors (by partition)
    uint32_t *istart;       // [S + 1] first item of every sub-bucket (valid when items != S)
    uint32_t *isub;         // [max_items] sub-bucket of every item (likewise)
    uint64_t *plan;         // chained scan of the planning workgroups
    uint32_t *ticket;
    uint32_t *plan_ticket;
    uint32_t *join_sync;    // kJoinSync counters of the global-table join
    // the plan's results: the number of items, and 1 if every build
    // sub-bucket fits an LDS table, else 0 (together, for one load)
    uint32_t *plan_out;
    int64_t S, max_items;
    int32_t P;
};

inline RJoinWs rjoin_ws(void *base, const RJoinLayout &L, int32_t P)
{
    char *b = (char *)base;
    RJoinWs w;
    w.status = (uint64_t *)(b + L.status_off);
    w.cursor = (uint64_t *)(b + L.cursor_off);
    w.istart = (uint32_t *)(b + L.istart_off);
    w.isub = (uint32_t *)(b + L.isub_off);
    w.plan = (uint64_t *)(b + L.plan_off);
    w.ticket = (uint32_t *)(b + L.misc_off);
    w.plan_ticket = w.ticket + 1;
    w.join_sync = w.ticket + 64;
    w.plan_out = w.ticket + 32;  // not on the tickets' cache line
    w.S = L.S;
    w.max_items = L.max_items;
    w.P = P;
    return w;
}

// ---- join table -------------------------------------------------------------
// Partition p of a view over partitions [pb, pe) owns slots
//   [sb(p), sb(p) + 2 n_p + 16),  sb(p) = 2 (off[p] - off[pb]) + 16 (p - pb),
// split into two halves of H_p = n_p + 8 slots.  A key whose hash has top
// bit t lives in half t; half 0 marks empty slots with ~0 and half 1 with 0,
// values no hash of that half can take, so no key value is reserved.
struct TableLayout {
    size_t off_off, flags_off, bump_off, slots_off, gstart_off, grouped_off, bytes;
    int64_t nslots;
};

inline TableLayout table_layout(int64_t n, int32_t P)
{
    TableLayout L;
    L.nslots = 2 * n + 16 * (int64_t)P;
    size_t o = 0;
    L.off_off = o;
    o += align_up((size_t)(P + 1) * sizeof(int64_t));
    L.flags_off = o;
    o += align_up((size_t)P * sizeof(int32_t));
    L.bump_off = o;
    o += align_up((size_t)P * sizeof(int64_t));
    L.slots_off = o;
    o += align_up((size_t)L.nslots * 2 * sizeof(uint64_t));
    L.gstart_off = o;
    o += align_up((size_t)L.nslots * sizeof(int64_t));
    L.grouped_off = o;
    o += align_up((size_t)(n > 0 ? n : 1) * sizeof(int64_t));
    L.bytes = o;
    return L;
}

// Device view of the tables of partitions [pb, pe).
struct TView {
    uint64_t *slots;
    int64_t *gstart;
    int64_t *grouped;
    const int64_t *off;  // build offsets [P+1] (absolute rows)
    int32_t *flags;      // [P]
    int64_t *bump;       // [P]
    int32_t pb, pe;
    Dest d;
    const int32_t *skip;  // optional: kernels do nothing while *skip != 0
};

// ---- probe ------------------------------------------------------------------
// Rows per thread of the probe, which walk together.  Staged build + probe of
// n x n rows, P = 8, in us: 1, 2, 4 (8: two groups of four) rows: n = 1E5 84,
// 89, 89, (106); 6E5 165, 148, 146, (166); 1E7 1563, 1413, 1356, (1478); all
// on a full device's workgroups (1E5 with one per tile: 74).
constexpr int kProbeRows = 4;
constexpr int kProbeTile = kBlock * kProbeRows;     // 2048 rows per tile

struct Deferred {
    int64_t rbeg, rend;  // probe rows of the tile
    int64_t base, count; // output rows [base, base + count)
    int64_t group;
};

struct ProbeLayout {
    int64_t max_tiles;
    size_t off_off, tile_start_off, status_off, ticket_off, ndefer_off, defer_off,
        row_pre_off, row_gs_off, bytes;
};

inline ProbeLayout probe_layout(int64_t n, int32_t P)
{
    ProbeLayout L;
    L.max_tiles = (n + kProbeTile - 1) / kProbeTile + P;
    size_t o = 0;
    L.off_off = o;
    o += align_up((size_t)(P + 1) * sizeof(int64_t));
    L.tile_start_off = o;
    o += align_up((size_t)(P + 1) * sizeof(int64_t));
    L.status_off = o;
    o += align_up((size_t)L.max_tiles * sizeof(uint64_t));
    L.ticket_off = o;
    o += align_up((size_t)P * sizeof(uint32_t));
    L.ndefer_off = o;
    o += align_up(sizeof(uint32_t));
    L.defer_off = o;
    o += align_up((size_t)L.max_tiles * sizeof(Deferred));
    L.row_pre_off = o;
    o += align_up((size_t)(n > 0 ? n : 1) * sizeof(int64_t));
    L.row_gs_off = o;
    o += align_up((size_t)(n > 0 ? n : 1) * sizeof(int64_t));
    L.bytes = o;
    return L;
}

struct ProbeWs {
    int64_t *off;  // [P+1] sanitized probe offsets
    int64_t *tile_start;
    uint64_t *status;
    uint32_t *ticket;
    uint32_t *ndefer;
    Deferred *defer;
    int64_t *row_pre;
    int64_t *row_gs;
    int64_t max_tiles;
};

inline ProbeWs probe_ws(void *base, const ProbeLayout &L)
{
    char *b = (char *)base;
    ProbeWs w;
    w.off = (int64_t *)(b + L.off_off);
    w.tile_start = (int64_t *)(b + L.tile_start_off);
    w.status = (uint64_t *)(b + L.status_off);
    w.ticket = (uint32_t *)(b + L.ticket_off);
    w.ndefer = (uint32_t *)(b + L.ndefer_off);
    w.defer = (Deferred *)(b + L.defer_off);
    w.row_pre = (int64_t *)(b + L.row_pre_off);
    w.row_gs = (int64_t *)(b + L.row_gs_off);
    w.max_tiles = L.max_tiles;
    return w;
}

struct ProbeOut {
    void *key;
    int64_t *lpay;
    int64_t *rpay;
    int64_t cap;
    int64_t *offsets;  // [P+1]
};

// Number of workgroups that fill the device for grid-stride kernels.
int device_fill_blocks();

// Benchmark tracing (mdx_trace_kernel): the launch wrappers call these
// around the launches of the kernels that can be traced.
void trace_begin(const char *kernel, hipStream_t s);
void trace_end(const char *kernel, hipStream_t s);

// A table as two columns, and as rows.
inline Cols cols_of(const void *keys, const int64_t *pay, int key_bytes)
{
    return Cols{(const char *)keys, (const char *)pay, key_bytes, 8};
}

inline Cols cols_of_rows(const void *rows, int64_t n, int key_bytes)
{
    const char *b = (const char *)rows;
    return key_bytes == 8 ? Cols{b, b + 8, 16, 16} : Cols{b, b + row_keys_bytes(n), 4, 8};
}

// Build a view of `rows` rows: init slots, insert rows, group repeated keys.
hipError_t launch_build(const Cols &table, int key_bytes, const TView &v,
                        int64_t rows, int32_t *status, hipStream_t s);

// Copy the build offsets (sanitized, for n build rows) into the table and
// clear per-partition flags.  off_in may be null (flags only).
hipError_t launch_table_setup(const int64_t *off_in, int64_t n, int64_t *off_tab, int32_t *flags,
                              int64_t *bump, int32_t P, hipStream_t s);

// A merge's global-table join: nothing when *v.skip, else per-partition
// offsets from the first pass's (offPL[p] = offAL[p stride], offPR[p] =
// offAR[p strideR]), the table built from `build`, probed with `probe`, the output and its
// offsets.  one: in one launch (for up to kOneLaunchRows rows of both sides, and
// wherever there is a ProbePart).  sync: kJoinSync zeroed counters, kSyncStride
// apart.
constexpr int64_t kOneLaunchRows = (int64_t)1 << 21;

struct GlobalJoin {
    const int64_t *offAL, *offAR;
    int64_t *offPL, *offPR, *off_tab;
    int64_t n_build, n_probe;
    int32_t stride, strideR, w_P;
    TView v;
    ProbeWs w;
    ProbeOut o;
    int32_t *status;
};

// The probe table's partition as a two-pass merge's first pass makes it, for
// a merge split in one pass: the global-table join's output rows follow this
// order whatever the split.  off null: not needed, `probe` has it already.
// ws: part_layout(n, d.ndest, kProbePartRows).bytes.
constexpr int kProbePartRows = 4;
constexpr int kProbePartMax = 256;  // destinations

struct ProbePart {
    const void *keys;
    const int64_t *pay;
    int64_t n;
    void *rows_out;  // Rows<K>: what `probe` reads
    int64_t *off;    // [d.ndest + 1]: g.offAR with g.strideR
    void *ws;
    Dest d;
};

hipError_t launch_global_join(const Cols &build, const Cols &probe, int key_bytes,
                              const GlobalJoin &g, const ProbePart &pp, bool one,
                              uint32_t *sync, hipStream_t s);

// Probe: plan tiles from the probe offsets (sanitized for n probe rows; zero
// output offsets when there are none), then probe and write the output and
// its offsets.
hipError_t launch_probe_plan(const int64_t *offR, int64_t n, int32_t P, const ProbeWs &w,
                             int64_t *offsets, hipStream_t s);
hipError_t launch_probe_group(const Cols &table, int key_bytes, const TView &v, int group,
                              const ProbeWs &w, const ProbeOut &o, int32_t *status, hipStream_t s);

// Count-only join of two partitioned tables (full views, pb = 0, pe = P):
// per-partition output counts into out_offsets (exclusive prefix, total at
// [P]).  v: a table view (off, slots; v.off is written with the sanitized
// build offsets); off_probe [P+1] and pcount [P] are workspace.
hipError_t launch_join_count(const void *lk, const int64_t *lofs, int64_t n_build, const void *rk,
                             const int64_t *rofs, int64_t n_probe, int key_bytes, const TView &v,
                             int64_t *off_probe, uint64_t *pcount, int64_t *out_offsets,
                             int32_t *status, hipStream_t s);

// Radix join: plan (the LDS-fit flag from the build sub-buckets, the items,
// the cleared chained scan), join (which writes the output offsets too,
// unless it places rows by partition).  chunked: a build sub-bucket larger
// than a table is joined in table-sized chunks (the flag stays set and no
// global-table join is needed); otherwise such a sub-bucket clears the flag
// and the join does nothing.
hipError_t launch_rjoin_plan(const int64_t *subL, const int64_t *subR, int64_t S,
                             const RJoinWs &w, bool chunked, int32_t *status, hipStream_t s);
hipError_t launch_rjoin(const void *lrows, int64_t nL, const int64_t *subL, const void *rrows,
                        int64_t nR, const int64_t *subR, int key_bytes, int qbits,
                        const RJoinWs &w, const ProbeOut &o, int32_t *status, bool chunked,
                        hipStream_t s);
// Radix join of every merge of a batch (one key width): record m describes
// merge m (its S sub-buckets, its chained scan jstatus of S entries and
// cursors jcursor of P, output); Spre [M + 1] prefix of the merges' S in device memory, S its
// total; ticket: a device counter; by_part: some merge places its rows by
// partition.  Clears the chained scans, joins (a build sub-bucket larger than
// an LDS table is joined in table-sized chunks), and writes every merge's
// output offsets.
struct JoinRec {
    const void *lrows;    // Rows<K> of nL rows
    const int64_t *subL;  // [S + 1]
    const void *rrows;    // Rows<K> of nR rows
    const int64_t *subR;  // [S + 1]
    int64_t nL, nR;
    uint64_t *jstatus;    // [S]
    uint64_t *jcursor;    // [P]
    int64_t S;
    ProbeOut o;
    int32_t *status;
    int32_t P, qbits;
    int32_t by_part;  // rjoin_by_partition: rows placed by partition cursor
    int32_t pad;
};

// Workgroups of a radix-join launch over S sub-buckets.
int rjoin_grid(int64_t S);

// Whether a radix join places its output rows by partition (a cursor per
// partition and a chained scan over partitions) rather than by sub-bucket
// (a chained scan over sub-buckets): when a partition's 2^qbits sub-buckets
// are many times the G workgroups working at once.
bool rjoin_by_partition(int qbits, int64_t G);

hipError_t launch_rjoin_batch(const JoinRec *recs, int M, const uint32_t *Spre, uint32_t S,
                              uint32_t *ticket, int key_bytes, bool by_part, hipStream_t s);

// A merge's output offsets from the partition cursors, if the radix join ran
// and placed its rows by partition (otherwise nothing is launched).
hipError_t launch_merge_finalize(int qbits, const RJoinWs &w, const ProbeOut &o, hipStream_t s);


// ---- transpose sum (y = x + x^T, float64) -------------------------------------------
hipError_t launch_transpose_sum(const double *x, double *y, int64_t n, hipStream_t s);

}  // namespace mdx
