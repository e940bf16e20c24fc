// Per-partition hash join (the local merge after the shuffle; arXiv
// 2101.08878, Section V-B "cuDF Merge": each worker merges the frames it
// received).  Inner equi-join, multiset semantics; left = build side.
//
// Table of partition p (see TableLayout): open addressing with linear
// probing over 16-byte slots (hash, value), split into two halves by the top
// bit of the hash so that each half has an empty marker no hash of that half
// can equal.  Hashes are stored instead of keys: fmix64 is a bijection, so
// equal hashes mean equal keys.
//
// Build (tbl_init, tbl_insert): every row claims a slot for its hash with a
// compare-and-swap; the first row of a key stores its payload in the value.
// A row that finds its hash already present marks the partition as holding
// a repeated key.  Only such partitions then run the grouped build
// (grp_reset, grp_count, grp_alloc, grp_scatter), which turns the value into
// a cursor and lays the partition's payloads out grouped by key
// ("grouped", with [gstart[s], value[s]) the group of slot s).  A key can
// hold millions of rows (a Zipf distribution's first key), so rows are
// counted and placed per workgroup first: a workgroup's rows of one slot
// meet in an LDS map and reach the slot with one global atomic, and group
// starts are allocated per chunk of slots, not per wave.
//
// Probe (probe_chain): tiles of 2048 probe rows, each inside one partition,
// are taken in order from a ticket counter.  A tile looks up its rows,
// counts its output rows, and obtains the number of output rows of all
// earlier tiles from a chained scan (each tile publishes its count, then its
// inclusive prefix; a successor sums predecessors' counts until it meets an
// inclusive prefix).  Tiles of unique-key partitions write their matches
// directly; tiles of repeated-key partitions record per-row prefixes and are
// expanded by probe_expand, which spreads a tile's output over the whole
// device in chunks (one right row can match millions of left rows).
#include <algorithm>

#include "mdx.h"
#include "mdx_internal.hpp"
#include "mdx_partition.hpp"

namespace mdx {
namespace {

typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint64_t empty_of_half(uint64_t t)
{
    return t ? 0ull : ~0ull;
}

// Slot range of partition p inside a view whose first row is o0.
__device__ __forceinline__ void part_slots(const TView &v, int64_t o0, int p, int64_t &sb,
                                           int64_t &H)
{
    const int64_t a = v.off[p], b = v.off[p + 1];
    sb = 2 * (a - o0) + 16 * (int64_t)(p - v.pb);
    H = b - a + 8;
}

// Partition of slot s: largest p in [pb, pe) with sb(p) <= s.
__device__ __forceinline__ int slot_part(const TView &v, int64_t o0, int64_t s)
{
    int l = v.pb, h = v.pe - 1;
    while (l < h) {
        const int mid = (l + h + 1) >> 1;
        if (2 * (v.off[mid] - o0) + 16 * (int64_t)(mid - v.pb) <= s)
            l = mid;
        else
            h = mid - 1;
    }
    return l;
}

// Slot of hash h in partition (sb, H), or -1.
__device__ __forceinline__ int64_t find_slot(const uint64_t *slots, int64_t sb, int64_t H,
                                             uint64_t h)
{
    const uint64_t t = h >> 63;
    const uint64_t empty = empty_of_half(t);
    const int64_t base = sb + (int64_t)t * H;
    uint64_t i = __umul64hi(h << 1, (uint64_t)H);
    for (int64_t k = 0; k < H; ++k) {
        const uint64_t w = slots[2 * (base + (int64_t)i)];
        if (w == h)
            return base + (int64_t)i;
        if (w == empty)
            return -1;
        if (++i == (uint64_t)H)
            i = 0;
    }
    return -1;
}

// A hash's place in the table: the half it walks, [lo, lo + H), is the top
// bit's half of its partition's slots [sb, sb + 2 H).
__device__ __forceinline__ int64_t half_of(int64_t sb, int64_t H, uint64_t h)
{
    return sb + (int64_t)(h >> 63) * H;
}

__device__ __forceinline__ int64_t home_slot(int64_t sb, int64_t H, uint64_t h)
{
    return half_of(sb, H, h) + (int64_t)__umul64hi(h << 1, (uint64_t)H);
}

__device__ __forceinline__ int64_t next_slot(int64_t at, int64_t sb, int64_t H, uint64_t h)
{
    const int64_t lo = half_of(sb, H, h);
    return at + 1 == lo + H ? lo : at + 1;
}

// Slots of a thread's R hashes (-1: absent) and their values, for the rows of
// mask `open`; the partition of row c owns slots sb(c) on, H(c) per half.  The
// rows walk together: every round issues the loads of all
// unfinished rows at once, so a round costs one memory latency whatever R
// is.  (One row after the other, as first written, a row's two or three
// dependent loads waited for the row before: the probe of 1E7 rows took 651
// us.)
template <int R, typename Sb, typename Hn>
__device__ __forceinline__ void find_slots(const uint64_t *slots, Sb sb, Hn H, const uint64_t *h,
                                           uint32_t open, int64_t *slot, uint64_t *val)
{
    const u64x2 *s2 = (const u64x2 *)slots;
    const uint32_t rows = open;
    uint32_t found = 0;
#pragma unroll
    for (int c = 0; c < R; ++c) {
        slot[c] = rows >> c & 1 ? home_slot(sb(c), H(c), h[c]) : -1;
        val[c] = 0;
    }
    // a half has 8 empty slots, so the walk ends within H steps
    for (int64_t k = 0; open; ++k) {
        u64x2 x[R];
#pragma unroll
        for (int c = 0; c < R; ++c) {
            x[c] = u64x2(0);
            if (open >> c & 1)
                x[c] = s2[slot[c]];
        }
#pragma unroll
        for (int c = 0; c < R; ++c) {
            if (open >> c & 1) {
                if (x[c].x == h[c]) {
                    val[c] = x[c].y;
                    found |= 1u << c;
                    open &= ~(1u << c);
                } else if (x[c].x == empty_of_half(h[c] >> 63) || k >= H(c)) {
                    open &= ~(1u << c);
                } else {
                    slot[c] = next_slot(slot[c], sb(c), H(c), h[c]);
                }
            }
        }
    }
#pragma unroll
    for (int c = 0; c < R; ++c)
        slot[c] = found >> c & 1 ? slot[c] : -1;
}

// Partition of every row of [r0, r1) when they share one (r0 < r1), else -1.
__device__ __forceinline__ int shared_part(const TView &v, int64_t r0, int64_t r1)
{
    const int p = upper_index(v.off, v.pb, v.pe, r0);
    return p + 1 == v.pe || r1 <= v.off[p + 1] ? p : -1;
}

// A workgroup's number and how many there are: of a launch, or of a step
// inside global_join's.
struct Blk {
    int64_t id, n;
};

__device__ __forceinline__ Blk this_block()
{
    return {(int64_t)blockIdx.x, (int64_t)gridDim.x};
}

__device__ __forceinline__ bool skipped(const int32_t *skip)
{
    return skip && *skip != 0;
}

__device__ __forceinline__ bool block_any_dup(const TView &v)
{
    int any = 0;
    for (int p = v.pb + (int)threadIdx.x; p < v.pe; p += kBlock)
        any |= v.flags[p];
    return __syncthreads_or(any) != 0;
}

// ---- build -----------------------------------------------------------------

// One block: the table's sanitized build offsets, cleared per-partition flags.
__device__ __forceinline__ void table_setup_block(const int64_t *off_in, int64_t n,
                                                  int64_t *off_tab, int32_t *flags, int64_t *bump,
                                                  int P, int64_t *scratch)
{
    if (off_in)
        sanitize_offsets(off_in, off_tab, P, n, scratch);
    for (int p = threadIdx.x; p < P; p += kBlock) {
        flags[p] = 0;
        bump[p] = 0;
    }
}

__global__ __launch_bounds__(kBlock) void table_setup(const int64_t *__restrict__ off_in, int64_t n,
                                                      int64_t *__restrict__ off_tab,
                                                      int32_t *__restrict__ flags,
                                                      int64_t *__restrict__ bump, int P)
{
    __shared__ int64_t scratch[kWavesPerBlock];
    table_setup_block(off_in, n, off_tab, flags, bump, P, scratch);
}

__device__ __forceinline__ void tbl_init_by(const Blk &b, const TView &v)
{
    const int64_t o0 = v.off[v.pb];
    const int64_t total = 2 * (v.off[v.pe] - o0) + 16 * (int64_t)(v.pe - v.pb);
    const int64_t stride = (int64_t)b.n * kBlock;
    u64x2 *slots = (u64x2 *)v.slots;
    for (int64_t s = (int64_t)b.id * kBlock + threadIdx.x; s < total; s += stride) {
        const int p = slot_part(v, o0, s);
        int64_t sb, H;
        part_slots(v, o0, p, sb, H);
        u64x2 e;
        e.x = (s - sb < H) ? ~0ull : 0ull;
        e.y = 0;
        slots[s] = e;
    }
}

__global__ __launch_bounds__(kBlock) void tbl_init(TView v)
{
    if (skipped(v.skip))
        return;
    tbl_init_by(this_block(), v);
}

// Inserts rows of the view: with `sample`, every 2^shift-th one; otherwise
// the others (all of them when shift < 0).  A slot's compare-and-swaps are
// made one after the other at the memory, 1 to 2 us each when they come from
// different workgroups, and at the start of a launch every workgroup finds a
// hot key's slot empty: 4E6 rows of which 10% hold one key took 1.8 ms.  So a
// few workgroups insert a sample first (sample_shift), which holds every key
// that repeats often, and its other rows then find it with a load: 0.26 ms.
// The rest runs at the rate of the device's compare-and-swaps (16E9 a second
// over distinct slots, in any order); four rows per thread at a time were
// slower (4E6 distinct keys: 305 against 245 us).
template <typename K>
__device__ __forceinline__ void tbl_insert_by(const Blk &b, const Cols &in, const TView &v,
                                              int shift, bool sample, int32_t *status)
{
    const int64_t o0 = v.off[v.pb], n = v.off[v.pe] - o0;
    const int64_t stride = (int64_t)b.n * kBlock;
    const int step = sample ? shift : 0;  // rows o0 + i 2^step
    const int64_t sampled = !sample && shift >= 0 ? ((int64_t)1 << shift) - 1 : -1;
    for (int64_t i = ((int64_t)b.id * kBlock + threadIdx.x) << step; i < n;
         i += stride << step) {
        if (sampled >= 0 && (i & sampled) == 0)
            continue;
        const int64_t r = o0 + i;
        const uint64_t h = fmix64(key_bits(key_at<K>(in, r)));
        const int p = upper_index(v.off, v.pb, v.pe, r);
        if ((int)part_of(h, v.d) != p) {
            or_status(status, MDX_DEV_BAD_PARTITIONING);
            continue;
        }
        int64_t sb, H;
        part_slots(v, o0, p, sb, H);
        const uint64_t empty = empty_of_half(h >> 63);
        int64_t at = home_slot(sb, H, h);
        // The half holds at most n_p of its H = n_p + 8 slots, so an empty
        // slot exists and the walk ends within H steps.
        for (int64_t k = 0; k < H; ++k) {
            uint64_t *sp = v.slots + 2 * at;
            uint64_t w = ld_agent(sp);
            if (w == empty) {
                uint64_t expect = empty;
                if (__hip_atomic_compare_exchange_strong(sp, &expect, h, __ATOMIC_RELAXED,
                                                         __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT)) {
                    sp[1] = (uint64_t)pay_at(in, r);
                    break;
                }
                w = expect;
            }
            if (w == h) {
                // repeated key: one store per partition suffices (a key can
                // repeat millions of times, each a store to one address)
                if (!v.flags[p])
                    v.flags[p] = 1;
                break;
            }
            at = next_slot(at, sb, H, h);
        }
    }
}

template <typename K>
__global__ __launch_bounds__(kBlock) void tbl_insert(Cols in, TView v, int shift, bool sample,
                                                     int32_t *status)
{
    if (skipped(v.skip))
        return;
    tbl_insert_by<K>(this_block(), in, v, shift, sample, status);
}

// Repeated-key partitions: value := 0 on every slot.
__device__ __forceinline__ void grp_reset_by(const Blk &b, const TView &v)
{
    if (!block_any_dup(v))
        return;
    const int64_t o0 = v.off[v.pb];
    const int64_t total = 2 * (v.off[v.pe] - o0) + 16 * (int64_t)(v.pe - v.pb);
    const int64_t stride = (int64_t)b.n * kBlock;
    for (int64_t s = (int64_t)b.id * kBlock + threadIdx.x; s < total; s += stride) {
        if (v.flags[slot_part(v, o0, s)])
            v.slots[2 * s + 1] = 0;
    }
}

__global__ __launch_bounds__(kBlock) void grp_reset(TView v)
{
    if (skipped(v.skip))
        return;
    grp_reset_by(this_block(), v);
}

// Slots of a thread's R rows r0, r0 + kBlock, ... (below r1): -1 where the row
// lies in no repeated-key partition.  pt: shared_part of the workgroup's rows.
template <typename K, int R>
__device__ __forceinline__ void dup_row_slots(const Cols &in, const TView &v, int64_t o0,
                                              int64_t r0, int64_t r1, int pt, int64_t *slot)
{
    uint64_t h[R], val[R];
    int64_t sb[R], H[R];
    uint32_t open = 0;
    K k[R];
#pragma unroll
    for (int c = 0; c < R; ++c) {
        const int64_t r = r0 + (int64_t)c * kBlock;
        k[c] = r < r1 ? key_at<K>(in, r) : K(0);
    }
#pragma unroll
    for (int c = 0; c < R; ++c) {
        const int64_t r = r0 + (int64_t)c * kBlock;
        h[c] = fmix64(key_bits(k[c]));
        if (r >= r1)
            continue;
        const int p = pt >= 0 ? pt : upper_index(v.off, v.pb, v.pe, r);
        if (!v.flags[p] || (int)part_of(h[c], v.d) != p)
            continue;
        part_slots(v, o0, p, sb[c], H[c]);
        open |= 1u << c;
    }
    find_slots<R>(
        v.slots, [&](int c) { return sb[c]; }, [&](int c) { return H[c]; }, h, open, slot, val);
}

// ---- per-workgroup aggregation of rows by slot ------------------------------------
constexpr int kAggPer = 8;   // rows per thread of grp_count / grp_scatter
constexpr int kAggWalk = 4;  // of them walking together
constexpr int kAggRows = kBlock * kAggPer;
constexpr int kAggMap = 2048;    // LDS map entries: slot -> rows of this workgroup
constexpr int kAggProbe = 8;     // map probes before a row goes to the slot directly
constexpr int64_t kAggNone = -1;

struct AggLds {
    int64_t mkey[kAggMap];   // slot
    int64_t mbase[kAggMap];  // grp_scatter: first place of this workgroup's rows
    uint32_t mcnt[kAggMap];  // rows of this workgroup
};

__device__ __forceinline__ uint32_t agg_home(int64_t s)
{
    return ((uint32_t)s * 0x9E3779B1u) >> (32 - 11);
}
static_assert(kAggMap == 1 << 11, "agg_home takes 11 bits");

// Entry of slot s in the map, inserting it if there is room within
// kAggProbe probes; -1 otherwise.  Entries are never removed, so every row of
// one slot gets the same answer.
__device__ __forceinline__ int agg_insert(int64_t *mkey, int64_t s)
{
    uint32_t h = agg_home(s);
    for (int k = 0; k < kAggProbe; ++k) {
        int64_t cur = mkey[h];
        if (cur == kAggNone) {
            cur = (int64_t)atomicCAS((unsigned long long *)&mkey[h], (unsigned long long)kAggNone,
                                     (unsigned long long)s);
            if (cur == kAggNone)
                return (int)h;
        }
        if (cur == s)
            return (int)h;
        h = (h + 1) & (kAggMap - 1);
    }
    return -1;
}

// Rows of workgroup b: [o0 + b kAggRows, ...) of the view's rows.
__device__ __forceinline__ void agg_rows(const Blk &b, const TView &v, int64_t &o0, int64_t &r0,
                                         int64_t &r1)
{
    o0 = v.off[v.pb];
    const int64_t o1 = v.off[v.pe];
    r0 = o0 + b.id * kAggRows;
    r1 = r0 + kAggRows < o1 ? r0 + kAggRows : o1;
}

// value[s] += rows of the slot's key.
template <typename K>
__device__ __forceinline__ void grp_count_by(const Blk &b, AggLds &lds, const Cols &in,
                                             const TView &v)
{
    if (!block_any_dup(v))
        return;
    int64_t *mkey = lds.mkey;
    uint32_t *mcnt = lds.mcnt;
    for (int i = threadIdx.x; i < kAggMap; i += kBlock) {
        mkey[i] = kAggNone;
        mcnt[i] = 0;
    }
    __syncthreads();
    int64_t o0, r0, r1;
    agg_rows(b, v, o0, r0, r1);
    if (r0 >= r1)
        return;
    int64_t slot[kAggPer];
    const int pt = shared_part(v, r0, r1);
#pragma unroll
    for (int c = 0; c < kAggPer; c += kAggWalk)
        dup_row_slots<K, kAggWalk>(in, v, o0, r0 + threadIdx.x + (int64_t)c * kBlock, r1, pt,
                                   slot + c);
#pragma unroll
    for (int c = 0; c < kAggPer; ++c) {
        if (slot[c] < 0)
            continue;
        const int e = agg_insert(mkey, slot[c]);
        if (e >= 0)
            atomicAdd(&mcnt[e], 1u);
        else
            atomicAdd((unsigned long long *)&v.slots[2 * slot[c] + 1], 1ull);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kAggMap; i += kBlock)
        if (mkey[i] != kAggNone)
            atomicAdd((unsigned long long *)&v.slots[2 * mkey[i] + 1], (unsigned long long)mcnt[i]);
}

template <typename K>
__global__ __launch_bounds__(kBlock) void grp_count(Cols in, TView v, int64_t shares)
{
    if (skipped(v.skip))
        return;
    __shared__ AggLds lds;
    for (Blk b = this_block(); b.id < shares; b.id += b.n, __syncthreads())
        grp_count_by<K>(b, lds, in, v);
}

// Give every key of a repeated-key partition its range of the grouped array:
// gstart[s] = value[s] = (partition's first row) + running total.  Workgroup b
// takes the slots [b kAllocSlots, (b+1) kAllocSlots), read once into
// registers: per partition in it, a scan of the threads' sums, one atomic on
// the partition's allocator, then every thread places its slots' groups from
// there.  (65536 slots per workgroup, read twice: 198 us for 8E6 slots, with
// half the CUs idle.)
constexpr int kAllocPer = 8;
constexpr int64_t kAllocSlots = (int64_t)kBlock * kAllocPer;

__device__ __forceinline__ void grp_alloc_by(const Blk &b, int64_t *scratch, int64_t &s_base,
                                             const TView &v)
{
    if (!block_any_dup(v))
        return;
    const int tid = threadIdx.x;
    const int64_t o0 = v.off[v.pb];
    const int64_t total = 2 * (v.off[v.pe] - o0) + 16 * (int64_t)(v.pe - v.pb);
    const int64_t c0 = (int64_t)b.id * kAllocSlots;
    const int64_t c1 = c0 + kAllocSlots < total ? c0 + kAllocSlots : total;
    if (c0 >= c1)
        return;
    const u64x2 *slots = (const u64x2 *)v.slots;
    u64x2 x[kAllocPer];
#pragma unroll
    for (int k = 0; k < kAllocPer; ++k) {
        const int64_t s = c0 + k * kBlock + tid;
        x[k] = slots[s < c1 ? s : c1 - 1];
    }
    for (int p = slot_part(v, o0, c0); p < v.pe; ++p) {
        int64_t sb, H;
        part_slots(v, o0, p, sb, H);
        if (sb >= c1)
            break;
        if (!v.flags[p])
            continue;
        const int64_t a = sb > c0 ? sb : c0, e = sb + 2 * H < c1 ? sb + 2 * H : c1;
        auto rows = [&](int k) {  // of slot k of this thread, if in p and taken
            const int64_t s = c0 + k * kBlock + tid;
            const bool in = s >= a && s < e && x[k].x != empty_of_half(s - sb >= H ? 1 : 0);
            return in ? (int64_t)x[k].y : 0;
        };
        int64_t sum = 0;
#pragma unroll
        for (int k = 0; k < kAllocPer; ++k)
            sum += rows(k);
        int64_t all;
        const int64_t ex = block_excl_scan(sum, scratch, &all);
        if (tid == 0)
            s_base = (int64_t)atomicAdd((unsigned long long *)&v.bump[p], (unsigned long long)all);
        __syncthreads();
        int64_t run = (v.off[p] - o0) + s_base + ex;
#pragma unroll
        for (int k = 0; k < kAllocPer; ++k) {
            const int64_t c = rows(k), s = c0 + k * kBlock + tid;
            if (c > 0) {
                v.gstart[s] = run;
                v.slots[2 * s + 1] = (uint64_t)run;
                run += c;
            }
        }
        __syncthreads();  // s_base is reused by the next partition
    }
}

__global__ __launch_bounds__(kBlock) void grp_alloc(TView v, int64_t shares)
{
    if (skipped(v.skip))
        return;
    __shared__ int64_t scratch[kWavesPerBlock];
    __shared__ int64_t s_base;
    for (Blk b = this_block(); b.id < shares; b.id += b.n, __syncthreads())
        grp_alloc_by(b, scratch, s_base, v);
}

// grouped[value[s]++] = payload, for every row of a repeated-key partition.
// First the workgroup counts its rows per slot in the map (a row's count so
// far is its rank) and reserves one range per slot; then every row takes its
// rank's place in its slot's range (rows the map could not hold take a place
// from the slot directly).  Slots and ranks stay in registers.
template <typename K>
__device__ __forceinline__ void grp_scatter_by(const Blk &b, AggLds &lds, const Cols &in,
                                               const TView &v)
{
    if (!block_any_dup(v))
        return;
    int64_t *mkey = lds.mkey, *mbase = lds.mbase;
    uint32_t *mcnt = lds.mcnt;
    for (int i = threadIdx.x; i < kAggMap; i += kBlock) {
        mkey[i] = kAggNone;
        mcnt[i] = 0;
    }
    __syncthreads();
    int64_t o0, r0, r1;
    agg_rows(b, v, o0, r0, r1);
    if (r0 >= r1)
        return;
    int64_t slot[kAggPer];
    const int pt = shared_part(v, r0, r1);
#pragma unroll
    for (int c = 0; c < kAggPer; c += kAggWalk)
        dup_row_slots<K, kAggWalk>(in, v, o0, r0 + threadIdx.x + (int64_t)c * kBlock, r1, pt,
                                   slot + c);
    int e[kAggPer];
    uint32_t rank[kAggPer];
#pragma unroll
    for (int c = 0; c < kAggPer; ++c) {
        e[c] = slot[c] >= 0 ? agg_insert(mkey, slot[c]) : -1;
        rank[c] = e[c] >= 0 ? atomicAdd(&mcnt[e[c]], 1u) : 0u;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kAggMap; i += kBlock) {
        if (mkey[i] != kAggNone)
            mbase[i] = (int64_t)atomicAdd((unsigned long long *)&v.slots[2 * mkey[i] + 1],
                                          (unsigned long long)mcnt[i]);
    }
    __syncthreads();
    int64_t at[kAggPer];
#pragma unroll
    for (int c = 0; c < kAggPer; ++c) {
        at[c] = -1;
        if (slot[c] >= 0)
            at[c] = e[c] >= 0 ? mbase[e[c]] + rank[c]
                              : (int64_t)atomicAdd(
                                    (unsigned long long *)&v.slots[2 * slot[c] + 1], 1ull);
    }
#pragma unroll
    for (int c = 0; c < kAggPer; ++c)
        if (slot[c] >= 0)
            v.grouped[at[c]] = pay_at(in, r0 + threadIdx.x + (int64_t)c * kBlock);
}

template <typename K>
__global__ __launch_bounds__(kBlock) void grp_scatter(Cols in, TView v, int64_t shares)
{
    if (skipped(v.skip))
        return;
    __shared__ AggLds lds;
    for (Blk b = this_block(); b.id < shares; b.id += b.n, __syncthreads())
        grp_scatter_by<K>(b, lds, in, v);
}

// ---- probe -----------------------------------------------------------------

// Block 0 plans the probe tiles; every block clears its share of the
// chained-scan status.
__device__ __forceinline__ void probe_plan_blocks(const Blk &b, const int64_t *offR, int64_t n,
                                                  int P, const ProbeWs &w, int64_t *offsets,
                                                  int64_t *scratch)
{
    if (b.id == 0) {
        sanitize_offsets(offR, w.off, P, n, scratch);
        int64_t carry = 0;
        for (int base = 0; base < P; base += kBlock) {
            const int p = base + threadIdx.x;
            const int64_t nt =
                p < P ? (w.off[p + 1] - w.off[p] + kProbeTile - 1) / kProbeTile : 0;
            int64_t tot;
            const int64_t ex = block_excl_scan(nt, scratch, &tot);
            if (p < P) {
                w.tile_start[p] = carry + ex;
                w.ticket[p] = 0;
            }
            carry += tot;
        }
        if (threadIdx.x == 0) {
            w.tile_start[P] = carry;
            *w.ndefer = 0;
        }
        if (carry == 0)  // no tile will write the output offsets
            for (int p = threadIdx.x; p <= P; p += kBlock)
                offsets[p] = 0;
    }
    const int64_t stride = (int64_t)b.n * kBlock;
    for (int64_t i = (int64_t)b.id * kBlock + threadIdx.x; i < w.max_tiles; i += stride)
        w.status[i] = 0;
}

__global__ __launch_bounds__(kBlock) void probe_plan(const int64_t *__restrict__ offR, int64_t n,
                                                     int P, ProbeWs w, int64_t *offsets)
{
    __shared__ int64_t scratch[kWavesPerBlock];
    probe_plan_blocks(this_block(), offR, n, P, w, offsets, scratch);
}

// Set-up of a merge's global-table join in one block: per-partition build
// and probe offsets taken from the first-pass offsets (every stride-th
// entry), the table's offsets and flags, the probe plan.
__device__ __forceinline__ void fallback_setup_by(const GlobalJoin &g, int64_t *scratch)
{
    const int P = g.w_P;
    for (int p = threadIdx.x; p <= P; p += kBlock) {
        g.offPL[p] = g.offAL[(int64_t)p * g.stride];
        g.offPR[p] = g.offAR[(int64_t)p * g.strideR];
    }
    __syncthreads();
    table_setup_block(g.offPL, g.n_build, g.off_tab, g.v.flags, g.v.bump, P, scratch);
    probe_plan_blocks(Blk{0, 1}, g.offPR, g.n_probe, P, g.w, g.o.offsets, scratch);
}

__global__ __launch_bounds__(kBlock) void fallback_setup(GlobalJoin g)
{
    if (skipped(g.v.skip))
        return;
    __shared__ int64_t scratch[kWavesPerBlock];
    fallback_setup_by(g, scratch);
}

// LDS of probe_chain and probe_expand.
struct ChainLds {
    int64_t tile, excl, total, cw[kProbeRows * kWavesPerBlock];
};

struct ExpandLds {
    int64_t pre[kProbeTile];  // row prefixes of the tile
    int64_t first[kBlock];    // first chunk of every tile of a batch
};


// One wave: the output offsets that tile `tile` of partition p settles, whose
// M output rows start at ex: its partition's and those of empty ones right
// before it when it starts p, those after p when it is the last tile.
__device__ __forceinline__ void tile_offsets(const ProbeWs &w, int P, int p, int64_t tile,
                                             int64_t ex, int64_t M, int lane, int64_t *offsets)
{
    if (tile == w.tile_start[p])
        for (int q = p - lane; q >= 0 && w.tile_start[q] == tile; q -= kWave)
            offsets[q] = ex;
    if (tile + 1 == w.tile_start[P])
        for (int q = p + 1 + lane; q <= P; q += kWave)
            offsets[q] = ex + M;
}

template <typename K>
__device__ __forceinline__ void probe_chain_by(ChainLds &lds, const Cols &in, const TView &v,
                                               int group, const ProbeWs &w, const ProbeOut &o,
                                               int32_t *status)
{
    constexpr int RP = kProbeRows;
    constexpr int kCells = RP * kWavesPerBlock;  // (row step, wave)
    static_assert(kCells <= kWave, "one wave scans the cells");
    static_assert(sizeof(lds.cw) == kCells * 8, "one sum per cell");
    int64_t &s_tile = lds.tile, &s_excl = lds.excl, &s_total = lds.total, *cw = lds.cw;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int64_t t_begin = w.tile_start[v.pb], t_end = w.tile_start[v.pe];
    const int64_t o0 = v.off[v.pb];
    K *out_key = (K *)o.key;

    for (;;) {
        if (tid == 0)
            s_tile = t_begin + (int64_t)atomicAdd(&w.ticket[group], 1u);
        __syncthreads();
        const int64_t tile = s_tile;
        if (tile >= t_end)
            break;
        const int p = upper_index(w.tile_start, v.pb, v.pe, tile);
        const int64_t rbeg = w.off[p] + (tile - w.tile_start[p]) * kProbeTile;
        const int64_t rlim = w.off[p + 1];
        const int64_t rend = rbeg + kProbeTile < rlim ? rbeg + kProbeTile : rlim;
        const bool dup = v.flags[p] != 0;
        int64_t sb, H;
        part_slots(v, o0, p, sb, H);

        K kk[RP];
        int64_t vv[RP];
#pragma unroll
        for (int c = 0; c < RP; ++c) {
            const int64_t r = rbeg + (int64_t)c * kBlock + tid;
            kk[c] = r < rend ? key_at<K>(in, r) : K(0);
        }
#pragma unroll
        for (int c = 0; c < RP; ++c) {
            const int64_t r = rbeg + (int64_t)c * kBlock + tid;
            vv[c] = r < rend ? pay_at(in, r) : 0;
        }
        int64_t slot[RP];
        uint64_t val[RP];
        bool bad = false;
        uint64_t h[RP];
        uint32_t open = 0;
#pragma unroll
        for (int c = 0; c < RP; ++c) {
            const int64_t r = rbeg + (int64_t)c * kBlock + tid;
            h[c] = fmix64(key_bits(kk[c]));
            const bool here = (int)part_of(h[c], v.d) == p;
            if (r < rend && here)
                open |= 1u << c;
            bad |= r < rend && !here;
        }
        find_slots<RP>(
            v.slots, [=](int) { return sb; }, [=](int) { return H; }, h, open, slot, val);
        if (bad)
            or_status(status, MDX_DEV_BAD_PARTITIONING);

        // Matches per (row step, wave) into cw, in row order.  In a
        // repeated-key partition slot[c] becomes the row's rank among its
        // wave's output rows of the step, and val[c] its group's start.
        uint32_t hit = 0;
        if (!dup) {
#pragma unroll
            for (int c = 0; c < RP; ++c) {
                const bool x = slot[c] >= 0;
                hit |= x ? 1u << c : 0u;
                const uint64_t b = ballot(x);
                if (lane == 0)
                    cw[c * kWavesPerBlock + wv] = __popcll(b);
            }
        } else {
#pragma unroll
            for (int c = 0; c < RP; ++c) {
                int64_t m = 0;
                if (slot[c] >= 0) {
                    const int64_t g0 = v.gstart[slot[c]];
                    m = (int64_t)val[c] - g0;
                    val[c] = (uint64_t)g0;
                }
                const int64_t inc = wave_incl_scan(m, lane);
                slot[c] = inc - m;
                if (lane == kWave - 1)
                    cw[c * kWavesPerBlock + wv] = inc;
            }
        }
        __syncthreads();
        if (wv == 0) {  // cw := exclusive prefix; the tile's rows placed
            const int64_t x = lane < kCells ? cw[lane] : 0;
            const int64_t inc = wave_incl_scan(x, lane);
            if (lane < kCells)
                cw[lane] = inc - x;
            const int64_t M = __shfl(inc, kWave - 1, kWave);
            const int64_t ex = lookback(w.status, tile, M, lane, status);
            if (lane == 0) {
                s_excl = ex;
                s_total = M;
            }
            tile_offsets(w, v.pe, p, tile, ex, M, lane, o.offsets);
        }
        __syncthreads();
        const int64_t E = s_excl, M = s_total;
        if (E + M > o.cap) {
            if (tid == 0 && M > 0)
                or_status(status, MDX_DEV_OUTPUT_OVERFLOW);
        } else if (!dup) {
#pragma unroll
            for (int c = 0; c < RP; ++c) {
                const bool x = hit >> c & 1;
                const uint64_t b = ballot(x);
                if (x) {
                    const int64_t at = E + cw[c * kWavesPerBlock + wv] + mbcnt(b);
                    out_key[at] = kk[c];
                    o.lpay[at] = (int64_t)val[c];
                    o.rpay[at] = vv[c];
                }
            }
        } else {
#pragma unroll
            for (int c = 0; c < RP; ++c) {
                const int64_t r = rbeg + (int64_t)c * kBlock + tid;
                if (r < rend) {
                    w.row_pre[r] = cw[c * kWavesPerBlock + wv] + slot[c];
                    w.row_gs[r] = (int64_t)val[c];
                }
            }
            if (tid == 0 && M > 0) {
                const uint32_t d = atomicAdd(w.ndefer, 1u);
                Deferred D;
                D.rbeg = rbeg;
                D.rend = rend;
                D.base = E;
                D.count = M;
                D.group = group;
                w.defer[d] = D;
            }
        }
        __syncthreads();
    }
}

template <typename K>
__global__ __launch_bounds__(kBlock) void probe_chain(Cols in, TView v, int group, ProbeWs w,
                                                      ProbeOut o, int32_t *status)
{
    if (skipped(v.skip))
        return;
    __shared__ ChainLds lds;
    probe_chain_by<K>(lds, in, v, group, w, o, status);
}

template <typename K>
__device__ __forceinline__ void probe_expand_by(const Blk &b, ExpandLds &lds, int64_t *scratch,
                                                const Cols &in, const TView &v, int group,
                                                const ProbeWs &w, const ProbeOut &o)
{
    // The deferred tiles' outputs are cut into chunks, numbered tile by tile;
    // workgroup b takes the chunks b, b + G, ...  The tiles' chunk counts are
    // read kBlock at a time (one after the other, 105 tiles took each
    // workgroup 100 us).
    constexpr int64_t CH = 4096;  // output rows per chunk
    int64_t *pre = lds.pre, *first = lds.first;
    const uint32_t nd = *w.ndefer;
    const int64_t G = b.n;
    K *out_key = (K *)o.key;
    int64_t acc = 0;  // chunks of the tiles before e0
    for (uint32_t e0 = 0; e0 < nd; e0 += kBlock) {
        const uint32_t e = e0 + threadIdx.x;
        int64_t nch = 0, all;
        if (e < nd && w.defer[e].group == group)
            nch = (w.defer[e].count + CH - 1) / CH;
        const int64_t ex = block_excl_scan(nch, scratch, &all);
        __syncthreads();  // `first` is no longer read
        first[threadIdx.x] = acc + ex;
        __syncthreads();
        const int ne = (int)(nd - e0 < (uint32_t)kBlock ? nd - e0 : (uint32_t)kBlock);
        int held = -1;  // the tile whose row prefixes are in pre
        Deferred D = {};
        for (int64_t j = acc + (((int64_t)b.id - acc) % G + G) % G; j < acc + all; j += G) {
            // the last tile that starts at or before j
            const int te = upper_index(first, 0, ne, j);
            if (te != held) {
                __syncthreads();  // pre is no longer read
                D = w.defer[e0 + te];
                const int rows = (int)(D.rend - D.rbeg);
                for (int i = threadIdx.x; i < rows; i += kBlock)
                    pre[i] = w.row_pre[D.rbeg + i];
                __syncthreads();
                held = te;
            }
            const int rows = (int)(D.rend - D.rbeg);
            const int64_t q0 = (j - first[te]) * CH;
            const int64_t lim = q0 + CH < D.count ? q0 + CH : D.count;
            for (int64_t q = q0 + threadIdx.x; q < lim; q += kBlock) {
                int l = 0, h = rows - 1;  // last row whose prefix <= q
                while (l < h) {
                    const int mid = (l + h + 1) >> 1;
                    if (pre[mid] <= q)
                        l = mid;
                    else
                        h = mid - 1;
                }
                const int64_t r = D.rbeg + l;
                const int64_t at = D.base + q;
                out_key[at] = key_at<K>(in, r);
                o.lpay[at] = v.grouped[w.row_gs[r] + (q - pre[l])];
                o.rpay[at] = pay_at(in, r);
            }
        }
        acc += all;
    }
}

template <typename K>
__global__ __launch_bounds__(kBlock) void probe_expand(Cols in, TView v, int group, ProbeWs w,
                                                       ProbeOut o)
{
    if (skipped(v.skip))
        return;
    __shared__ ExpandLds lds;
    __shared__ int64_t scratch[kWavesPerBlock];
    probe_expand_by<K>(this_block(), lds, scratch, in, v, group, w, o);
}

// ---- the whole global-table join in one launch --------------------------------
// A merge launches its global-table join always and almost never needs it:
// ten launches that return at once cost it 20 to 25 us of 62 (1E5 x 1E5) to 88
// (1E6 x 1E6).  Up to kOneLaunchRows, and where the probe rows are partitioned
// again (ProbePart, up to 3.2E6 rows: those steps are here alone), they are one
// launch: a step's workgroups are items, handed out in order by a ticket
// counter, and an item of a step first waits until every item of the steps
// before it is done (they were all handed out before, to running workgroups, so
// the wait ends).  Merges that do need the join then take up to 1.6 times as
// long (1E6 x 1E5 with hot build keys: 260 us with ten launches, 392 with one;
// 4E6 x 4E5: 565 and 846): every item writes its L2 back.
enum JoinStep {
    kPartHist,
    kPartScan,
    kPartOffsets,
    kPartScatter,
    kSetup,
    kInit,
    kSample,
    kInsert,
    kReset,
    kCount,
    kAlloc,
    kScatter,
    kProbe,
    kExpand,
    kJoinSteps
};

struct JoinSteps {
    uint32_t first[kJoinSteps + 1];  // first item of every step
    // ticket, items done, items done at the end of the last finished step
    // (zero before the launch; kSyncStride apart)
    uint32_t *sync;
    // workgroups' shares of the rows (kCount, kScatter) and slots (kAlloc)
    int64_t shares_rows, shares_slots;
};

template <typename K>
__global__ __launch_bounds__(kBlock, 4) void global_join(GlobalJoin g, Cols build, Cols probe,
                                                         int shift, PartTable<K> pt, Dest pd,
                                                         JoinSteps t)
{
    if (skipped(g.v.skip))
        return;
    __shared__ union {
        AggLds agg;
        ChainLds chain;
        ExpandLds expand;
        uint32_t hist[kProbePartMax];
        alignas(16) unsigned char tile[scatter_lds(kBlock * kProbePartRows, kProbePartMax,
                                                   (int)sizeof(K), false)
                                           .total];
    } lds;
    __shared__ int64_t scratch[kWavesPerBlock];
    __shared__ int64_t s_base;
    __shared__ uint32_t s_item;
    __shared__ int s_ok;
    int ready = 0;  // the steps before this one are done
    for (;;) {
        if (threadIdx.x == 0)
            s_item = atomicAdd(t.sync, 1u);
        __syncthreads();
        const uint32_t item = s_item;
        if (item >= t.first[kJoinSteps])
            return;
        int step = 0;
        while (item >= t.first[step + 1])
            ++step;
        if (step > ready) {
            if (threadIdx.x == 0) {
                s_ok = 1;
                int64_t polls = 0;
                // (not the count itself: reads of it would slow its additions)
                while (__hip_atomic_load(t.sync + 2 * kSyncStride, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT) < t.first[step]) {
                    __builtin_amdgcn_s_sleep(8);
                    if (++polls > kSpinLimit) {
                        or_status(g.status, MDX_DEV_SCAN_TIMEOUT);
                        s_ok = 0;
                        break;
                    }
                }
            }
            // what the steps before wrote is read afresh
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            __syncthreads();
            if (!s_ok)
                return;
            ready = step;
        }
        const Blk b = {(int64_t)(item - t.first[step]),
                       (int64_t)(t.first[step + 1] - t.first[step])};
        switch (step) {
        case kPartHist:
            for (int64_t k = b.id; k < pt.ntiles; k += b.n, __syncthreads())
                hist_tile<K, kProbePartRows, false>(pt, k, pd, lds.hist);
            break;
        case kPartScan: {
            const int lane = threadIdx.x & (kWave - 1);
            for (int64_t d = b.id * kWavesPerBlock + threadIdx.x / kWave; d < pd.ndest;
                 d += b.n * kWavesPerBlock) {
                const int64_t total = wave_scan_row(pt.cnt + d * pt.ntiles, pt.ntiles, lane);
                if (lane == 0)
                    pt.totals[d] = total;
            }
            break;
        }
        case kPartOffsets: offsets_of(pt.totals, pt.off, pd.ndest, scratch); break;
        case kPartScatter:
            for (int64_t k = b.id; k < pt.ntiles; k += b.n, __syncthreads())
                part_scatter_tile<K, kProbePartRows, true, false>(pt, k, pd, 0, 0, lds.tile);
            break;
        case kSetup: fallback_setup_by(g, scratch); break;
        case kInit: tbl_init_by(b, g.v); break;
        case kSample: tbl_insert_by<K>(b, build, g.v, shift, true, g.status); break;
        case kInsert: tbl_insert_by<K>(b, build, g.v, shift, false, g.status); break;
        case kReset: grp_reset_by(b, g.v); break;
        case kCount:
            for (Blk k = b; k.id < t.shares_rows; k.id += b.n, __syncthreads())
                grp_count_by<K>(k, lds.agg, build, g.v);
            break;
        case kAlloc:
            for (Blk k = b; k.id < t.shares_slots; k.id += b.n, __syncthreads())
                grp_alloc_by(k, scratch, s_base, g.v);
            break;
        case kScatter:
            for (Blk k = b; k.id < t.shares_rows; k.id += b.n, __syncthreads())
                grp_scatter_by<K>(k, lds.agg, build, g.v);
            break;
        case kProbe: probe_chain_by<K>(lds.chain, probe, g.v, 0, g.w, g.o, g.status); break;
        default: probe_expand_by<K>(b, lds.expand, scratch, probe, g.v, 0, g.w, g.o); break;
        }
        // every wave's writes have reached the L2, then they are written
        // back, before the item counts as done
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (threadIdx.x == 0) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            if (atomicAdd(t.sync + kSyncStride, 1u) + 1 == t.first[step + 1]) {
                // the last item of the step passes on what it has seen of the
                // others: those who wait read only the word that it stores
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
                __hip_atomic_store(t.sync + 2 * kSyncStride, t.first[step + 1], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

// ---- count-only join --------------------------------------------------------------
// The table of the build side holds, per distinct hash, the number of build
// rows with that hash (slot value; tbl_init sets it to 0).  Both sides'
// rows are first counted per workgroup in an LDS map of hashes, so a key
// repeated millions of times costs one global update per workgroup; rows
// the map cannot take go to the table one by one.
//
// A workgroup's share of the rows: kCountWgRows, halved for smaller sides
// until kCountFill workgroups run.  5E7 x 5E7 Zipf(1.1) keys (P = 16): the
// table's updates, one per distinct hash and share, go at the rate of the
// device's atomics on random lines, which more aggregation lowers (a share
// holds 22% distinct hashes, one four times as large 16%) and fewer waves in
// flight do not reach: 40 KB of LDS and 512 threads keep a CU's 32 waves
// in cnt_insert (in cnt_probe, with its sums per partition, 24),
// 2.75 ms a count with its partitions; 32-bit counts (24 waves) 2.81; 256
// threads 3.20, 1024 2.90; 8192 entries for 32768 rows 3.48, 2048 for 8192
// 2.99.  Four entries' slots walked at once by each thread were slower (3.03).
// (Figures from before count_rows left out the search per row: 2.50 now.)
// 2E5 x 1E5 keys: 197 us with shares of 16384 rows (13 workgroups), 72 with
// 1024; 3E6 x 2E6 int32: 309 and 189.
constexpr int kCountBlock = 512;
constexpr int kCountRows = 4;  // rows per thread loaded together
constexpr int kCountMapBits = 12;
constexpr int kCountMap = 1 << kCountMapBits;  // LDS map entries
constexpr int kCountWgRows = 16384;            // a share
static_assert(kCountWgRows <= 0xffff, "a share's counts fit the map's 16 bits");
constexpr int kCountMinRows = 1024;
constexpr int kCountFill = 384;

// The LDS map of a workgroup: hashes and their rows in the share (two
// 16-bit counts per word).
struct CountMap {
    uint64_t key[kCountMap];
    uint32_t cnt[kCountMap / 2];
    __device__ __forceinline__ void clear()
    {
        for (int i = threadIdx.x; i < kCountMap; i += kCountBlock) {
            key[i] = ~0ull;
            if (i < kCountMap / 2)
                cnt[i] = 0;
        }
    }
    __device__ __forceinline__ void add(int e)
    {
        atomicAdd(&cnt[e >> 1], 1u << 16 * (e & 1));
    }
    // fn(hash, rows) for every entry.  Each workgroup starts elsewhere, so
    // that those of one partition do not come to a hot hash's slot together.
    template <typename Fn>
    __device__ __forceinline__ void each(Fn fn) const
    {
        const int turn = (int)((blockIdx.x * 0x9E3779B1u) >> (32 - kCountMapBits));
        for (int i = threadIdx.x; i < kCountMap; i += kCountBlock) {
            const int e = i ^ turn;
            if (key[e] != ~0ull)
                fn(key[e], cnt[e >> 1] >> 16 * (e & 1) & 0xffffu);
        }
    }
};

// Entry of hash h in the LDS map (inserted if there is room within
// kAggProbe probes), or -1.  ~0 marks an empty entry, so a row whose hash is
// ~0 is never mapped.
__device__ __forceinline__ int hmap_insert(uint64_t *mkey, uint64_t h)
{
    if (h == ~0ull)
        return -1;
    // the top bits, as a slot's home in the table: the map's order is nearly the
    // slots' order (the partition takes the low bits)
    uint32_t i = (uint32_t)(h >> 32) >> (32 - kCountMapBits);
    for (int k = 0; k < kAggProbe; ++k) {
        uint64_t cur = mkey[i];
        if (cur == ~0ull) {
            cur = atomicCAS((unsigned long long *)&mkey[i], ~0ull, (unsigned long long)h);
            if (cur == ~0ull)
                return (int)i;
        }
        if (cur == h)
            return (int)i;
        i = (i + 1) & (kCountMap - 1);
    }
    return -1;
}

// value[slot of h] += c in partition p, claiming the slot if h is new.  The
// half holds at most n_p distinct hashes in its H = n_p + 8 slots.
__device__ __forceinline__ void slot_add(const TView &v, int64_t o0, int p, uint64_t h,
                                         uint64_t c)
{
    int64_t sb, H;
    part_slots(v, o0, p, sb, H);
    const uint64_t t = h >> 63;
    const uint64_t empty = empty_of_half(t);
    const int64_t base = sb + (int64_t)t * H;
    uint64_t i = __umul64hi(h << 1, (uint64_t)H);
    for (int64_t k = 0; k < H; ++k) {
        uint64_t *sp = v.slots + 2 * (base + (int64_t)i);
        uint64_t w = __hip_atomic_load(sp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (w == empty) {
            uint64_t expect = empty;
            if (__hip_atomic_compare_exchange_strong(sp, &expect, h, __ATOMIC_RELAXED,
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                atomicAdd((unsigned long long *)(sp + 1), (unsigned long long)c);
                return;
            }
            w = expect;
        }
        if (w == h) {
            atomicAdd((unsigned long long *)(sp + 1), (unsigned long long)c);
            return;
        }
        if (++i == (uint64_t)H)
            i = 0;
    }
}

// Rows [r0, r1) of the workgroup's share, kCountRows per thread loaded
// together; fn(hash, partition) for every row in its partition, the others
// reported.
template <typename K, typename Fn>
__device__ __forceinline__ void count_rows(const K *__restrict__ keys, const int64_t *off, int P,
                                           const Dest &d, int64_t r0, int64_t r1, int32_t *status,
                                           Fn fn)
{
    if (r0 >= r1)
        return;
    // the share mostly lies in one partition: no search per row then (2.50 ms
    // for the 5E7 x 5E7 rows above, with it 2.75)
    const int p0 = upper_index(off, 0, P, r0);
    const bool one = p0 + 1 == P || r1 <= off[p0 + 1];
    bool bad = false;
    for (int64_t b = r0; b < r1; b += (int64_t)kCountRows * kCountBlock) {
        K k[kCountRows];
#pragma unroll
        for (int j = 0; j < kCountRows; ++j) {
            const int64_t r = b + (int64_t)j * kCountBlock + threadIdx.x;
            k[j] = r < r1 ? __builtin_nontemporal_load(keys + r) : K(0);
        }
#pragma unroll
        for (int j = 0; j < kCountRows; ++j) {
            const int64_t r = b + (int64_t)j * kCountBlock + threadIdx.x;
            if (r < r1) {
                const uint64_t h = fmix64(key_bits(k[j]));
                const int p = one ? p0 : upper_index(off, 0, P, r);
                if ((int)part_of(h, d) != p)
                    bad = true;
                else
                    fn(h, p);
            }
        }
    }
    if (bad)
        or_status(status, MDX_DEV_BAD_PARTITIONING);
}

// Block: the sanitized build offsets into the table, the sanitized probe
// offsets, per-partition counts cleared.
__global__ __launch_bounds__(kBlock) void cnt_setup(const int64_t *__restrict__ lofs,
                                                    int64_t n_build,
                                                    const int64_t *__restrict__ rofs,
                                                    int64_t n_probe, int64_t *off_tab,
                                                    int64_t *off_probe, uint64_t *pcount, int P)
{
    __shared__ int64_t scratch[kWavesPerBlock];
    sanitize_offsets(lofs, off_tab, P, n_build, scratch);
    sanitize_offsets(rofs, off_probe, P, n_probe, scratch);
    for (int p = threadIdx.x; p < P; p += kBlock)
        pcount[p] = 0;
}

template <typename K>
__global__ __launch_bounds__(kCountBlock) void cnt_insert(const K *__restrict__ keys, TView v,
                                                          int share, int32_t *status)
{
    __shared__ CountMap map;
    map.clear();
    __syncthreads();
    const int64_t o0 = v.off[0], o1 = v.off[v.pe];
    const int64_t r0 = o0 + (int64_t)blockIdx.x * share;
    const int64_t r1 = r0 + share < o1 ? r0 + share : o1;
    count_rows(keys, v.off, v.pe, v.d, r0, r1, status, [&](uint64_t h, int p) {
        const int e = hmap_insert(map.key, h);
        if (e >= 0)
            map.add(e);
        else
            slot_add(v, o0, p, h, 1);
    });
    __syncthreads();
    map.each([&](uint64_t h, uint64_t c) { slot_add(v, o0, (int)part_of(h, v.d), h, c); });
}

// Build rows of hash h in partition p (0 when absent).
__device__ __forceinline__ uint64_t slot_count(const TView &v, int64_t o0, int p, uint64_t h)
{
    int64_t sb, H;
    part_slots(v, o0, p, sb, H);
    const int64_t s = find_slot(v.slots, sb, H, h);
    return s >= 0 ? v.slots[2 * s + 1] : 0;
}

template <typename K>
__global__ __launch_bounds__(kCountBlock) void cnt_probe(const K *__restrict__ keys,
                                                    const int64_t *__restrict__ off_probe,
                                                    TView v, uint64_t *pcount, int share,
                                                    int32_t *status)
{
    extern __shared__ unsigned long long psum[];  // [P]
    __shared__ CountMap map;
    const int P = v.pe;
    map.clear();
    for (int p = threadIdx.x; p < P; p += kCountBlock)
        psum[p] = 0;
    __syncthreads();
    const int64_t o0 = v.off[0];
    const int64_t n = off_probe[P];
    const int64_t r0 = off_probe[0] + (int64_t)blockIdx.x * share;
    const int64_t r1 = r0 + share < n ? r0 + share : n;
    count_rows(keys, off_probe, P, v.d, r0, r1, status, [&](uint64_t h, int p) {
        const int e = hmap_insert(map.key, h);
        if (e >= 0) {
            map.add(e);
        } else {
            const uint64_t c = slot_count(v, o0, p, h);
            if (c)
                atomicAdd(&psum[p], (unsigned long long)c);
        }
    });
    __syncthreads();
    map.each([&](uint64_t h, uint64_t rows) {
        const int p = (int)part_of(h, v.d);
        const uint64_t c = slot_count(v, o0, p, h);
        if (c)
            atomicAdd(&psum[p], (unsigned long long)(c * rows));
    });
    __syncthreads();
    for (int p = threadIdx.x; p < P; p += kCountBlock)
        if (psum[p])
            atomicAdd((unsigned long long *)&pcount[p], psum[p]);
}

// Block: out_offsets = exclusive prefix of the per-partition counts.
__global__ __launch_bounds__(kBlock) void cnt_finalize(const uint64_t *__restrict__ pcount, int P,
                                                       int64_t *out_offsets)
{
    __shared__ int64_t scratch[kWavesPerBlock];
    int64_t carry = 0;
    for (int base = 0; base < P; base += kBlock) {
        const int p = base + threadIdx.x;
        const int64_t c = p < P ? (int64_t)pcount[p] : 0;
        int64_t tot;
        const int64_t ex = block_excl_scan(c, scratch, &tot);
        if (p < P)
            out_offsets[p] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0)
        out_offsets[P] = carry;
}

// Rows of a build's sample, every 2^shift-th; -1: no sample (few workgroups
// insert the rows at all).
constexpr int64_t kSampleRows = 32768;
constexpr int kSampleBlocks = kSampleRows / kBlock;

static int sample_shift(int64_t rows)
{
    int shift = 0;
    while (rows >> shift > kSampleRows)
        ++shift;
    return rows <= 4 * kSampleRows ? -1 : shift;
}

// Rows per workgroup of a count's kernel over `rows` rows.
static int count_share(int64_t rows)
{
    int share = kCountWgRows;
    while (share > kCountMinRows && rows < (int64_t)share * kCountFill)
        share /= 2;
    return share;
}

// G: the most workgroups of a kernel.
template <typename K>
hipError_t run_build(const Cols &in, const TView &v, int64_t rows, int32_t *status, int G,
                     hipStream_t s)
{
    // the grouping kernels take fixed shares of the rows and of the slots
    const int64_t P = v.pe - v.pb;
    const int64_t rshares = std::max<int64_t>(1, (rows + kAggRows - 1) / kAggRows);
    const int64_t sshares =
        std::max<int64_t>(1, (2 * rows + 16 * P + kAllocSlots - 1) / kAllocSlots);
    const unsigned Gr = (unsigned)std::min<int64_t>(rshares, G);
    const unsigned Gs = (unsigned)std::min<int64_t>(sshares, G);
    const int shift = sample_shift(rows);
    trace_begin("tbl_init", s);
    hipLaunchKernelGGL(tbl_init, dim3(G), dim3(kBlock), 0, s, v);
    trace_end("tbl_init", s);
    trace_begin("tbl_insert", s);
    if (shift >= 0)
        hipLaunchKernelGGL((tbl_insert<K>), dim3(kSampleBlocks), dim3(kBlock), 0, s, in, v, shift,
                           true, status);
    hipLaunchKernelGGL((tbl_insert<K>), dim3(G), dim3(kBlock), 0, s, in, v, shift, false, status);
    trace_end("tbl_insert", s);
    hipLaunchKernelGGL(grp_reset, dim3(G), dim3(kBlock), 0, s, v);
    trace_begin("grp_count", s);
    hipLaunchKernelGGL((grp_count<K>), dim3(Gr), dim3(kBlock), 0, s, in, v, rshares);
    trace_end("grp_count", s);
    trace_begin("grp_alloc", s);
    hipLaunchKernelGGL(grp_alloc, dim3(Gs), dim3(kBlock), 0, s, v, sshares);
    trace_end("grp_alloc", s);
    trace_begin("grp_scatter", s);
    hipLaunchKernelGGL((grp_scatter<K>), dim3(Gr), dim3(kBlock), 0, s, in, v, rshares);
    trace_end("grp_scatter", s);
    return hipGetLastError();
}

template <typename K>
hipError_t run_probe_group(const Cols &in, const TView &v, int group,
                           const ProbeWs &w, const ProbeOut &o, int32_t *status, int G,
                           hipStream_t s)
{
    trace_begin("probe_chain", s);
    hipLaunchKernelGGL((probe_chain<K>), dim3(G), dim3(kBlock), 0, s, in, v, group, w, o,
                       status);
    trace_end("probe_chain", s);
    // The expansion's work is the output rows, which can be millions for one
    // probe row: it always gets a full device (it returns at once when no
    // tile deferred rows).
    trace_begin("probe_expand", s);
    hipLaunchKernelGGL((probe_expand<K>), dim3(device_fill_blocks()), dim3(kBlock), 0, s, in, v,
                       group, w, o);
    trace_end("probe_expand", s);
    return hipGetLastError();
}

template <typename K>
hipError_t run_count(const K *lk, const int64_t *lofs, int64_t n_build, const K *rk,
                     const int64_t *rofs, int64_t n_probe, const TView &v, int64_t *off_probe,
                     uint64_t *pcount, int64_t *out_offsets, int32_t *status, hipStream_t s)
{
    const int P = v.pe;
    const int bs = count_share(n_build), ps = count_share(n_probe);
    hipLaunchKernelGGL(cnt_setup, dim3(1), dim3(kBlock), 0, s, lofs, n_build, rofs, n_probe,
                       (int64_t *)v.off, off_probe, pcount, P);
    trace_begin("tbl_init", s);
    hipLaunchKernelGGL(tbl_init, dim3(device_fill_blocks()), dim3(kBlock), 0, s, v);
    trace_end("tbl_init", s);
    if (n_build > 0) {
        trace_begin("cnt_insert", s);
        hipLaunchKernelGGL((cnt_insert<K>),
                           dim3((unsigned)((n_build + bs - 1) / bs)),
                           dim3(kCountBlock), 0, s, lk, v, bs, status);
        trace_end("cnt_insert", s);
    }
    if (n_probe > 0) {
        trace_begin("cnt_probe", s);
        hipLaunchKernelGGL((cnt_probe<K>),
                           dim3((unsigned)((n_probe + ps - 1) / ps)),
                           dim3(kCountBlock), (size_t)P * 8, s, rk, off_probe, v, pcount, ps,
                           status);
        trace_end("cnt_probe", s);
    }
    hipLaunchKernelGGL(cnt_finalize, dim3(1), dim3(kBlock), 0, s, pcount, P, out_offsets);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_join_count(const void *lk, const int64_t *lofs, int64_t n_build, const void *rk,
                             const int64_t *rofs, int64_t n_probe, int key_bytes, const TView &v,
                             int64_t *off_probe, uint64_t *pcount, int64_t *out_offsets,
                             int32_t *status, hipStream_t s)
{
    if (key_bytes == 8)
        return run_count<int64_t>((const int64_t *)lk, lofs, n_build, (const int64_t *)rk, rofs,
                                  n_probe, v, off_probe, pcount, out_offsets, status, s);
    return run_count<int32_t>((const int32_t *)lk, lofs, n_build, (const int32_t *)rk, rofs,
                              n_probe, v, off_probe, pcount, out_offsets, status, s);
}

hipError_t launch_table_setup(const int64_t *off_in, int64_t n, int64_t *off_tab, int32_t *flags,
                              int64_t *bump, int32_t P, hipStream_t s)
{
    hipLaunchKernelGGL(table_setup, dim3(1), dim3(kBlock), 0, s, off_in, n, off_tab, flags, bump,
                       P);
    return hipGetLastError();
}

hipError_t launch_build(const Cols &table, int key_bytes, const TView &v, int64_t rows,
                        int32_t *status, hipStream_t s)
{
    if (key_bytes == 8)
        return run_build<int64_t>(table, v, rows, status, device_fill_blocks(), s);
    return run_build<int32_t>(table, v, rows, status, device_fill_blocks(), s);
}

template <typename K>
hipError_t run_global_join(const Cols &build, const Cols &probe, const GlobalJoin &g,
                           const ProbePart &pp, bool one, uint32_t *sync, hipStream_t s)
{
    // workgroups of 2048 rows (16384 left most of the device idle at 4E6
    // rows: 725 against 567 us), at most four per CU, which fill it: merges that
    // do not need the join pay for every workgroup that starts and returns
    // (5E6 x 5E6 int32: 250 us a merge with eight, 247 with four, 246 with two;
    // hot keys, 4E6 x 4E5: 547, 539, 559; 2.5E6 x 2.5E6: 574, 547, 588)
    const int full = std::max(1, device_fill_blocks() / 2);
    auto blocks = [&](int64_t rows) { return (int)std::min<int64_t>((rows >> 11) + 1, full); };
    if (!one) {
        hipLaunchKernelGGL(fallback_setup, dim3(1), dim3(kBlock), 0, s, g);
        hipError_t e = run_build<K>(build, g.v, g.n_build, g.status, blocks(g.n_build), s);
        if (e != hipSuccess)
            return e;
        return run_probe_group<K>(probe, g.v, 0, g.w, g.o, g.status, blocks(g.n_probe), s);
    }
    // All steps in one launch on at most kMost workgroups.  The ticket and the
    // count of done items are one address each, so more workgroups make every
    // step's end longer (1E6 rows: 506 us with 512 of them, 406 with 256, 445
    // with 128).
    constexpr int64_t kMost = 256;
    auto cap = [&](int64_t items) { return std::min(items, kMost); };
    PartTable<K> pt = {};
    if (pp.off) {
        const PartLayout L = part_layout(pp.n, pp.d.ndest, kProbePartRows);
        pt.keys = (const K *)pp.keys;
        pt.pay = pp.pay;
        pt.n = pp.n;
        pt.ntiles = L.ntiles;
        pt.rows_out = make_rows<K>(pp.rows_out, pp.n);
        pt.off = pp.off;
        pt.cnt = (int64_t *)((char *)pp.ws + L.cnt_off);
        pt.totals = (int64_t *)((char *)pp.ws + L.totals_off);
    }
    const int shift = sample_shift(g.n_build);
    const int64_t slots = 2 * g.n_build + 16 * (int64_t)g.w_P;
    JoinSteps t;
    t.sync = sync;
    t.shares_rows = std::max<int64_t>(1, (g.n_build + kAggRows - 1) / kAggRows);
    t.shares_slots = std::max<int64_t>(1, (slots + kAllocSlots - 1) / kAllocSlots);
    const int64_t again = pp.off ? 1 : 0;
    // (the expansion's work is the output rows, which can be many for few probe
    // rows)
    const int64_t n[kJoinSteps] = {cap(pt.ntiles),
                                   again * ((pp.d.ndest + kWavesPerBlock - 1) / kWavesPerBlock),
                                   again,
                                   cap(pt.ntiles),
                                   1,
                                   cap(blocks(slots)),
                                   shift >= 0 ? kSampleBlocks : 0,
                                   cap(blocks(g.n_build)),
                                   cap(blocks(slots)),
                                   cap(t.shares_rows),
                                   cap(t.shares_slots),
                                   cap(t.shares_rows),
                                   cap(blocks(g.n_probe)),
                                   kMost};
    t.first[0] = 0;
    for (int i = 0; i < kJoinSteps; ++i)
        t.first[i + 1] = t.first[i] + (uint32_t)n[i];
    const int64_t G = cap(std::max(blocks(g.n_build), blocks(g.n_probe)));
    trace_begin("global_join", s);
    hipLaunchKernelGGL((global_join<K>), dim3((unsigned)G), dim3(kBlock), 0, s, g, build, probe,
                       shift, pt, pp.d, t);
    trace_end("global_join", s);
    return hipGetLastError();
}

hipError_t launch_global_join(const Cols &build, const Cols &probe, int key_bytes,
                              const GlobalJoin &g, const ProbePart &pp, bool one, uint32_t *sync,
                              hipStream_t s)
{
    if (pp.off && (!one || pp.d.ndest > kProbePartMax))
        return hipErrorInvalidValue;
    return key_bytes == 8 ? run_global_join<int64_t>(build, probe, g, pp, one, sync, s)
                          : run_global_join<int32_t>(build, probe, g, pp, one, sync, s);
}

hipError_t launch_probe_plan(const int64_t *offR, int64_t n, int32_t P, const ProbeWs &w,
                             int64_t *offsets, hipStream_t s)
{
    const int G = device_fill_blocks() / 4 > 0 ? device_fill_blocks() / 4 : 1;
    hipLaunchKernelGGL(probe_plan, dim3(G), dim3(kBlock), 0, s, offR, n, P, w, offsets);
    return hipGetLastError();
}

hipError_t launch_probe_group(const Cols &table, int key_bytes, const TView &v, int group,
                              const ProbeWs &w, const ProbeOut &o, int32_t *status, hipStream_t s)
{
    // A workgroup for every tile, at most a full device: one without a tile only
    // takes a ticket, and those of a full device, made one after the other at one
    // address, set the time of a small probe (build and probe of 1E4 x 3333 rows
    // 70 us, so 53).
    const int G = (int)std::min<int64_t>(device_fill_blocks(), w.max_tiles);
    if (key_bytes == 8)
        return run_probe_group<int64_t>(table, v, group, w, o, status, G, s);
    return run_probe_group<int32_t>(table, v, group, w, o, status, G, s);
}

}  // namespace mdx
