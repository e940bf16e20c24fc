// Radix join: the per-partition inner join (arXiv 2101.08878, Section V-B
// "cuDF Merge": every worker merges the frames it received) with every table
// held in LDS.
//
// Both sides arrive split into sub-buckets (partition p, top hash bits q), so
// that a sub-bucket's build rows fit one workgroup's LDS.  A workgroup takes
// sub-buckets in order from a ticket counter; for each it
//   1. loads the build rows into LDS: key, payload, and a chain link; bucket
//      heads hold the last row inserted per bucket (LDS atomic exchange), so
//      equal keys share a chain and repeated keys need nothing special;
//   2. counts the output rows of all its probe rows (walking each row's
//      chain) and takes the output row of its first one (output placement,
//      below);
//   3. writes (key, left payload, right payload) rows; the probe rows stay
//      in registers between 2 and 3.  A merge's sub-bucket with more probe
//      rows than one batch (4096: a probe key repeated very often) is taken
//      one batch per workgroup, each building the table again.  (One
//      workgroup for all of a sub-bucket's batches, reading them once to
//      count and once to write, took 16.3 ms of a 1E7 x 5E7 merge whose
//      probe keys are Zipf(1.1).)  The fused batch joins such a sub-bucket in
//      one workgroup.
// Sub-buckets are numbered partition-major, and partition p's output is the
// contiguous range [out_off[p], out_off[p+1]).  Global memory is only
// streamed: the random accesses of the join all hit LDS.  The partition
// already sent each key to its sub-bucket by fmix64, so inside a sub-bucket a
// key's chain is chosen by a one-multiply hash of the key itself and keys are
// compared directly: fmix64 (six 32-bit multiplies, quarter-rate
// instructions) is not computed again here.
//
// Latency hiding: two workgroups per CU, one running while the other waits
// on the dependent steps of its sub-bucket; inside a sub-bucket the loads
// are issued in the order they are needed (count_one_batch), and the hash
// chains of a thread's probe rows are walked two (the fused batch: four) at a
// time without branches, so that their LDS reads are in flight together.
#include <algorithm>

#include "mdx.h"
#include "mdx_internal.hpp"

namespace mdx {
namespace {

constexpr int kJoinWaves = kJoinThreads / kWave;
constexpr int kCells = kJoinRows * kJoinWaves;  // (row step, wave) partial sums
constexpr int kCellsPerLane = kCells / kWave;
static_assert(kCells % kWave == 0, "one wave scans the partial sums");

// A table of geometry G (G::cap build rows, G::heads chain heads).  Chains
// end at the sentinel row `sent` (one slot past the table), whose link
// points to itself.
template <class G>
struct Tab {
    static constexpr uint32_t sent = G::cap;
    static constexpr int log_heads = __builtin_ctz(G::heads);
    // build rows per thread, loaded together: what a full table takes (a
    // merge's 3456 rows: 7; with 8, one load and insert more per item, 3E7 x
    // 3E7 int32 rows took 1209 us, so 1198)
    static constexpr int build_rows = (G::cap + kJoinThreads - 1) / kJoinThreads;
    static_assert(G::cap <= 0xffff, "chain links are 16-bit");
    static_assert((G::heads & (G::heads - 1)) == 0, "power-of-two heads");
    static_assert(kJoinRows % G::walk == 0, "walk groups tile the thread's rows");
};

// Chain of a key inside its sub-bucket: multiplicative (Fibonacci) hashing
// of the key's two 32-bit halves folded together.
template <class G>
__device__ __forceinline__ uint32_t bucket_of(int64_t key)
{
    const uint32_t x = (uint32_t)key ^ (uint32_t)((uint64_t)key >> 32);
    return (x * 0x9E3779B1u) >> (32 - Tab<G>::log_heads);
}

// Values every lane of the workgroup holds alike, in scalar registers.
__device__ __forceinline__ int64_t uniform(int64_t x)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)x >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// ---- output placement ------------------------------------------------------
// Partition p's output rows form one range, [base(p), base(p+1)); the order
// of its sub-buckets' rows inside that range is free (row order inside a
// partition is implementation-defined).  Two ways to place them:
//  - by sub-bucket: a chained scan over all items in ticket order (pst[t]
//    the status of item t).  An item waits until every item ticketed before
//    it has been counted.
//  - by partition: an item takes its rows from its partition's cursor with
//    one atomic add (the low kDoneBits count the items counted, the bits
//    above the rows taken), and base(p) is the exclusive prefix of the
//    partition totals, a chained scan over the P entries of pst: the last
//    item of p to be counted publishes p's total.  An item then waits only
//    while an earlier partition still has items being counted.  The items of
//    earlier partitions were all ticketed before this one, to running
//    workgroups, so the wait ends.
// By partition pays when partitions hold many more sub-buckets than there
// are workgroups: then few sub-buckets wait at all (1E8 x 1E8 at P = 1:
// 13.7 instead of 18.4 us per sub-bucket and workgroup).  With partitions
// of ~2 workgroups' worth (P = 32), half the sub-buckets in flight wait for
// the partition before and are all released at once when it completes, and
// their output writes then contend (21 us per sub-bucket): by sub-bucket.
struct Place {
    uint64_t *cursor;        // by partition: [P] rows taken << kDoneBits | items counted
    uint64_t *pst;           // [P] or [items]: chained-scan status
    const uint32_t *istart;  // [S + 1] first item of every sub-bucket; null: item = sub-bucket
    int64_t nitems;
    int64_t *offsets;        // [P + 1] output offsets (written here unless by partition)
    int32_t qbits;           // 2^qbits sub-buckets per partition
    int32_t by_part;         // 1: by partition, 0: by sub-bucket
};
// A merge has at most 2^20 sub-buckets and 2^22 further probe batches, so the
// count of a partition's items never carries into its rows; the rows taken
// are kept modulo 2^41 (a carry out of them is lost), and a partition
// reaching 2^41 output rows (far beyond any output buffer) is reported as an
// output overflow.
constexpr int kDoneBits = 23;
static_assert((int64_t)MDX_MAX_P * kSegMaxDest + MDX_MAX_ROWS / kJoinBatch < 1ll << kDoneBits,
              "a partition's items fit their count");
constexpr uint64_t kDoneMask = (1ull << kDoneBits) - 1;
constexpr uint64_t kRowsLimit = 1ull << (64 - kDoneBits);

// Wave 0 of a workgroup: the output row of the first row of item t, a batch
// of sub-bucket s (its first one: `first`), for its `total` rows.  By
// sub-bucket, the item that starts a partition writes the partition's output
// offset, and the last one the total.  (cp, cb): the workgroup's last
// partition and that partition's base, kept across items (cp = -1: none yet).
__device__ inline int64_t place_rows(const Place &pl, int64_t t, int64_t s, bool first,
                                     int64_t total, int &cp, int64_t &cb, int lane,
                                     int32_t *status)
{
    const int p = (int)(s >> pl.qbits);
    if (!pl.by_part) {
        const int64_t ex = lookback(pl.pst, t, total, lane, status);
        if (lane == 0) {
            if (first && s == (int64_t)p << pl.qbits)
                pl.offsets[p] = ex;
            if (t == pl.nitems - 1)
                pl.offsets[p + 1] = ex + total;
        }
        return ex;
    }
    uint64_t old = 0;
    if (lane == 0)
        old = atomicAdd((unsigned long long *)(pl.cursor + p), ((uint64_t)total << kDoneBits) + 1);
    old = __shfl(old, 0, kWave);
    const uint64_t before = old >> kDoneBits;  // rows of p taken before these
    if (lane == 0) {
        if ((uint64_t)total >= kRowsLimit || before + (uint64_t)total >= kRowsLimit)
            or_status(status, MDX_DEV_OUTPUT_OVERFLOW);
        const int64_t s0 = (int64_t)p << pl.qbits, s1 = (int64_t)(p + 1) << pl.qbits;
        const uint64_t items = pl.istart ? pl.istart[s1] - pl.istart[s0] : (uint64_t)(s1 - s0);
        if ((old & kDoneMask) + 1 == items)
            st_agent(pl.pst + p, kFlagAgg | (before + (uint64_t)total));
    }
    if (p != cp) {
        bool ok;
        cb = prefix_before(pl.pst, p, lane, status, &ok);
        // p - 1's inclusive prefix is base(p): later look-backs stop there
        if (ok && p > 0 && lane == 0)
            st_agent(pl.pst + p - 1, kFlagIncl | (uint64_t)cb);
        cp = p;
    }
    return cb + (int64_t)before;
}

// ---- plan --------------------------------------------------------------------
// Items of a sub-bucket: its probe batches, one when there is at most one
// or nothing to match.
__device__ __forceinline__ uint32_t items_of(int64_t nb, int64_t nr)
{
    return nb > 0 && nr > kJoinBatch ? (uint32_t)((nr + kJoinBatch - 1) / kJoinBatch) : 1u;
}

// Sub-buckets per thread of a planning workgroup: rj_plan_one's does up to
// kPlanOneMax alone, rj_plan's kPlanChunk each.
constexpr int kPlanOnePer = 8, kPlanPer = 2;
constexpr int64_t kPlanOneMax = (int64_t)kBlock * kPlanOnePer;
static_assert(kPlanChunk == (int64_t)kBlock * kPlanPer, "chunks of rj_plan");

// Block: sub-buckets [s0, s0 + m), m <= kBlock PER: exclusive prefix of their
// items into pre[0..m] (LDS); over: some build side exceeds a table.  Returns
// the items.  The items are counted with consecutive lanes on consecutive
// sub-buckets; the prefix is formed only when some sub-bucket has several.
template <int PER>
__device__ __forceinline__ int64_t plan_prefix(const int64_t *subL, const int64_t *subR,
                                               int64_t s0, int m, uint32_t *pre,
                                               int64_t *scratch, bool &over)
{
    const int tid = threadIdx.x;
    int64_t nb[PER], nr[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        // indices past the end are clamped: no load behind a branch
        const int i = k * kBlock + tid;
        const int64_t c = s0 + (i < m ? i : m - 1);
        nb[k] = subL[c + 1] - subL[c];
        nr[k] = subR[c + 1] - subR[c];
    }
    int big = 0, over_ = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = k * kBlock + tid;
        const uint32_t ni = items_of(nb[k], nr[k]);
        big |= ni > 1;
        over_ |= nb[k] > kJoinCap;
        if (i < m)
            pre[i] = ni;
    }
    over = __syncthreads_or(over_) != 0;
    if (!__syncthreads_or(big)) {
        for (int i = tid; i <= m; i += kBlock)
            pre[i] = (uint32_t)i;
        __syncthreads();
        return m;
    }
    uint32_t ni[PER], sum = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = tid * PER + k;
        ni[k] = i < m ? pre[i] : 0u;
        sum += ni[k];
    }
    int64_t total;  // (the scan's barriers: every item count has been read)
    uint32_t run = (uint32_t)block_excl_scan((int64_t)sum, scratch, &total);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = tid * PER + k;
        if (i < m)
            pre[i] = run;
        run += ni[k];
    }
    if (tid == 0)
        pre[m] = (uint32_t)total;
    __syncthreads();
    return total;
}

// Block: the item list of those sub-buckets, whose first item is `base`.
__device__ void plan_list(const RJoinWs &w, int64_t s0, int m, int64_t base, const uint32_t *pre)
{
    const int total = (int)pre[m];
    for (int k = threadIdx.x; k < m; k += kBlock)
        w.istart[s0 + k] = (uint32_t)base + pre[k];
    for (int i = threadIdx.x; i < total; i += kBlock) {
        int l = 0, h = m - 1;  // the last k with pre[k] <= i
        if (total == m)
            l = i;
        else
            while (l < h) {
                const int mid = (l + h + 1) >> 1;
                if (pre[mid] <= (uint32_t)i)
                    l = mid;
                else
                    h = mid - 1;
            }
        w.isub[base + i] = (uint32_t)(s0 + l);
    }
}

// Chained scan and cursors cleared (whole grid).
__device__ __forceinline__ void plan_clear(const RJoinWs &w)
{
    const int64_t stride = (int64_t)gridDim.x * kBlock, i0 = (int64_t)blockIdx.x * kBlock;
    for (int64_t i = i0 + threadIdx.x; i < w.max_items; i += stride)
        w.status[i] = 0;
    for (int64_t i = i0 + threadIdx.x; i < w.P; i += stride)
        w.cursor[i] = 0;
}

// chunked: oversized build sub-buckets are joined in chunks (the LDS-fit
// flag stays 1).
__global__ __launch_bounds__(kBlock) void rj_plan(const int64_t *__restrict__ subL,
                                                  const int64_t *__restrict__ subR, RJoinWs w,
                                                  int chunked, int32_t *status)
{
    __shared__ uint32_t pre[kPlanChunk + 1];
    __shared__ int64_t scratch[kWavesPerBlock];
    __shared__ int64_t s_base;
    __shared__ uint32_t s_chunk;
    plan_clear(w);
    if (threadIdx.x == 0)
        s_chunk = atomicAdd(w.plan_ticket, 1u);
    __syncthreads();
    const int64_t b = s_chunk, s0 = b * kPlanChunk;
    if (s0 >= w.S)
        return;  // a workgroup that only clears
    const int m = (int)(w.S - s0 < kPlanChunk ? w.S - s0 : kPlanChunk);
    bool over;
    const int64_t total = plan_prefix<kPlanPer>(subL, subR, s0, m, pre, scratch, over);
    if (over && !chunked)
        w.plan_out[1] = 0;  // rj_plan_init set it to 1 before this kernel
    if (threadIdx.x < kWave) {
        const int64_t base = lookback(w.plan, b, total, threadIdx.x, status);
        if (threadIdx.x == 0)
            s_base = base;
    }
    __syncthreads();
    plan_list(w, s0, m, s_base, pre);
    if (s0 + m == w.S && threadIdx.x == 0) {
        w.istart[w.S] = (uint32_t)(s_base + total);
        w.plan_out[0] = (uint32_t)(s_base + total);
    }
}

__global__ __launch_bounds__(kBlock) void rj_plan_init(RJoinWs w, int chunks)
{
    for (int i = threadIdx.x; i < chunks; i += kBlock)
        w.plan[i] = 0;
    if (threadIdx.x < kJoinSync)
        w.join_sync[threadIdx.x * kSyncStride] = 0;
    if (threadIdx.x == 0) {
        w.plan_out[1] = 1;
        *w.ticket = 0;
        *w.plan_ticket = 0;
    }
}

// One block for the whole plan when there are few sub-buckets: the flag is
// decided by a block-wide OR, so it needs no earlier kernel to set it.
__global__ __launch_bounds__(kBlock) void rj_plan_one(const int64_t *__restrict__ subL,
                                                      const int64_t *__restrict__ subR, RJoinWs w,
                                                      int chunked)
{
    __shared__ uint32_t pre[kPlanOneMax + 1];
    __shared__ int64_t scratch[kWavesPerBlock];
    const int m = (int)w.S;
    bool over;
    const int64_t total = plan_prefix<kPlanOnePer>(subL, subR, 0, m, pre, scratch, over);
    if (threadIdx.x < kJoinSync)
        w.join_sync[threadIdx.x * kSyncStride] = 0;
    if (threadIdx.x == 0) {
        w.plan_out[1] = over && !chunked ? 0 : 1;
        *w.ticket = 0;
        w.plan_out[0] = (uint32_t)total;
        w.istart[m] = (uint32_t)total;
    }
    plan_clear(w);
    if (total != m)
        plan_list(w, 0, m, 0, pre);
}

// This thread's rows of the batch starting at rb (the same on every lane),
// up to re (rb < re): rb + j kJoinThreads + tid.  Rows past re load the
// batch's last row instead (no branch per load) and are ignored by the
// callers, which check r < re.  KEYS: only what holds the keys (int64 rows
// come whole).
template <bool KEYS, typename K>
__device__ __forceinline__ void load_batch(Rows<K> rrows, int64_t rb, int64_t re,
                                           K *kk, int64_t *vv)
{
    const Rows<K> b = rrows.from(rb);
    const int64_t left = re - rb;
    const uint32_t last = (uint32_t)((left < kJoinBatch ? left : kJoinBatch) - 1);
    const auto index = [&](int j) {
        const uint32_t r = (uint32_t)(j * kJoinThreads) + threadIdx.x;
        return r < last ? r : last;
    };
    if (KEYS)
        b.template load_keys<kJoinRows>(index, kk, vv);
    else
        b.template load<kJoinRows>(index, kk, vv);
}

// Per row: the number of matches (high 16 bits; at most G::cap) and the
// first matching build row in chain order (low 16 bits; meaningful when the
// count is not 0).  The chains of G::walk rows are walked together without
// branches: a finished chain sits on the sentinel row, whose link points to
// itself, so every step issues all G::walk rows' LDS reads at once.
template <class G, typename K>
__device__ __forceinline__ void match_batch(int64_t rb, int64_t re, const int64_t *tkey,
                                            const uint16_t *tn, const uint32_t *head, const K *kk,
                                            uint32_t *mf)
{
    constexpr uint32_t kSent = Tab<G>::sent;
    constexpr int kWalk = G::walk;
    const int64_t left = re - rb;
    const uint32_t n = (uint32_t)(left < kJoinBatch ? left : kJoinBatch);
#pragma unroll
    for (int g = 0; g < kJoinRows; g += kWalk) {
        int64_t h[kWalk];
        uint32_t e[kWalk];
        bool live = false;
#pragma unroll
        for (int i = 0; i < kWalk; ++i) {
            const int j = g + i;
            const uint32_t r = (uint32_t)(j * kJoinThreads) + threadIdx.x;
            mf[j] = 0;
            h[i] = (int64_t)kk[j];
            e[i] = r < n ? head[bucket_of<G>(h[i])] : kSent;
            live |= e[i] != kSent;
        }
        while (ballot(live)) {
            int64_t x[kWalk];
            uint32_t nx[kWalk];
#pragma unroll
            for (int i = 0; i < kWalk; ++i) {
                x[i] = tkey[e[i]];
                nx[i] = tn[e[i]];
            }
            live = false;
#pragma unroll
            for (int i = 0; i < kWalk; ++i) {
                const int j = g + i;
                if (x[i] == h[i] && e[i] != kSent)
                    mf[j] = mf[j] == 0 ? ((1u << 16) | e[i]) : mf[j] + (1u << 16);
                e[i] = nx[i];
                live |= e[i] != kSent;
            }
        }
    }
}

// Per-(row step, wave) sums of the match counts into cw (row order =
// step-major).  When no row of the step matches twice, the sum is a
// population count.
__device__ __forceinline__ void cell_sums(const uint32_t *mf, int64_t *cw, int lane, int wv)
{
#pragma unroll
    for (int j = 0; j < kJoinRows; ++j) {
        const uint32_t cnt = mf[j] >> 16;
        const uint64_t one = ballot(cnt == 1), many = ballot(cnt > 1);
        const int64_t s = many ? wave_sum((int64_t)cnt) : (int64_t)__popcll(one);
        if (lane == 0)
            cw[j * kJoinWaves + wv] = s;
    }
}

// Wave 0: total of the cells.
__device__ __forceinline__ int64_t cell_total(const int64_t *cw, int lane)
{
    int64_t loc = 0;
#pragma unroll
    for (int i = 0; i < kCellsPerLane; ++i)
        loc += cw[lane * kCellsPerLane + i];
    return wave_sum(loc);
}

// Wave 0: cw := exclusive prefix of cw (step-major), returns the total.
__device__ __forceinline__ int64_t cell_scan(int64_t *cw, int lane)
{
    int64_t v[kCellsPerLane], loc = 0;
#pragma unroll
    for (int i = 0; i < kCellsPerLane; ++i) {
        v[i] = cw[lane * kCellsPerLane + i];
        loc += v[i];
    }
    const int64_t inc = wave_incl_scan(loc, lane);
    int64_t run = inc - loc;
#pragma unroll
    for (int i = 0; i < kCellsPerLane; ++i) {
        cw[lane * kCellsPerLane + i] = run;
        run += v[i];
    }
    return __shfl(inc, kWave - 1, kWave);
}

// Write the output rows of the batch held in registers; base = output row of
// the batch's first match; cw holds the exclusive cell prefixes.
template <class G, typename K>
__device__ __forceinline__ void emit_batch(const K *kk, const int64_t *vv, const uint32_t *mf,
                                           const int64_t *cw, int64_t base, const int64_t *tkey,
                                           const int64_t *tp, const uint16_t *tn, K *out_key,
                                           int64_t *out_l, int64_t *out_r, int lane, int wv)
{
    constexpr uint32_t kSent = Tab<G>::sent;
#pragma unroll
    for (int j = 0; j < kJoinRows; ++j) {
        const uint32_t cnt = mf[j] >> 16, fst = mf[j] & 0xffffu;
        const uint64_t one = ballot(cnt == 1), many = ballot(cnt > 1);
        if (!(one | many))
            continue;
        const int64_t before =
            many ? wave_incl_scan((int64_t)cnt, lane) - (int64_t)cnt : (int64_t)mbcnt(one);
        // the wave's first output row of this step: a scalar base; lanes add
        // a 32-bit offset (a step of a wave has at most 64 G::cap rows)
        const int64_t wb = uniform(base + cw[j * kJoinWaves + wv]);
        K *ok = out_key + wb;
        int64_t *ol = out_l + wb, *orr = out_r + wb;
        uint32_t at = (uint32_t)before;
        if (cnt == 1) {
            ok[at] = kk[j];
            ol[at] = tp[fst];
            orr[at] = vv[j];
        } else if (cnt > 1) {
            const int64_t h = (int64_t)kk[j];
            for (uint32_t e = fst; e != kSent; e = tn[e]) {
                if (tkey[e] == h) {
                    ok[at] = kk[j];
                    ol[at] = tp[e];
                    orr[at] = vv[j];
                    ++at;
                }
            }
        }
    }
}

// Insert build rows [b0, b0 + n) (0 < n <= G::cap) into the LDS table.  Rows
// past n load the last row (no branch per load) and are not inserted.
template <class G, typename K>
__device__ __forceinline__ void build_table(Rows<K> lrows, int64_t b0,
                                            int64_t n, int64_t *tkey, int64_t *tp, uint16_t *tn,
                                            uint32_t *head)
{
    const int tid = threadIdx.x;
    for (int i = tid; i < G::heads; i += kJoinThreads)
        head[i] = Tab<G>::sent;
    __syncthreads();
    const Rows<K> b = lrows.from(b0);
    const uint32_t last = (uint32_t)n - 1;
    constexpr int kBuild = Tab<G>::build_rows;
    K bk[kBuild];
    int64_t bv[kBuild];
    b.template load<kBuild>(
        [&](int j) {
            const uint32_t i = (uint32_t)(j * kJoinThreads) + tid;
            return i < last ? i : last;
        },
        bk, bv);
#pragma unroll
    for (int j = 0; j < kBuild; ++j) {
        const int i = j * kJoinThreads + tid;
        if (i < n) {
            const int64_t k = (int64_t)bk[j];
            tkey[i] = k;
            tp[i] = bv[j];
            tn[i] = (uint16_t)atomicExch(&head[bucket_of<G>(k)], (uint32_t)i);
        }
    }
    __syncthreads();
}

// The LDS of a join workgroup.
struct JoinLds {
    int64_t *tkey;  // [G::cap + 1] key of build row i
    int64_t *tp;    // [G::cap] payload of build row i
    uint16_t *tn;   // [G::cap + 1] next row in i's chain
    uint32_t *head; // [G::heads] last row inserted per bucket
    int64_t *cw;    // [kCells]
    int64_t *s_excl, *s_total;
};

// The common item: its build rows fit one table and its probe rows one batch
// (0 < nb <= G::cap, 0 < eR - bR <= kJoinBatch): builds the table and counts
// the matches of every probe row (mf; per-wave sums in L.cw).  A wave's loads
// complete in the order they were issued, and waiting for one waits for all
// issued before it; so they are issued in the order they are needed, with
// no branch around any of them (so that the compiler counts them exactly):
// the build rows (the inserts wait for these alone), the probe rows' keys
// (the match), then, once the table is built, payloads that do not come with
// their keys (needed only to write the output).
template <class G, typename K>
__device__ __forceinline__ void count_one_batch(Rows<K> lrows, int64_t bL,
                                                int64_t nb, Rows<K> rrows, int64_t bR,
                                                int64_t eR, const JoinLds &L, K *kk, int64_t *vv,
                                                uint32_t *mf)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const uint32_t blast = (uint32_t)nb - 1, plast = (uint32_t)(eR - bR) - 1;
    constexpr int kBuild = Tab<G>::build_rows;
    K bk[kBuild];
    int64_t bv[kBuild];
    auto clamped = [tid](uint32_t last) {
        return [tid, last](int j) {
            const uint32_t i = (uint32_t)(j * kJoinThreads + tid);
            return i < last ? i : last;
        };
    };
    lrows.from(bL).template load<kBuild>(clamped(blast), bk, bv);
    rrows.from(bR).template load_keys<kJoinRows>(clamped(plast), kk, vv);
    for (int i = tid; i < G::heads; i += kJoinThreads)
        L.head[i] = Tab<G>::sent;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kBuild; ++j) {
        const int i = j * kJoinThreads + tid;
        if (i < nb) {
            const int64_t k = (int64_t)bk[j];
            L.tkey[i] = k;
            L.tp[i] = bv[j];
            L.tn[i] = (uint16_t)atomicExch(&L.head[bucket_of<G>(k)], (uint32_t)i);
        }
    }
    __syncthreads();
    rrows.from(bR).template load_rest<kJoinRows>(clamped(plast), vv);
    match_batch<G>(bR, eR, L.tkey, L.tn, L.head, kk, mf);
    cell_sums(mf, L.cw, lane, wv);
}

// Item t of one merge, of sub-bucket s (its first item: `first`): build rows
// [bL, bL + nb), probe rows [bR, eR).  Counts its output rows, takes them
// (place_rows), then writes them.  Without LOOPS, the build rows fit one
// table and the probe rows one batch.  With LOOPS a larger build side is
// joined one table-sized chunk at a time, every chunk against every probe
// batch (each pair of rows meets once), counting first and writing in a
// second round.
template <class G, typename K, bool LOOPS>
__device__ __forceinline__ void join_item(Rows<K> lrows, int64_t bL, int64_t nb,
                                          Rows<K> rrows, int64_t bR, int64_t eR,
                                          const Place &pl, int64_t t, int64_t s, bool first,
                                          int &cp, int64_t &cb, const ProbeOut &o, int32_t *status,
                                          const JoinLds &L)
{
    constexpr int64_t kCap = G::cap;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    K *out_key = (K *)o.key;
    const bool any = nb > 0 && eR > bR;
    const bool loops = LOOPS && any && (nb > kCap || eR - bR > kJoinBatch);
    K kk[kJoinRows];
    int64_t vv[kJoinRows];
    uint32_t mf[kJoinRows];

    int64_t counted = 0;  // the rows of a looped item
    if (loops) {
        for (int64_t c0 = 0; c0 < nb; c0 += kCap) {
            build_table<G>(lrows, bL + c0, nb - c0 < kCap ? nb - c0 : kCap, L.tkey, L.tp, L.tn,
                           L.head);
            for (int64_t b = bR; b < eR; b += kJoinBatch) {
                load_batch<true>(rrows, b, eR, kk, vv);
                match_batch<G>(b, eR, L.tkey, L.tn, L.head, kk, mf);
                cell_sums(mf, L.cw, lane, wv);
                __syncthreads();
                if (wv == 0) {
                    const int64_t all = cell_total(L.cw, lane);
                    if (lane == 0)
                        *L.s_total = all;
                }
                __syncthreads();
                counted += *L.s_total;
            }
        }
    } else if (any) {
        count_one_batch<G, K>(lrows, bL, nb, rrows, bR, eR, L, kk, vv, mf);
        __syncthreads();
    }
    if (wv == 0) {
        const int64_t rows = loops ? counted : (any ? cell_scan(L.cw, lane) : 0);
        const int64_t ex = place_rows(pl, t, s, first, rows, cp, cb, lane, status);
        if (lane == 0) {
            *L.s_excl = ex;
            *L.s_total = rows;
        }
    }
    __syncthreads();
    const int64_t E = *L.s_excl, total = *L.s_total;
    if (total == 0)
        return;
    if (E + total > o.cap) {
        if (tid == 0)
            or_status(status, MDX_DEV_OUTPUT_OVERFLOW);
        return;
    }
    if (!loops) {
        emit_batch<G>(kk, vv, mf, L.cw, E, L.tkey, L.tp, L.tn, out_key, o.lpay, o.rpay, lane, wv);
        return;
    }
    int64_t run = E;
    for (int64_t c0 = 0; c0 < nb; c0 += kCap) {
        __syncthreads();  // s_total has been read, the last chunk's table used
        if (nb > kCap)    // (a single table is still there)
            build_table<G>(lrows, bL + c0, nb - c0 < kCap ? nb - c0 : kCap, L.tkey, L.tp, L.tn,
                           L.head);
        for (int64_t b = bR; b < eR; b += kJoinBatch) {
            load_batch<false>(rrows, b, eR, kk, vv);
            match_batch<G>(b, eR, L.tkey, L.tn, L.head, kk, mf);
            cell_sums(mf, L.cw, lane, wv);
            __syncthreads();
            if (wv == 0) {
                const int64_t all = cell_scan(L.cw, lane);
                if (lane == 0)
                    *L.s_total = all;
            }
            __syncthreads();
            emit_batch<G>(kk, vv, mf, L.cw, run, L.tkey, L.tp, L.tn, out_key, o.lpay, o.rpay, lane,
                          wv);
            run += *L.s_total;
            __syncthreads();  // cw, s_total and the table are reused
        }
    }
}

// The kernel's kJoinPerCu workgroups of kJoinThreads fill a CU's 4 SIMDs
// with kJoinSimdWaves waves each.
constexpr int kJoinSimdWaves = kJoinPerCu * kJoinThreads / (4 * kWave);

// Items are taken strictly in ticket order, just before each is
// started: a ticket taken ahead of time would make later sub-buckets wait
// for it in the chained scan.
#define MDX_JOIN_LDS(G)                                                                    \
    __shared__ int64_t tkey[G::cap + 1];                                                   \
    __shared__ int64_t tp[G::cap];                                                         \
    __shared__ uint16_t tn[G::cap + 1];                                                    \
    __shared__ uint32_t head[G::heads];                                                    \
    __shared__ int64_t cw[kCells];                                                         \
    __shared__ int64_t s_next, s_excl, s_total;                                            \
    const JoinLds L = {tkey, tp, tn, head, cw, &s_excl, &s_total};                         \
    if (threadIdx.x == 0) {                                                                \
        tkey[G::cap] = 0;                                                                  \
        tn[G::cap] = (uint16_t)G::cap;                                                     \
    }

// Next ticket, the same on every lane.
__device__ __forceinline__ int64_t take_ticket(uint32_t *ticket, int64_t *s_next)
{
    if (threadIdx.x == 0)
        *s_next = (int64_t)atomicAdd(ticket, 1u);
    __syncthreads();
    const int64_t t = uniform(*s_next);
    __syncthreads();  // everyone has read s_next before it is replaced
    return t;
}

// CHUNKED: oversized build sub-buckets are joined in chunks; otherwise the
// kernel does nothing unless the plan found that every one fits a table.
template <typename K, bool CHUNKED>
__global__ __launch_bounds__(kJoinThreads)
__attribute__((amdgpu_waves_per_eu(kJoinSimdWaves, kJoinSimdWaves))) void rj_join(
    Rows<K> lrows, const int64_t *__restrict__ subL, Rows<K> rrows,
    const int64_t *__restrict__ subR, const uint32_t *__restrict__ istart,
    const uint32_t *__restrict__ isub, RJoinWs w, int qbits, int by_part, ProbeOut o,
    int32_t *status)
{
    MDX_JOIN_LDS(MergeJoin)
    // no items when the plan found a build side too large; the first ticket is
    // taken while these loads are under way
    const int64_t n = !CHUNKED && w.plan_out[1] == 0 ? 0 : w.plan_out[0];
    const bool split = n != w.S;  // some sub-bucket is several items
    const Place pl = {w.cursor, w.status, split ? istart : nullptr, n, o.offsets, qbits, by_part};
    int cp = -1;
    int64_t cb = 0;
    for (;;) {
        const int64_t t = take_ticket(w.ticket, &s_next);
        if (t >= n)
            break;
        const int64_t s = split ? isub[t] : t;
        // The item's bounds, loaded together (nothing that uses the first of
        // them passes the empty asm) and, as the list is only read here,
        // through the scalar cache.  One after the other, with the list in
        // vector loads, an item of a list began 0.4 us later: 51663 x 13.9E6
        // int32 rows with a few sub-buckets of several batches took 411 us,
        // so 405; 1E8 x 1E8 4054 and 4038.  (Without a list its entry is read
        // too, inside the workspace, and not used.)
        int64_t bL = subL[s], eL = subL[s + 1], bR = subR[s], eR = subR[s + 1];
        uint32_t i0 = istart[s];
        asm volatile("" : "+s"(bL), "+s"(eL), "+s"(bR), "+s"(eR), "+s"(i0));
        const int64_t nb = eL - bL;
        bool first = true;
        if (split) {
            const int64_t c = t - i0;
            first = c == 0;
            bR += c * kJoinBatch;
            eR = nb > 0 && bR + kJoinBatch < eR ? bR + kJoinBatch : eR;
        }
        join_item<MergeJoin, K, CHUNKED>(lrows, bL, nb, rrows, bR, eR, pl, t, s, first, cp, cb, o,
                                         status, L);
        __syncthreads();  // the table is reused by the next item
    }
}

// Every merge of a batch: tickets run over all merges' sub-buckets (merge m
// owns tickets [Spre[m], Spre[m+1])), so the workgroups stay busy across
// merges; each merge has its own partition cursors and chained scan.
template <typename K>
__global__ __launch_bounds__(kJoinThreads)
__attribute__((amdgpu_waves_per_eu(kJoinSimdWaves, kJoinSimdWaves))) void rj_join_batch(
    const JoinRec *__restrict__ B, const uint32_t *__restrict__ Spre, int M, uint32_t *ticket)
{
    MDX_JOIN_LDS(BatchJoin)
    const int64_t total = Spre[M];
    int64_t c0 = 0, c1 = 0;  // tickets of the merge whose record is loaded
    JoinRec r = {};
    int cp = -1;  // place_rows' cache, per merge
    int64_t cb = 0;
    for (;;) {
        const int64_t t = take_ticket(ticket, &s_next);
        if (t >= total)
            break;
        if (t < c0 || t >= c1) {
            const int m = find_range(Spre, M, (uint32_t)t);
            c0 = Spre[m];
            c1 = Spre[m + 1];
            r = B[m];
            cp = -1;
        }
        const int64_t s = t - c0;
        const int64_t *subL = r.subL, *subR = r.subR;
        const int64_t bL = subL[s];
        const Rows<K> lrows = make_rows<K>(r.lrows, r.nL), rrows = make_rows<K>(r.rrows, r.nR);
        const Place pl = {r.jcursor, r.jstatus, nullptr, r.S, r.o.offsets, r.qbits, r.by_part};
        join_item<BatchJoin, K, true>(lrows, bL, subL[s + 1] - bL, rrows, subR[s], subR[s + 1], pl,
                                      s, s, true, cp, cb, r.o, r.status, L);
        __syncthreads();  // the table is reused by the next sub-bucket
    }
}

// Block m: clear merge m's partition cursors and chained scan.  Block 0
// also resets the ticket.
__global__ __launch_bounds__(kBlock) void rj_clear_batch(const JoinRec *__restrict__ B,
                                                         uint32_t *ticket)
{
    const JoinRec &r = B[blockIdx.x];
    for (int64_t s = threadIdx.x; s < r.S; s += kBlock)
        r.jstatus[s] = 0;
    for (int p = threadIdx.x; p < r.P; p += kBlock)
        r.jcursor[p] = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0)
        *ticket = 0;
}

// offsets[0..P] of a placement by partition, one block: the exclusive prefix
// of the rows each partition's cursor took.
__device__ inline void offsets_from_cursors(const uint64_t *cursor, int P, int64_t *offsets)
{
    __shared__ int64_t scratch[kWavesPerBlock];
    int64_t carry = 0;
    for (int b = 0; b < P; b += kBlock) {
        const int p = b + threadIdx.x;
        const int64_t v = p < P ? (int64_t)(ld_agent(cursor + p) >> kDoneBits) : 0;
        int64_t all;
        const int64_t ex = block_excl_scan(v, scratch, &all);
        if (p < P)
            offsets[p] = carry + ex;
        carry += all;
    }
    if (threadIdx.x == 0)
        offsets[P] = carry;
}

// Block m: merge m's output offsets (those placed by partition).
__global__ __launch_bounds__(kBlock) void rj_finalize_batch(const JoinRec *__restrict__ B)
{
    const JoinRec &r = B[blockIdx.x];
    if (r.by_part)
        offsets_from_cursors(r.jcursor, r.P, r.o.offsets);
}

// Output offsets of a merge placed by partition, if the radix join ran.
__global__ __launch_bounds__(kBlock) void merge_finalize(RJoinWs w, ProbeOut o)
{
    if (w.plan_out[1] != 0)
        offsets_from_cursors(w.cursor, w.P, o.offsets);
}

}  // namespace

int rjoin_grid(int64_t S)
{
    // kJoinPerCu workgroups per CU (all resident at once), or one per
    // sub-bucket when there are fewer: a workgroup holds half a CU's LDS,
    // which other merges' kernels may need meanwhile.
    const int64_t cus = device_fill_blocks() / 8 > 0 ? device_fill_blocks() / 8 : 1;
    return (int)std::max<int64_t>(1, std::min<int64_t>(cus * kJoinPerCu, S));
}

bool rjoin_by_partition(int qbits, int64_t G)
{
    return ((int64_t)1 << qbits) >= 8 * G;
}

hipError_t launch_rjoin_plan(const int64_t *subL, const int64_t *subR, int64_t S,
                             const RJoinWs &w, bool chunked, int32_t *status, hipStream_t s)
{
    if (S <= kPlanOneMax) {
        hipLaunchKernelGGL(rj_plan_one, dim3(1), dim3(kBlock), 0, s, subL, subR, w, (int)chunked);
        return hipGetLastError();
    }
    // a workgroup per chunk of sub-buckets, and more to clear the items' status
    const int chunks = (int)((S + kPlanChunk - 1) / kPlanChunk);
    const int G = (int)std::max<int64_t>(chunks, std::min<int64_t>(256, w.max_items / kBlock));
    hipLaunchKernelGGL(rj_plan_init, dim3(1), dim3(kBlock), 0, s, w, chunks);
    hipLaunchKernelGGL(rj_plan, dim3(G), dim3(kBlock), 0, s, subL, subR, w, (int)chunked, status);
    return hipGetLastError();
}

template <typename K>
void launch_rjoin_kernel(int G, const void *lrows, int64_t nL, const int64_t *subL,
                         const void *rrows, int64_t nR, const int64_t *subR, const RJoinWs &w,
                         int qbits, const ProbeOut &o, int32_t *status, bool chunked,
                         hipStream_t s)
{
    const int by_part = rjoin_by_partition(qbits, rjoin_grid(w.S)) ? 1 : 0;
    const auto fn = chunked ? rj_join<K, true> : rj_join<K, false>;
    hipLaunchKernelGGL(fn, dim3(G), dim3(kJoinThreads), 0, s, make_rows<K>(lrows, nL), subL,
                       make_rows<K>(rrows, nR), subR, w.istart, w.isub, w, qbits, by_part, o,
                       status);
}

hipError_t launch_rjoin(const void *lrows, int64_t nL, const int64_t *subL, const void *rrows,
                        int64_t nR, const int64_t *subR, int key_bytes, int qbits,
                        const RJoinWs &w, const ProbeOut &o, int32_t *status, bool chunked,
                        hipStream_t s)
{
    const auto run = key_bytes == 8 ? launch_rjoin_kernel<int64_t> : launch_rjoin_kernel<int32_t>;
    trace_begin("rj_join", s);
    run(rjoin_grid(w.max_items), lrows, nL, subL, rrows, nR, subR, w, qbits, o, status, chunked, s);
    trace_end("rj_join", s);
    return hipGetLastError();
}

hipError_t launch_rjoin_batch(const JoinRec *recs, int M, const uint32_t *Spre, uint32_t S,
                              uint32_t *ticket, int key_bytes, bool by_part, hipStream_t s)
{
    if (M <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(rj_clear_batch, dim3((unsigned)M), dim3(kBlock), 0, s, recs, ticket);
    const int G = rjoin_grid(S);
    trace_begin("rj_join", s);
    if (key_bytes == 8)
        hipLaunchKernelGGL(rj_join_batch<int64_t>, dim3(G), dim3(kJoinThreads), 0, s, recs, Spre,
                           M, ticket);
    else
        hipLaunchKernelGGL(rj_join_batch<int32_t>, dim3(G), dim3(kJoinThreads), 0, s, recs, Spre,
                           M, ticket);
    trace_end("rj_join", s);
    if (by_part)
        hipLaunchKernelGGL(rj_finalize_batch, dim3((unsigned)M), dim3(kBlock), 0, s, recs);
    return hipGetLastError();
}

hipError_t launch_merge_finalize(int qbits, const RJoinWs &w, const ProbeOut &o, hipStream_t s)
{
    if (!rjoin_by_partition(qbits, rjoin_grid(w.S)))
        return hipSuccess;
    hipLaunchKernelGGL(merge_finalize, dim3(1), dim3(kBlock), 0, s, w, o);
    return hipGetLastError();
}

}  // namespace mdx
