// Device bodies of the partition's steps on one tile or one row of counts,
// shared by the partition kernels (partition.hip) and the global-table join
// (join.hip).
#pragma once

#include "mdx_internal.hpp"

namespace mdx {
namespace {

template <typename K>
struct PartTable {
    const K *keys;
    const int64_t *pay;
    int64_t n, ntiles;
    K *keys_out;      // two columns, or
    int64_t *pay_out;
    Rows<K> rows_out; // rows
    int64_t *off;     // [D + 1]
    uint8_t *dig;     // optional: one digit byte per output row
    int64_t *cnt;     // [D][ntiles]: counts, then exclusive prefixes
    int64_t *totals;  // [D]
};

// Histograms of at most this many destinations count by ballot: a whole
// wave's LDS atomics on a few addresses serialize.
constexpr int kFewDest = 4;

// Counts of tile `tile` of table tb per destination into tb.cnt.  FEW: the
// destinations may be few enough to count by ballot.
template <typename K, int R, bool FEW>
__device__ __forceinline__ void hist_tile(const PartTable<K> &tb, int64_t tile, const Dest &d,
                                          uint32_t *hist)
{
    const int tid = threadIdx.x;
    const int P = d.ndest;  // destinations
    for (int p = tid; p < P; p += kBlock)
        hist[p] = 0;
    const int64_t row0 = tile * (int64_t)(kBlock * R);
    const bool few = FEW && P <= kFewDest;
    uint32_t wc[kFewDest] = {};  // with few destinations: the wave's counts
    auto count = [&](bool valid, uint32_t p) {
        if (few) {
#pragma unroll
            for (int q = 0; q < kFewDest; ++q)
                if (q < P)
                    wc[q] += (uint32_t)__popcll(ballot(valid && p == (uint32_t)q));
        } else if (valid) {
            atomicAdd(&hist[p], 1u);
        }
    };
    // Keys are read 16 bytes per lane when the column is 16-byte aligned
    // (the counts do not depend on which thread reads which row).
    constexpr int V = 16 / (int)sizeof(K);  // keys per 16-byte load
    if (R % V == 0 && ((uintptr_t)tb.keys & 15) == 0) {
        // Thread tid, load j: rows row0 + (j kBlock + tid) V + [0, V).
        typedef K KV __attribute__((ext_vector_type(V)));
        K k[R];
#pragma unroll
        for (int j = 0; j < R / V; ++j) {
            const int64_t r = row0 + ((int64_t)j * kBlock + tid) * V;
            if (r + V <= tb.n) {
                const KV x = __builtin_nontemporal_load((const KV *)(tb.keys + r));
#pragma unroll
                for (int v = 0; v < V; ++v)
                    k[j * V + v] = x[v];
            } else {
#pragma unroll
                for (int v = 0; v < V; ++v)
                    k[j * V + v] = r + v < tb.n ? tb.keys[r + v] : K(0);
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < R / V; ++j) {
            const int64_t r = row0 + ((int64_t)j * kBlock + tid) * V;
#pragma unroll
            for (int v = 0; v < V; ++v)
                count(r + v < tb.n, dest_of(fmix64(key_bits(k[j * V + v])), d));
        }
    } else {
        K k[R];
#pragma unroll
        for (int c = 0; c < R; ++c) {
            const int64_t r = row0 + (int64_t)c * kBlock + tid;
            k[c] = r < tb.n ? __builtin_nontemporal_load(tb.keys + r) : K(0);
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < R; ++c) {
            const int64_t r = row0 + (int64_t)c * kBlock + tid;
            count(r < tb.n, dest_of(fmix64(key_bits(k[c])), d));
        }
    }
    if (few && (tid & (kWave - 1)) == 0) {
#pragma unroll
        for (int q = 0; q < kFewDest; ++q)
            if (q < P && wc[q] != 0)
                atomicAdd(&hist[q], wc[q]);
    }
    __syncthreads();
    for (int p = tid; p < P; p += kBlock)
        tb.cnt[(int64_t)p * tb.ntiles + tile] = hist[p];
}

// One wave: exclusive prefix of a row of tile counts in place; returns its
// total.  64 kScanLane counts at a time, each lane kScanLane consecutive ones.
__device__ __forceinline__ int64_t wave_scan_row(int64_t *row, int64_t ntiles, int lane)
{
    constexpr int kScanLane = 8;
    int64_t carry = 0;
    for (int64_t base = 0; base < ntiles; base += (int64_t)kWave * kScanLane) {
        const int64_t i0 = base + (int64_t)lane * kScanLane;
        int64_t v[kScanLane], sum = 0;
#pragma unroll
        for (int j = 0; j < kScanLane; ++j) {
            v[j] = i0 + j < ntiles ? row[i0 + j] : 0;
            sum += v[j];
        }
        const int64_t inc = wave_incl_scan(sum, lane);
        int64_t run = carry + inc - sum;
#pragma unroll
        for (int j = 0; j < kScanLane; ++j) {
            if (i0 + j < ntiles)
                row[i0 + j] = run;
            run += v[j];
        }
        carry += __shfl(inc, kWave - 1, kWave);
    }
    return carry;
}

// One table's destination offsets from its totals.
__device__ __forceinline__ void offsets_of(const int64_t *totals, int64_t *off, int P,
                                           int64_t *scratch)
{
    int64_t carry = 0;
    for (int base = 0; base < P; base += kBlock) {
        const int p = base + threadIdx.x;
        const int64_t v = p < P ? totals[p] : 0;
        int64_t tot;
        const int64_t ex = block_excl_scan(v, scratch, &tot);
        if (p < P)
            off[p] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0)
        off[P] = carry;
}

// Exclusive prefix over a[0..P) in LDS, in place (all threads call).
__device__ inline void lds_excl_scan_u32(uint32_t *a, int P, int64_t *scratch)
{
    int64_t carry = 0;
    for (int base = 0; base < P; base += kBlock) {
        const int p = base + threadIdx.x;
        const int64_t v = p < P ? a[p] : 0;
        int64_t tot;
        const int64_t ex = block_excl_scan(v, scratch, &tot);
        if (p < P)
            a[p] = (uint32_t)(carry + ex);
        carry += tot;
    }
    __syncthreads();
}

// A tile's input: two columns (keys first, then payloads, which are needed
// only for staging), or rows.
template <typename K>
struct FromCols {
    const K *__restrict__ keys;
    const int64_t *__restrict__ pay;
    template <int R>
    __device__ __forceinline__ void load(int64_t r0, int64_t row_end, K *kr, int64_t *vr) const
    {
#pragma unroll
        for (int c = 0; c < R; ++c) {
            const int64_t r = r0 + (int64_t)c * kWave;
            kr[c] = r < row_end ? __builtin_nontemporal_load(keys + r) : K(0);
        }
#pragma unroll
        for (int c = 0; c < R; ++c) {
            const int64_t r = r0 + (int64_t)c * kWave;
            vr[c] = r < row_end ? __builtin_nontemporal_load(pay + r) : 0;
        }
    }
};

template <typename K>
struct FromRows {
    Rows<K> rows;
    template <int R>
    __device__ __forceinline__ void load(int64_t r0, int64_t row_end, K *kr, int64_t *vr) const
    {
        rows.template load_if<R>([&](int c) { return r0 + (int64_t)c * kWave; },
                                 [&](int c) { return r0 + (int64_t)c * kWave < row_end; }, kr, vr);
    }
};

// A tile's output as two columns (or Rows<K>).
template <typename K>
struct ToCols {
    K *__restrict__ keys;
    int64_t *__restrict__ pay;
    __device__ __forceinline__ void store(int64_t r, K k, int64_t v) const
    {
        keys[r] = k;
        pay[r] = v;
    }
};

// Stable scatter of one tile, rows [row0, row_end) (at most kBlock R of them).
// A row's destination in [0, D) is dfn(fmix64(key)); with DIG_OUT every
// output row's next-pass digit digit_of(h, dshift, dbits) is written beside
// it (from the same hash).  base_of(d) is the output position of the tile's
// first row with destination d.  Wave w owns the contiguous rows
// [row0 + 64 R w, row0 + 64 R (w+1)); step c reads 64 consecutive rows.
// (The second pass hashes its keys again rather than reading the digit
// bytes: byte loads, 64 bytes per wave instruction, slowed it by a quarter.)
template <typename K, int R, bool DIG_OUT, typename From, typename To, typename DestFn,
          typename BaseFn>
__device__ __forceinline__ void scatter_tile(const From &from, int64_t row0, int64_t row_end, int D,
                                             int nbits, DestFn dfn, BaseFn base_of, const To &to,
                                             unsigned char *smem, uint8_t *__restrict__ dig_out,
                                             int dshift, int dbits)
{
    constexpr int T = kBlock * R;
    static_assert(T <= 65535, "per-wave tile counts are 16-bit");
    const ScatterLds L = scatter_lds(T, D, (int)sizeof(K), DIG_OUT);
    int64_t *stage_v = (int64_t *)(smem + L.stage_v);
    K *stage_k = (K *)(smem + L.stage_k);
    uint16_t *stage_p = (uint16_t *)(smem + L.stage_p);
    uint8_t *stage_d = (uint8_t *)(smem + L.stage_d);
    uint16_t *whist = (uint16_t *)(smem + L.whist);
    uint32_t *tstart = (uint32_t *)(smem + L.tstart);
    int64_t *gbase = (int64_t *)(smem + L.gbase);
    int64_t *scratch = (int64_t *)(smem + L.scratch);

    const int tid = threadIdx.x, w = tid / kWave, lane = tid & (kWave - 1);

    // The row loads go first, so that the destination bases' loads and the
    // ranking overlap them.
    const int64_t wrow0 = row0 + (int64_t)w * kWave * R;
    K kr[R];
    int64_t vr[R];
    from.template load<R>(wrow0 + lane, row_end, kr, vr);
    for (int i = tid; i < kWavesPerBlock * D; i += kBlock)
        whist[i] = 0;
    for (int p = tid; p < D; p += kBlock)
        gbase[p] = base_of(p);
    __syncthreads();

    // Rank every row among the earlier rows of its wave with its destination.
    uint16_t *wh = whist + w * D;
    uint32_t pr[R], rk[R];
    uint8_t dg[R];
#pragma unroll
    for (int c = 0; c < R; ++c) {
        const int64_t r = wrow0 + (int64_t)c * kWave + lane;
        const bool valid = r < row_end;
        const uint64_t h = fmix64(key_bits(kr[c]));
        const uint32_t p = valid ? dfn(h) : 0u;
        if (DIG_OUT)
            dg[c] = (uint8_t)digit_of(h, dshift, dbits);
        uint64_t m = ballot(valid);
        for (int b = 0; b < nbits; ++b) {
            const bool bit = (p >> b) & 1u;
            const uint64_t bb = ballot(bit);
            m &= bit ? bb : ~bb;
        }
        const uint32_t rank = mbcnt(m);
        uint32_t prev = 0;
        if (valid)
            prev = wh[p];
        if (valid && rank == 0)
            wh[p] = (uint16_t)(prev + (uint32_t)__popcll(m));
        pr[c] = valid ? p : 0xffffffffu;
        rk[c] = prev + rank;
    }
    __syncthreads();

    // Per destination: tile count, and every wave's offset inside it.
    for (int p = tid; p < D; p += kBlock) {
        uint32_t acc = 0;
#pragma unroll
        for (int ww = 0; ww < kWavesPerBlock; ++ww) {
            const uint32_t c = whist[ww * D + p];
            whist[ww * D + p] = (uint16_t)acc;
            acc += c;
        }
        tstart[p] = acc;
    }
    __syncthreads();
    lds_excl_scan_u32(tstart, D, scratch);  // tstart[p]: first staged row of p
    for (int p = tid; p < D; p += kBlock) {
        const uint32_t t0 = tstart[p];
#pragma unroll
        for (int ww = 0; ww < kWavesPerBlock; ++ww)
            whist[ww * D + p] = (uint16_t)(whist[ww * D + p] + t0);
    }
    __syncthreads();

#pragma unroll
    for (int c = 0; c < R; ++c) {
        if (pr[c] != 0xffffffffu) {
            const uint32_t s = wh[pr[c]] + rk[c];
            stage_k[s] = kr[c];
            stage_v[s] = vr[c];
            stage_p[s] = (uint16_t)pr[c];
            if (DIG_OUT)
                stage_d[s] = dg[c];
        }
    }
    __syncthreads();

    const int rows = (int)((row_end - row0) < (int64_t)T ? (row_end - row0) : (int64_t)T);
    for (int s = tid; s < rows; s += kBlock) {
        const uint32_t p = stage_p[s];
        const int64_t dst = gbase[p] + (s - (int)tstart[p]);
        // Ordinary stores: a run's first and last cache lines are shared
        // with the neighbouring tiles' runs and must meet them in L2 (the
        // XCD-contiguous tile order keeps those tiles on one L2).  With
        // streaming stores the partial lines went to HBM separately: 25% more
        // bytes written, 26% slower at a fan-out of 128.
        to.store(dst, stage_k[s], stage_v[s]);
        if (DIG_OUT)
            dig_out[dst] = stage_d[s];
    }
}

// First-pass scatter of tile `tile` of table tb.
template <typename K, int R, bool ROWS, bool DIG>
__device__ __forceinline__ void part_scatter_tile(const PartTable<K> &tb, int64_t tile,
                                                  const Dest &d, int dshift, int dbits,
                                                  unsigned char *smem)
{
    auto scatter = [&](const auto &to) {
        scatter_tile<K, R, DIG>(
            FromCols<K>{tb.keys, tb.pay}, tile * (int64_t)(kBlock * R), tb.n, d.ndest, d.nbits,
            [&](uint64_t h) { return dest_of(h, d); },
            [&](int p) { return tb.off[p] + tb.cnt[(int64_t)p * tb.ntiles + tile]; }, to, smem,
            tb.dig, dshift, dbits);
    };
    if constexpr (ROWS)
        scatter(tb.rows_out);
    else
        scatter(ToCols<K>{tb.keys_out, tb.pay_out});
}

}  // namespace
}  // namespace mdx
