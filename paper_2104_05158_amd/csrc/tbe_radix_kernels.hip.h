// Radix sort by (table, row) and run-length segmentation of a batch's lookups, for the calls in which the partition of
// tbe_sort_kernels.hip.h loses (use_radix_sort in tbe_rules.h): a few very tall tables, whose buckets do not fit a
// workgroup's LDS and are too few for the chip, and very many tables, each of which takes that sort a plan of its own.
//
// The input is table-major, so the lookups of table t already occupy one contiguous range of
// positions: sorting by (table, row) is a SEGMENTED sort in which every table is sorted by its own
// row index.  That needs only ceil(log2 max_t H_t) key bits instead of ceil(log2 sum_t H_t), the first
// pass can read the caller's indices directly as keys (the payload b, the bag's position inside its
// table's batch, is derived from the offsets on the fly), and the last pass adds the table's row base
// so that the result is sorted by the linear row id.
//
// Tiles of kSortTile positions never cross a table border.  A small plan (two launches) turns the
// table borders offsets[t*B] into: the first tile of every table, the first position of every
// table, and the table of every tile.  The per-tile digit histograms are laid out table by table,
// digit-major inside a table: hist[tile_base[t]*nd + d*ntiles_t + local_tile].  One exclusive scan
// over the whole array then yields global output positions, because every table's counts add up to
// exactly its number of lookups.
//
// Every table is sorted over its own ceil(log2 H_t) index bits in ceil(bits / 8) passes of equal-as-possible
// digit widths.  A launch serves all tables; a table that needs fewer passes than the tallest one sits out
// the first launches (its tiles report all their keys under digit 0, so the scan still yields global
// positions, and move nothing) and makes its first pass -- the one that reads the caller's indices -- later,
// so that every table finishes in the same launch and in the same buffer.
//
// Per pass: (1) per-tile digit histogram, (2) the scan, (3) scatter: every wavefront ranks its
// 16 x 64 keys with ballot-based digit matching into per-wave LDS counters, the tile is reordered by
// digit inside LDS and then written out in runs that are contiguous in global memory.  Order inside
// a tile is (wavefront, round, lane) = ascending position, so equal digits keep their input order
// and the whole sort is stable.
#pragma once

#include "tbe_sort_kernels.hip.h"

namespace tbe {

constexpr int kScanThreads = 256;
constexpr int kScanPerThread = 16;
constexpr int kScanTile = kScanThreads * kScanPerThread;      // 4096
constexpr int kRlThreads = 256;
constexpr int kRlPerThread = 16;
constexpr int kRlTile = kRlThreads * kRlPerThread;            // 4096 sorted positions

struct TileDesc {        // 32 bytes: everything a workgroup needs to know about its tile, in one load
    int32_t t;           // table, -1 past the last tile
    int32_t first;       // first position of the tile
    int32_t cnt;         // positions in the tile (1..kSortTile)
    int32_t hstride;     // tiles of the table = distance between consecutive digits in the histogram
    int32_t tbase;       // first tile of the table
    int32_t local;       // index of the tile inside its table
    int32_t bag_lo;      // bag (inside the table's batch) of the tile's first position ...
    int32_t bag_hi;      // ... and of its last one
};

struct SortPlan {
    const int32_t* tile_base;    // [T+1] first tile of table t; [T] = number of tiles
    const int32_t* tstart;       // [T+1] first position of table t; [T] = n
    const TileDesc* tiles;       // [max_tiles]
};

// one workgroup: table borders -> tile_base / tstart; also clears the per-call counters
__global__ __launch_bounds__(256) void sort_plan_tables_kernel(const int64_t* __restrict__ offsets, int32_t B,
                                                               int32_t T, int32_t* __restrict__ tile_base,
                                                               int32_t* __restrict__ tstart,
                                                               Counters* __restrict__ counters)
{
    __shared__ uint32_t s_wave[4];
    if (threadIdx.x == 0)
        counters->num_unique = 0;
    uint32_t carry = 0;
    for (int base = 0; base < T; base += 256) {
        const int t = base + threadIdx.x;
        int32_t lo = 0, cnt = 0;
        if (t < T) {
            lo = (int32_t)offsets[(int64_t)t * B];
            cnt = (int32_t)offsets[(int64_t)(t + 1) * B] - lo;
        }
        const uint32_t tiles = (uint32_t)((cnt + kSortTile - 1) / kSortTile);
        uint32_t tot;
        const uint32_t ex = block_exclusive_scan_256(tiles, s_wave, tot);
        if (t < T) {
            tile_base[t] = (int32_t)(carry + ex);
            tstart[t] = lo;
        }
        carry += tot;
    }
    if (threadIdx.x == 0) {
        tile_base[T] = (int32_t)carry;
        tstart[T] = (int32_t)offsets[(int64_t)T * B];
    }
}

// last bag b in [0, B) of table t with offsets[t*B + b] <= q
__device__ __forceinline__ int bag_of_position(const int64_t* __restrict__ offsets, int64_t j0, int B, int64_t q)
{
    int a = 0, c = B;
    while (c - a > 1) {
        const int mid = (a + c) >> 1;
        if (offsets[j0 + mid] <= q)
            a = mid;
        else
            c = mid;
    }
    return a;
}

__global__ __launch_bounds__(256) void sort_plan_tiles_kernel(const int32_t* __restrict__ tile_base,
                                                              const int32_t* __restrict__ tstart,
                                                              const int64_t* __restrict__ offsets, int32_t B,
                                                              int32_t T, TileDesc* __restrict__ tiles,
                                                              int32_t max_tiles)
{
    const int g = blockIdx.x * 256 + threadIdx.x;
    if (g >= max_tiles)
        return;
    TileDesc d;
    d.t = -1; d.first = 0; d.cnt = 0; d.hstride = 0; d.tbase = 0; d.local = 0; d.bag_lo = d.bag_hi = 0;
    if (g < tile_base[T]) {
        int a = 0, c = T;  // last a in [0, T) with tile_base[a] <= g
        while (c - a > 1) {
            const int mid = (a + c) >> 1;
            if (tile_base[mid] <= g)
                a = mid;
            else
                c = mid;
        }
        const int tb = tile_base[a];
        d.t = a;
        d.tbase = tb;
        d.local = g - tb;
        d.first = tstart[a] + d.local * kSortTile;
        d.cnt = min(kSortTile, tstart[a + 1] - d.first);
        d.hstride = tile_base[a + 1] - tb;
        d.bag_lo = bag_of_position(offsets, (int64_t)a * B, B, d.first);
        d.bag_hi = bag_of_position(offsets, (int64_t)a * B, B, d.first + d.cnt - 1);
    }
    tiles[g] = d;
}

struct TileGeom {
    int t;          // table
    int first;      // first position of the tile
    int cnt;        // positions in the tile (1..kSortTile)
    int64_t hbase;  // index of this tile's digit-0 histogram entry
    int hstride;    // distance between consecutive digits (tiles of the table)
};

__device__ __forceinline__ bool tile_geom(const SortPlan& pl, int g, int nd, TileGeom& tg)
{
    const int4 a = *reinterpret_cast<const int4*>(&pl.tiles[g]);            // t, first, cnt, hstride
    const int2 b = *reinterpret_cast<const int2*>(&pl.tiles[g].tbase);      // tbase, local
    if (a.x < 0)
        return false;
    tg.t = a.x;
    tg.first = a.y;
    tg.cnt = a.z;
    tg.hstride = a.w;
    tg.hbase = (int64_t)b.x * nd + b.y;
    return true;
}

// Where table t stands in launch p of P: P_t = ceil(bits / 8) passes, the last P_t launches; pass lp orders
// `width` bits starting at `shift` (the bits are split as evenly as possible, wider digits first).
struct PassGeom {
    bool active;     // the table takes part in this launch
    bool first;      // this is the table's first pass: keys come from the caller's indices
    int shift, width;
};

__device__ __forceinline__ PassGeom pass_geom(int key_bits, int p, int P)
{
    const int pt = (key_bits + 7) >> 3;
    const int lp = p - (P - pt);
    PassGeom g;
    g.active = lp >= 0;
    g.first = lp == 0;
    const int q = key_bits / pt, rem = key_bits - q * pt;
    const int l = max(lp, 0);
    g.width = q + (l < rem ? 1 : 0);
    g.shift = l * q + min(l, rem);
    return g;
}

// Lanes of the wavefront whose digit equals this lane's (valid lanes only).  Bit b of every lane is
// broadcast by a ballot; a lane keeps the lanes whose bit agrees with its own.  The loop is unrolled
// for the largest digit width with a uniform guard, so no bit position costs a loop iteration.
__device__ __forceinline__ uint64_t match_digit(uint32_t dg, bool valid, int bits)
{
    uint32_t lo, hi;
    {
        const uint64_t v = __ballot(valid);
        lo = (uint32_t)v;
        hi = (uint32_t)(v >> 32);
    }
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        if (b < bits) {
            const uint32_t m = (uint32_t)(((int32_t)(dg << (31 - b))) >> 31);   // all ones if bit b is set
            const uint64_t bal = __ballot(m != 0u);
            // lanes whose bit differs from mine drop out: peers &= ~(bal ^ m)
            lo &= ~((uint32_t)bal ^ m);
            hi &= ~((uint32_t)(bal >> 32) ^ m);
        }
    }
    return ((uint64_t)hi << 32) | lo;
}

__global__ __launch_bounds__(kSortThreads) void radix_hist_kernel(
    SortPlan pl, const TableMeta* __restrict__ meta, const uint32_t* __restrict__ keys_cur,
    const uint32_t* __restrict__ indices, uint32_t* __restrict__ hist, int p, int P, int nd_bits)
{
    __shared__ uint32_t s_hist[256];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x >> 6;
    const int nd = 1 << nd_bits;
    TileGeom tg;
    if (!tile_geom(pl, blockIdx.x, nd, tg))
        return;
    const PassGeom pg = pass_geom(meta[tg.t].key_bits, p, P);
    if (!pg.active) {
        // the table sits this launch out: all its keys count under digit 0
        if ((int)threadIdx.x < nd)
            hist[tg.hbase + (int64_t)threadIdx.x * tg.hstride] = threadIdx.x == 0 ? (uint32_t)tg.cnt : 0u;
        return;
    }
    const uint32_t* __restrict__ keys = pg.first ? indices : keys_cur;
    const int shift = pg.shift;
    const uint32_t mask = (1u << pg.width) - 1u;
    const int base = tg.first + wave * (kSortTile / (kSortThreads / kWave));
    const int end = tg.first + tg.cnt;
    // all 16 key loads are issued before the first one is used (positions past the tile are clamped);
    // 16-byte loads of four keys per lane were measured and are not faster
    uint32_t key[kSortPerThread];
#pragma unroll
    for (int r = 0; r < kSortPerThread; ++r)
        key[r] = keys[min(base + r * kWave + lane, end - 1)];
    if ((int)threadIdx.x < nd)
        s_hist[threadIdx.x] = 0;
    __syncthreads();
    // Counting needs no ranks: when the 64 keys of a round share one digit (identical rows are adjacent
    // from the second pass on) one lane adds the whole count, otherwise every lane adds 1; LDS integer
    // atomics, so the totals do not depend on the order.
#pragma unroll
    for (int r = 0; r < kSortPerThread; ++r) {
        const int q = base + r * kWave + lane;
        const bool valid = q < end;                   // valid lanes are a prefix of the wavefront
        const uint32_t dg = (key[r] >> shift) & mask;
        const uint64_t vm = __ballot(valid);
        const uint32_t d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)dg);
        const uint64_t same = __ballot(dg == d0);
        if ((same & vm) == vm) {
            if (lane == 0 && vm != 0ull)
                atomicAdd(&s_hist[d0], (uint32_t)__popcll(vm));
        } else if (valid) {
            atomicAdd(&s_hist[dg], 1u);
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < nd)
        hist[tg.hbase + (int64_t)threadIdx.x * tg.hstride] = s_hist[threadIdx.x];
}

// A table's first pass reads the caller's index array as keys and computes the payload from the offsets;
// LAST (the launch in which every table makes its last pass): the table's row base is added to the keys
// that are written out.  V16 (batch <= 65536): between the passes the payload, a bag number below 2^16,
// travels as 16 bits (in the same buffers); the last launch writes the int32 payloads the update reads.
template <bool LAST, bool V16>
__global__ __launch_bounds__(kSortThreads) void radix_scatter_kernel(
    SortPlan pl, const TableMeta* __restrict__ meta, const uint32_t* __restrict__ keys_cur,
    const int32_t* __restrict__ vals_in, const uint32_t* __restrict__ indices,
    uint32_t* __restrict__ keys_out, int32_t* __restrict__ vals_out,
    const uint32_t* __restrict__ hist_scanned, const int64_t* __restrict__ offsets,
    const uint32_t* __restrict__ row_base, int32_t B, int p, int P, int nd_bits)
{
    constexpr int kWaves = kSortThreads / kWave;
    __shared__ uint32_t s_keys[kSortTile];
    __shared__ int32_t s_vals[kSortTile];
    __shared__ uint32_t s_whist[kWaves][256];
    __shared__ uint32_t s_dstart[256];
    __shared__ uint32_t s_goff[256];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x >> 6;
    const int nd = 1 << nd_bits;
    TileGeom tg;
    if (!tile_geom(pl, blockIdx.x, nd, tg))
        return;
    const PassGeom pg = pass_geom(meta[tg.t].key_bits, p, P);
    if (!pg.active)
        return;                                  // the table sits this launch out: nothing moves
    const bool FIRST = pg.first;
    const int shift = pg.shift, bits = pg.width;
    const uint32_t mask = (1u << bits) - 1u;
    const uint32_t* __restrict__ keys_in = FIRST ? indices : keys_cur;
    const int tile_cnt = tg.cnt;
    const int end = tg.first + tile_cnt;

    for (int i = threadIdx.x; i < kWaves * 256; i += kSortThreads)
        (&s_whist[0][0])[i] = 0;
    __syncthreads();

    uint32_t key[kSortPerThread];
    int32_t val[kSortPerThread];
    uint32_t rank[kSortPerThread];
    const int base = tg.first + wave * (kSortTile / kWaves);
#pragma unroll
    for (int r = 0; r < kSortPerThread; ++r) {
        const int q = min(base + r * kWave + lane, end - 1);
        key[r] = keys_in[q];
        if (!FIRST)
            val[r] = V16 ? (int32_t)reinterpret_cast<const uint16_t*>(vals_in)[q] : vals_in[q];
    }
    if (FIRST) {
        // payload = bag of the position: the borders of the bags the tile touches are staged in
        // LDS (in the space the reordered payloads use later) and searched there
        const int2 bags = *reinterpret_cast<const int2*>(&pl.tiles[blockIdx.x].bag_lo);
        const int b_lo = bags.x, b_hi = bags.y;
        const int nb = b_hi - b_lo + 1;
        const int64_t j0 = (int64_t)tg.t * B + b_lo;
        if (nb <= kSortTile) {
            for (int i = threadIdx.x; i < nb; i += kSortThreads)
                s_vals[i] = (int32_t)offsets[j0 + i];
            __syncthreads();
            int steps = 0;
            while ((1 << steps) < nb)
                ++steps;
#pragma unroll
            for (int r = 0; r < kSortPerThread; ++r) {
                const int q = min(base + r * kWave + lane, end - 1);
                int a = 0, c = nb;  // last a with s_vals[a] <= q
                for (int st = 0; st < steps; ++st) {
                    const int mid = (a + c) >> 1;
                    const bool up = s_vals[mid] <= q;
                    a = up ? mid : a;
                    c = up ? c : max(mid, a + 1);
                }
                val[r] = b_lo + a;
            }
        } else {
#pragma unroll 1
            for (int r = 0; r < kSortPerThread; ++r) {
                const int q = min(base + r * kWave + lane, end - 1);
                int a = 0, c = nb;
                while (c - a > 1) {
                    const int mid = (a + c) >> 1;
                    if (offsets[j0 + mid] <= q)
                        a = mid;
                    else
                        c = mid;
                }
                val[r] = b_lo + a;
            }
        }
    }
    // The wavefront's private counters are indexed as the LDS array they are (a pointer to the row would be
    // a generic pointer: flat loads and stores, each waited for).  LDS operations of one wavefront execute
    // in order and the compiler keeps a load behind a store that may alias it, so a round sees the counts
    // of the rounds before it.
    const uint64_t lt = (1ull << lane) - 1ull;
#pragma unroll
    for (int r = 0; r < kSortPerThread; ++r) {
        const int q = base + r * kWave + lane;
        const bool valid = q < end;
        const uint32_t dg = (key[r] >> shift) & mask;
        const uint64_t peers = match_digit(dg, valid, bits);
        const uint32_t pre = s_whist[wave][dg];
        const uint32_t below = (uint32_t)__popcll(peers & lt);
        if (valid && below == 0)
            s_whist[wave][dg] = pre + (uint32_t)__popcll(peers);
        rank[r] = pre + below;
    }
    __syncthreads();

    // per digit: exclusive prefix over the wavefronts, and the tile total
    if ((int)threadIdx.x < nd) {
        uint32_t run = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const uint32_t c = s_whist[w][threadIdx.x];
            s_whist[w][threadIdx.x] = run;
            run += c;
        }
        s_dstart[threadIdx.x] = run;
    }
    __syncthreads();
    // exclusive scan of the (up to 256) digit totals by wavefront 0: 4 digits per lane
    if (wave == 0) {
        uint32_t c[4];
        uint32_t s = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int d = lane * 4 + i;
            c[i] = d < nd ? s_dstart[d] : 0u;
            s += c[i];
        }
        uint32_t incl = s;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const uint32_t up = __shfl_up(incl, o);
            if (lane >= o)
                incl += up;
        }
        uint32_t ex = incl - s;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int d = lane * 4 + i;
            if (d < nd) {
                s_dstart[d] = ex;
                s_goff[d] = hist_scanned[tg.hbase + (int64_t)d * tg.hstride] - ex;
            }
            ex += c[i];
        }
    }
    __syncthreads();

#pragma unroll
    for (int r = 0; r < kSortPerThread; ++r) {
        const int q = base + r * kWave + lane;
        if (q < end) {
            const uint32_t dg = (key[r] >> shift) & mask;
            const uint32_t pos = s_dstart[dg] + s_whist[wave][dg] + rank[r];
            s_keys[pos] = key[r];
            s_vals[pos] = val[r];
        }
    }
    __syncthreads();
    const uint32_t add = LAST ? row_base[tg.t] : 0u;
#pragma unroll
    for (int i = 0; i < kSortPerThread; ++i) {
        const int p = threadIdx.x + i * kSortThreads;
        if (p < tile_cnt) {
            const uint32_t k = s_keys[p];
            const uint32_t g = s_goff[(k >> shift) & mask] + (uint32_t)p;
            keys_out[g] = k + add;
            if (V16 && !LAST)
                reinterpret_cast<uint16_t*>(vals_out)[g] = (uint16_t)s_vals[p];
            else
                vals_out[g] = s_vals[p];
        }
    }
}

// ---------------------------------------------------------------- device-wide exclusive scan (uint32)

__global__ __launch_bounds__(kScanThreads) void scan_reduce_kernel(
    const uint32_t* __restrict__ data, uint32_t* __restrict__ block_sums, int64_t n)
{
    __shared__ uint32_t s_wave[4];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPerThread;
    uint32_t s = 0;
    if (base + kScanPerThread <= n) {
        const uint4* p = reinterpret_cast<const uint4*>(data + base);
#pragma unroll
        for (int i = 0; i < kScanPerThread / 4; ++i) {
            const uint4 v = p[i];
            s += v.x + v.y + v.z + v.w;
        }
    } else {
        for (int i = 0; i < kScanPerThread; ++i)
            if (base + i < n)
                s += data[base + i];
    }
    uint32_t tot;
    (void)block_exclusive_scan_256(s, s_wave, tot);
    if (threadIdx.x == 0)
        block_sums[blockIdx.x] = tot;
}

// single workgroup: exclusive scan of block_sums[nb] in place
__global__ __launch_bounds__(kScanThreads) void scan_top_kernel(uint32_t* __restrict__ block_sums, int32_t nb)
{
    __shared__ uint32_t s_wave[4];
    uint32_t carry = 0;
    for (int base = 0; base < nb; base += kScanThreads) {
        const int i = base + threadIdx.x;
        const uint32_t v = i < nb ? block_sums[i] : 0u;
        uint32_t tot;
        const uint32_t ex = block_exclusive_scan_256(v, s_wave, tot);
        if (i < nb)
            block_sums[i] = carry + ex;
        carry += tot;
    }
}

__global__ __launch_bounds__(kScanThreads) void scan_apply_kernel(
    uint32_t* __restrict__ data, const uint32_t* __restrict__ block_sums, int64_t n)
{
    __shared__ uint32_t s_wave[4];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPerThread;
    uint32_t v[kScanPerThread];
    const bool full = base + kScanPerThread <= n;
    if (full) {
        const uint4* p = reinterpret_cast<const uint4*>(data + base);
#pragma unroll
        for (int i = 0; i < kScanPerThread / 4; ++i) {
            const uint4 x = p[i];
            v[4 * i] = x.x; v[4 * i + 1] = x.y; v[4 * i + 2] = x.z; v[4 * i + 3] = x.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < kScanPerThread; ++i)
            v[i] = base + i < n ? data[base + i] : 0u;
    }
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < kScanPerThread; ++i)
        s += v[i];
    uint32_t tot;
    uint32_t run = block_exclusive_scan_256(s, s_wave, tot) + block_sums[blockIdx.x];
#pragma unroll
    for (int i = 0; i < kScanPerThread; ++i) {
        const uint32_t c = v[i];
        v[i] = run;
        run += c;
    }
    if (full) {
        uint4* p = reinterpret_cast<uint4*>(data + base);
#pragma unroll
        for (int i = 0; i < kScanPerThread / 4; ++i)
            p[i] = make_uint4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
    } else {
#pragma unroll
        for (int i = 0; i < kScanPerThread; ++i)
            if (base + i < n)
                data[base + i] = v[i];
    }
}

// ---------------------------------------------------------------- run-length segmentation (Section 5.1)
//
// A sorted position q is a run head when q == 0 or key[q] != key[q-1].  Pass 1 counts heads per
// tile, a scan turns the counts into the index of each tile's first run, pass 2 writes
// unique_keys / seg_offsets and, for every kSpanUnit-aligned position, the number of heads before it.

__device__ __forceinline__ void rl_load(const uint32_t* __restrict__ keys, int32_t n, int base,
                                        uint32_t (&k)[kRlPerThread], uint32_t& prev)
{
    if (base + kRlPerThread <= n) {
        const uint4* p = reinterpret_cast<const uint4*>(keys + base);
#pragma unroll
        for (int i = 0; i < kRlPerThread / 4; ++i) {
            const uint4 x = p[i];
            k[4 * i] = x.x; k[4 * i + 1] = x.y; k[4 * i + 2] = x.z; k[4 * i + 3] = x.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < kRlPerThread; ++i)
            k[i] = base + i < n ? keys[base + i] : 0u;
    }
    prev = (base > 0 && base < n) ? keys[base - 1] : 0u;
}

__global__ __launch_bounds__(kRlThreads) void runlength_count_kernel(
    const uint32_t* __restrict__ keys, uint32_t* __restrict__ tile_heads, int32_t n)
{
    __shared__ uint32_t s_wave[4];
    const int base = blockIdx.x * kRlTile + threadIdx.x * kRlPerThread;
    uint32_t k[kRlPerThread], prev;
    rl_load(keys, n, base, k, prev);
    uint32_t c = 0;
#pragma unroll
    for (int i = 0; i < kRlPerThread; ++i) {
        const int q = base + i;
        const bool head = q < n && (q == 0 || k[i] != (i == 0 ? prev : k[i - 1]));
        c += head ? 1u : 0u;
    }
    uint32_t tot;
    (void)block_exclusive_scan_256(c, s_wave, tot);
    if (threadIdx.x == 0)
        tile_heads[blockIdx.x] = tot;
}

__global__ __launch_bounds__(kRlThreads) void runlength_write_kernel(
    const uint32_t* __restrict__ keys, const uint32_t* __restrict__ tile_first_run,
    uint32_t* __restrict__ unique_keys, int32_t* __restrict__ seg_offsets,
    int32_t* __restrict__ unit_first_run, Counters* __restrict__ counters, int32_t n)
{
    __shared__ uint32_t s_wave[4];
    const int base = blockIdx.x * kRlTile + threadIdx.x * kRlPerThread;
    uint32_t k[kRlPerThread], prev;
    rl_load(keys, n, base, k, prev);
    bool head[kRlPerThread];
    uint32_t c = 0;
#pragma unroll
    for (int i = 0; i < kRlPerThread; ++i) {
        const int q = base + i;
        head[i] = q < n && (q == 0 || k[i] != (i == 0 ? prev : k[i - 1]));
        c += head[i] ? 1u : 0u;
    }
    uint32_t tot;
    uint32_t r = block_exclusive_scan_256(c, s_wave, tot) + tile_first_run[blockIdx.x];
#pragma unroll
    for (int i = 0; i < kRlPerThread; ++i) {
        const int q = base + i;
        if (q < n) {
            if ((q & (kSpanUnit - 1)) == 0)
                unit_first_run[q / kSpanUnit] = (int32_t)r;
            if (head[i]) {
                unique_keys[r] = k[i];
                seg_offsets[r] = q;
                ++r;
            }
            if (q == n - 1) {
                seg_offsets[r] = n;
                unit_first_run[(n + kSpanUnit - 1) / kSpanUnit] = (int32_t)r;
                counters->num_unique = (int64_t)r;
            }
        }
    }
}

}  // namespace tbe
