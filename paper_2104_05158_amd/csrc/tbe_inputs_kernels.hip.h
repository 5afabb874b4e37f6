// Device kernels of the input-side operations that sit next to the embedding operator
// (arxiv 2104.05158, Section 7.1: combined lengths format, (W,T,B) -> (T,W,B) permute; Section 4
// "Row-wise parallelism" + Section 7.1: bucketize).  gfx950, wave64.
//
// All of it is integer streaming work bound by memory bandwidth: coalesced 4-byte or 16-byte
// accesses, wavefront ballots for ranks, no atomics except integer counters (whose result does not
// depend on their order), so every output is exact and identical run to run.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace tbe_in {

constexpr int kWave = 64;
constexpr int kThreads = 256;
constexpr int kScanGroups = 4;                         // int4 groups per thread
constexpr int kScanTile = kThreads * 4 * kScanGroups;  // 4096 lengths per workgroup
constexpr int kCopyPerThread = 16;
constexpr int kCopyTile = kThreads * kCopyPerThread;   // 4096 index positions per workgroup
constexpr int kMaxShards = 1024;

// ---------------------------------------------------------------- lengths -> offsets (Section 7.1)
//
// Exclusive prefix sum of int32 lengths into int64 offsets, a tile of kScanTile lengths per workgroup.  Inside a
// tile a thread owns one int4 of each of kScanGroups consecutive 1024-length groups, so loads are 16 bytes per lane
// and contiguous across the wavefront.  How a tile gets the sum of the lengths before it goes by the number of tiles:
//   up to kScanSelf     it adds them up itself: one launch (256 lengths: 3.0 us instead of 6.8 in three launches)
//   up to kScanSums     a first launch writes the tiles' totals and every workgroup adds up those before its own
//   more                a single workgroup scans the totals in between (8 M lengths: 27.4 us with that
//                       launch, 26 when every workgroup adds up totals; 12 M: 41 either way; 16 M: 52 and 55)

__device__ __forceinline__ int64_t block_exclusive_scan64(int64_t v, int64_t* s_wave /*[4]*/, int64_t& block_total)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x >> 6;
    int64_t incl = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int64_t up = __shfl_up(incl, o);
        if (lane >= o)
            incl += up;
    }
    if (lane == kWave - 1)
        s_wave[wave] = incl;
    __syncthreads();
    int64_t woff = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kThreads / kWave; ++w) {
        const int64_t c = s_wave[w];
        if (w < wave)
            woff += c;
        tot += c;
    }
    block_total = tot;
    __syncthreads();
    return woff + incl - v;
}

// sum over the workgroup, to all threads (s_wave must not be in use; one barrier)
__device__ __forceinline__ int64_t block_sum64(int64_t v, int64_t* s_wave)
{
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1)
        v += __shfl_xor(v, o);
    if ((threadIdx.x & (kWave - 1)) == 0)
        s_wave[threadIdx.x >> 6] = v;
    __syncthreads();
    int64_t tot = 0;
#pragma unroll
    for (int w = 0; w < kThreads / kWave; ++w)
        tot += s_wave[w];
    return tot;
}

// Inclusive sums over the wavefront of kScanGroups values at once, each below 2^25 in every lane if `small`: then a
// 32-bit scan by data-parallel moves does, otherwise 64-bit shuffles.
__device__ __forceinline__ void wave_scan_groups(int64_t (&v)[kScanGroups], bool small)
{
    const int lane = threadIdx.x & (kWave - 1);
    if (small) {
#pragma unroll
        for (int g = 0; g < kScanGroups; ++g) {
            int x = (int)v[g];
            x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr 1, 2, 4, 8
            x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
            x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
            x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
            x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast 15, 31
            x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
            v[g] = (int64_t)x;
        }
        return;
    }
#pragma unroll
    for (int g = 0; g < kScanGroups; ++g) {
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int64_t up = __shfl_up(v[g], o);
            if (lane >= o)
                v[g] += up;
        }
    }
}

__device__ __forceinline__ int4 load_lengths4(const int32_t* __restrict__ lengths, int64_t i, int64_t n)
{
    if (i + 4 <= n)
        return *reinterpret_cast<const int4*>(lengths + i);
    int4 v = make_int4(0, 0, 0, 0);
    if (i < n) v.x = lengths[i];
    if (i + 1 < n) v.y = lengths[i + 1];
    if (i + 2 < n) v.z = lengths[i + 2];
    return v;
}

__global__ __launch_bounds__(kThreads) void scan64_reduce_kernel(const int32_t* __restrict__ lengths,
                                                                 int64_t* __restrict__ block_sums, int64_t n)
{
    __shared__ int64_t s_wave[kThreads / kWave];
    const int64_t tile = (int64_t)blockIdx.x * kScanTile;
    int64_t s = 0;
#pragma unroll
    for (int g = 0; g < kScanGroups; ++g) {
        const int4 v = load_lengths4(lengths, tile + g * (kThreads * 4) + threadIdx.x * 4, n);
        s += (int64_t)v.x + v.y + v.z + v.w;
    }
    int64_t tot;
    (void)block_exclusive_scan64(s, s_wave, tot);
    if (threadIdx.x == 0)
        block_sums[blockIdx.x] = tot;
}

// one workgroup: exclusive scan of block_sums[nb] in place, kTopPerThread consecutive sums per thread
constexpr int kTopPerThread = 8;
__global__ __launch_bounds__(kThreads) void scan64_top_kernel(int64_t* __restrict__ block_sums, int32_t nb)
{
    __shared__ int64_t s_wave[kThreads / kWave];
    int64_t carry = 0;
    for (int base = 0; base < nb; base += kThreads * kTopPerThread) {
        const int i0 = base + threadIdx.x * kTopPerThread;
        int64_t v[kTopPerThread];
        int64_t s = 0;
#pragma unroll
        for (int k = 0; k < kTopPerThread; ++k) {
            v[k] = i0 + k < nb ? block_sums[i0 + k] : 0;
            s += v[k];
        }
        int64_t tot;
        int64_t run = carry + block_exclusive_scan64(s, s_wave, tot);
#pragma unroll
        for (int k = 0; k < kTopPerThread; ++k) {
            if (i0 + k < nb)
                block_sums[i0 + k] = run;
            run += v[k];
        }
        carry += tot;
    }
}

constexpr int kScanSelf = 8;
constexpr int kScanSums = 3072;
enum { kBeforeSelf = 0, kBeforeSums = 1, kBeforePrefix = 2 };   // where the sum of the lengths before a tile comes from

template <int BEFORE>
__global__ __launch_bounds__(kThreads) void scan64_apply_kernel(const int32_t* __restrict__ lengths,
                                                                const int64_t* __restrict__ block_sums,
                                                                int64_t* __restrict__ offsets, int64_t n)
{
    constexpr int kWaves = kThreads / kWave;
    __shared__ int64_t s_wave[kWaves], s_tot[kScanGroups][kWaves];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const int64_t tile = (int64_t)blockIdx.x * kScanTile;
    int4 v[kScanGroups];
    int64_t s[kScanGroups], incl[kScanGroups];
    int most = 0;
#pragma unroll
    for (int g = 0; g < kScanGroups; ++g)
        v[g] = load_lengths4(lengths, tile + g * (kThreads * 4) + threadIdx.x * 4, n);
    int64_t before = 0;
    if (BEFORE == kBeforePrefix) {
        before = block_sums[blockIdx.x];
    } else {
        if (BEFORE == kBeforeSelf) {
            for (int64_t i = threadIdx.x * 4; i < tile; i += kThreads * 4) {     // whole tiles: no ragged end
                const int4 x = *reinterpret_cast<const int4*>(lengths + i);
                before += (int64_t)x.x + x.y + x.z + x.w;
            }
        } else {
            for (int i = threadIdx.x; i < (int)blockIdx.x; i += kThreads)
                before += block_sums[i];
        }
        before = block_sum64(before, s_wave);
    }
#pragma unroll
    for (int g = 0; g < kScanGroups; ++g) {
        s[g] = incl[g] = (int64_t)v[g].x + v[g].y + v[g].z + v[g].w;
        most = max(max(most, v[g].x), max(v[g].y, max(v[g].z, v[g].w)));
    }
    wave_scan_groups(incl, __ballot(most >= (1 << 23)) == 0ull);
    if (lane == kWave - 1) {
#pragma unroll
        for (int g = 0; g < kScanGroups; ++g)
            s_tot[g][wave] = incl[g];
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < kScanGroups; ++g) {
        int64_t o0 = before + incl[g] - s[g];
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const int64_t c = s_tot[g][w];
            o0 += w < wave ? c : 0;
            before += c;
        }
        const int64_t i = tile + g * (kThreads * 4) + threadIdx.x * 4;
        const int64_t o1 = o0 + v[g].x, o2 = o1 + v[g].y, o3 = o2 + v[g].z, o4 = o3 + v[g].w;
        if (i + 4 <= n) {
            // offsets + i is 32-byte aligned (i is a multiple of 4)
            *reinterpret_cast<longlong2*>(offsets + i) = make_longlong2(o0, o1);
            *reinterpret_cast<longlong2*>(offsets + i + 2) = make_longlong2(o2, o3);
            if (i + 4 == n)
                offsets[n] = o4;
        } else if (i < n) {
            offsets[i] = o0;
            if (i + 1 < n) offsets[i + 1] = o1; else offsets[n] = o1;
            if (i + 2 < n) offsets[i + 2] = o2; else if (i + 2 == n) offsets[n] = o2;
            if (i + 3 == n) offsets[n] = o3;
        }
    }
}

__global__ void write_zero_offset_kernel(int64_t* __restrict__ offsets) { offsets[0] = 0; }

// ---------------------------------------------------------------- (W,T,B) -> (T,W,B) permute (Section 7.1)
//
// Bags (w,t,0..B-1) are consecutive on both sides, so the lengths move in rows of B and the indices
// move as W*T contiguous blocks whose borders are offsets[q*B].  The blocks of the input have the same sizes, so
// their starts follow from the output's offsets alone and the input's bags need no prefix sum of their own.

// One tile of kScanTile bags of the output per workgroup: moves their lengths and writes the tile's total.
// VEC = 4 (16-byte accesses) needs B % 4 == 0.
template <int VEC>
__global__ __launch_bounds__(kThreads) void permute_lengths_kernel(const int32_t* __restrict__ lengths_in,
                                                                   int32_t* __restrict__ lengths_out,
                                                                   int64_t* __restrict__ block_sums, int32_t W,
                                                                   int32_t T, int32_t B, int32_t n)
{
    __shared__ int64_t s_wave[kThreads / kWave];
    constexpr int kSteps = kScanTile / (kThreads * VEC);
    const int64_t tile = (int64_t)blockIdx.x * kScanTile;
    int64_t sum = 0;
#pragma unroll
    for (int k = 0; k < kSteps; ++k) {
        const int64_t i = tile + (int64_t)(k * kThreads + (int)threadIdx.x) * VEC;
        if (i >= n)
            continue;
        const int q = (int)i / B, b = (int)i - q * B;
        const int t = q / W, w = q - t * W;
        const int64_t src = ((int64_t)w * T + t) * B + b;
        if (VEC == 4) {
            const int4 v = *reinterpret_cast<const int4*>(lengths_in + src);
            *reinterpret_cast<int4*>(lengths_out + i) = v;
            sum += (int64_t)v.x + v.y + v.z + v.w;
        } else {
            const int32_t v = lengths_in[src];
            lengths_out[i] = v;
            sum += v;
        }
    }
    sum = block_sum64(sum, s_wave);
    if (threadIdx.x == 0)
        block_sums[blockIdx.x] = sum;
}

// one workgroup: first position of every input block (input order (w, t)), from the output's offsets
__global__ __launch_bounds__(kThreads) void permute_starts_kernel(const int64_t* __restrict__ offsets_out,
                                                                  int64_t* __restrict__ starts, int32_t W, int32_t T, int32_t B)
{
    __shared__ int64_t s_wave[kThreads / kWave];
    int64_t carry = 0;
    for (int base = 0; base < W * T; base += kThreads) {
        const int p = base + threadIdx.x;
        int64_t size = 0;
        if (p < W * T) {
            const int64_t q = (int64_t)(p % T) * W + p / T;
            size = offsets_out[(q + 1) * B] - offsets_out[q * B];
        }
        int64_t tot;
        const int64_t ex = block_exclusive_scan64(size, s_wave, tot);
        if (p < W * T)
            starts[p] = carry + ex;
        carry += tot;
    }
}

// the same for many blocks: their sizes, in input order, for the prefix sum of lengths
__global__ __launch_bounds__(kThreads) void permute_sizes_kernel(const int64_t* __restrict__ offsets_out,
                                                                 int32_t* __restrict__ sizes, int32_t W, int32_t T, int32_t B)
{
    const int p = (int)blockIdx.x * kThreads + (int)threadIdx.x;
    if (p >= W * T)
        return;
    const int64_t q = (int64_t)(p % T) * W + p / T;
    sizes[p] = (int32_t)(offsets_out[(q + 1) * B] - offsets_out[q * B]);
}

// last q in [lo, hi] with offsets[q*B] <= p   (offsets[lo*B] <= p is given)
__device__ __forceinline__ int find_block(const int64_t* __restrict__ offsets, int64_t B, int lo, int hi, int64_t p)
{
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (offsets[(int64_t)mid * B] <= p)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// the same among all `rows` blocks for a whole wavefront: 64 borders per step
__device__ __forceinline__ int find_block_wave(const int64_t* __restrict__ offsets, int64_t B, int rows, int64_t p)
{
    const int lane = threadIdx.x & (kWave - 1);
    int lo = 0, n = rows;
    while (n > 1) {
        const int step = (n + kWave - 1) / kWave;
        const int i = lane * step;
        const uint64_t le = __ballot(i < n && offsets[(int64_t)(lo + min(i, n - 1)) * B] <= p);
        const int k = (__popcll(le) - 1) * step;
        lo += k;
        n = min(step, n - k);
    }
    return lo;
}

// Every workgroup copies kCopyTile consecutive OUTPUT positions.  The output rows the tile touches
// are bracketed once per workgroup; when they are few (the usual case: a row holds B bags) their
// borders and source shifts are staged in LDS, so a position costs a short LDS search, one load and
// one store, all loads of a thread issued before its stores.  starts: first position of every input block, or null
// (at most kCopyLdsRows rows): then the workgroup sums the sizes of the blocks before each of its rows itself.
constexpr int kCopyLdsRows = 256;
__global__ __launch_bounds__(kThreads) void permute_indices_kernel(const int32_t* __restrict__ indices_in,
                                                                   const int64_t* __restrict__ starts,
                                                                   const int64_t* __restrict__ offsets_out,
                                                                   int32_t* __restrict__ indices_out, int32_t W,
                                                                   int32_t T, int32_t B, int64_t n)
{
    __shared__ int s_q[2];
    __shared__ int64_t s_wave[2][kThreads / kWave];
    __shared__ int64_t s_start[kCopyLdsRows];   // first output position of row q_lo + i
    __shared__ int64_t s_shift[kCopyLdsRows];   // source position minus output position inside that row
    const int64_t tile = (int64_t)blockIdx.x * kCopyTile;
    const int64_t tile_end = min(tile + kCopyTile, n);
    const int rows = W * T;
    if (threadIdx.x < 2 * kWave) {
        const int q = find_block_wave(offsets_out, B, rows, threadIdx.x < kWave ? tile : tile_end - 1);
        if ((threadIdx.x & (kWave - 1)) == 0)
            s_q[threadIdx.x >> 6] = q;
    }
    __syncthreads();
    const int q_lo = s_q[0], q_hi = s_q[1];
    const int nrows = q_hi - q_lo + 1;
    const bool staged = nrows <= kCopyLdsRows;
    if (starts != nullptr) {
        if (staged && (int)threadIdx.x < nrows) {
            const int q = q_lo + threadIdx.x;
            const int t = q / W;
            const int w = q - t * W;
            const int64_t start = offsets_out[(int64_t)q * B];
            s_start[threadIdx.x] = start;
            s_shift[threadIdx.x] = starts[(int64_t)w * T + t] - start;
        }
    } else {
        for (int q = q_lo; q <= q_hi; ++q) {
            const int t = q / W;
            const int w = q - t * W;
            int64_t sum = 0;
            for (int p = threadIdx.x; p < w * T + t; p += kThreads) {
                const int64_t o = (int64_t)(p % T) * W + p / T;
                sum += offsets_out[(o + 1) * B] - offsets_out[o * B];
            }
            sum = block_sum64(sum, s_wave[q & 1]);
            if (threadIdx.x == 0) {
                const int64_t start = offsets_out[(int64_t)q * B];
                s_start[q - q_lo] = start;
                s_shift[q - q_lo] = sum - start;
            }
        }
    }
    __syncthreads();
    int64_t src[kCopyPerThread];
#pragma unroll
    for (int i = 0; i < kCopyPerThread; ++i) {
        const int64_t p = min(tile + i * kThreads + threadIdx.x, tile_end - 1);
        if (staged) {
            int lo = 0, hi = nrows - 1;   // last row with s_start <= p
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (s_start[mid] <= p)
                    lo = mid;
                else
                    hi = mid - 1;
            }
            src[i] = p + s_shift[lo];
        } else {
            const int q = find_block(offsets_out, B, q_lo, q_hi, p);
            const int t = q / W;
            const int w = q - t * W;
            src[i] = starts[(int64_t)w * T + t] + (p - offsets_out[(int64_t)q * B]);
        }
    }
    int32_t v[kCopyPerThread];
#pragma unroll
    for (int i = 0; i < kCopyPerThread; ++i)
        v[i] = indices_in[src[i]];
#pragma unroll
    for (int i = 0; i < kCopyPerThread; ++i) {
        const int64_t p = tile + i * kThreads + threadIdx.x;
        if (p < tile_end)
            indices_out[p] = v[i];
    }
}

// ---------------------------------------------------------------- row-wise bucketize (Section 4, Section 7.1)
//
// Shard w of table t owns rows [w*blk_t, (w+1)*blk_t), blk_t = ceil(H_t / W).  The output order
// (w, t, b), with the input order kept inside every bag, makes the region of shard w a STABLE
// FILTER of the input stream: the elements of shard w, in input order.  So bucketize is one stable
// multi-way split of the index stream by shard, plus per-(shard, bag) counts:
//
//   pass 1 (count):  a workgroup owns `nbags` consecutive bags of ONE table, walks their positions and counts
//                    (shard, bag) pairs with integer LDS atomics; the counts go out as rows of lengths_out
//                    (consecutive b for each shard).
//   prefix sum:      lengths_out -> offsets_out (the scan kernels above).
//   pass 2 (place):  the same bags per workgroup.  offsets_out at the workgroup's first bag is,
//                    for every shard, exactly where the workgroup's elements of that shard start.
//                    Positions are handled in sub-tiles: ballot-matched stable ranks per wavefront,
//                    prefix over wavefronts and shards in LDS, the sub-tile is reordered by shard
//                    inside LDS and written out in contiguous runs.
//
// Both passes are bound by vector instructions (one per element is 0.8 us at 31 M indices), not by their bytes.  One
// table per workgroup leaves one divisor, as a multiplication by its reciprocal, and pass 2 needs no bag at all (a
// workgroup of bags of any table looked every element's bag up in LDS to find its divisor); the number of shard bits
// is a template parameter.  64 tables x 16384 bags x 30 over 8 shards: 233 -> 135 us for the call, count 35
// (65 with 4-byte loads and without the border read ahead) and place 60 of it: 4.1 TB/s, what a copy reaches here.

// floor(r / blk) for r < 2^31, exactly: r * mul / 2^(31 + l) with mul = floor(2^(31 + l) / blk) + 1, l = ceil(log2 blk)
// (mul * blk exceeds 2^(31 + l) by at most blk <= 2^l).  Invalid rows may give a wrong value; callers clamp.
struct ShardSize {
    uint32_t blk;    // rows per shard
    uint32_t mul;
    int32_t sh;      // l - 1; < 0: blk is 1
    __device__ __forceinline__ ShardSize(int64_t rows, int32_t W)
    {
        blk = max(1u, (uint32_t)((rows + W - 1) / W));
        const int l = blk == 1u ? 0 : 32 - __clz((int)(blk - 1u));
        const uint64_t one = 1ull << (31 + l);
        uint64_t q = (uint64_t)((double)one / (double)blk);      // off by at most one, upwards
        q -= q * blk > one ? 1u : 0u;
        mul = (uint32_t)q + 1u;
        sh = l - 1;
    }
    __device__ __forceinline__ uint32_t shard(uint32_t r, uint32_t last) const
    {
        const uint32_t q = sh < 0 ? r : __umulhi(r, mul) >> sh;
        return min(q, last);
    }
};

constexpr int kBuckMaxBags = 256;   // bags per workgroup (fewer when W is large: nbags * W <= 8192)
constexpr int kBuckCount = 8;       // consecutive positions per thread of the counting pass
constexpr int kBuckPerThread = 8;
constexpr int kBuckTile = kThreads * kBuckPerThread;  // 2048 positions per sub-tile

// last a in [0, nb) with off[a] <= p; nb <= 256: eight branch-free halvings
__device__ __forceinline__ int find_bag(const int32_t* off, int nb, int p)
{
    int a = 0, c = nb;
#pragma unroll
    for (int step = 0; step < 8; ++step) {
        const int mid = (a + c) >> 1;
        const bool up = off[mid] <= p;       // mid == a once c - a <= 1: then a stays
        a = up ? mid : a;
        c = up ? c : max(mid, a + 1);
    }
    return a;
}

// four words at any 4-byte aligned address (one 16-byte load)
struct __attribute__((packed, aligned(4))) Words4 {
    uint32_t x, y, z, w;
};

// work items: T * per_table, per_table = ceil(B / nbags), nbags = 1 << lg_nbags; dynamic LDS: W * nbags counters
__global__ __launch_bounds__(kThreads) void bucketize_count_kernel(const int64_t* __restrict__ rows,
                                                                   const int32_t* __restrict__ indices,
                                                                   const int64_t* __restrict__ offsets,
                                                                   int32_t* __restrict__ lengths_out, int32_t T,
                                                                   int32_t B, int32_t W, int32_t lg_nbags,
                                                                   int32_t per_table, int32_t num_items)
{
    __shared__ int32_t s_off[kBuckMaxBags + 2];     // (the last one is read ahead, never used)
    extern __shared__ int32_t s_cnt[];  // [W][nbags]
    const int nbags = 1 << lg_nbags;
    for (uint32_t item = blockIdx.x; item < (uint32_t)num_items; item += gridDim.x) {
        const int t = (int)(item / (uint32_t)per_table);
        const int b0 = ((int)item - t * per_table) << lg_nbags;
        const int nb = min(nbags, B - b0);
        const int64_t* off = offsets + ((int64_t)t * B + b0);
        const int64_t base = off[0];
        const ShardSize size(rows[t], W);
        for (int i = threadIdx.x; i < W << lg_nbags; i += kThreads)
            s_cnt[i] = 0;
        for (int i = threadIdx.x; i <= nb; i += kThreads)
            s_off[i] = (int32_t)(off[i] - base);
        __syncthreads();
        const int total = s_off[nb];
        const uint32_t last = (uint32_t)(W - 1);
        // Counting does not depend on the order, so a thread takes kBuckCount CONSECUTIVE positions: one bag
        // search for the first of them, then it only steps over the bag borders it meets (the border after the next
        // one is on its way meanwhile: some lane steps at nearly every position).
        for (int p0 = threadIdx.x * kBuckCount; p0 < total; p0 += kThreads * kBuckCount) {
            uint32_t r[kBuckCount];
            if (p0 + kBuckCount <= total) {
#pragma unroll
                for (int u = 0; u < kBuckCount; u += 4) {
                    const Words4 v = *reinterpret_cast<const Words4*>(indices + base + p0 + u);
                    r[u] = v.x, r[u + 1] = v.y, r[u + 2] = v.z, r[u + 3] = v.w;
                }
            } else {
#pragma unroll
                for (int u = 0; u < kBuckCount; ++u)
                    r[u] = (uint32_t)indices[base + min(p0 + u, total - 1)];
            }
            int a = find_bag(s_off, nb, p0);
            int next = s_off[a + 1], next2 = s_off[a + 2];
#pragma unroll
            for (int u = 0; u < kBuckCount; ++u) {
                const int p = p0 + u;
                if (p < total) {
                    while (p >= next && a + 1 < nb) {   // p < total = off[nb]: a stays below nb even for bad offsets
                        ++a;
                        next = next2;
                        next2 = s_off[a + 2];
                    }
                    atomicAdd(&s_cnt[(size.shard(r[u], last) << lg_nbags) + a], 1);
                }
            }
        }
        __syncthreads();
        for (int i = threadIdx.x; i < W << lg_nbags; i += kThreads) {
            const int w = i >> lg_nbags;
            const int a = i & (nbags - 1);
            if (a < nb)
                lengths_out[((int64_t)w * T + t) * B + (b0 + a)] = s_cnt[i];
        }
        __syncthreads();
    }
}

// BITS: W <= 1 << BITS
template <int BITS>
__global__ __launch_bounds__(kThreads) void bucketize_place_kernel(const int64_t* __restrict__ rows,
                                                                   const int32_t* __restrict__ indices,
                                                                   const int64_t* __restrict__ offsets,
                                                                   const int64_t* __restrict__ offsets_out,
                                                                   int32_t* __restrict__ indices_out, int32_t T,
                                                                   int32_t B, int32_t W, int32_t nbags,
                                                                   int32_t per_table, int32_t num_items)
{
    constexpr int kShards = 1 << BITS;
    constexpr int kWaves = kThreads / kWave;
    constexpr int kScanThreads = kShards <= kWave ? kWave : kThreads;           // threads of the prefix over the shards
    constexpr int kDpt = (kShards + kScanThreads - 1) / kScanThreads;           // shards per thread there
    using Digit = typename std::conditional<BITS <= 8, uint8_t, uint16_t>::type;
    __shared__ uint32_t s_slot[kWaves][kShards];   // counts of a wavefront, then the slot of its first element
    __shared__ int32_t s_goff[kShards];            // output position of slot 0 of the shard, minus the slot
    __shared__ int32_t s_next[kShards];            // output position of the shard's next element
    __shared__ int32_t s_val[kBuckTile];
    __shared__ Digit s_dig[kBuckTile];
    __shared__ uint32_t s_wave[kWaves];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x >> 6;
    for (uint32_t item = blockIdx.x; item < (uint32_t)num_items; item += gridDim.x) {
        const int t = (int)(item / (uint32_t)per_table);
        const int b0 = ((int)item - t * per_table) * nbags;
        const int64_t j0 = (int64_t)t * B + b0;
        const int64_t base = offsets[j0];
        const int total = (int)(offsets[j0 + min(nbags, B - b0)] - base);
        const int32_t* __restrict__ in = indices + base;
        const ShardSize size(rows[t], W);
        const uint32_t last = (uint32_t)(W - 1);
        // (s_next is written and read by the same threads, those of the prefix below)
        if (threadIdx.x < kScanThreads)
#pragma unroll
            for (int i = 0; i < kDpt; ++i) {
                const int d = threadIdx.x * kDpt + i;
                if (d < W)
                    s_next[d] = (int32_t)offsets_out[((int64_t)d * T + t) * B + b0];
            }

        for (int tile0 = 0; tile0 < total; tile0 += kBuckTile) {
            const int tile_cnt = min(kBuckTile, total - tile0);
            // order inside the sub-tile: (wavefront, round, lane) = ascending position
            const int wbase = tile0 + wave * (kBuckTile / kWaves);
            uint32_t r[kBuckPerThread];
#pragma unroll
            for (int k = 0; k < kBuckPerThread; ++k)
                r[k] = (uint32_t)in[min(wbase + k * kWave + lane, total - 1)];
            for (int i = lane; i < kShards; i += kWave)
                s_slot[wave][i] = 0;
            uint32_t dig[kBuckPerThread], rank[kBuckPerThread];
#pragma unroll
            for (int k = 0; k < kBuckPerThread; ++k) {
                const bool valid = wbase + k * kWave + lane < total;
                const uint32_t w = size.shard(r[k], last);
                dig[k] = w;
                // lanes of the same shard: one ballot per bit, lanes whose bit differs drop out
                const uint64_t alive = __ballot(valid);
                uint32_t lo = (uint32_t)alive, hi = (uint32_t)(alive >> 32);
#pragma unroll
                for (int b = 0; b < BITS; ++b) {
                    const int32_t mk = (int32_t)(w << (31 - b)) >> 31;
                    const uint64_t bal = __ballot(mk != 0);
                    lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)bal, (uint32_t)mk, 0x90);
                    hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(bal >> 32), (uint32_t)mk, 0x90);
                }
                const uint32_t below = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
                rank[k] = s_slot[wave][w] + below;       // LDS operations of a wavefront execute in order
                if (valid && below == 0)
                    atomicAdd(&s_slot[wave][w], (uint32_t)(__popc(lo) + __popc(hi)));
            }
            __syncthreads();

            // exclusive prefix of the counts over shards and, inside a shard, over wavefronts
            uint32_t tot[kDpt], mine = 0, incl = 0;
            if (threadIdx.x < kScanThreads) {
#pragma unroll
                for (int i = 0; i < kDpt; ++i) {
                    const int d = threadIdx.x * kDpt + i;
                    tot[i] = 0;
                    if (d < W)
#pragma unroll
                        for (int w = 0; w < kWaves; ++w)
                            tot[i] += s_slot[w][d];
                    mine += tot[i];
                }
                incl = mine;
#pragma unroll
                for (int o = 1; o < kWave && o < kShards; o <<= 1) {
                    const uint32_t up = __shfl_up(incl, o);
                    if (lane >= o)
                        incl += up;
                }
            }
            uint32_t ex = incl - mine;
            if constexpr (kScanThreads > kWave) {
                if (lane == kWave - 1)
                    s_wave[wave] = incl;
                __syncthreads();
                for (int w = 0; w < wave; ++w)
                    ex += s_wave[w];
            }
            if (threadIdx.x < kScanThreads) {
#pragma unroll
                for (int i = 0; i < kDpt; ++i) {
                    const int d = threadIdx.x * kDpt + i;
                    if (d < W) {
                        const int32_t nxt = s_next[d];
                        s_goff[d] = nxt - (int32_t)ex;
                        s_next[d] = nxt + (int32_t)tot[i];
#pragma unroll
                        for (int w = 0; w < kWaves; ++w) {
                            const uint32_t c = s_slot[w][d];
                            s_slot[w][d] = ex;
                            ex += c;
                        }
                    }
                }
            }
            __syncthreads();

#pragma unroll
            for (int k = 0; k < kBuckPerThread; ++k) {
                if (wbase + k * kWave + lane < total) {
                    const uint32_t pos = s_slot[wave][dig[k]] + rank[k];
                    s_val[pos] = (int32_t)(r[k] - dig[k] * size.blk);
                    s_dig[pos] = (Digit)dig[k];
                }
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < kBuckPerThread; ++k) {
                const int q = threadIdx.x + k * kThreads;
                if (q < tile_cnt)
                    indices_out[s_goff[s_dig[q]] + q] = s_val[q];
            }
        }
    }
}

}  // namespace tbe_in
