// Sort by (table, row) and run-length segmentation of a batch's lookups (Section 5.1 of arxiv 2104.05158,
// "gradient sorting by rows"), for gfx950.
//
// The input is table-major, so the lookups of a table already occupy one contiguous range of positions: only the
// row index has to be sorted, table by table.  Every table is partitioned once into buckets that fit a workgroup's
// LDS, and every bucket is sorted there -- the lookups cross HBM twice, whatever the number of index bits, where a
// digit-by-digit radix sort crosses it once per eight bits and once more for the run lengths.  That holds up to about 6 M
// lookups in a table; the buckets of a taller one exceed a tile and take the digits through memory one bucket per workgroup.
// (use_radix_sort in tbe_rules.h names the calls that are better off with the radix sort of tbe_radix_kernels.hip.h.)
//
//   sort_plan_kernel     one workgroup per table: sorts a sample of its indices and picks the borders of its
//                        buckets so that a bucket holds about `target` lookups whatever their distribution.  A row
//                        that is looked up more often than that gets a bucket of its own, which needs no sorting.
//   sort_hist_kernel     lookups per bucket and chunk (a chunk is a few tiles of kSortTile positions)
//   sort_columns_kernel  positions of every chunk inside its buckets, lookups of every bucket
//   sort_units_kernel    bucket starts and work units
//   sort_scatter_kernel  stable partition: a lookup becomes one word, (row - first row of the bucket) and bag
//                        number packed in 32 bits
//   sort_local_kernel    one workgroup per unit: sorts the words in LDS, writes keys and payloads, counts the runs
//   sort_runs_kernel     bucket borders are run borders, so a unit's runs start at a known index: unique_keys,
//                        seg_offsets, and the first run of every span unit
// A call of up to 8 M lookups in words of 32 bits leaves out histogram, columns and units: its chunks are put in order of
// their buckets where they lie, and a unit collects its piece of each (use_pieces_sort).  One of up to 2^18, and few a table,
// leaves out the partition, too: sort_select_kernel sorts units that it finds itself (use_select_sort).  One of at most
// kSortTile lookups is sorted by (table, row) at once, by one workgroup (sort_small_kernel).
//
// (The runs' first index could also come from a look-back over the units' counts inside sort_local_kernel; at
// 38,000 units its polling took 6 ms where the extra kernel takes 0.2.)
//
// The word is 32 bits while the rows of every table can be cut into at most kMaxRangeCuts ranges whose row offset
// and bag number fit 32 bits (always for batch <= 65536 and tables below 2^25 rows); otherwise 64 bits.
//
// Stability (equal rows keep the order of their bags) comes from ranks formed by ballots in position order; nothing
// depends on scheduling: the artefacts are bit-identical run to run.
#pragma once

#include <type_traits>

#include "tbe_kernels.hip.h"

namespace tbe {

constexpr int kSortThreads = 512;                 // 8 wavefronts
constexpr int kSortWaves = kSortThreads / kWave;
constexpr int kSortPerThread = 16;
constexpr int kSortTile = kSortThreads * kSortPerThread;   // 8192 words: what a workgroup sorts in LDS
static_assert(kSamplesMax <= kSortTile, "one workgroup sorts a table's samples");
constexpr int kMaxBuckets = 1024;                 // per table
constexpr int kMaxRangeCuts = 512;                // of those, bucket borders at multiples of the packed key range
constexpr int kLutBits = 12;
constexpr int kLutSize = (1 << kLutBits) + 8;
constexpr int kLocalDigits = 256;
constexpr int kUnitsThreads = 1024;
constexpr int kColThreads = 1024;                 // 16 wavefronts that share the chunks of a table ...
constexpr int kColBuckets = kWave;                // ... for 64 of its buckets ...
constexpr int kColAhead = 16;                     // ... and read this many at a time
constexpr int kColChunks = 32;                    // a table of no more chunks needs no such workgroups

struct SortTable {       // 32 bytes
    int32_t start, n;    // first position, lookups
    int32_t chunk_base;  // first chunk
    int32_t nchunks;
    int32_t nb;          // buckets (0: no lookups)
    int16_t lut_shift;   // of its lookup table
    int16_t lut_span;    // most borders inside a cell
    int32_t part;        // index of its border / lookup tables
    int32_t pad;
};

struct SortChunk {       // 16 bytes
    int32_t t, first, cnt, pad;
};

struct SortUnit {        // 32 bytes
    int32_t start, m;    // positions
    uint32_t key0;       // linear row id that row offset 0 stands for
    int32_t bits;        // bits of the row offsets to sort
    uint16_t t, bucket;  // (bucket: pieces)
    int32_t flags;       // kUnit...; select: the part's number in the bits from 8 on; pieces: there, and the last's from 20 on
    int32_t first;       // the table's first unit (they are numbered one after the other)
    uint32_t last;       // select: offset of the unit's last row from key0 (of the last unit: of any index); pieces: the table's first chunk
};
static_assert(kPiecesChunk == kSortTile, "sort_scatter_kernel<.., true> orders one tile");
static_assert(sizeof(SortUnit) == 32 && kManyTables <= 65536, "");
constexpr int kUnitContinued = 1;     // further part of a one-row bucket: its first lookup starts no run
constexpr int kUnitNone = 2;          // (select, pieces) no bucket; until the unit is sorted its start and m are those of the table
constexpr int kUnitMore = 4;          // (select) further parts follow

// How the lookups come to their units: by a partition with known places (histogram, units, scatter), every unit finding its
// own among all of the table's (use_select_sort), or every chunk sorted by bucket where it lies and the units collecting
// their piece of each (use_pieces_sort).
enum SortMode { kSortPartition, kSortSelect, kSortPieces };
constexpr int kPieceStarts = kMaxBuckets + 8;     // first positions of the buckets in a chunk, as many words of 16 bits

struct SortArgs {
    const int64_t* offsets;
    const uint32_t* indices;
    const TableMeta* meta;
    const uint32_t* row_base;
    SortTable* tables;       // [T]
    SortChunk* chunks;
    SortUnit* units;
    uint32_t* split;         // [parts][kMaxBuckets] first row of every bucket
    uint16_t* lut;           // [parts][kLutSize] bucket of the first row of every cell of rows (and of the row past the last)
    uint32_t* bstart;        // [parts][kMaxBuckets] lookups, then first position of every bucket
    uint32_t* hist;          // [chunks][kMaxBuckets]; pieces: [chunks][kPieceStarts], as uint16_t (piece_starts)
    int32_t* multi;          // tables of more than col_chunks chunks
    int32_t* tile_bag;       // [chunks * tiles_per_chunk] bag of the first position of every tile
    uint32_t* unit_runs;     // [slots] runs of every unit
    uint32_t* table_runs;    // [T]
    int32_t* tstart;         // [T + 1]
    Counters* counters;
    void* words[2];          // words, and the second buffer of units larger than a tile
    uint32_t* keys;
    int32_t* vals;
    uint32_t* unique_keys;
    int32_t* seg_offsets;
    int32_t* unit_first_run;
    uint32_t* small_long;    // indices of a small call's runs of more than kPosPiece lookups, their number in front
    int32_t n, B, T;
    int32_t vb;              // bits of the bag number in a word
    int32_t kb;              // bits left for the row offset
    int32_t target;          // lookups per bucket
    int32_t lg_chunk;        // (pieces: a chunk is a power of two)
    int32_t chunk;           // positions of a chunk: tiles_per_chunk tiles, or in a small call less than one
    int32_t tiles_per_chunk;
    int32_t col_chunks;      // chunks of a table up to which sort_units_kernel adds them up itself
    int32_t mode;            // SortMode
};
// A launch's arguments are new to the caches, and a kernel of a few us waits for every line of them: with 260 bytes here and
// the learning rate of the update behind its first 256, a step of 256 bags of 8 took 17.31 us; within 256 both, 17.09.
static_assert(sizeof(SortArgs) + sizeof(int) <= 256, "with the one-workgroup sort's key_bits");

// first positions of the buckets in a chunk
__device__ __forceinline__ uint16_t* piece_starts(const SortArgs& a, int chunk)
{
    return reinterpret_cast<uint16_t*>(a.hist) + (int64_t)chunk * kPieceStarts;
}

// ---------------------------------------------------------------- wavefront and workgroup primitives

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp0(uint32_t v)     // lanes without a source get 0
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xf, false);
}

__device__ __forceinline__ uint32_t wave_scan_add(uint32_t v)   // inclusive
{
    v += dpp0<0x111, 0xf>(v);
    v += dpp0<0x112, 0xf>(v);
    v += dpp0<0x114, 0xf>(v);
    v += dpp0<0x118, 0xf>(v);
    v += dpp0<0x142, 0xa>(v);
    v += dpp0<0x143, 0xc>(v);
    return v;
}

template <int N>
__device__ __forceinline__ uint32_t first_lanes_scan_add(uint32_t v)   // inclusive, over the first N lanes
{
    static_assert(N == 8, "");
    v += dpp0<0x111, 0xf>(v);
    v += dpp0<0x112, 0xf>(v);
    v += dpp0<0x114, 0xf>(v);
    return v;
}

__device__ __forceinline__ uint32_t wave_scan_max(uint32_t v)   // inclusive
{
    v = max(v, dpp0<0x111, 0xf>(v));
    v = max(v, dpp0<0x112, 0xf>(v));
    v = max(v, dpp0<0x114, 0xf>(v));
    v = max(v, dpp0<0x118, 0xf>(v));
    v = max(v, dpp0<0x142, 0xa>(v));
    v = max(v, dpp0<0x143, 0xc>(v));
    return v;
}

__device__ __forceinline__ uint32_t last_lane(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, kWave - 1);
}

// exclusive scan over the workgroup's NT threads; one barrier (s_wsum must not be in use), total to all threads
template <int NT>
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* s_wsum, uint32_t& total)
{
    const uint32_t incl = wave_scan_add(v);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & (kWave - 1)) == kWave - 1)
        s_wsum[wave] = incl;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < NT / kWave; ++w) {
        const uint32_t c = s_wsum[w];
        off += w < wave ? c : 0u;
        tot += c;
    }
    total = tot;
    return off + incl - v;
}

// last i in [0, n) with p[i] <= q for a whole wavefront (p[0] <= q, ascending): 64 probes per step
__device__ __forceinline__ int wave_upper(const int64_t* __restrict__ p, int n, int64_t q)
{
    const int lane = threadIdx.x & (kWave - 1);
    int lo = 0;
    while (n > 1) {
        const int step = (n + kWave - 1) / kWave;
        const int i = lane * step;
        const uint64_t le = __ballot(i < n && p[lo + min(i, n - 1)] <= q);
        const int k = (__popcll(le) - 1) * step;
        lo += k;
        n = min(step, n - k);
    }
    return lo;
}

__device__ __forceinline__ int ceil_log2(uint32_t x) { return x <= 1 ? 0 : 32 - __clz((int)(x - 1)); }

// The digit counters are counted as words and read as their halves.
typedef uint16_t __attribute__((may_alias)) u16_alias;
typedef uint32_t __attribute__((may_alias)) u32_alias;

// element i of an array: 32-bit byte offset to a uniform base, so that unrolled accesses share one address register
template <typename T>
__device__ __forceinline__ T load_at(const T* base, uint32_t i, uint32_t plus)
{
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + i * (uint32_t)sizeof(T) + plus * sizeof(T));
}
template <typename T>
__device__ __forceinline__ void store_at(T* base, uint32_t i, uint32_t plus, T v)
{
    *reinterpret_cast<T*>(reinterpret_cast<char*>(base) + i * (uint32_t)sizeof(T) + plus * sizeof(T)) = v;
}

// digit of `width` bits from `sh` on
__device__ __forceinline__ uint32_t digit_of(uint32_t w, int sh, int width) { return __builtin_amdgcn_ubfe(w, sh, width); }
__device__ __forceinline__ uint32_t digit_of(uint64_t w, int sh, int width) { return __builtin_amdgcn_ubfe((uint32_t)(w >> sh), 0, width); }

// A value the compiler may not carry over from one phase to the next: sixteen positions per thread, or the masks
// of their comparisons, kept in registers across the phases of a tile spill.
__device__ __forceinline__ int opaque(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// Ranks of the wavefront's words among those of the same digit, in position order: rank[r] counts the earlier
// words of the wavefront's own row of counters.  Lanes with the same digit find each other with one ballot per
// digit bit; the first of them adds the count.  The counters are 16-bit halves of words, read and added to by LDS
// operations, which execute in order.
// Rounds come in groups whose counter reads are waited for together.  Every position of every round counts: positions past the end hold words whose digit is the largest, so they
// come out last.  BITS is a template parameter: with a test per bit and round the kernels spend as long on scalar
// branches as on ballots.
template <int BITS, int GROUP, int ND, int PER, typename Digit>
__device__ __forceinline__ void rank_bits(Digit digit, int groups, uint16_t (&s_cnt)[kSortWaves][ND], uint32_t (&rank)[PER])
{
    const int wave = uniform(threadIdx.x >> 6);
#pragma unroll
    for (int r0 = 0; r0 < PER; r0 += GROUP) {
        if (r0 >= groups * GROUP)
            break;
        uint32_t lo[GROUP], hi[GROUP], dg[GROUP];
#pragma unroll
        for (int x = 0; x < GROUP; ++x) {
            dg[x] = digit(r0 + x);
            lo[x] = hi[x] = ~0u;
#pragma unroll
            for (int b = 0; b < BITS; ++b) {
                int32_t mk;                                  // all ones if bit b is set
                asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(mk) : "v"(dg[x]), "n"(b));
                const uint64_t bal = __ballot(mk != 0);
                // x &= ~(ballot ^ mk): lanes whose bit differs drop out (left to itself the compiler takes 3/2 as many)
                lo[x] = __builtin_amdgcn_bitop3_b32(lo[x], (uint32_t)bal, (uint32_t)mk, 0x90);
                hi[x] = __builtin_amdgcn_bitop3_b32(hi[x], (uint32_t)(bal >> 32), (uint32_t)mk, 0x90);
            }
        }
        uint32_t pre[GROUP];
#pragma unroll
        for (int x = 0; x < GROUP; ++x) {
            const uint32_t below = __builtin_amdgcn_mbcnt_hi(hi[x], __builtin_amdgcn_mbcnt_lo(lo[x], 0u));
            pre[x] = reinterpret_cast<const u16_alias*>(s_cnt[wave])[dg[x]];
            if (below == 0)
                atomicAdd(reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(s_cnt[wave]) + (2u * dg[x] & ~3u)),
                          (uint32_t)(__popc(lo[x]) + __popc(hi[x])) << ((dg[x] & 1u) * 16u));
            rank[r0 + x] = below;
        }
#pragma unroll
        for (int x = 0; x < GROUP; ++x)
            rank[r0 + x] += pre[x];
    }
}

// groups: of GROUP rounds each
template <int GROUP, int ND, int PER, typename Digit>
__device__ __forceinline__ void rank_rounds(Digit digit, int groups, int bits, uint16_t (&s_cnt)[kSortWaves][ND],
                                            uint32_t (&rank)[PER])
{
    static_assert(ND == 256 || ND == 1024, "digit tables");
    switch (bits) {
        case 0:
        case 1: rank_bits<1, GROUP>(digit, groups, s_cnt, rank); break;
        case 2: rank_bits<2, GROUP>(digit, groups, s_cnt, rank); break;
        case 3: rank_bits<3, GROUP>(digit, groups, s_cnt, rank); break;
        case 4: rank_bits<4, GROUP>(digit, groups, s_cnt, rank); break;
        case 5: rank_bits<5, GROUP>(digit, groups, s_cnt, rank); break;
        case 6: rank_bits<6, GROUP>(digit, groups, s_cnt, rank); break;
        case 7: rank_bits<7, GROUP>(digit, groups, s_cnt, rank); break;
        case 8: rank_bits<8, GROUP>(digit, groups, s_cnt, rank); break;
        default:
            if constexpr (ND > 256) {
                if (bits == 9)
                    rank_bits<9, GROUP>(digit, groups, s_cnt, rank);
                else
                    rank_bits<10, GROUP>(digit, groups, s_cnt, rank);
            }
    }
}

// Turns the wavefronts' digit counts into the slots of their first words (digit-major, wavefront by wavefront):
// slot = s_cnt[wave][digit] + rank.  A thread owns two neighbouring digits as the halves of one word (no count
// exceeds kSortTile).  Returns the thread's pair of digit starts; counts: its pair of digit totals.  One barrier
// inside; the caller synchronises before the slots are read.
template <int ND>
__device__ __forceinline__ uint32_t digit_starts(uint16_t (&s_cnt)[kSortWaves][ND], uint32_t* s_wsum, uint32_t& counts)
{
    uint32_t c[kSortWaves], sum = 0;
    const bool mine = 2 * (int)threadIdx.x < ND;
    if (mine) {
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w) {
            c[w] = reinterpret_cast<const u32_alias*>(s_cnt[w])[threadIdx.x];
            sum += c[w];
        }
    }
    uint32_t total;
    const uint32_t ex = block_scan<kSortThreads>((sum & 0xffffu) + (sum >> 16), s_wsum, total);
    uint32_t run = ex | ((ex + (sum & 0xffffu)) << 16);
    const uint32_t starts = run;
    if (mine) {
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w) {
            reinterpret_cast<u32_alias*>(s_cnt[w])[threadIdx.x] = run;
            run += c[w];
        }
    }
    counts = sum;
    return starts;
}

template <int ND>
__device__ __forceinline__ void zero_counts(uint16_t (&s_cnt)[kSortWaves][ND])
{
    for (int i = threadIdx.x; i < kSortWaves * ND / 8; i += kSortThreads)
        reinterpret_cast<uint4*>(&s_cnt[0][0])[i] = make_uint4(0u, 0u, 0u, 0u);
}

constexpr int kSortGroup = 2;      // rounds per group of the sorts in LDS (units differ in size) ...
constexpr int kPartGroup = 4;      // ... and of the partition (tiles are full)

// rounds of 64 words per wavefront that hold m words, in whole groups
template <int GROUP>
__device__ __forceinline__ int group_count(int m) { return (m + kSortThreads * GROUP - 1) / (kSortThreads * GROUP); }

// One pass of a stable sort of the words w, in registers at positions wavefront * rounds * 64 + r * 64 + lane: by
// `width` bits from `sh` on; the result is in s_w, barrier included.  s_cnt: cleared, and synchronised since.
template <typename W, int PER, int ND>
__device__ __forceinline__ void block_sort_pass(W (&w)[PER], int groups, int sh, int width, W* s_w,
                                                uint16_t (&s_cnt)[kSortWaves][ND], uint32_t* s_wsum)
{
    const int wave = uniform(threadIdx.x >> 6);
    uint32_t rank[PER];
    rank_rounds<kSortGroup>([&](int r) { return digit_of(w[r], sh, width); }, groups, width, s_cnt, rank);
    __syncthreads();
    uint32_t counts;
    (void)digit_starts<ND>(s_cnt, s_wsum, counts);
    __syncthreads();
#pragma unroll
    for (int r0 = 0; r0 < PER; r0 += kSortGroup)
        if (r0 < groups * kSortGroup) {
#pragma unroll
            for (int r = r0; r < r0 + kSortGroup; ++r)
                rank[r] += s_cnt[wave][digit_of(w[r], sh, width)];
        }
#pragma unroll
    for (int r = 0; r < PER; ++r)
        if (r < groups * kSortGroup)
            s_w[rank[r]] = w[r];
    __syncthreads();
}

// the digits of pass p of P over `bits` bits
__device__ __forceinline__ int pass_width(int bits, int P, int p) { return bits / P + (p < bits % P ? 1 : 0); }

// s_cnt: cleared, and synchronised since (between other work of the caller's: clearing and a barrier take 0.3 to 0.5 us).
template <typename W, int PER, int ND>
__device__ __forceinline__ void block_sort(W (&w)[PER], int groups, int shift, int bits, W* s_w,
                                           uint16_t (&s_cnt)[kSortWaves][ND], uint32_t* s_wsum)
{
    const int p0 = (int)(threadIdx.x >> 6) * groups * kSortGroup * kWave + (int)(threadIdx.x & (kWave - 1));
    constexpr int kBits = ND == 256 ? 8 : 10;
    const int passes = (bits + kBits - 1) / kBits;
    for (int p = 0; p < passes; ++p) {
        const int width = pass_width(bits, passes, p);
        if (p > 0) {
            zero_counts(s_cnt);
            const int q = opaque(p0);
#pragma unroll
            for (int r = 0; r < PER; ++r)
                if (r < groups * kSortGroup)
                    w[r] = s_w[q + r * kWave];
            __syncthreads();
        }
        block_sort_pass(w, groups, shift, width, s_w, s_cnt, s_wsum);
        shift += width;
    }
}

// Makes every mark the largest at or before it in its wavefront's stretch, position p = wavefront * rounds * 64 + r * 64 +
// lane, and returns the largest before the stretch.  Two barriers, the last one before the caller may read.
__device__ __forceinline__ uint32_t carry_marks(int rounds, uint32_t* s_mark, uint32_t* s_wsum)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x >> 6;
    const int p0 = wave * rounds * kWave + lane;
    __syncthreads();
    uint32_t top = 0;
    for (int r = 0; r < rounds; r += 2) {
        const uint32_t v = wave_scan_max(s_mark[p0 + r * kWave]), x = wave_scan_max(s_mark[p0 + (r + 1) * kWave]);
        const uint32_t mid = max(top, last_lane(v));
        s_mark[p0 + r * kWave] = max(v, top);
        s_mark[p0 + (r + 1) * kWave] = max(x, mid);
        top = max(mid, last_lane(x));
    }
    if (lane == 0)
        s_wsum[wave] = top;
    __syncthreads();
    uint32_t carry = 0;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w)
        carry = max(carry, w < wave ? s_wsum[w] : 0u);
    return carry;
}

// Bags of the positions [first, first + m) of a table (offsets: its B + 1 bag borders; bags lo..hi are the ones
// that can hold them): every bag that is not empty marks its first position, and a position's bag is the largest
// mark at or before it, for position p = wavefront * rounds * 64 + r * 64 + lane
//     max(s_mark[p], returned carry of the wavefront) - 1.
// s_mark: rounds * kSortThreads words of LDS, rounds a multiple of 2.  Barriers inside, the last one before the
// caller may read.
__device__ __forceinline__ uint32_t bags_of_positions(const int64_t* __restrict__ offsets, int lo, int hi, int first, int m,
                                                      int rounds, uint32_t* s_mark, uint32_t* s_wsum)
{
    for (int i = threadIdx.x; i < rounds * (kSortThreads / 4); i += kSortThreads)
        reinterpret_cast<uint4*>(s_mark)[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    for (int i = lo + (int)threadIdx.x; i <= hi; i += kSortThreads) {
        const int o = (int)offsets[i], e = (int)offsets[i + 1];
        const int p = max(o - first, 0);
        if (e > o && e > first && p < m)
            s_mark[p] = (uint32_t)i + 1u;
    }
    return carry_marks(rounds, s_mark, s_wsum);
}

// ---------------------------------------------------------------- plan

struct TablePlan {
    int want, cuts;      // buckets asked for, ranges of the packed key
    int chunks;
    int units;           // select, pieces: most there can be, of all buckets and rows of several units
};

// lookups of a unit of a row that has several
__device__ __forceinline__ int unit_part(int mode) { return mode == kSortSelect ? kSelectPart : kSortTile; }

__device__ __forceinline__ TablePlan table_plan(const SortArgs& a, int n, uint32_t rows)
{
    TablePlan p;
    p.cuts = a.kb >= 31 ? 1 : (int)((rows + (1u << a.kb) - 1) >> a.kb);
    p.want = min(max((n + a.target - 1) / a.target, 1), kMaxBuckets - p.cuts);
    p.chunks = n == 0 || a.mode == kSortSelect ? 0 : (n + a.chunk - 1) / a.chunk;
    p.units = n == 0 || a.mode == kSortPartition ? 0 : p.want + p.cuts - 1 + n / unit_part(a.mode);
    return p;
}

// first i in [0, n) with p[i] >= v (n if none); p ascending, in LDS
__device__ __forceinline__ int lds_lower(const uint32_t* p, int n, uint32_t v)
{
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (p[mid] < v)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// Up to kRankSamples samples are sorted by counting for each how many go before it, every thread a stretch of them: two passes of the
// sort in LDS cost 3.8 us however few there are, this 0.5 for 64 and 1.3 for 256.
constexpr int kRankBits = 8;
constexpr int kRankSamples = 1 << kRankBits;

// w: the thread's words, at positions p0 + r * 64 (behind n: any), of at most 32 - kRankBits bits; the result is in s_out, barrier
// included.  s_tmp: 2 * kRankSamples words, cleared, and synchronised since.
template <int PER>
__device__ __forceinline__ void rank_sort(const uint32_t (&w)[PER], int n, int p0, uint32_t* s_out, uint32_t* s_tmp)
{
    uint32_t* s_in = s_tmp;
    uint32_t* s_rank = s_tmp + kRankSamples;
    const int lg = max(2, ceil_log2((uint32_t)n)), size = 1 << lg;
    static_assert(kSortGroup * kSortThreads >= kRankSamples, "the first rounds hold all of them");
#pragma unroll
    for (int r = 0; r < kSortGroup; ++r) {
        const int p = p0 + r * kWave;                    // (the position makes every word another)
        if (p < size)
            s_in[p] = p < n ? w[r] << kRankBits | (uint32_t)p : ~0u;
    }
    __syncthreads();
    const int i = (int)threadIdx.x & (size - 1), part = (int)threadIdx.x >> lg, each = max(4, size * size / kSortThreads);
    const uint32_t mine = s_in[i];
    uint32_t before = 0;
    for (int j = part * each; j < min((part + 1) * each, size); j += 4) {
        const uint4 x = *reinterpret_cast<const uint4*>(s_in + j);
        before += (x.x < mine ? 1u : 0u) + (x.y < mine ? 1u : 0u) + (x.z < mine ? 1u : 0u) + (x.w < mine ? 1u : 0u);
    }
    if (before > 0)
        atomicAdd(&s_rank[i], before);
    __syncthreads();
    if ((int)threadIdx.x < n)
        s_out[s_rank[threadIdx.x]] = s_in[threadIdx.x] >> kRankBits;
    __syncthreads();
}

// MODE: a.mode (in one kernel the partition's plan took 0.3 us longer)
template <int MODE>
__global__ __launch_bounds__(kSortThreads) void sort_plan_kernel(SortArgs a)
{
    __shared__ __align__(16) uint32_t s_key[kSortTile];
    __shared__ __align__(16) uint16_t s_cnt[kSortWaves][1024];     // (samples are few: two passes of ten bits)
    __shared__ uint32_t s_list[kMaxBuckets + 2], s_cut[kMaxRangeCuts];
    __shared__ uint32_t s_wsum[kSortWaves];
    __shared__ uint32_t s_sum[4], s_hot;             // (s_hot: a row may have several units)
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int t = blockIdx.x;
    const int64_t o0 = a.offsets[(int64_t)t * a.B], o1 = a.offsets[(int64_t)(t + 1) * a.B];
    const int start = (int)o0, n = (int)(o1 - o0);
    const uint32_t rbase = a.row_base[t], rows = a.row_base[t + 1] - rbase;
    const int bits = a.meta[t].key_bits;
    if (tid < 4)
        s_sum[tid] = 0;
    if (tid == 0)
        s_hot = 0;
    zero_counts(s_cnt);
    const TablePlan p = table_plan(a, n, rows);
    // ---- a sample: one lookup from each of S equal stretches of the table's positions.  Requested before the tables before this
    // one are counted: bound by the misses a CU has in flight (1000 samples 2 us, 7700 samples, of 2 M lookups, 23 of 45).
    const int q = samples_per_bucket(p.want, a.target);
    const int S = p.want * q;
    const int groups = group_count<kSortGroup>(S), rounds = groups * kSortGroup;
    uint32_t w[kSortPerThread];
    const int prior = min(tid, t - 1);               // (of up to kSortThreads tables, requested before the sample)
    int64_t prior_end = 0, prior_start = 0;
    uint32_t prior_rows = 0;
    if (t > 0) {
        prior_end = a.offsets[(int64_t)(prior + 1) * a.B];
        prior_start = a.offsets[(int64_t)prior * a.B];
        prior_rows = a.row_base[prior + 1] - a.row_base[prior];
    }
    if (n > 0) {
        const uint64_t stretch = ((uint64_t)n << 32) / (uint32_t)S;      // 32.32
        const uint32_t* __restrict__ idx = a.indices + start;
        const int first = wave * rounds * kWave + lane;
#pragma unroll
        for (int r = 0; r < kSortPerThread; r += kSortGroup)
            if (r < rounds) {
#pragma unroll
                for (int x = 0; x < kSortGroup; ++x)
                    w[r + x] = idx[sample_position(stretch, (uint32_t)min(first + (r + x) * kWave, S - 1), n)];
            }
    }
    __syncthreads();
    {   // what the tables before this one take
        uint32_t multi = 0, chunks = 0, parts = 0, units = 0;
        for (int i = tid; i < t; i += kSortThreads) {
            if (i >= kSortThreads) {
                prior_end = a.offsets[(int64_t)(i + 1) * a.B];
                prior_start = a.offsets[(int64_t)i * a.B];
                prior_rows = a.row_base[i + 1] - a.row_base[i];
            }
            const int n = (int)(prior_end - prior_start);
            const TablePlan p = table_plan(a, n, prior_rows);
            multi += p.chunks > a.col_chunks; chunks += p.chunks; parts += n > 0; units += p.units;
        }
        multi = last_lane(wave_scan_add(multi));
        chunks = last_lane(wave_scan_add(chunks));
        parts = last_lane(wave_scan_add(parts));
        units = last_lane(wave_scan_add(units));
        if (lane == 0 && parts > 0) {
            atomicAdd(&s_sum[0], multi); atomicAdd(&s_sum[1], chunks); atomicAdd(&s_sum[2], parts); atomicAdd(&s_sum[3], units);
        }
    }
    __syncthreads();
    SortTable st;
    st.start = start; st.n = n;
    st.pad = 0; st.chunk_base = (int)s_sum[1]; st.part = (int)s_sum[2];
    st.nchunks = p.chunks;
    st.nb = 0; st.lut_shift = 0; st.lut_span = 0;
    if (tid == 0) {
        a.tstart[t] = start;
        a.table_runs[t] = 0;
        if (p.chunks > a.col_chunks)
            a.multi[s_sum[0]] = t;
        if (t == a.T - 1) {
            a.tstart[a.T] = (int)o1;
            a.counters->sort_chunks = st.chunk_base + p.chunks;
            a.counters->sort_multi = (int)s_sum[0] + (p.chunks > a.col_chunks);
            a.counters->sort_units = s_sum[3] + (uint32_t)p.units;
            a.counters->sort_ticket = 0;
        }
    }
    for (int i = tid; i < p.chunks; i += kSortThreads) {
        SortChunk c;
        c.t = t;
        c.first = start + i * a.chunk;
        c.cnt = min(a.chunk, start + n - c.first);
        c.pad = 0;
        a.chunks[st.chunk_base + i] = c;
    }
    if (n == 0) {
        if (tid == 0)
            a.tables[t] = st;
        return;
    }
    if (MODE == kSortSelect && p.units == 1) {                 // one bucket
        if (tid == 0)
            a.units[s_sum[3]] = SortUnit{start, n, rbase, ceil_log2(rows), (uint16_t)t, 0, 0, (int32_t)s_sum[3], ~0u};
        return;
    }

    // ---- sorted: past the sample the largest key, behind it
#pragma unroll
    for (int r = 0; r < kSortPerThread; ++r)
        w[r] = r < rounds && wave * rounds * kWave + r * kWave + lane < S ? min(w[r], rows - 1) : ~0u;
    if (S <= kRankSamples && bits <= 32 - kRankBits)
        rank_sort(w, S, wave * rounds * kWave + lane, s_key, reinterpret_cast<uint32_t*>(&s_cnt[0][0]));
    else
        block_sort(w, groups, 0, bits, s_key, s_cnt, s_wsum);
    // ---- borders: row 0, every q-th sample once, and the row after one that fills a whole stretch of samples
    // (a bucket of its own).  Thread j owns candidates 2 j and 2 j + 1.
    uint32_t cand[2], emit[2];
    const int part = unit_part(MODE);
    const int part_samples = (int)((uint32_t)part * (uint32_t)S / (uint32_t)n);      // so many hold lookups for a unit more
    static_assert((int64_t)kSortTile * kSamplesMax < (int64_t)1 << 32, "");
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int j = 2 * tid + k;
        emit[k] = 0;
        cand[k] = 0;
        if (j < p.want) {
            const uint32_t c = j == 0 ? 0u : s_key[j * q];
            const uint32_t before = j <= 1 ? 0u : s_key[(j - 1) * q];
            const bool fresh = j == 0 || c != before;
            cand[k] = c;
            emit[k] = fresh ? (j + 1 < p.want && s_key[(j + 1) * q] == c ? 2u : 1u) : 0u;
            if (MODE != kSortPartition && emit[k] > 1 && s_key[min(j * q + part_samples, S) - 1] == c)
                s_hot = 1;
        }
    }
    uint32_t total;
    uint32_t at = block_scan<kSortThreads>(emit[0] + emit[1], s_wsum, total);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        if (emit[k] > 0)
            s_list[at] = cand[k];
        if (emit[k] > 1)
            s_list[at + 1] = cand[k] + 1;
        at += emit[k];
    }
    __syncthreads();
    // distinct borders below the number of rows
    uint32_t* s_uniq = reinterpret_cast<uint32_t*>(&s_cnt[0][0]);      // (the counters are done with)
    const int n_list = (int)total;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int i = 2 * tid + k;
        emit[k] = i < n_list && s_list[i] < rows && (i == 0 || s_list[i] != s_list[i - 1]) ? 1u : 0u;
    }
    at = block_scan<kSortThreads>(emit[0] + emit[1], s_wsum, total);
#pragma unroll
    for (int k = 0; k < 2; ++k)
        if (emit[k])
            s_uniq[at++] = s_list[2 * tid + k];
    const int na = (int)total;
    __syncthreads();
    // multiples of the packed key range that are no border yet (cuts <= kMaxRangeCuts = kSortThreads)
    uint32_t cut = 0;
    bool keep = false;
    if (tid >= 1 && tid < p.cuts) {
        cut = (uint32_t)tid << a.kb;
        const int i = lds_lower(s_uniq, na, cut);
        keep = i == na || s_uniq[i] != cut;
    }
    at = block_scan<kSortThreads>(keep ? 1u : 0u, s_wsum, total);
    if (keep)
        s_cut[at] = cut;
    const int nc = (int)total;
    __syncthreads();
    uint32_t* split = a.split + (int64_t)st.part * kMaxBuckets;
    if (keep)
        s_list[at + lds_lower(s_uniq, na, cut)] = cut;
    for (int i = tid; i < na; i += kSortThreads)
        s_list[i + lds_lower(s_cut, nc, s_uniq[i])] = s_uniq[i];
    const int nb = na + nc;
    __syncthreads();
    if (MODE != kSortPartition) {
        // ---- units: one per bucket, and for a bucket of one row as many as its samples say it has lookups for
        uint32_t lo[2], hi[2], parts[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int i = 2 * tid + k;
            lo[k] = hi[k] = 0;
            parts[k] = 0;
            if (i < nb) {
                lo[k] = s_list[i];
                hi[k] = i + 1 < nb ? s_list[i + 1] : rows;
                parts[k] = 1;
                if (s_hot && hi[k] - lo[k] == 1) {
                    const int before = lds_lower(s_key, S, lo[k]);
                    parts[k] = (uint32_t)unit_parts((uint32_t)lds_lower(s_key + before, S - before, hi[k]), n, S, part);
                }
            }
        }
        at = s_sum[3] + block_scan<kSortThreads>(parts[0] + parts[1], s_wsum, total);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int i = 2 * tid + k;
            SortUnit u{start, n, rbase + lo[k], ceil_log2(hi[k] - lo[k]), (uint16_t)t, (uint16_t)i, 0, (int32_t)s_sum[3], 0};
            // (an index that is no row of the table is the last bucket's)
            u.last = MODE == kSortPieces ? (uint32_t)st.chunk_base : i + 1 < nb ? hi[k] - lo[k] - 1u : ~0u - lo[k];
            static_assert((int64_t)kPiecesMax * kPiecesChunk / kSortTile < 1 << 12, "a part's number");
            for (uint32_t j = 0; j < parts[k]; ++j) {
                const uint32_t last = MODE == kSortPieces ? (parts[k] - 1u) << 20 : j + 1 < parts[k] ? (uint32_t)kUnitMore : 0u;
                u.flags = (int32_t)(last | j << 8);
                a.units[at++] = u;
            }
        }
        for (int i = (int)total + tid; i < p.units; i += kSortThreads)
            a.units[s_sum[3] + i] = SortUnit{start, n, 0, 0, (uint16_t)t, 0, kUnitNone, (int32_t)s_sum[3], (uint32_t)st.chunk_base};
        if (MODE == kSortSelect)
            return;
        __syncthreads();                             // (the samples make room for the cells)
    }
    for (int i = tid; i < nb; i += kSortThreads)
        split[i] = s_list[i];
    // ---- lookup table: the bucket of every cell's first row, the last border at or before it.  A border counts in the
    // first cell that starts at or behind it; the low halves add up to the buckets, the high ones count the borders that
    // do not start their cell, which lie inside the one before.  (A bisection of the borders per cell took 2 to 9 us.)
    const int lut_bits = min(min(kLutBits, bits), ceil_log2((uint32_t)nb) + 3);
    const int shift = bits - lut_bits, cells = 1 << lut_bits;
    uint32_t* s_cell = s_key;
    static_assert((1 << kLutBits) < kSortTile && (1 << kLutBits) % kSortThreads == 0, "");
    for (int i = tid; i <= cells; i += kSortThreads)
        s_cell[i] = 0;
    if (tid == 0)
        s_sum[0] = 0;
    __syncthreads();
    for (int i = tid; i < nb; i += kSortThreads) {
        const uint32_t row = s_list[i], cell = (row >> shift) + ((row & ((1u << shift) - 1u)) != 0 ? 1u : 0u);
        atomicAdd(&s_cell[cell], cell << shift == row ? 1u : 0x10001u);
    }
    __syncthreads();
    uint16_t* lut = a.lut + (int64_t)st.part * kLutSize;
    const int each = max(cells / kSortThreads, 1), c0 = tid * each;
    uint32_t borders = 0;
    if (c0 < cells)
        for (int i = 0; i < each; ++i)
            borders += s_cell[c0 + i] & 0xffffu;
    uint32_t bucket = block_scan<kSortThreads>(borders, s_wsum, total) - 1u, span = 0;
    if (c0 < cells)
        for (int i = 0; i < each; ++i) {
            bucket += s_cell[c0 + i] & 0xffffu;
            lut[c0 + i] = (uint16_t)bucket;
            span = max(span, s_cell[c0 + i + 1] >> 16);
        }
    if (tid == 0)
        lut[cells] = (uint16_t)(nb - 1);
    span = last_lane(wave_scan_max(span));
    if (lane == 0)
        atomicMax(&s_sum[0], span);
    __syncthreads();
    if (tid == 0) {
        st.nb = nb;
        st.lut_shift = (int16_t)shift;
        st.lut_span = (int16_t)s_sum[0];
        a.tables[t] = st;
    }
}

// ---------------------------------------------------------------- partition

// A table's borders and lookup table in LDS (synchronise before use), and the bucket of a row: the bucket of the
// first row of its cell, moved on over the borders inside the cell.  Cells of hashed ids hold one border or, for
// a row with a bucket of its own, two: up to kLinear borders are compared one after the other, all at once; ids
// that crowd in a few cells are bisected.
struct Borders {
    static constexpr int kLinear = 4;
    uint32_t below[kMaxBuckets + kLinear];     // first row of the bucket, minus 1
    uint16_t lut[kLutSize];

    __device__ __forceinline__ void load(const SortArgs& a, const SortTable& st, int bits)
    {
        const uint32_t* from = a.split + (int64_t)st.part * kMaxBuckets;
        for (int i = threadIdx.x; i < st.nb + kLinear; i += kSortThreads)
            below[i] = i < st.nb ? from[i] - 1u : ~0u;
        const uint32_t* cells = reinterpret_cast<const uint32_t*>(a.lut + (int64_t)st.part * kLutSize);
        const int n = (1 << (bits - st.lut_shift)) / 2 + 1;
        for (int i = threadIdx.x; i < n; i += kSortThreads)
            reinterpret_cast<uint32_t*>(lut)[i] = cells[i];
    }

    // SPAN: most borders inside a cell; 0: more than kLinear
    template <int SPAN>
    __device__ __forceinline__ uint32_t bucket(uint32_t row, int shift, uint32_t last_cell) const
    {
        if constexpr (SPAN > 0) {
            return linear_bucket<SPAN>(below, lut, row, shift, last_cell);
        } else {
            const uint32_t cell = min(row >> shift, last_cell);
            uint32_t d = lut[cell], hi = lut[cell + 1];
            while (__ballot(d < hi) != 0ull) {
                const uint32_t mid = (d + hi + 1) >> 1;
                const bool up = below[mid] < row;
                d = up ? mid : d;
                hi = up ? hi : max(mid, 1u) - 1u;
            }
            return d;
        }
    }

    // f(the SPAN of the table)
    template <typename F>
    __device__ __forceinline__ static void with_span(int span, F f)
    {
        switch (span) {
            case 0:
            case 1: f(std::integral_constant<int, 1>()); break;
            case 2: f(std::integral_constant<int, 2>()); break;
            case 3: f(std::integral_constant<int, 3>()); break;
            case 4: f(std::integral_constant<int, 4>()); break;
            default: f(std::integral_constant<int, 0>()); break;
        }
    }
};

__global__ __launch_bounds__(kSortThreads) void sort_hist_kernel(SortArgs a)
{
    __shared__ uint32_t s_hist[kMaxBuckets];
    __shared__ Borders s_borders;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const SortChunk c = a.chunks[blockIdx.x];        // (requested together with the number of chunks; there is room for the grid)
    if ((int)blockIdx.x >= a.counters->sort_chunks)
        return;
    const SortTable st = a.tables[c.t];
    const int bits = a.meta[c.t].key_bits;
    const int shift = st.lut_shift, span = st.lut_span;
    const uint32_t last_cell = (1u << (bits - shift)) - 1u;
    const int end = c.first + c.cnt;
    s_borders.load(a, st, bits);
    for (int i = threadIdx.x; i < kMaxBuckets; i += kSortThreads)
        s_hist[i] = 0;
    // the bag of every tile's first position, one tile per wavefront (the partition starts from it)
    static_assert(kSortWaves >= 8, "a chunk has at most 8 tiles");
    if (c.first + wave * kSortTile < end) {
        const int b = wave_upper(a.offsets + (int64_t)c.t * a.B, a.B, c.first + wave * kSortTile);
        if (lane == 0)
            a.tile_bag[(int)blockIdx.x * a.tiles_per_chunk + wave] = b;
    }
    __syncthreads();
    const uint32_t* __restrict__ idx = a.indices + c.first;
    Borders::with_span(span, [&](auto sp) {
        constexpr int kSpan = decltype(sp)::value;
        int first = 0;
        for (; first + kSortTile <= c.cnt; first += kSortTile) {
            uint32_t key[kSortPerThread];
#pragma unroll
            for (int r = 0; r < kSortPerThread; ++r)
                key[r] = load_at(idx, (uint32_t)(first + (int)threadIdx.x), r * kSortThreads);
#pragma unroll
            for (int r = 0; r < kSortPerThread; ++r)
                atomicAdd(&s_hist[s_borders.bucket<kSpan>(key[r], shift, last_cell)], 1u);
        }
        for (int i = first + (int)threadIdx.x; i - (int)threadIdx.x < c.cnt; i += kSortThreads) {   // whole wavefronts: bucket() may ballot
            const uint32_t d = s_borders.bucket<kSpan>(idx[min(i, c.cnt - 1)], shift, last_cell);
            if (i < c.cnt)
                atomicAdd(&s_hist[d], 1u);
        }
    });
    __syncthreads();
    for (int i = threadIdx.x; i < st.nb; i += kSortThreads)
        a.hist[(int64_t)blockIdx.x * kMaxBuckets + i] = s_hist[i];
}

// Counts of the chunks -> positions of the chunks inside the bucket, and the bucket's lookups, for a table of many chunks.
// A lane has a bucket and the wavefronts of a workgroup share the chunks out, kColAhead of them at a time: bound by trips
// to the histogram one after the other.  (sort_units_kernel walked them with one thread per bucket, eight chunks a trip:
// 49 / 152 / 783 us for one table of 3 M / 10 M / 100 M lookups, now 13 / 24 / 76 in the two.)
__global__ __launch_bounds__(kColThreads) void sort_columns_kernel(SortArgs a)
{
    constexpr int kWaves = kColThreads / kWave;
    __shared__ uint32_t s_sum[kWaves][kColBuckets];
    if ((int)(blockIdx.x / (kMaxBuckets / kColBuckets)) >= a.counters->sort_multi)
        return;
    const SortTable st = a.tables[a.multi[blockIdx.x / (kMaxBuckets / kColBuckets)]];
    const int d = (int)(blockIdx.x % (kMaxBuckets / kColBuckets)) * kColBuckets + (int)(threadIdx.x & (kWave - 1));
    const int wave = uniform(threadIdx.x >> 6);
    if (d - (int)(threadIdx.x & (kWave - 1)) >= st.nb)
        return;
    const bool mine = d < st.nb;
    const int each = (st.nchunks + kWaves - 1) / kWaves;
    const int c0 = min(wave * each, st.nchunks), c1 = min(c0 + each, st.nchunks);
    uint32_t* col = a.hist + (int64_t)st.chunk_base * kMaxBuckets + min(d, st.nb - 1);
    uint32_t x[kColAhead], sum = 0;
    for (int c = c0; c < c1; c += kColAhead) {
#pragma unroll
        for (int i = 0; i < kColAhead; ++i)
            x[i] = col[(int64_t)min(c + i, c1 - 1) * kMaxBuckets];
#pragma unroll
        for (int i = 0; i < kColAhead; ++i)
            sum += c + i < c1 ? x[i] : 0u;
    }
    s_sum[wave][threadIdx.x & (kWave - 1)] = sum;
    __syncthreads();
    uint32_t run = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const uint32_t c = s_sum[w][threadIdx.x & (kWave - 1)];
        run += w < wave ? c : 0u;
        tot += c;
    }
    if (mine && wave == 0)
        a.bstart[(int64_t)st.part * kMaxBuckets + d] = tot;
    for (int c = c0; c < c1; c += kColAhead) {
        if (each > kColAhead) {                      // (otherwise x still holds them)
#pragma unroll
            for (int i = 0; i < kColAhead; ++i)
                x[i] = col[(int64_t)min(c + i, c1 - 1) * kMaxBuckets];
        }
#pragma unroll
        for (int i = 0; i < kColAhead; ++i) {
            if (mine && c + i < c1)
                col[(int64_t)(c + i) * kMaxBuckets] = run;
            run += x[i];
        }
    }
}

// One workgroup per table, one thread per bucket: bucket starts and work units (and, for a table of few chunks, what
// sort_columns_kernel does for the others).  A table takes the next unit numbers there are: which ones depends on the
// order of the workgroups, but nothing else does -- units are independent, and runs are counted table by table.  (Numbers
// in the order of the tables took a last workgroup that waited for all others behind two fences, 13 us of 27.)
__global__ __launch_bounds__(kUnitsThreads) void sort_units_kernel(SortArgs a)
{
    __shared__ uint32_t s_wsum[2][kUnitsThreads / kWave];
    __shared__ uint32_t s_first;
    const int t = blockIdx.x;
    const int d = threadIdx.x;
    const SortTable st = a.tables[t];
    if (st.nb == 0)
        return;
    uint32_t* bstart = a.bstart + (int64_t)st.part * kMaxBuckets;
    const uint32_t* split = a.split + (int64_t)st.part * kMaxBuckets;
    uint32_t run = 0;
    if (st.nchunks > a.col_chunks) {
        run = d < st.nb ? bstart[d] : 0u;
    } else if (d < st.nb) {
        uint32_t* col = a.hist + (int64_t)st.chunk_base * kMaxBuckets + d;
        for (int c = 0; c < st.nchunks; c += kColAhead) {
            uint32_t x[kColAhead];
#pragma unroll
            for (int i = 0; i < kColAhead; ++i)
                x[i] = col[(int64_t)min(c + i, st.nchunks - 1) * kMaxBuckets];
#pragma unroll
            for (int i = 0; i < kColAhead; ++i) {
                if (c + i < st.nchunks) {
                    col[(int64_t)(c + i) * kMaxBuckets] = run;
                    run += x[i];
                }
            }
        }
    }
    uint32_t tot;
    const uint32_t start = (uint32_t)st.start + block_scan<kUnitsThreads>(run, s_wsum[0], tot);
    uint32_t lo = 0, range = 1, pieces = 0;
    if (d < st.nb) {
        bstart[d] = start;
        lo = split[d];
        range = (d + 1 < st.nb ? split[d + 1] : a.row_base[t + 1] - a.row_base[t]) - lo;
        pieces = run == 0 ? 0u : range == 1 ? (run + kSortTile - 1) / kSortTile : 1u;
    }
    const uint32_t before = block_scan<kUnitsThreads>(pieces, s_wsum[1], tot);
    if (d == 0)
        s_first = atomicAdd(&a.counters->sort_units, tot);
    __syncthreads();
    SortUnit u;
    u.key0 = a.row_base[t] + lo;
    u.bits = ceil_log2(range);
    u.t = (uint16_t)t;
    u.bucket = (uint16_t)d;
    u.first = (int32_t)s_first;
    u.last = 0;
    for (uint32_t i = 0; i < pieces; ++i) {
        u.start = (int32_t)(start + i * kSortTile);
        u.m = (int32_t)(range == 1 ? min((uint32_t)kSortTile, run - i * kSortTile) : run);
        u.flags = i > 0 ? kUnitContinued : 0;
        a.units[s_first + before + i] = u;
    }
}

// PIECES (a.mode is kSortPieces): the words stay where the chunk's lookups lie, in order of their buckets, and the buckets' first
// positions in it are written down.  A chunk is a chain of trips and barriers (4096 lookups 9.4 us: descriptors 1.3, borders and
// lookups 1.3, the bags of its ends 1.0, of all positions 1.3, buckets 1.4, ranks 2.2, order and writing 1.1).
template <typename W, bool PIECES>
__global__ __launch_bounds__(kSortThreads, sizeof(W) == 4 ? 4 : 2) void sort_scatter_kernel(SortArgs a)
{
    __shared__ __align__(16) W s_w[kSortTile];
    // digit counters while ranking, then the digits of the reordered words
    __shared__ __align__(16) uint16_t s_cnt[kSortWaves][kMaxBuckets];
    static_assert(kSortWaves * kMaxBuckets == kSortTile, "the digits of a tile replace its counters");
    __shared__ uint32_t s_next[PIECES ? 1 : kMaxBuckets], s_delta[PIECES ? 1 : kMaxBuckets];
    __shared__ int s_bag[2];
    __shared__ Borders s_borders;
    __shared__ uint32_t s_wsum[kSortWaves];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = uniform(tid >> 6);
    const SortChunk c = a.chunks[blockIdx.x];        // (requested together with the number of chunks; there is room for the grid)
    if ((int)blockIdx.x >= a.counters->sort_chunks)
        return;
    const SortTable st = a.tables[c.t];
    const int bits = a.meta[c.t].key_bits;
    const int shift = st.lut_shift, span = st.lut_span;
    const uint32_t last_cell = (1u << (bits - shift)) - 1u;
    const int digit_bits = ceil_log2((uint32_t)st.nb + 1u);   // bucket nb: positions past the end
    const int end = c.first + c.cnt;
    const int64_t* __restrict__ offsets = a.offsets + (int64_t)c.t * a.B;
    W* __restrict__ out = static_cast<W*>(a.words[0]);
    uint16_t* s_dig = &s_cnt[0][0];
    const uint32_t* s_mark = reinterpret_cast<const uint32_t*>(s_w);
    uint32_t dg[kSortPerThread];                     // rows of the lookups, then their buckets
    auto load_rows = [&](int first) {
        const int m = min(kSortTile, end - first);
        const int q = opaque(wave * group_count<kPartGroup>(m) * kPartGroup * kWave + lane);
        const uint32_t* __restrict__ idx = a.indices + first;
        if (m == kSortTile) {
#pragma unroll
            for (int r = 0; r < kSortPerThread; ++r)
                dg[r] = load_at(idx, (uint32_t)q, r * kWave);
        } else {
#pragma unroll
            for (int r = 0; r < kSortPerThread; ++r)
                dg[r] = idx[min(q + r * kWave, m - 1)];
        }
    };
    load_rows(c.first);
    s_borders.load(a, st, bits);
    if constexpr (PIECES) {                          // bags of the chunk's first and last position
        if (wave < 2) {
            const int b = wave_upper(offsets, a.B, wave == 0 ? c.first : end - 1);
            if (lane == 0)
                s_bag[wave] = b;
        }
        __syncthreads();
    } else {
        for (int i = tid; i < st.nb; i += kSortThreads)
            s_next[i] = a.bstart[(int64_t)st.part * kMaxBuckets + i] + a.hist[(int64_t)blockIdx.x * kMaxBuckets + i];
    }

    for (int k = 0; c.first + k * kSortTile < end; ++k) {
        const int first = c.first + k * kSortTile;
        const int m = min(kSortTile, end - first);
        const int groups = group_count<kPartGroup>(m), rounds = groups * kPartGroup;
        const int p0 = wave * rounds * kWave + lane;
        int lo, hi;
        if constexpr (PIECES) {
            lo = s_bag[0];
            hi = s_bag[1];
        } else {
            lo = a.tile_bag[(int)blockIdx.x * a.tiles_per_chunk + k];
            // the next tile's first bag bounds this one's; the last tile of a chunk looks at the next chunk's first tile
            const bool more = first + m < st.start + st.n;
            hi = more ? a.tile_bag[first + m < end ? (int)blockIdx.x * a.tiles_per_chunk + k + 1
                                                   : ((int)blockIdx.x + 1) * a.tiles_per_chunk]
                      : a.B - 1;
        }
        const uint32_t carry = bags_of_positions(offsets, lo, hi, first, m, rounds, reinterpret_cast<uint32_t*>(s_w), s_wsum);
        zero_counts(s_cnt);
        W w[kSortPerThread];
        uint32_t rank[kSortPerThread];
        Borders::with_span(span, [&](auto sp) {
            constexpr int kSpan = decltype(sp)::value;
            const int q = opaque(p0);
#pragma unroll
            for (int r0 = 0; r0 < kSortPerThread; r0 += kPartGroup) {
                if (r0 < rounds) {
#pragma unroll
                    for (int r = r0; r < r0 + kPartGroup; ++r) {
                        const uint32_t row = dg[r], d = s_borders.bucket<kSpan>(row, shift, last_cell);
                        w[r] = ((W)(row + ~s_borders.below[d]) << a.vb) + (W)(max(s_mark[q + r * kWave], carry) - 1u);
                        dg[r] = d;
                    }
                }
            }
            if (m < kSortTile) {
#pragma unroll
                for (int r = 0; r < kSortPerThread; ++r)
                    dg[r] = q + r * kWave < m ? dg[r] : (uint32_t)st.nb;
            }
        });
        __syncthreads();
        rank_rounds<kPartGroup>([&](int r) { return dg[r]; }, groups, digit_bits, s_cnt, rank);
        __syncthreads();
        uint32_t counts;
        const uint32_t starts = digit_starts<kMaxBuckets>(s_cnt, s_wsum, counts);
        if constexpr (PIECES) {
            if (2 * tid <= st.nb)                     // (bucket nb starts behind the last word)
                reinterpret_cast<uint32_t*>(piece_starts(a, (int)blockIdx.x))[tid] = starts;
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int d = 2 * tid + i;
                if (d < st.nb) {
                    const uint32_t nx = s_next[d];
                    s_delta[d] = nx - (i ? starts >> 16 : starts & 0xffffu);
                    s_next[d] = nx + (i ? counts >> 16 : counts & 0xffffu);
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int r0 = 0; r0 < kSortPerThread; r0 += kPartGroup)
            if (r0 < rounds) {
#pragma unroll
                for (int r = r0; r < r0 + kPartGroup; ++r)
                    rank[r] += s_cnt[wave][dg[r]];    // slot of the word in the reordered tile
            }
        if constexpr (!PIECES)
            __syncthreads();                          // the counters become the slots' digits
#pragma unroll
        for (int r0 = 0; r0 < kSortPerThread; r0 += kPartGroup)
            if (r0 < rounds) {
#pragma unroll
                for (int r = r0; r < r0 + kPartGroup; ++r) {
                    s_w[rank[r]] = w[r];
                    if constexpr (!PIECES)
                        s_dig[rank[r]] = (uint16_t)dg[r];
                }
            }
        __syncthreads();
        if constexpr (PIECES) {
#pragma unroll
            for (int i = 0; i < kSortPerThread; ++i)
                if (i * kSortThreads + tid < m)
                    out[first + i * kSortThreads + tid] = s_w[i * kSortThreads + tid];
            return;                                   // a chunk is one tile
        }
        if (first + m < end)
            load_rows(first + m);                     // in flight while this tile is written
        // the words of a bucket are written together; four at a time so that the LDS reads overlap
        for (int i0 = 0; i0 < rounds; i0 += 4) {
            uint32_t to[4];
            W x[4];
            const int q = i0 * kSortThreads + tid;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                to[i] = s_dig[q + i * kSortThreads];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                to[i] = s_delta[to[i]] + (uint32_t)(q + i * kSortThreads);
                x[i] = s_w[q + i * kSortThreads];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (q + i * kSortThreads < m)
                    out[to[i]] = x[i];
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------- units: sort in LDS, runs

// One workgroup per unit.  A unit of more than kSortTile words -- a bucket the sample undersized, or of a table with
// more than kMaxBuckets * kSortTile lookups -- takes the same passes tile by tile through global memory.
//
// PIECES (a.mode is kSortPieces): the unit's words are collected first, its piece of every chunk of the table in turn.  Where the
// pieces start says how many lookups of the table go before the unit: no histogram, no second walk over the indices.  A unit
// that does not fit is collected in memory, where its keys will be.  8 tables, 0.66 M lookups: 16.7 us instead of 14.7, for 9.1
// of the histogram and 6.0 of the units; 64 tables, 6.2 M: 56 instead of 49, for 27 (the words of a unit are collected four a
// thread at a time: with eight, registers spill and every reload is a trip to memory, 22 us instead of 16.7).  Collecting is
// one pass more for a unit of several rows that does not fit: where the sample misses 1000 rows that have nearly all of
// 0.9 M lookups, the sort takes 4.3 ms instead of 3.7.
constexpr int kCollect = 4;

template <typename W, bool PIECES>
__global__ __launch_bounds__(kSortThreads, sizeof(W) == 4 ? 6 : 4) void sort_local_kernel(SortArgs a)
{
    static_assert(!PIECES || sizeof(W) == 4, "a unit is collected where its keys go");
    __shared__ uint32_t s_slot[PIECES ? kPiecesMax : 1];           // first slot of every chunk's piece in the unit ...
    __shared__ uint32_t s_from[PIECES ? kPiecesMax : 1];           // ... and where slot 0 would lie if all of the unit lay there
    __shared__ __align__(16) W s_w[kSortTile];
    __shared__ __align__(16) uint16_t s_cnt[kSortWaves][kLocalDigits];
    __shared__ uint32_t s_run[kLocalDigits];         // units larger than a tile: next slot of every digit
    __shared__ uint32_t s_wsum[kSortWaves];
    __shared__ uint32_t s_heads;
    __shared__ int s_ticket;
    __shared__ SortUnit s_unit;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = uniform(tid >> 6);
    const int total_units = (int)a.counters->sort_units;
    const W vmask = ((W)1 << a.vb) - 1;

    // Units beyond the grid are handed out one at a time (their sizes differ); the next number is asked for a unit ahead.
    // (All workgroups add to one word, at 6 ns each: no unit that has a workgroup of its own waits for that.)
    const bool tickets = total_units > (int)gridDim.x;
    for (int u = blockIdx.x; u < total_units;) {
        __syncthreads();
        if (tid < 8) {
            const int i = opaque(tid);
            reinterpret_cast<int*>(&s_unit)[i] = reinterpret_cast<const int*>(&a.units[u])[i];
        }
        if (tid == 0)
            s_heads = 0;
        __syncthreads();
        if (tid == 0)
            s_ticket = tickets ? (int)(gridDim.x + atomicAdd(&a.counters->sort_ticket, 1u)) : total_units;
        int start = uniform(s_unit.start), m_all = uniform(s_unit.m);
        const int bits = uniform(s_unit.bits);
        const uint32_t key0 = (uint32_t)uniform((int)s_unit.key0);
        bool large = m_all > kSortTile;
        int from_slot = 0;                           // (PIECES) first of the unit's slots, not 0 for a further part of a row
        const W* pieces = static_cast<const W*>(a.words[0]);
        if constexpr (PIECES) {
            const int table_start = start, flags = uniform(s_unit.flags);
            const int nchunks = flags & kUnitNone ? 0 : (m_all + a.chunk - 1) >> a.lg_chunk;
            const uint16_t* starts = piece_starts(a, uniform((int)s_unit.last)) + uniform((int)s_unit.bucket);
            uint32_t before = 0, slots = 0;
            for (int c0 = 0; c0 < nchunks; c0 += kSortThreads) {
                // (up to 64 chunks: every wavefront for itself)
                const bool few = nchunks <= kWave;
                const int c = few ? lane : c0 + tid;
                uint32_t s = 0, e = 0, sum;
                if (c < nchunks) {
                    s = starts[(int64_t)c * kPieceStarts];
                    e = starts[(int64_t)c * kPieceStarts + 1];
                }
                uint32_t slot = slots;
                if (few) {
                    const uint32_t incl = wave_scan_add(e - s);
                    slot = incl - (e - s);
                    sum = last_lane(incl);
                    before = last_lane(wave_scan_add(s));
                } else {
                    uint32_t ahead;
                    slot += block_scan<kSortThreads>(e - s, s_wsum, sum);
                    __syncthreads();
                    (void)block_scan<kSortThreads>(s, s_wsum, ahead);
                    __syncthreads();
                    before += ahead;
                }
                slots += sum;
                if (c < nchunks && (!few || wave == 0)) {
                    s_slot[c] = slot;
                    s_from[c] = (uint32_t)(table_start + c * a.chunk) + s - slot;
                }
            }
            __syncthreads();
            start = table_start + uniform((int)before);
            m_all = uniform((int)slots);
            // Of a row with several units this one's share.  Their number is the sample's guess: a tile each with the rest for
            // the last one, that one had a few tiles too many every other time (16 tables of 300 rows, 2 M Zipf lookups 58.4 us,
            // 54.5 with shares).  A row that the sample has missed altogether stays with one workgroup, 0.8 us for 1000
            // lookups of it: no input whose rows do not depend on mix_bits of their positions has one.
            if (bits == 0) {
                const uint32_t part = (uint32_t)flags >> 8 & 0xfffu, parts = ((uint32_t)flags >> 20) + 1u;
                from_slot = (int)((uint64_t)(uint32_t)m_all * part / parts);
                m_all = (int)((uint64_t)(uint32_t)m_all * (part + 1u) / parts) - from_slot;
                start += from_slot;
            }
            large = m_all > kSortTile;
            // The words go to LDS, those of a unit that does not fit where its keys will be, or are keys and payloads already if they
            // are of one row.  A wavefront has a stretch of the slots and walks the chunks that have them, the next 64 in its lanes.
#pragma unroll 1
            for (int first = 0; first < m_all; first += kSortTile) {
                const int m = min(kSortTile, m_all - first), rounds = group_count<kSortGroup>(m) * kSortGroup;
                const int q = wave * rounds * kWave, end = from_slot + first + m - 1;
                const int p0 = min(from_slot + first + q, end);
                int c = -1;                          // chunk of slot p0, the last one whose piece starts at or before it
                for (int i = 0; i < nchunks; i += kWave)
                    c += __popcll(__ballot(i + lane < nchunks && (int)s_slot[min(i + lane, nchunks - 1)] <= p0));
                int ahead = c;                       // lane i: chunk ahead + i
                uint32_t slot = s_slot[min(c + lane, nchunks - 1)], from = s_from[min(c + lane, nchunks - 1)];
                uint32_t here = (uint32_t)__builtin_amdgcn_readfirstlane((int)from);
#pragma unroll 1
                for (int r0 = 0; r0 < rounds; r0 += kCollect) {
                    W w[kCollect];
#pragma unroll
                    for (int r = 0; r < kCollect; ++r) {
                        if (r0 + r < rounds) {
                            const int p1 = p0 + (r0 + r) * kWave, p = min(p1 + lane, end);
                            uint32_t at = here;
                            while (c + 1 < nchunks) {
                                if (c + 1 - ahead == kWave) {
                                    ahead = c + 1;
                                    slot = s_slot[min(ahead + lane, nchunks - 1)];
                                    from = s_from[min(ahead + lane, nchunks - 1)];
                                }
                                const int next = __builtin_amdgcn_readlane((int)slot, c + 1 - ahead);
                                if (next >= p1 + kWave)
                                    break;
                                ++c;
                                here = (uint32_t)__builtin_amdgcn_readlane((int)from, c - ahead);
                                at = p >= next ? here : at;
                            }
                            w[r] = pieces[at + (uint32_t)p];
                        }
                    }
#pragma unroll
                    for (int r = 0; r < kCollect; ++r) {
                        const int i = q + (r0 + r) * kWave + lane;
                        if (r0 + r < rounds) {
                            if (!large)
                                s_w[i] = i < m ? w[r] : ~(W)0;
                            else if (i < m && bits > 0)
                                a.keys[start + first + i] = (uint32_t)w[r];
                            else if (i < m) {
                                a.keys[start + first + i] = key0 + (uint32_t)(w[r] >> a.vb);
                                a.vals[start + first + i] = (int32_t)(w[r] & vmask);
                            }
                        }
                    }
                }
            }
            __syncthreads();
        }
        const int passes = (bits + 7) >> 3;
        W* src = (PIECES ? reinterpret_cast<W*>(a.keys) : static_cast<W*>(a.words[0])) + start;
        W* dst = (PIECES ? reinterpret_cast<W*>(a.vals) : static_cast<W*>(a.words[1])) + start;
        int sh = a.vb;
        for (int p = 0; p < passes; ++p) {
            const int width = pass_width(bits, passes, p);
            const uint32_t mask = (1u << width) - 1u;
            if (large) {                             // first slot of every digit in the unit
                if (tid < kLocalDigits)
                    s_run[tid] = 0;
                __syncthreads();
#pragma unroll 1
                for (int i = tid; i < m_all; i += kSortThreads)
                    atomicAdd(&s_run[(uint32_t)(src[i] >> sh) & mask], 1u);
                __syncthreads();
                uint32_t tot;
                const uint32_t ex = block_scan<kSortThreads>(tid < kLocalDigits ? s_run[tid] : 0u, s_wsum, tot);
                if (tid < kLocalDigits)
                    s_run[tid] = ex;
                __syncthreads();
            }
#pragma unroll 1
            for (int first = 0; first < m_all; first += kSortTile) {
                const int m = min(kSortTile, m_all - first);
                const int groups = group_count<kSortGroup>(m);
                const int p0 = wave * groups * kSortGroup * kWave + lane;
                W w[kSortPerThread];
                zero_counts(s_cnt);
                {
                    const int q = opaque(p0);
                    const W* from = src + first;
                    if ((large || (!PIECES && p == 0)) && (wave + 1) * groups * kSortGroup * kWave <= m) {   // all of the wavefront's words
#pragma unroll
                        for (int r = 0; r < kSortPerThread; ++r)
                            if (r < groups * kSortGroup)
                                w[r] = load_at(from, (uint32_t)q, r * kWave);
                    } else if (large || (!PIECES && p == 0)) {
#pragma unroll
                        for (int r = 0; r < kSortPerThread; ++r)
                            if (r < groups * kSortGroup)
                                w[r] = q + r * kWave < m ? from[q + r * kWave] : ~(W)0;
                    } else {
#pragma unroll
                        for (int r = 0; r < kSortPerThread; ++r)
                            if (r < groups * kSortGroup)
                                w[r] = s_w[q + r * kWave];
                    }
                }
                __syncthreads();
                block_sort_pass(w, groups, sh, width, s_w, s_cnt, s_wsum);
                if (large) {
                    // The tile is in digit order in s_w and the digits' last wavefront row ends where the next digit
                    // starts: slot in the tile -> slot in the unit
                    uint32_t counts_lo = 0, counts_hi = 0, first_lo = 0, first_hi = 0;
                    if (2 * tid < kLocalDigits) {
                        const uint32_t f = reinterpret_cast<const u32_alias*>(s_cnt[0])[tid];
                        first_lo = f & 0xffffu;
                        first_hi = f >> 16;
                        const uint32_t f2 = 2 * tid + 2 < kLocalDigits ? s_cnt[0][2 * tid + 2] : (uint32_t)(groups * kSortGroup * kSortThreads);
                        counts_lo = first_hi - first_lo;
                        counts_hi = f2 - first_hi;
                    }
                    __syncthreads();
                    if (2 * tid < kLocalDigits) {
                        const uint32_t r_lo = s_run[2 * tid], r_hi = s_run[2 * tid + 1];
                        reinterpret_cast<u32_alias*>(s_cnt)[2 * tid] = r_lo - first_lo;       // (the counters are done with)
                        reinterpret_cast<u32_alias*>(s_cnt)[2 * tid + 1] = r_hi - first_hi;
                        s_run[2 * tid] = r_lo + counts_lo;
                        s_run[2 * tid + 1] = r_hi + counts_hi;
                    }
                    __syncthreads();
#pragma unroll 1
                    for (int i = tid; i < m; i += kSortThreads) {
                        const W x = s_w[i];
                        dst[reinterpret_cast<const u32_alias*>(s_cnt)[(uint32_t)(x >> sh) & mask] + (uint32_t)i] = x;
                    }
                    __syncthreads();
                }
            }
            if (large) {
                W* x = src; src = dst; dst = x;
            }
            sh += width;
        }
        // ---- keys and payloads; words that lie in LDS (sorted here) or in memory (large units, and buckets of one
        // row, which are sorted as they are)
        uint32_t heads = 0;
        if ((PIECES || bits > 0) && !large) {
            const int groups = group_count<kSortGroup>(m_all);
            const int q = opaque(wave * groups * kSortGroup * kWave + lane);
            uint32_t* keys = a.keys + start;
            int32_t* vals = a.vals + start;
            auto emit = [&](auto all) {
                constexpr bool kAll = decltype(all)::value;      // the wavefront has words in every round
#pragma unroll
                for (int r = 0; r < kSortPerThread; ++r) {
                    if (r < groups * kSortGroup) {
                        const int p = q + r * kWave;
                        const W x = s_w[p], before = s_w[r == 0 ? max(p, 1) - 1 : p - 1];
                        const bool other = ((x ^ before) >> a.vb) != 0 || (r == 0 && p == 0);
                        heads += (kAll || p < m_all) && other ? 1u : 0u;
                        if (kAll || p < m_all) {
                            store_at(keys, (uint32_t)q, r * kWave, key0 + (uint32_t)(x >> a.vb));
                            store_at(vals, (uint32_t)q, r * kWave, (int32_t)(x & vmask));
                        }
                    }
                }
            };
            if ((wave + 1) * groups * kSortGroup * kWave <= m_all)
                emit(std::true_type());
            else
                emit(std::false_type());
        } else {
            if (large && bits > 0) {
#pragma unroll 1
                for (int i = opaque(tid); i < m_all; i += kSortThreads)
                    heads += i == 0 || (src[i] >> a.vb) != (src[i - 1] >> a.vb) ? 1u : 0u;
                __syncthreads();                     // 32-bit words lie where keys or payloads go
            } else if (!PIECES && tid == 0 && !(s_unit.flags & kUnitContinued)) {
                heads = 1;
            }
#pragma unroll 4
            for (int i = PIECES && bits == 0 ? m_all : opaque(tid); i < m_all; i += kSortThreads) {
                const W x = src[i];
                a.keys[start + i] = key0 + (uint32_t)(x >> a.vb);
                a.vals[start + i] = (int32_t)(x & vmask);
            }
        }
        if (PIECES && bits == 0)                     // one run, of the row's first unit
            heads = tid == 0 && m_all > 0 && from_slot == 0 ? 1u : 0u;
        heads = last_lane(wave_scan_add(heads));
        if (lane == 0 && heads > 0)
            atomicAdd(&s_heads, heads);
        __syncthreads();
        if (tid == 0) {
            a.unit_runs[u] = s_heads;
            if (PIECES) {
                a.units[u].start = start;
                a.units[u].m = m_all;
            }
            atomicAdd(&a.table_runs[s_unit.t], s_heads);
        }
        u = s_ticket;                                // (written before the barrier above, at the latest)
    }
}

// ---------------------------------------------------------------- middle calls: every unit finds its lookups itself
//
// In a call of some 100,000 lookups the launches of the partition (histogram, units, scatter) each cost their latency and
// little else.  Here the workgroup of a unit reads all indices of the unit's table instead, out of L2, and keeps those
// of its own rows: table lookups x units index reads in all, but nothing to wait for between the plan and the sort.
// It reads them twice.  The first time every wavefront counts the lookups of its own rows and of earlier ones in a stretch of
// the table, which says where the unit starts and where the stretch's go; the second time they are put there, in order.
// Neither waits for the other wavefronts.  Read once, in steps whose counts all wavefronts exchange, 4096 positions took 1.3 us;
// now 0.6.  Bound by latency and, from some 20,000 lookups of a table on, by that walk.  40 tables, 0.17 M lookups: 15 us, where
// histogram, units, scatter and bucket sort took 47; 11 tables, one with 200,000 lookups: 45 us, 53 (in steps 75).
constexpr int kSelectWords = kSelectCap / kSortThreads;
constexpr int kSelectPer = 12;                    // positions per thread and block (200,000 lookups of a table: 16 are 4 us slower, 8 the same)
constexpr int kSelectCoarse = kSortThreads;       // bag borders in LDS: every (B / 512)-th (every (B / 4096)-th: no faster)

template <typename W>
__global__ __launch_bounds__(kSortThreads, sizeof(W) == 4 ? 4 : 2) void sort_select_kernel(SortArgs a)
{
    static_assert(kSelectCap % (kSortGroup * kSortThreads) == 0 && kSelectCap <= kSortTile, "");
    // positions of the unit's lookups in the table, then their row offsets and later their words; the positions of a single
    // row's take all of it, kSelectRow at a time
    __shared__ __align__(16) uint32_t s_pos[kSelectCap * (1 + sizeof(W) / 4)];
    W* s_w = reinterpret_cast<W*>(s_pos + kSelectCap);
    constexpr int kSelectRow = kSelectCap * (1 + sizeof(W) / 4);
    __shared__ __align__(16) uint16_t s_cnt[kSortWaves][kLocalDigits];
    __shared__ int32_t s_coarse[kSelectCoarse];
    __shared__ uint32_t s_below[kSortWaves], s_hits[kSortWaves], s_wsum[kSortWaves];
    __shared__ uint32_t s_heads;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = uniform(tid >> 6);
    const int total_units = (int)a.counters->sort_units;
    const W vmask = ((W)1 << a.vb) - 1;
    for (int u = blockIdx.x; u < total_units; u += gridDim.x) {
        const SortUnit un = a.units[u];
        if (un.flags & kUnitNone) {                  // fewer buckets than there could be
            if (tid == 0) {
                a.units[u].m = 0;
                a.unit_runs[u] = 0;
            }
            continue;
        }
        const int n = uniform(un.m), t = uniform(un.t), table_start = uniform(un.start);
        const uint32_t unit_key = (uint32_t)uniform((int)un.key0), unit_last = (uint32_t)uniform((int)un.last);
        const __amdgpu_buffer_rsrc_t idx = row_buffer(a.indices + table_start, 4ull * (uint32_t)n);
        const int64_t* __restrict__ offsets = a.offsets + (int64_t)t * a.B;
        const int lg_each = max(0, ceil_log2((uint32_t)a.B) - 9);      // bags per coarse border
        static_assert(kSelectCoarse == 1 << 9, "");
        __syncthreads();
        s_coarse[tid] = (int64_t)tid << lg_each < a.B ? (int)offsets[tid << lg_each] - table_start : INT32_MAX;
        if (tid == 0)
            s_heads = 0;
        // bag of a position: the last one that starts at or before it
        auto bag_of = [&](int pos) {
            int c = 0;
#pragma unroll
            for (int s = kSelectCoarse / 2; s > 0; s >>= 1)
                c += s_coarse[c + s] <= pos ? s : 0;
            int b = c << lg_each, lg = lg_each;
            auto starts = [&](int bag) { return (int)offsets[min(bag, a.B)] - table_start <= pos ? 1 : 0; };
            for (; lg > 1; lg -= 2) {
                const int quarter = 1 << (lg - 2);
                b += (starts(b + quarter) + starts(b + 2 * quarter) + starts(b + 3 * quarter)) * quarter;
            }
            if (lg > 0)
                b += starts(b + 1);
            return (uint32_t)b;
        };
        // Every wavefront reads a stretch of the table's positions, block by block, the first out of registers: use(key, at, full)
        // with its positions from `at` on, all of them or (full false) those before `end`.
        constexpr int kBlock = kSelectPer * kWave;
        const int each = (n + kSortWaves * kWave - 1) / (kSortWaves * kWave) * kWave;
        const int begin = min(wave * each, n), end = min(begin + each, n);
        uint32_t first_block[kSelectPer];
        auto load = [&](uint32_t (&key)[kSelectPer], int at) {     // behind the table: 0
            const int from = opaque((at + lane) * 4) & 0x7fffff;        // (seen not to be negative, the rest goes into the instruction)
            static_assert(kSelectLookups + 2 * kBlock <= 0x7fffff / 4, "");
#pragma unroll
            for (int r = 0; r < kSelectPer; ++r)
                key[r] = __builtin_amdgcn_raw_buffer_load_b32(idx, from + r * kWave * 4, 0, 0);
            __builtin_amdgcn_sched_barrier(0);                     // (not behind the block before it)
        };
        auto walk = [&](auto use) {
            uint32_t even[kSelectPer], odd[kSelectPer];
#pragma unroll
            for (int r = 0; r < kSelectPer; ++r)
                even[r] = first_block[r];
            int at = begin;
            for (; at + 2 * kBlock <= end; at += 2 * kBlock) {
                load(odd, at + kBlock);
                use(even, at, std::true_type());
                load(even, at + 2 * kBlock);
                use(odd, at + kBlock, std::true_type());
            }
            if (at + kBlock <= end) {
                load(odd, at + kBlock);
                use(even, at, std::true_type());
                at += kBlock;
#pragma unroll
                for (int r = 0; r < kSelectPer; ++r)
                    even[r] = odd[r];
            }
            use(even, at, std::false_type());
        };
        // keys and payloads of a single row's m lookups in LDS
        auto emit_row = [&](uint32_t key, int at, int m) {
#pragma unroll 4
            for (int i = tid; i < m; i += kSortThreads) {
                a.keys[at + i] = key;
                a.vals[at + i] = (int32_t)bag_of((int)s_pos[i]);
            }
        };
        // One part for all rows of the unit as a rule.  If they have more lookups than fit the LDS (the sample undersized the
        // bucket) they are cut; the lookups of a single row need no sorting and leave in as many turns as it takes.
        const uint32_t table_key = (uint32_t)uniform((int)a.row_base[t]);
        const uint32_t table_rows = (uint32_t)uniform((int)a.row_base[t + 1]) - table_key;
        const uint32_t first_row = unit_key - table_key;
        const uint32_t unit_rows = min(unit_last, table_rows - first_row - 1u) + 1u;
        uint32_t lo = 0, rows = unit_rows, heads = 0;             // the rows [lo, lo + rows) of the unit
        int unit_start = 0, unit_m = 0, all = -1;
        while (lo < unit_rows) {
            const uint32_t row0 = first_row + lo, key0 = unit_key + lo;
            const uint32_t last = lo + rows == unit_rows ? unit_last - lo : rows - 1u;
            const uint32_t top = row0 + last;
            const bool single = rows == 1;
            load(first_block, begin);
            uint32_t below = 0, upto = 0;
            walk([&](const uint32_t (&key)[kSelectPer], int at, auto full) {
#pragma unroll
                for (int r = 0; r < kSelectPer; ++r) {
                    const bool valid = full || at + r * kWave + lane < end;
                    below += valid && key[r] < row0 ? 1u : 0u;
                    upto += valid && key[r] <= top ? 1u : 0u;
                }
            });
            below = last_lane(wave_scan_add(below));
            upto = last_lane(wave_scan_add(upto));
            __syncthreads();
            if (lane == 0) {
                s_below[wave] = below;
                s_hits[wave] = upto - below;
            }
            __syncthreads();
            below = first_lanes_scan_add<kSortWaves>(lane < kSortWaves ? s_below[lane] : 0u);
            const uint32_t hits = first_lanes_scan_add<kSortWaves>(lane < kSortWaves ? s_hits[lane] : 0u);
            const int start = table_start + __builtin_amdgcn_readlane((int)below, kSortWaves - 1);
            const int m = __builtin_amdgcn_readlane((int)hits, kSortWaves - 1);
            const int next_slot = __builtin_amdgcn_readlane((int)hits, wave);
            const int first_slot = wave == 0 ? 0 : __builtin_amdgcn_readlane((int)hits, max(wave, 1) - 1);
            if (all < 0)
                all = m;
            if (m > kSelectCap && !single) {
                rows = select_fewer_rows(rows, m);
                continue;
            }
            // put(slot, row offset, position) for each of them, in position order
            auto select = [&](auto put) {
                uint32_t slot = (uint32_t)first_slot;
                // (compared again: no masks are kept of the first block)
                const uint32_t from = (uint32_t)uniform(opaque((int)row0)), to = (uint32_t)uniform(opaque((int)top));
                walk([&](const uint32_t (&key)[kSelectPer], int at, auto full) {
                    const int from_pos = opaque(at + lane);
#pragma unroll
                    for (int r = 0; r < kSelectPer; ++r) {
                        const int pos = from_pos + r * kWave;
                        const uint64_t mine = __ballot(key[r] <= to) & ~__ballot(key[r] < from) & (full ? ~0ull : __ballot(pos < end));
                        if (mine != 0) {
                            if (__builtin_amdgcn_inverse_ballot_w64(mine))
                                put(__builtin_amdgcn_mbcnt_hi((uint32_t)(mine >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mine, slot)),
                                    key[r] - row0, (uint32_t)pos);
                            slot += (uint32_t)__popcll(mine);
                        }
                    }
                });
            };
            // (of a row with several units this one's part, the last takes the rest)
            const int part = un.flags >> 8;
            const int from_slot = min(part * kSelectPart, m), to_slot = un.flags & kUnitMore ? min((part + 1) * kSelectPart, m) : m;
            if (single) {
                for (int done = from_slot; done < to_slot; done += kSelectRow) {
                    if (first_slot < min(done + kSelectRow, to_slot) && next_slot > done)
                        select([&](uint32_t slot, uint32_t, uint32_t pos) {
                            if (slot - (uint32_t)done < (uint32_t)kSelectRow)
                                s_pos[slot - done] = pos;
                        });
                    __syncthreads();
                    emit_row(key0, start + done, min(kSelectRow, to_slot - done));
                    __syncthreads();
                }
            } else if (m > 0) {
                zero_counts(s_cnt);
                select([&](uint32_t slot, uint32_t row, uint32_t pos) {
                    s_pos[slot] = pos;
                    s_w[slot] = (W)row;
                });
                __syncthreads();
#pragma unroll 4
                for (int i = tid; i < m; i += kSortThreads)
                    s_pos[i] = bag_of((int)s_pos[i]);
                __syncthreads();
                uint32_t* keys = a.keys + start;
                int32_t* vals = a.vals + start;
                const int groups = group_count<kSortGroup>(m);
                const int p0 = opaque(wave * groups * kSortGroup * kWave + lane);
                W w[kSelectWords];
#pragma unroll
                for (int r = 0; r < kSelectWords; ++r) {
                    if (r < groups * kSortGroup) {
                        const int p = p0 + r * kWave;
                        w[r] = p < m ? (s_w[p] << a.vb) | (W)s_pos[p] : ~(W)0;
                    }
                }
                __syncthreads();
                block_sort(w, groups, a.vb, ceil_log2(rows), s_w, s_cnt, s_wsum);
#pragma unroll
                for (int r = 0; r < kSelectWords; ++r) {
                    const int p = p0 + r * kWave;
                    if (r < groups * kSortGroup && p < m) {
                        const W x = s_w[p], before = s_w[max(p, 1) - 1];
                        heads += p == 0 || ((x ^ before) >> a.vb) != 0 ? 1u : 0u;
                        keys[p] = key0 + (uint32_t)(x >> a.vb);
                        vals[p] = (int32_t)(x & vmask);
                    }
                }
            }
            heads += single && tid == 0 && part == 0 && m > 0 ? 1u : 0u;
            if (lo == 0)
                unit_start = start + from_slot;
            unit_m += to_slot - from_slot;
            lo += rows;
            if (unit_m == all)
                break;
            rows = select_next_rows(rows, m, unit_rows - lo, all - unit_m);
        }
        heads = last_lane(wave_scan_add(heads));
        if (lane == 0 && heads > 0)
            atomicAdd(&s_heads, heads);
        __syncthreads();
        if (tid == 0) {
            a.units[u].start = unit_m > 0 ? unit_start : 0;
            a.units[u].m = unit_m;
            a.unit_runs[u] = s_heads;
            atomicAdd(&a.table_runs[t], s_heads);
        }
    }
}

// ---------------------------------------------------------------- small calls: all of it in one workgroup
//
// At most kSortTile lookups in at most kSmallBags bags: one workgroup finds every lookup's bag, sorts (linear row id,
// bag) words in LDS and writes keys, payloads and runs.  A small call is a chain of launches of 2 to 5 us each, most
// of them with nothing to do: 2048 lookups took 13 launches and 55 us, then three and 20 us with the kernels above.
constexpr int kSmallBags = 1 << 15;

__global__ __launch_bounds__(kSortThreads) void sort_small_kernel(SortArgs a, int key_bits)
{
    __shared__ __align__(16) uint64_t s_w[kSortTile];
    __shared__ __align__(16) uint16_t s_cnt[kSortWaves][kLocalDigits];
    __shared__ uint32_t s_wsum[kSortWaves], s_long;
    __shared__ uint16_t s_starts[kSortTile + 1];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int n = a.n;
    const int groups = group_count<kSortGroup>(n), rounds = groups * kSortGroup;
    const int p0 = wave * rounds * kWave + lane;
    const int table_start = tid <= a.T ? (int)a.offsets[(int64_t)tid * a.B] : 0;
    uint32_t index[kSortPerThread];                  // on their way while the bags are found
#pragma unroll
    for (int r = 0; r < kSortPerThread; r += kSortGroup)
        if (r < rounds) {
#pragma unroll
            for (int x = 0; x < kSortGroup; ++x)
                index[r + x] = a.indices[min(p0 + (r + x) * kWave, n - 1)];
        }
    zero_counts(s_cnt);
    const uint32_t* s_mark = reinterpret_cast<const uint32_t*>(s_w);
    const uint32_t carry = bags_of_positions(a.offsets, 0, a.T * a.B - 1, 0, n, rounds, reinterpret_cast<uint32_t*>(s_w), s_wsum);
    uint64_t w[kSortPerThread];
    {
        const int q = opaque(p0);
#pragma unroll
        for (int r = 0; r < kSortPerThread; ++r) {
            if (r < rounds) {
                const int p = q + r * kWave;
                const uint32_t bag = max(s_mark[p], carry) - 1u;
                const uint32_t t = a.T == 1 ? 0u : bag / (uint32_t)a.B;
                w[r] = p < n ? (uint64_t)((a.T == 1 ? 0u : a.row_base[t]) + index[r]) << 32 | (bag - t * (uint32_t)a.B) : ~0ull;
            }
        }
    }
    __syncthreads();
    block_sort(w, groups, 32, key_bits, s_w, s_cnt, s_wsum);
    uint32_t mask = 0, mine = 0;
    const int q = opaque(p0);
#pragma unroll
    for (int r = 0; r < kSortPerThread; ++r) {
        if (r < rounds) {
            const int p = q + r * kWave;
            w[r] = s_w[p];
            const bool head = p < n && (p == 0 || (uint32_t)(s_w[max(p, 1) - 1] >> 32) != (uint32_t)(w[r] >> 32));
            mask |= (head ? 1u : 0u) << r;
            mine += (uint32_t)__popcll(__ballot(head));
        }
    }
    __syncthreads();
    if (lane == 0)
        s_wsum[wave] = mine;
    __syncthreads();
    uint32_t run = 0, total = 0;
#pragma unroll
    for (int i = 0; i < kSortWaves; ++i) {
        run += i < wave ? s_wsum[i] : 0u;
        total += s_wsum[i];
    }
#pragma unroll
    for (int r = 0; r < kSortPerThread; ++r) {
        if (r < rounds) {
            const int p = q + r * kWave;
            const uint64_t hm = __ballot((mask >> r & 1u) != 0u);
            const uint32_t x = run + __builtin_amdgcn_mbcnt_hi((uint32_t)(hm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hm, 0u));
            if (p < n) {
                a.keys[p] = (uint32_t)(w[r] >> 32);
                a.vals[p] = (int32_t)w[r];
                if ((p & (kSpanUnit - 1)) == 0)
                    a.unit_first_run[p / kSpanUnit] = (int32_t)x;
                if (mask >> r & 1u) {
                    a.unique_keys[x] = (uint32_t)(w[r] >> 32);
                    a.seg_offsets[x] = p;
                    s_starts[x] = (uint16_t)p;
                }
            }
            run += (uint32_t)__popcll(hm);
        }
    }
    // the long runs, for the update
    if (tid == 0) {
        s_starts[total] = (uint16_t)n;
        s_long = 0;
    }
    __syncthreads();
    for (uint32_t x = tid; x < total; x += kSortThreads)
        if (s_starts[x + 1] - s_starts[x] > kPosPiece)
            a.small_long[1 + atomicAdd(&s_long, 1u)] = x;
    __syncthreads();
    for (int t = tid; t <= a.T; t += kSortThreads)
        a.tstart[t] = t < kSortThreads ? table_start : (int)a.offsets[(int64_t)t * a.B];
    if (tid == 0) {
        a.small_long[0] = s_long;
        a.seg_offsets[total] = n;
        a.unit_first_run[(n + kSpanUnit - 1) / kSpanUnit] = (int32_t)total;
        a.counters->num_unique = (int64_t)total;
    }
}

// Runs: a run starts where the key changes; a unit's first run is the runs of the tables before its own plus those
// of the units before it in its table, so a workgroup sums those counts itself.  A thread owns 16 consecutive
// positions (one count per thread to scan instead of a ballot per 64 positions); the runs are collected in LDS and
// written together.
constexpr int kRunThreads = 256;
constexpr int kRunPer = 16;
constexpr int kRunTile = kRunThreads * kRunPer;
static_assert(kRunPer <= kSpanUnit, "a thread writes the first run of one span unit at most");
__global__ __launch_bounds__(kRunThreads) void sort_runs_kernel(SortArgs a)
{
    __shared__ uint32_t s_key[kRunTile];
    __shared__ int32_t s_pos[kRunTile];
    __shared__ uint32_t s_wsum[2][kRunThreads / kWave];
    const int tid = threadIdx.x;
    const int total_units = (int)a.counters->sort_units;
    for (int u = blockIdx.x; u < total_units; u += gridDim.x) {
        const SortUnit un = a.units[u];
        const uint32_t unit_runs = a.unit_runs[u];
        if (un.m == 0)
            continue;
        uint32_t part = 0, run;
        for (int i = tid; i < un.t; i += kRunThreads)
            part += a.table_runs[i];
        for (int i = un.first + tid; i < u; i += kRunThreads)
            part += a.unit_runs[i];
        __syncthreads();
        (void)block_scan<kRunThreads>(part, s_wsum[0], run);
        if (tid == 0 && un.start + un.m == a.n) {    // the last unit of the last table
            const uint32_t all = run + unit_runs;
            a.seg_offsets[all] = a.n;
            a.unit_first_run[(a.n + kSpanUnit - 1) / kSpanUnit] = (int32_t)all;
            a.counters->num_unique = (int64_t)all;
        }
        if (un.bits == 0) {                          // one row: at most one run, and nothing to compare
            if (tid == 0 && unit_runs > 0) {
                a.unique_keys[run] = un.key0;
                a.seg_offsets[run] = un.start;
            }
            const int first = (un.start + kSpanUnit - 1) / kSpanUnit, last = (un.start + un.m - 1) / kSpanUnit;
            for (int i = first + tid; i <= last; i += kRunThreads)
                a.unit_first_run[i] = (int32_t)(run + (i * kSpanUnit > un.start ? unit_runs : 0u));
            continue;
        }
        for (int first = 0; first < un.m; first += kRunTile) {
            const int m = min(kRunTile, un.m - first);
            const int g0 = un.start + first + tid * kRunPer;
            const int mine = min(max(m - tid * kRunPer, 0), kRunPer);
            uint32_t key[kRunPer], before = 0, mask = 0;
            if (mine == kRunPer) {
#pragma unroll
                for (int i = 0; i < kRunPer; ++i)    // (combined into 16-byte loads)
                    key[i] = a.keys[g0 + i];
            } else {
#pragma unroll
                for (int i = 0; i < kRunPer; ++i)
                    key[i] = i < mine ? a.keys[g0 + i] : 0u;
            }
            if (mine > 0 && first + tid > 0)
                before = a.keys[g0 - 1];
#pragma unroll
            for (int i = 0; i < kRunPer; ++i)
                mask |= (key[i] != (i == 0 ? before : key[i - 1]) ? 1u : 0u) << i;
            if (first + tid == 0)
                mask |= 1u;                          // borders of buckets are borders of runs
            mask &= (1u << mine) - 1u;
            uint32_t tile_runs;
            uint32_t at = block_scan<kRunThreads>((uint32_t)__popc(mask), s_wsum[1], tile_runs);
            // runs before the first position of this thread's that starts a span unit
            const int k = (0 - g0) & (kSpanUnit - 1);
            if (k < mine)
                a.unit_first_run[(g0 + k) / kSpanUnit] = (int32_t)(run + at + (uint32_t)__popc(mask & ((1u << k) - 1u)));
#pragma unroll
            for (int i = 0; i < kRunPer; ++i) {
                if (mask >> i & 1u) {
                    s_key[at] = key[i];
                    s_pos[at] = g0 + i;
                    ++at;
                }
            }
            __syncthreads();
            for (int i = tid; i < (int)tile_runs; i += kRunThreads) {
                a.unique_keys[run + i] = s_key[i];
                a.seg_offsets[run + i] = s_pos[i];
            }
            run += tile_runs;
            __syncthreads();
        }
    }
}

}  // namespace tbe
