// Launch rules and index arithmetic of the embedding library in plain C++: used by the host code and the kernels, and
// checked on the CPU at sizes and values that a GPU test could not take (tests/test_rules.py).
#pragma once

#include <algorithm>
#include <cstdint>

#ifdef __HIPCC__
#define TBE_BOTH __host__ __device__ __forceinline__
#else
#define TBE_BOTH inline
#endif

namespace tbe {

constexpr int kWave = 64;

// A launch holds fewer than 2^32 threads.
constexpr int64_t kMaxLaunchThreads = ((int64_t)1 << 32) - 1;

// ---------------------------------------------------------------- forward

constexpr int kFwdThreads = 256;          // 4 wavefronts per workgroup, each with its own block of bags
constexpr int kFwdMaxBagsPerWave = 8;     // measured best on configs 2-4 (4..32 tried)
// forward_bag_kernel (one bag per wavefront) takes a call ...
// ... of fewer than kFewBags bags that hold few_bags_lookups() lookups on average.  forward_kernel has one bag per wavefront
//     there too and leaves all lane groups but one idle; from 32,768 bags it packs several (fp32 dim 64, 8 lookups:
//     24,000 bags 15.0 against 11.6 us, 40,000 bags 15.0 against 17.6).  Shorter bags have little to spread and pay for the
//     sum over the lane groups: a step of it moves 4 or 8 values per lane, and there are the more steps the narrower the
//     rows.  8000 bags, forward_kernel / this one: fp32 dim 16, 4 lookups 3.5 / 4.1 us, 6 lookups 4.5 / 4.1; dim 128, 4 lookups
//     4.4 / 4.7; fp16 dim 64, 4 lookups 3.9 / 4.6, 6 lookups 4.9 / 4.6; dim 8, 8 lookups 5.2 / 6.2, 12 lookups 6.6 / 6.2;
// ... of any size if every table's row fills the wavefront and a bag holds kWideBagLookups lookups on average: there
//     is no lane group to spread over, but up to 8 rows in flight instead of 4.  131,072 bags: fp32 dim 256, 16 lookups
//     174 against 154 us, dim 512, 24 lookups 463 against 400; fp16 dim 384, 16 lookups 179 against 166.
//     Its launch has 64 threads per bag: kMaxLaunchThreads ends that at 2^26 bags.
constexpr int kFewBags = 32768;
constexpr int kWideBagLookups = 16;

// epl: elements per lane; narrowest: log2 of the fewest lanes that a table's row takes
inline int few_bags_lookups(int epl, int narrowest) { return epl == 8 && narrowest < 2 ? 9 : 6; }

struct ForwardLaunch {
    bool one_bag;          // forward_bag_kernel
    int bags_per_wave;     // of forward_kernel, which holds a wavefront's borders in its lanes: at most kWave - 1
    int64_t blocks;
};

// few: few_bags_lookups(); wide: every table's row takes all lanes of a wavefront
inline ForwardLaunch forward_launch(int64_t num_bags, int64_t lookups, int few, bool wide)
{
    constexpr int64_t kMaxBlocks = kMaxLaunchThreads / kFwdThreads, kWaves = kFwdThreads / kWave;
    ForwardLaunch f;
    f.one_bag = ((num_bags < kFewBags && lookups >= few * num_bags) || (wide && lookups >= kWideBagLookups * num_bags)) &&
                num_bags <= kMaxBlocks * kWaves;
    // enough bags to amortise the per-block prologue, few enough to keep >= ~16k wavefronts in the grid when the batch
    // is small; beyond 2^29 bags as many as the largest launch needs
    const int64_t fewest = (num_bags + kMaxBlocks * kWaves - 1) / (kMaxBlocks * kWaves);
    const int64_t per_wave = std::min<int64_t>(kFwdMaxBagsPerWave, num_bags / 16384);
    f.bags_per_wave = f.one_bag ? 1 : (int)std::max<int64_t>({1, fewest, per_wave});
    const int64_t per_block = kWaves * f.bags_per_wave;
    f.blocks = (num_bags + per_block - 1) / per_block;
    return f;
}

// ---------------------------------------------------------------- update: spans

// Sorted positions that a wavefront of the update kernel owns.  What a span costs is a chain: its descriptors, then steps of
// 64 / lanes rows or a few times that (lanes: of a row, 8 columns each), so a call that leaves the chip room for more
// wavefronts takes shorter spans, the shorter the wider its rows.  Short spans of narrow rows only fill their steps worse
// and stage more often.  kSpanWaves wavefronts per lane of a row (mean of the tables) is where the two meet; update
// kernel, us, spans of 16 / 32 / 64 / 128: dims 4..512, 0.17 M lookups 34 / 37 / 61 / 112; 384 columns, 3444
// lookups 20 / 32 / 56 / 100; 128 columns, 0.65 M 142 / 144 / 151 / 157, 2 M in fp16 114 / 100 / 108 / 121, 6.2 M in 16 bits
// 423 / 355 / 320 / 305; 256 columns, 1 M 157 / 165 / 178 / 200; 512, 4 M 625 / 631 / 641 / 644; 64, 1.2 M 65 / 52 / 48 / 53;
// 16, 1 M 64 / 40 / 33 / 33; 8, 0.16 M 15 / 13 / 13 / 14.
// The mean is over tables whatever their share of the lookups: seven tables of 8 columns with 25,000 each beside one of 512 with
// 1000 take spans of 16, 22 us (64 with spans of 64 and long runs in launches of their own).
constexpr int64_t kSpanWaves = 4096;

// lanes: of a row, added up over the tables
inline int update_span(int64_t lookups, int64_t lanes, int64_t tables)
{
    for (int span = 16; span < 128; span *= 2)
        if (lookups <= span * kSpanWaves * lanes / tables)
            return span;
    return 128;
}

// ---------------------------------------------------------------- update: long runs

constexpr int kLongRun = 512;             // a run of more lookups is long: other kernels than the update kernel sum it, in pieces
// Largest gradient block of a table (bytes) up to which long runs are cut by position, beyond it by bag window.  While the
// block fits the 4 MiB of an L2 the windows bring no locality: batch 611, dims to 512: 28 us for all long runs instead of
// 245; batch 8191, 128 bf16 columns (2 MiB): 81 instead of 236.  Beyond it gathering loses: batch 16384, 128 fp32 columns
// (8 MiB): 754 us instead of 410.
constexpr int64_t kPositionBlock = 4 << 20;
// Gathered gradient (lookups x bytes of an element) from which a call cut by position leaves the runs beyond the dense
// threshold to counts x gradient block and calls a run long from kLongRun on, as the calls beyond kPositionBlock do.  A
// smaller call is a matter of latency: it has too few slices of bags to fill the chip, and a wavefront that sums 512
// lookups by itself is a long chain (1 table of 1000 rows, batch 2048, 128 columns, 0.1 M lookups: the whole update 28 us,
// 84 with dense rows; 8 tables, batch 16384, 64 columns, 3.9 M: 135 / 152; 64 tables of 1 M rows, batch 8191, 128 bf16 columns,
// 5.2 M: 430 / 456).  A larger one gathers most of a skewed batch by position and adds every run to one list, 6 ns each:
// 64 tables of 1000 rows, batch 8191, 128 columns, 26 M lookups 1586 us, 724 with dense rows (790 by window); batch 16384,
// 32 columns, 52 M 1502 / 513 (615); of 1 M rows, 21 M 1668 / 1464 (1586).  Wide rows take the matrix cores several
// passes: 512 bf16 columns, 64 tables, 6.6 M 699 / 767; fp32, 128 tables, 13 M 2733 / 2262.
constexpr int64_t kManyLongBytes = 16000000, kManyLongPerColumn = 65536;

// Lookups up to which the long runs of a call without dense ones are found by position instead of listed: every partial row
// there could be takes a wavefront that looks for it, and the one that sums the last piece of a run finishes it; a list takes
// two launches more.  Update, us, listed / found: 8 tables of 128 fp32 columns, 60,000 lookups uniform 22.5 / 18.6, Zipf 1.05
// 26.3 / 15.0; 0.5 M 121 / 116, 67.8 / 61.1; 4..512 columns, 0.15 M 51.0 / 47.3, 59.8 / 34.9; 256, 0.5 M 225 / 222, 112.6 /
// 111.8; 64 of 128, 16-bit, 0.5 M 83.9 / 77.6, 60.3 / 47.3.  Beyond the line (uniform within the spread of the runs, Zipf):
// 8 of 128 fp32 columns, 0.66 M 78.8 / 73.4, 1 M 109 / 107, 1.5 M 154 / 155, 3.9 M 314 / 318; 16 of 128, 1 M 134 / 128, 2 M 204 /
// 202; 64 of 128, 16-bit, 1 M 125 / 107, 1.5 M 151 / 151; but 8 of 256, 1 M 189 / 192, 1.5 M 247 / 254.  Up to the line no call
// loses; calls of up to 1 M and 128 columns would still gain 2 to 15 %.  Narrow rows (longer spans) have short chains and stay
// listed.
constexpr int64_t kFoundLookups = 1 << 19;

constexpr int kPosPiece = 128;            // a piece by position has at most this many lookups (and fewer than that is never long) ...
constexpr int kPosPiecesMax = 256;        // ... unless that would make more pieces of a run than this
// Partial row of a piece: its first position / kPosSlot.  A piece has at least kPosSlot lookups, so no two share one, and a
// dense run's rows are those of the 128-position chunks that it covers completely, in which no other run has a position.
constexpr int kPosSlot = 64;

struct LongRunRule {
    bool by_position, dense;   // dense: runs beyond the dense threshold are summed as dense rows
    bool found;                // by position, and by wavefronts that look for them
    int long_run;              // a run of more lookups is long
};

// widest: columns of the widest table
inline LongRunRule long_run_rule(int64_t lookups, int64_t batch, int64_t widest, int grad_bytes)
{
    LongRunRule r;
    r.by_position = batch * widest * grad_bytes <= kPositionBlock;
    r.dense = !r.by_position || lookups * grad_bytes >= std::max(kManyLongBytes, kManyLongPerColumn * widest);
    r.found = !r.dense && lookups <= kFoundLookups;
    r.long_run = r.dense ? kLongRun : kPosPiece;
    return r;
}

// Whether the workgroups of the update kernel sum the long runs of a call of at most a tile of lookups themselves: the four
// wavefronts of one take 16 rows of the widest table per lane group and trip together, four each, and the longest run there can be,
// all lookups of the call, should take no more than 32 trips.
constexpr int kSmallLongTrips = 32;

// lanes: of a row of the widest table
inline bool small_long_runs(int64_t lookups, int lanes) { return lookups <= (int64_t)kSmallLongTrips * 16 * (kWave / lanes); }

TBE_BOTH int position_pieces(int len)
{
    const int np = (len + kPosPiece - 1) / kPosPiece;
    return np < kPosPiecesMax ? np : kPosPiecesMax;
}

// first position of piece i of the np pieces of a run of `len` lookups from position s (i = np: the end of the run)
TBE_BOTH int position_of_piece(int s, int len, int np, int i)
{
    const int each = len / np, more = len - each * np;    // the first `more` pieces are one longer
    return s + i * each + (i < more ? i : more);
}

// first of the np pieces of a run of `len` lookups that starts `from` positions behind the run's start, or later (np: none)
TBE_BOTH int first_piece_from(int len, int np, int from)
{
    const int each = len / np, more = len - each * np;
    const int longer = more * (each + 1);
    return from <= 0 ? 0 : from <= longer ? (from + each) / (each + 1) : more + (from - longer + each - 1) / each;
}

// ---------------------------------------------------------------- sort

// Which sort a call takes: that of tbe_sort_kernels.hip.h, or the digit-by-digit one of tbe_radix_kernels.hip.h.
// - Tables of at most 256 rows take one pass of the latter; the former's plan is wasted on them (100 rows: 8 tables, 50,000
//   lookups 52 us by digits, 51 by partition; 200,000 55 / 54; 800,000 56 / 63; 4 M 74 / 105; 16 M 164 / 175).
// - A table has at most 1024 buckets.  From 3.6 M lookups in it they grow beyond what a workgroup sorts well in LDS, from 8 M
//   all of them take passes through memory, and the buckets of few tables are too few for 768 resident workgroups.  The
//   lookups from which that costs more than the passes saved grow with about the third power of the number of tables: 10 M
//   rows, uniform, 1 table of 10 M lookups 288 us by digits, 328 by partition; 2 of 16 M 745 / 735, of 60 M 2540 / 2730; 3 of
//   30 M 1920 / 1840, of 60 M 3600 / 3820; 4 of 30 M 2600 / 2380, of 60 M 4650 / 4560; 8 of 30 M 4860 / 4220.  The fewer the
//   passes the sooner: 1 table, 60,000 rows, 800,000 lookups 88 / 91, 2 M 99 / 110; 1 M rows, 800,000 115 / 98, 2 M 128 / 137;
//   and with two passes two tables lose by 2 M already (60,000 rows: 2 M 97 / 95, 4 M 116 / 134, 16 M 280 / 320).
// - The partition takes a plan and 20 KiB of memory per table: 4000 tables of 100 lookups 253 / 249 us, 10,000 557 / 661.
constexpr int64_t kOnePassMin = 200000;
constexpr int kManyTables = 4096;

// passes: eight-bit digits of the tallest table's row index
inline bool use_radix_sort(int64_t tables, int64_t lookups, int passes)
{
    constexpr int64_t kTallTable[] = {0, 0, 1000000, 2000000, 3500000};
    const int64_t power = passes == 2 && tables == 2 ? tables : tables * tables * tables;
    return tables > kManyTables || (passes <= 1 && lookups >= kOnePassMin) ||
           (passes > 1 && tables <= 16 && lookups >= kTallTable[std::min(passes, 4)] * power);
}

// Lookups per bucket: a small call has some 512 units, two a CU, but none is worth less than kSortTargetMin.  From 5/16 of a
// tile each on, units come in rounds of the 768 resident workgroups (less some for the last, smaller one of every table and
// for rows with a unit of their own), in as few rounds as units of at most 7/16 of a tile make.  A bucket spreads by 1/4
// around that; beyond a tile it takes the slow path through memory, which one bucket in 1,000 did at half a tile (64 tables,
// 5.5 M lookups: 76 us for the units, 55 without such a straggler).  Sort with 512 units in a smaller call and 7/16 of a tile
// in a larger one -> this: 1000 rows, 8 tables, 2 M lookups 95 -> 81 us; 60,000 rows 105 -> 87; 64 tables, 4 M 108 -> 105; 4
// tables of 1000 rows, 4 M 117 -> 107.  Whole steps with 512 units / in a round of 704: 0.66 M lookups 320 / 324 us, 0.71 M
// 330 / 337, 0.84 M 253 / 257, 1.1 to 1.6 M the same, 1.8 M 998 / 977.
constexpr int kSortTargetMin = 1024, kSortTargetFew = 2560, kSortTargetMax = 3584;
constexpr int64_t kSortUnitsFew = 512, kSortUnitsRound = 704;

// rounds of units of a call that is not small
inline int64_t sort_rounds(int64_t lookups) { return (lookups + kSortTargetMax * kSortUnitsRound - 1) / (kSortTargetMax * kSortUnitsRound); }

inline int sort_target(int64_t lookups)
{
    if (lookups <= kSortTargetFew * kSortUnitsFew)
        return (int)std::max<int64_t>(kSortTargetMin, lookups / kSortUnitsFew);
    const int64_t units = sort_rounds(lookups) * kSortUnitsRound;
    return (int)((lookups + units - 1) / units);
}

// Most full buckets, rounded up, that calls of at most this many lookups can ask for (a table's last one comes on top)
inline int64_t sort_buckets_max(int64_t lookups) { return std::max<int64_t>(1, sort_rounds(lookups)) * kSortUnitsRound; }

// Samples per bucket of a table's plan.  A bucket's size spreads by 1/4 around the target with 16 of them; with 8, by 1/3, which
// a target of at most 5/16 of a tile leaves room for where a workgroup would sort thousands of samples (1 table, 0.49 M lookups,
// 480 buckets: plan of 31 us, 39 with 16).
constexpr int kSamplesMax = 8192;

TBE_BOTH int samples_per_bucket(int buckets, int target)
{
    const int room = kSamplesMax / buckets;
    const int want = target <= kSortTargetFew && buckets > 128 ? 8 : 16;
    return room < want ? room : want;
}

// Middle calls: the units find their lookups themselves, each among all of its table's (sort_select_kernel), instead of
// having them brought by histogram, units and scatter.  That reads a table's indices twice per unit: while tables have
// kSelectMean lookups on average the three launches cost more.  Sort, us, with them / without: 40 tables of 4300 lookups 41 /
// 26, 60 of 4300 43 / 28, 1 of 20,000 39 / 29, 11 of 23,800 43 / 35.  The host does not know how the lookups spread over the
// tables.  One table with 60,000 of 3 tables' 42 / 36 (Zipf 42 / 37), 100,000 of 40 47 / 43 (47 / 45), 120,000 of 16 48 / 46
// (48 / 49), 200,000 of 11 53 / 57 (52 / 63), 251,000 of 11 52 / 64 (53 / 73; in 16,384 bags 57 / 83): kSelectLookups ends what a
// call can lose.
constexpr int kSelectCap = 6144;           // words of a unit that is sorted in LDS
constexpr int64_t kSelectMean = 4 * kSelectCap, kSelectLookups = 1 << 18;

// Units of a row of which `sampled` of a table's `samples` samples are.  One workgroup would place all lookups of a hot row, and
// walk the table once more for every 12,288 of them (11 tables, one of 200,000 Zipf lookups: sort of 100 us, 62 with parts).
// Together the rows of a table have at most lookups / kSelectPart units more than one each.
constexpr int kSelectPart = 4096;

TBE_BOTH int unit_parts(uint32_t sampled, int lookups, int samples, int part)
{
    return 1 + (int)((uint64_t)sampled * (uint32_t)lookups / (uint32_t)samples / (uint32_t)part);
}

TBE_BOTH int select_parts(uint32_t sampled, int lookups, int samples) { return unit_parts(sampled, lookups, samples, kSelectPart); }

// A unit whose lookups do not fit the LDS (its rows have more of them than the sample said) is taken in parts.  Rows to try
// after `rows` turned out to have `found` lookups, too many, ...
TBE_BOTH uint32_t select_fewer_rows(uint32_t rows, int found)
{
    const uint32_t half = rows / 2 + (rows & 1u), even = (uint32_t)((uint64_t)rows * kSelectCap / (uint32_t)found);
    return even < half ? (even > 0 ? even : 1u) : half;
}

// ... and after a part of `rows` rows with `found` lookups that did fit, of the `rest_rows` that follow with `rest` lookups.  Each
// try walks the whole table, so what was learnt stays (200,000 lookups of which the sample missed 1000 rows with 198,000: trying
// all that was left again took 766 walks and 38 ms; this takes 37, and 2.3 ms).
TBE_BOTH uint32_t select_next_rows(uint32_t rows, int found, uint32_t rest_rows, int rest)
{
    const uint32_t more = found <= kSelectCap / 2 && rows < 1u << 31 ? 2 * rows : rows;
    return rest <= kSelectCap || rest_rows < more ? rest_rows : more;
}

inline bool use_select_sort(int64_t tables, int64_t lookups) { return lookups <= kSelectLookups && lookups <= kSelectMean * tables; }

// Other calls of 32-bit words, up to kPiecesMax chunks: every chunk's words are put in order of their buckets where they lie and a
// unit collects its piece of each chunk of its table, where the partition of larger ones counts first (histogram, starts, units).
// Sort, us, uniform / Zipf 1.05 indices, counted -> collected: 1 table, 40,000 lookups 39 / 39 -> 32 / 32, 0.6 M 70 / 65 -> 54 / 61; 8
// tables, 0.66 M 48 / 47 -> 42 / 42; 16, 2.6 M 95 / 93 -> 77 / 78; 64, 2 M 73 / 69 -> 64 / 61, 6.2 M 124 / 118 -> 113 / 109, 8 M 140 /
// 137 -> 133 / 129; 600, 2 M 105 / 103 -> 81 / 78; 16, of which one has 4 M, 140 / 145 -> 133 / 146; 64, one 8 M 234 / 252 -> 209 /
// 231.  Beyond, a table's units read the starts of hundreds of chunks for pieces of a few words (64 tables, 19 M lookups: the
// units 208 us, 119 and 55 for the count).  kPiecesMax is also what a workgroup holds of them in LDS.
// There is no smallest call: the smallest this gets, one table of 24,577 lookups (use_select_sort has the others), takes 39 counted
// and 33 collected, of 32,768 38 and 32 (1 M rows).
constexpr int kPiecesMax = 1024;
constexpr int kPiecesChunk = 8192;         // a chunk is ordered by one workgroup at once, in LDS; its length is a power of two

inline bool use_pieces_sort(bool words32, int64_t lookups, int chunk)
{
    return words32 && chunk <= kPiecesChunk && (chunk & (chunk - 1)) == 0 && lookups <= (int64_t)kPiecesMax * chunk;
}

// Workgroups of the bucket sort: one per unit there can be (and no fewer than are resident: tables cut by the packed range have
// more units) while those are at most kUnitsDispatched, otherwise as many as are resident, which take the units one by one.  An
// atomic on one word and a descriptor wait in front of every unit (sort, us, with 768 workgroups -> one each: 64 tables, 2 M
// lookups 74 -> 64, 8 M 139 -> 133, 20 M 286 -> 283; words of 64 bits, 512 workgroups: 8 tables, 1 M 77 -> 74, 4 M 133 -> 127, 16 M
// 388 -> 391, 24 M 557 -> 552; 32 tables, 2 M 100 -> 95, 8 M 207 -> 204, 20 M 455 -> 456), but a workgroup's start costs more
// once there are tens of thousands (128 tables, 100 M lookups 1285 -> 1319).
constexpr int64_t kUnitsDispatched = 8192;

inline int64_t sort_local_blocks(int64_t lookups, int64_t tables, int target, int tile, int64_t resident)
{
    const int64_t units = lookups / target + lookups / tile + 2 * tables;
    return units <= kUnitsDispatched ? std::max(units, resident) : resident;
}

// A published integer hash: lowbias32 of Wellons' hash-prospector (public domain).
TBE_BOTH uint32_t mix_bits(uint32_t x)
{
    x ^= x >> 16; x *= 0x7feb352du;
    x ^= x >> 15; x *= 0x846ca68bu;
    return x ^ (x >> 16);
}

// Where sample i of a table of n lookups lies: one from each of the equal stretches of `stretch` positions (32.32),
// at a random place of it, for which 8 bits are enough.  The product takes up to 40 bits more than n.
TBE_BOTH int sample_position(uint64_t stretch, uint32_t i, int n)
{
    const uint64_t pos = (uint64_t)(((unsigned __int128)stretch * (i * 256u + (mix_bits(i) & 255u))) >> 40);
    return pos < (uint64_t)n ? (int)pos : n - 1;
}

// Bucket of a row: that of the first row of its cell (lut), moved on over the SPAN borders that can lie inside one, all
// compared at once.  below: the row before the first row of every bucket (0 - 1 for the first bucket), then SPAN entries of
// all ones: those are below no 32-bit word, so an index that is no row of the table finds one of its buckets all the same.
template <int SPAN, typename Cell>
TBE_BOTH uint32_t linear_bucket(const uint32_t* below, const Cell* lut, uint32_t row, int shift, uint32_t last_cell)
{
    const uint32_t cell = row >> shift;
    const uint32_t first = lut[cell < last_cell ? cell : last_cell];
    uint32_t border[SPAN + 1], d = first;
#pragma unroll
    for (int k = 1; k <= SPAN; ++k)
        border[k] = below[first + k];
#pragma unroll
    for (int k = 1; k <= SPAN; ++k)
        d += border[k] < row ? 1u : 0u;
    return d;
}

}  // namespace tbe
