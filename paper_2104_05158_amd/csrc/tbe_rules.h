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
// ... of fewer than kFewBagsShort bags whatever their length: 2048 bags of 2 lookups, dim 128: 3.5 against 3.2 us;
// ... of fewer than kFewBags bags that hold kFewBagsLookups lookups on average.  forward_kernel has one bag per
//     wavefront there too and leaves all lane groups but one idle; from 32,768 bags it packs several (fp32 dim 64, 8
//     lookups: 24,000 bags 15.0 against 11.6 us, 40,000 bags 15.0 against 17.6).  Bags of 2 lookups have nothing to
//     spread (fp32 dim 128, 16,384 bags: 8.3 against 8.5);
// ... of any size if every table's row fills the wavefront and a bag holds kWideBagLookups lookups on average: there
//     is no lane group to spread over, but up to 8 rows in flight instead of 4.  131,072 bags: fp32 dim 256, 16 lookups
//     174 against 154 us, dim 512, 24 lookups 463 against 400; fp16 dim 384, 16 lookups 179 against 166.
//     Its launch has 64 threads per bag: kMaxLaunchThreads ends that at 2^26 bags.
constexpr int kFewBagsShort = 8192;
constexpr int kFewBags = 32768;
constexpr int kFewBagsLookups = 4;
constexpr int kWideBagLookups = 16;

struct ForwardLaunch {
    bool one_bag;          // forward_bag_kernel
    int bags_per_wave;     // of forward_kernel, which holds a wavefront's borders in its lanes: at most kWave - 1
    int64_t blocks;
};

// wide: every table's row takes all lanes of a wavefront
inline ForwardLaunch forward_launch(int64_t num_bags, int64_t lookups, bool wide)
{
    constexpr int64_t kMaxBlocks = kMaxLaunchThreads / kFwdThreads, kWaves = kFwdThreads / kWave;
    ForwardLaunch f;
    f.one_bag = (num_bags < kFewBagsShort || (num_bags < kFewBags && lookups >= kFewBagsLookups * num_bags) ||
                 (wide && lookups >= kWideBagLookups * num_bags)) && num_bags <= kMaxBlocks * kWaves;
    // enough bags to amortise the per-block prologue, few enough to keep >= ~16k wavefronts in the grid when the batch
    // is small; beyond 2^29 bags as many as the largest launch needs
    const int64_t fewest = (num_bags + kMaxBlocks * kWaves - 1) / (kMaxBlocks * kWaves);
    const int64_t per_wave = std::min<int64_t>(kFwdMaxBagsPerWave, num_bags / 16384);
    f.bags_per_wave = f.one_bag ? 1 : (int)std::max<int64_t>({1, fewest, per_wave});
    const int64_t per_block = kWaves * f.bags_per_wave;
    f.blocks = (num_bags + per_block - 1) / per_block;
    return f;
}

// ---------------------------------------------------------------- sort

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
