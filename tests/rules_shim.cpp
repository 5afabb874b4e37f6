// C entry points to the library's launch rules and index arithmetic for tests/test_rules.py.
#include "tbe_rules.h"

extern "C" {

void forward_launch(int64_t num_bags, int64_t lookups, int wide, int64_t* out /*[3]*/)
{
    const tbe::ForwardLaunch f = tbe::forward_launch(num_bags, lookups, wide != 0);
    out[0] = f.one_bag;
    out[1] = f.bags_per_wave;
    out[2] = f.blocks;
}

void sample_positions(int n, int samples, int32_t* out)
{
    const uint64_t stretch = ((uint64_t)n << 32) / (uint32_t)samples;
    for (int i = 0; i < samples; ++i)
        out[i] = tbe::sample_position(stretch, (uint32_t)i, n);
}

// buckets of n indices in a table of `rows` rows, as the partition finds them; lut: first bucket of every cell
void partition_buckets(const uint32_t* split, const uint16_t* lut, int shift, int span, uint32_t rows, const uint32_t* index, int n, uint32_t* out)
{
    for (int i = 0; i < n; ++i) {
        const uint32_t row = tbe::sort_row(index[i], rows - 1);
        out[i] = span == 1 ? tbe::linear_bucket<1>(split, lut, row, shift) : span == 2 ? tbe::linear_bucket<2>(split, lut, row, shift)
               : span == 3 ? tbe::linear_bucket<3>(split, lut, row, shift) : tbe::linear_bucket<4>(split, lut, row, shift);
    }
}

}
