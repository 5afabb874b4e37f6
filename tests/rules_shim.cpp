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

}
