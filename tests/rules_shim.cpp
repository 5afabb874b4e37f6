// C entry points to the library's launch rules and index arithmetic for tests/test_rules.py.
#include "tbe_rules.h"

extern "C" {

int few_bags_lookups(int epl, int narrowest) { return tbe::few_bags_lookups(epl, narrowest); }

void forward_launch(int64_t num_bags, int64_t lookups, int few, int wide, int64_t* out /*[3]*/)
{
    const tbe::ForwardLaunch f = tbe::forward_launch(num_bags, lookups, few, wide != 0);
    out[0] = f.one_bag;
    out[1] = f.bags_per_wave;
    out[2] = f.blocks;
}

void long_run_rule(int64_t lookups, int64_t batch, int64_t widest, int grad_bytes, int32_t* out /*[4]*/)
{
    const tbe::LongRunRule r = tbe::long_run_rule(lookups, batch, widest, grad_bytes);
    out[0] = r.by_position;
    out[1] = r.dense;
    out[2] = r.long_run;
    out[3] = r.found;
}

// borders of the pieces of a run; returns their number
int position_pieces(int s, int len, int32_t* out /*[257]*/)
{
    const int np = tbe::position_pieces(len);
    for (int i = 0; i <= np; ++i)
        out[i] = tbe::position_of_piece(s, len, np, i);
    return np;
}

int first_piece_from(int len, int np, int from) { return tbe::first_piece_from(len, np, from); }

int update_span(int64_t lookups, int64_t lanes, int64_t tables) { return tbe::update_span(lookups, lanes, tables); }

int use_radix_sort(int64_t tables, int64_t lookups, int passes) { return tbe::use_radix_sort(tables, lookups, passes); }

int small_long_runs(int64_t lookups, int lanes) { return tbe::small_long_runs(lookups, lanes); }

int use_select_sort(int64_t tables, int64_t lookups) { return tbe::use_select_sort(tables, lookups); }

int use_pieces_sort(int words32, int64_t lookups, int chunk) { return tbe::use_pieces_sort(words32 != 0, lookups, chunk); }

int64_t sort_local_blocks(int64_t lookups, int64_t tables, int target, int tile, int64_t resident)
{
    return tbe::sort_local_blocks(lookups, tables, target, tile, resident);
}

int unit_parts(int sampled, int lookups, int samples, int part) { return tbe::unit_parts((uint32_t)sampled, lookups, samples, part); }

int select_parts(int sampled, int lookups, int samples) { return tbe::select_parts((uint32_t)sampled, lookups, samples); }

uint32_t select_fewer_rows(uint32_t rows, int found) { return tbe::select_fewer_rows(rows, found); }
uint32_t select_next_rows(uint32_t rows, int found, uint32_t rest_rows, int rest) { return tbe::select_next_rows(rows, found, rest_rows, rest); }

int sort_target(int64_t lookups) { return tbe::sort_target(lookups); }
int64_t sort_buckets_max(int64_t lookups) { return tbe::sort_buckets_max(lookups); }

void sample_positions(int n, int samples, int32_t* out)
{
    const uint64_t stretch = ((uint64_t)n << 32) / (uint32_t)samples;
    for (int i = 0; i < samples; ++i)
        out[i] = tbe::sample_position(stretch, (uint32_t)i, n);
}

// buckets of n indices, as the partition finds them; lut: first bucket of every cell
void partition_buckets(const uint32_t* below, const uint16_t* lut, int shift, uint32_t last_cell, int span, const uint32_t* index, int n, uint32_t* out)
{
    for (int i = 0; i < n; ++i)
        out[i] = span == 1 ? tbe::linear_bucket<1>(below, lut, index[i], shift, last_cell)
               : span == 2 ? tbe::linear_bucket<2>(below, lut, index[i], shift, last_cell)
               : span == 3 ? tbe::linear_bucket<3>(below, lut, index[i], shift, last_cell)
                           : tbe::linear_bucket<4>(below, lut, index[i], shift, last_cell);
}

}
