"""GPU parity of the sort whose units find their lookups themselves (calls of at most 2^18 lookups, 24,576 a table on average):
sizes on both sides of its borders, tables of one bucket and of many, rows with more lookups than a workgroup's LDS holds
positions (12,288), units that have to be cut because the sample missed their rows, empty tables, and bags by the thousand.  Bit-exact."""
import numpy as np
import pytest

from test_gpu_sort_paths import _check, _lens, _mix

pytestmark = pytest.mark.gpu
MEAN, MOST = 24_576, 1 << 18

CASES = {
    # name: (rows, batch, lookups per table, share of the hottest row)
    "one_table_at_the_border": ([1_000_000], 700, [MEAN], 0.0),
    "one_table_beyond_it": ([1_000_000], 700, [MEAN + 1], 0.0),
    "most_lookups": ([30_000, 9, 500_000] * 5, 300, [MOST // 15] * 14 + [MOST - MOST // 15 * 14], 0.01),
    "more_than_that": ([30_000, 9, 500_000] * 5, 300, [MOST // 15] * 14 + [MOST + 1 - MOST // 15 * 14], 0.01),
    "steps_of_the_scan": ([5000] * 8, 40, [4095, 4096, 4097, 8191, 8192, 8193, 1, 12_289], 0.05),
    "one_bucket_each": ([700, 70_000, 3] * 9, 1000, [1023, 1024, 1025, 1, 0, 640, 511, 512, 513] * 3, 0.0),
    "one_table_has_nearly_all": ([100_000] * 9, 800, [200_000, 3, 0, 17, 0, 0, 1, 1000, 0], 0.1),
    "row_that_fills_the_lds": ([1_000_000, 40], 900, [40_000, 100], 12_288 / 40_000),
    "row_beyond_the_lds": ([1_000_000, 40], 900, [40_000, 100], 0.9),
    "tables_of_one_row": ([1, 1, 2], 65536, [30_000, 13_000, 9_000], 0.0),
    "words_of_64_bits": ([40_000_000, 500], 70_001, [45_000, 4_000], 0.3),
    "bags_by_the_thousand": ([50_000] * 3, 65536, [24_000, 100, 30_000], 0.02),
    "one_bag_a_table": ([50_000] * 5, 1, [24_000, 100, 0, 30_000, 2], 0.02),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_units_that_find_their_lookups_themselves(gpu_device, case):
    rows, batch, per_table, hot = CASES[case]
    rng = np.random.default_rng(len(case))
    lens = np.concatenate([_lens(rng, batch, n) for n in per_table])
    parts = []
    for h, n in zip(rows, per_table):
        x = rng.integers(0, h, n)
        x[rng.permutation(n)[:round(hot * n)]] = h * 2 // 3
        parts.append(x)
    print(f"{case}: N={sum(per_table)}", flush=True)
    _check(gpu_device, rows, batch, lens, np.concatenate(parts), case)


PARTS = {
    # name: (rows, batch, lookups per table, per table the rows that are looked up oftenest and their shares)
    "two_units": ([1_000_000, 300], 900, [24_000, 500], [{500_000: 0.2}, {}]),
    "five_rows_beside_each_other": ([1_000_000] * 8, 1024, [150_000] + [100] * 7, [{70 + i: 0.19 for i in range(5)}] + [{}] * 7),
    "first_and_last_row": ([77_777] * 6, 300, [60_000, 0, 40_000, 1, 2, 3], [{0: 0.4, 77_776: 0.4}, {}, {77_776: 0.5, 0: 0.3}, {}, {}, {}]),
    "one_row_of_a_large_call": ([1_000_000] * 11, 16_384, [261_000] + [10] * 10, [{999_999: 0.98}] + [{}] * 10),
    "words_of_64_bits": ([40_000_000, 500], 70_001, [45_000, 4_000], [{39_999_999: 0.3, 5: 0.5}, {}]),
}


@pytest.mark.parametrize("order", ["spread", "first"])
@pytest.mark.parametrize("case", sorted(PARTS))
def test_rows_of_several_units(gpu_device, case, order):
    """A row that the sample holds often enough is placed by several workgroups, 4096 of its lookups each; where all of them lie
    in the first positions of the table a wavefront has more of them than it would of an even spread."""
    rows, batch, per_table, hot = PARTS[case]
    rng = np.random.default_rng(len(case))
    lens = np.concatenate([_lens(rng, batch, n) for n in per_table])
    parts = []
    for h, n, most in zip(rows, per_table, hot):
        x = rng.integers(0, h, n)
        at = rng.permutation(n) if order == "spread" else np.arange(n)
        for row, share in most.items():
            x[at[:int(share * n)]] = row
            at = at[int(share * n):]
        parts.append(x)
    print(f"{case} {order}: N={sum(per_table)}", flush=True)
    _check(gpu_device, rows, batch, lens, np.concatenate(parts), case)


CUT = {
    # name: lookups that the sample misses: (first row, rows, lookups) each
    "many_parts": [(0, 2000, 38_000)],
    "last_part_is_a_row_beyond_the_lds": [(0, 1999, 20_000), (1999, 1, 18_000)],
    "first_part_is_a_row_beyond_the_lds": [(0, 1, 18_000), (1, 1999, 20_000)],
    "rows_beyond_the_lds_beside_each_other": [(0, 700, 5000), (700, 1, 12_289), (701, 1, 12_288), (702, 1298, 8000)],
    "a_few_rows_of_a_wide_unit": [(1990, 10, 38_000)],
    "just_fits": [(0, 2000, 6144)],
    "just_too_many": [(0, 2000, 6145)],
}


@pytest.mark.parametrize("second", [False, True])                                  # the table's unit starts behind another table
@pytest.mark.parametrize("rows,batch", [(300_000, 500), (40_000_000, 70_001)])     # words of 32 and of 64 bits
@pytest.mark.parametrize("case", sorted(CUT))
def test_units_that_have_to_be_cut(gpu_device, case, rows, batch, second):
    rng = np.random.default_rng(3)
    n = 40_000
    want = -(-n // 1024)
    samples = 16 * want
    stretch = (n << 32) // samples
    at = np.array([min((stretch * (i * 256 + (_mix(i) & 255))) >> 40, n - 1) for i in range(samples)])
    assert len(np.unique(at)) == samples
    # the sample holds row 2000 often enough for it to be a border, and rows behind it
    idx = rng.integers(2001, rows, n)
    idx[at[:48]] = 2000
    missed = np.concatenate([rng.integers(first, first + count, m) for first, count, m in CUT[case]])
    idx[rng.permutation(np.setdiff1d(np.arange(n), at))[:missed.size]] = missed
    # the plan's borders: row 0, every 16th sample, and the row behind one that fills a stretch of samples
    sampled = np.sort(idx[at])[::16]
    borders = np.unique(np.concatenate([[0], sampled[1:], sampled[:-1][sampled[:-1] == sampled[1:]] + 1]))
    assert borders[1] == 2000 and np.count_nonzero(idx < 2000) == missed.size and (missed.size > 6144) == (case != "just_fits")
    tables = [(rows, _lens(rng, batch, n), idx), (900, _lens(rng, batch, 5000), rng.integers(0, 900, 5000))]
    heights, lens, parts = zip(*(tables[::-1] if second else tables))
    print(f"{case} rows={rows} second={second}", flush=True)
    _check(gpu_device, list(heights), batch, np.concatenate(lens), np.concatenate(parts), case)


@pytest.mark.parametrize("n", [1 << 17, (1 << 17) + 1, 3 << 18, (3 << 18) + 1])
@pytest.mark.parametrize("tables", [1, 3])
def test_chunks_of_less_than_a_tile(gpu_device, tables, n):
    # a quarter of a tile up to 2^17 lookups, half of one up to 3 x 2^18; one table of more than 128 buckets has 8 samples each
    rng = np.random.default_rng(n + tables)
    per_table = [n] if tables == 1 else [n - 2047 - n // 3, 2047, n // 3]
    lens = np.concatenate([_lens(rng, 5000, m) for m in per_table])
    idx = np.concatenate([np.minimum(rng.zipf(1.3, m) * 2_654_435_761 % 2_000_000, 1_999_999) for m in per_table])
    _check(gpu_device, [2_000_000] * tables, 5000, lens, idx, "short chunks")
