"""GPU parity of the sort whose chunks are ordered by bucket where they lie and whose units collect their pieces: calls at the
borders of the chunk sizes, tables of up to 64, of up to 512 and of more chunks, rows of several units, units that do not
fit a tile because the sample missed their rows, empty tables, tables cut by the packed range, and both sides of the
largest call.  Bit-exact."""
import numpy as np
import pytest

from test_gpu_sort_paths import _check, _lens, _mix

pytestmark = pytest.mark.gpu
TILE = 8192
MOST = 1024 * TILE

CASES = {
    # name: (rows, batch, lookups per table, per table the rows that are looked up oftenest and their shares)
    "smallest_call": ([1_000_000], 100, [24_577], [{}]),
    "no_more_than_a_few_chunks": ([5000], 611, [32_768], [{4999: 0.4}]),
    "quarter_tiles": ([1_000_000], 700, [1 << 17], [{}]),
    "half_tiles": ([1_000_000], 700, [(1 << 17) + 1], [{}]),
    "most_half_tiles": ([1_000_000, 5000], 4096, [(3 << 18) - 3, 3], [{}, {}]),
    "tiles": ([1_000_000, 5000], 4096, [(3 << 18) - 3, 4], [{}, {}]),
    "chunks_of_64_and_65": ([900_000] * 4, 300, [64 * TILE, 64 * TILE + 1, 65 * TILE, 63 * TILE - 1], [{}] * 4),
    "chunks_of_512_and_513": ([1_500_000] * 2, 2000, [512 * TILE, 512 * TILE - 5], [{}, {3: 0.01}]),
    "more_than_512_chunks": ([1_500_000] * 2, 2000, [1, 513 * TILE + 7], [{}, {1_499_999: 0.01}]),
    "rows_of_several_units": ([1_000_000, 300], 900, [400_000, 90_000], [{0: 0.3, 999_999: 0.3, 500_000: 0.1}, {299: 0.9}]),
    "tables_of_one_row": ([1, 1, 2, 700_000], 65_536, [300_000, 16_384, 9_000, 60_000], [{}] * 4),
    "cut_by_the_packed_range": ([30_000_000, 70_000], 65_536, [150_000, 300_000], [{29_999_999: 0.2}, {}]),
    "empty_tables": ([50_000] * 7, 1000, [0, 40_000, 0, 100_000, 1, 270_000, 0], [{}] * 7),
    "more_tables_than_threads": ([3000] * 700, 30, [1500] * 700, [{}] * 700),
    "largest_call": ([400_000] * 20, 4000, [MOST // 20] * 19 + [MOST - MOST // 20 * 19], [{}] * 20),
    "beyond_it": ([400_000] * 20, 4000, [MOST // 20] * 19 + [MOST - MOST // 20 * 19 + 1], [{}] * 20),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_units_that_collect_their_pieces(gpu_device, case):
    rows, batch, per_table, hot = CASES[case]
    rng = np.random.default_rng(len(case))
    lens = np.concatenate([_lens(rng, batch, n) for n in per_table])
    parts = []
    for h, n, often in zip(rows, per_table, hot):
        x = rng.integers(0, h, n)
        where, at = rng.permutation(n), 0
        for row, share in often.items():
            x[where[at:at + round(share * n)]] = row
            at += round(share * n)
        parts.append(x)
    print(f"{case}: N={sum(per_table)}", flush=True)
    _check(gpu_device, rows, batch, lens, np.concatenate(parts), case)


@pytest.mark.parametrize("n,missed", [(300_000, 5), (900_000, 5), (900_000, 1)])
def test_units_that_do_not_fit_a_tile(gpu_device, n, missed):
    """The sampled lookups hit other rows than all others do: one bucket holds nearly everything, for two
    passes through memory."""
    rng = np.random.default_rng(n)
    want = -(-n // max(1024, n // 512))
    s = want * (8 if want > 128 else 16)
    stretch = (n << 32) // s
    at = [min((stretch * (i * 256 + (_mix(i) & 255))) >> 40, n - 1) for i in range(s)]
    idx = rng.integers(0, missed, n)
    idx[at] = rng.integers(1000, 200_000, s)
    _check(gpu_device, [200_000], 611, _lens(rng, 611, n), idx, "large unit")


def _sample(n, call):
    """Positions of a table's samples, buckets it asks for, samples per bucket; n of the call's lookups are the table's."""
    units = -(-call // (3584 * 704)) * 704
    target = max(1024, call // 512) if call <= 2560 * 512 else -(-call // units)
    want = -(-n // target)
    per = min(8 if target <= 2560 and want > 128 else 16, 8192 // want)
    stretch = (n << 32) // (want * per)
    return [min((stretch * (i * 256 + (_mix(i) & 255))) >> 40, n - 1) for i in range(want * per)], want, per


def _bucket_of(row, samples, want, per, rows):
    """First and end row of a row's bucket, from the samples of its table."""
    s = np.sort(samples)
    borders = {0}
    for j in range(1, want):
        borders.add(int(s[j * per]))
        if j + 1 < want and s[(j + 1) * per] == s[j * per]:
            borders.add(int(s[j * per]) + 1)
    borders = np.array(sorted(b for b in borders if b < rows) + [rows])
    i = int(np.searchsorted(borders, row, side="right")) - 1
    return int(borders[i]), int(borders[i + 1])


@pytest.mark.parametrize("n", [270_000, 900_000])
@pytest.mark.parametrize("missed,passes", [(100, 1), (300_000, 3)])
def test_large_units_after_an_odd_number_of_passes(gpu_device, n, missed, passes):
    """One bucket holds nearly everything and is sorted through memory; after one pass or three its words lie where its payloads go."""
    rng = np.random.default_rng(n + passes)
    rows = 1_000_000
    at, want, per = _sample(n, n)
    idx = rng.integers(0, missed, n)
    idx[at] = missed + rng.permutation(rows - missed)[:len(at)] if passes > 1 else missed + np.arange(len(at))
    lo, hi = _bucket_of(0, idx[at], want, per, rows)
    assert lo == 0 and hi >= missed and 8 * (passes - 1) < (hi - 1).bit_length() <= 8 * passes and (idx < hi).sum() > 10 * TILE
    _check(gpu_device, [rows], 611, _lens(rng, 611, n), idx, "large unit")


@pytest.mark.parametrize("n", [270_000, 2_000_000])
@pytest.mark.parametrize("samples_of_it", [3, 40])
def test_one_row_that_the_sample_undersizes(gpu_device, n, samples_of_it):
    """A row that has a bucket of its own, and with it nearly all lookups of its table, though few samples say so: its units, one
    or a few, do not fit a tile."""
    rng = np.random.default_rng(n)
    rows, call = 300_000, n + 40_000
    at, want, per = _sample(n, call)
    idx = np.full(n, 77_777)
    idx[at] = rng.integers(0, rows, len(at))
    idx[at[5:5 + samples_of_it * per]] = 77_777
    assert _bucket_of(77_777, idx[at], want, per, rows) == (77_777, 77_778)
    units = 1 + int((idx[at] == 77_777).sum()) * n // len(at) // TILE
    assert units * TILE * 2 < (idx == 77_777).sum()
    other = rng.integers(0, 999, 40_000)
    lens = np.concatenate([_lens(rng, 500, n), _lens(rng, 500, 40_000)])
    _check(gpu_device, [rows, 999], 500, lens, np.concatenate([idx, other]), "one row")
