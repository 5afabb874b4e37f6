"""GPU test of the sort that counts its buckets, partitions the lookups in words of 32 bits and sorts the buckets: only calls of more
than 2^23 lookups take it, so tables with little to sort make up the size, and beside them lie the tables that the
branches are for.  Bit-exact."""
import numpy as np
import pytest

from test_gpu_sort_paths import _check, _lens
from test_gpu_sort_pieces import TILE, _bucket_of, _sample

pytestmark = pytest.mark.gpu
FILLERS, EACH = 17, 500_000


def _missed(n, call, rows, below):
    """Lookups of a table whose sample sees none of the rows below `below`, which have nearly all of them."""
    rng = np.random.default_rng(below)
    at, want, per = _sample(n, call)
    idx = rng.integers(0, below, n)
    idx[at] = below + np.arange(len(at))
    lo, hi = _bucket_of(0, idx[at], want, per, rows)
    assert lo == 0 and hi >= below and (idx < hi).sum() > 2 * TILE
    return idx


CASES = {
    # name: (batch, [(rows, lookups, kind)] of the tables beside the fillers)
    "buckets_that_do_not_fit": (611, [(50_000, 90_000, 200), (400_000, 90_000, 50_000), (2_000_000, 90_000, 200_000)]),
    "rows_of_several_tiles": (900, [(1_000_000, 400_000, {0: 0.3, 999_999: 0.3, 500_000: 0.1}), (300, 90_000, {299: 0.9}), (1, 30_000, {})]),
    "chunks_around_32": (300, [(150_000, 31 * TILE, {}), (150_000, 32 * TILE, {}), (9000, 32 * TILE + 1, {5: 0.5}), (150_000, 33 * TILE + 1, {})]),
    "empty_tables": (300, [(7, 0, {}), (120_000, 1, {}), (50, 0, {}), (900_000, 33 * TILE, {})]),
    "cut_by_the_packed_range": (65_536, [(30_000_000, 150_000, {29_999_999: 0.2}), (70_000, 33 * TILE, {})]),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_partition_of_32_bit_words(gpu_device, case):
    batch, special = CASES[case]
    rng = np.random.default_rng(len(case))
    tables = [(3000, EACH, {})] * 9 + special + [(3000, EACH, {})] * (FILLERS - 9)
    call = sum(n for _, n, _ in tables)
    assert call > 1 << 23 and len(tables) > 16           # (few tall tables are sorted by digits)
    parts = []
    for rows, n, kind in tables:
        if isinstance(kind, int):
            parts.append(_missed(n, call, rows, kind))
            continue
        x, where, at = rng.integers(0, rows, n), rng.permutation(n), 0
        for row, share in kind.items():
            x[where[at:at + round(share * n)]] = row
            at += round(share * n)
        parts.append(x)
    lens = np.concatenate([_lens(rng, batch, n) for _, n, _ in tables])
    _check(gpu_device, [rows for rows, _, _ in tables], batch, lens, np.concatenate(parts), case)
