"""GPU test of every path of the backward's sort: the one-workgroup sort of small calls and its size limits, buckets of
one row, crowded row ids, tables cut by the range of a packed word, 64-bit words, a bucket larger than a tile (the
sample is made to miss its rows), more tables than lookups, empty tables and empty bags.  Words of 64 bits are partitioned here;
those of 32 only in calls of more than 2^23 lookups (test_gpu_sort_partition.py), and the calls of this size have units that find
(test_gpu_sort_select.py) or collect (test_gpu_sort_pieces.py) their lookups.  Keys, payloads, unique keys
and segment offsets must equal a stable argsort by (table, row) bit for bit."""
import numpy as np
import pytest
import torch

from paper_2104_05158_amd import tbe

pytestmark = pytest.mark.gpu

TILE = 8192


def _check(dev, rows, batch, lens, idx, what):
    """lens [T * batch] bag lengths, idx the lookups, table-major"""
    T = len(rows)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n = int(off[-1])
    assert idx.size == n
    bag = np.repeat(np.arange(T * batch), lens)
    base = np.concatenate([[0], np.cumsum(rows)]).astype(np.int64)
    key = base[bag // batch] + idx
    order = np.argsort(key, kind="stable")
    ref_key, ref_val = key[order].astype(np.uint32), (bag % batch)[order].astype(np.int32)
    head = np.flatnonzero(np.concatenate([[True], ref_key[1:] != ref_key[:-1]]))
    print(f"{what}: n={n} T={T} batch={batch} runs={head.size}", flush=True)
    op = tbe.TableBatchedEmbeddingBags(rows, [4] * T, 0, batch, n, device=dev)
    d_idx, d_off = torch.from_numpy(idx.astype(np.int32)).to(dev), torch.from_numpy(off).to(dev)
    for _ in range(2):                                   # the second sort starts from the first one's workspace
        op.backward_sort(d_idx, d_off, batch)
    art = op.artifacts()
    assert art["num_unique"] == head.size
    assert np.array_equal(art["sorted_keys"].cpu().numpy().view(np.uint32), ref_key)
    assert np.array_equal(art["sorted_vals"].cpu().numpy(), ref_val)
    assert np.array_equal(art["unique_keys"].cpu().numpy().view(np.uint32), ref_key[head])
    assert np.array_equal(art["seg_offsets"].cpu().numpy(), np.concatenate([head, [n]]))
    op.close()


def _lens(rng, bags, n):
    return np.bincount(rng.integers(0, bags, n), minlength=bags)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1024, 1025, TILE - 1, TILE, TILE + 1, 3 * TILE])
@pytest.mark.parametrize("tables,batch", [(1, 7), (3, 100), (40, 1000)])
def test_sizes_around_the_one_workgroup_sort(gpu_device, n, tables, batch):
    rng = np.random.default_rng(n + tables)
    rows = rng.integers(1, 5000, tables)
    lens = _lens(rng, tables * batch, n)                 # 40 tables x 1000 bags is beyond the small sort's bags
    t = np.repeat(np.arange(tables), lens.reshape(tables, batch).sum(1))
    _check(gpu_device, rows, batch, lens, (rng.random(n) * rows[t]).astype(np.int64), "small")


CASES = {
    # name: (rows, batch, lookups per table, ids)
    "hot_rows": ([100_000, 3], 300, [200_000, 50_000], "zipf"),
    "one_row": ([1, 1_000_000], 50, [90_000, 30_000], "first"),
    "crowded_low_ids": ([10_000_000], 500, [300_000], "crowded"),
    "tall_tables_large_batch": ([10_000_000, 70_000, 33_000_000], 65536, [70_000, 9_000, 100_000], "uniform"),
    "words_of_64_bits": ([34_000_000, 500], 65536, [120_000, 40_000], "zipf"),
    "batch_beyond_16_bits": ([50_000, 20], 70_001, [250_000, 100_000], "zipf"),
    "empty_tables": ([50, 300_000, 7, 120, 900_000], 4096, [0, 150_000, 0, 1, 20_000], "uniform"),
    "many_tables": ([900] * 600, 24, [40] * 600, "uniform"),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_paths_of_the_partition(gpu_device, case):
    """What the borders of the buckets have to cope with, whichever way the lookups come to them."""
    rows, batch, per_table, ids = CASES[case]
    rng = np.random.default_rng(len(case))
    lens = np.concatenate([_lens(rng, batch, n) for n in per_table])
    parts = []
    for h, n in zip(rows, per_table):
        if ids == "uniform":
            parts.append(rng.integers(0, h, n))
        elif ids == "zipf":
            parts.append(np.minimum(rng.zipf(1.2, n) * 2_654_435_761 % h, h - 1))
        elif ids == "crowded":
            parts.append(rng.integers(0, min(h, 3000), n))
        else:
            parts.append(np.zeros(n, np.int64))
    _check(gpu_device, rows, batch, lens, np.concatenate(parts), case)


def _mix(x):
    x = np.uint32(x)
    with np.errstate(over="ignore"):
        x ^= x >> np.uint32(16); x *= np.uint32(0x7feb352d)
        x ^= x >> np.uint32(15); x *= np.uint32(0x846ca68b)
    return int(x ^ (x >> np.uint32(16)))


@pytest.mark.parametrize("rows,batch", [(200_000, 611), (34_000_000, 65536)])     # words of 32 and of 64 bits
@pytest.mark.parametrize("n", [20_000, 90_000])
def test_bucket_larger_than_a_tile(gpu_device, n, rows, batch):
    # the sampled lookups hit rows from 1000 on, all others the 1000 rows below: one bucket holds nearly everything
    rng = np.random.default_rng(n)
    want = -(-n // 1024)
    s = want * 16
    stretch = (n << 32) // s
    at = [min((stretch * (i * 256 + (_mix(i) & 255))) >> 40, n - 1) for i in range(s)]
    idx = rng.integers(0, 1000, n)
    idx[at] = rng.integers(1000, 200_000, s)
    _check(gpu_device, [rows], batch, _lens(rng, batch, n), idx, "large bucket")


@pytest.mark.parametrize("chunks,extra", [(16, 0), (32, 0), (32, 1), (75, 0), (76, 0), (257, -1)])
def test_tables_of_few_and_of_many_chunks(gpu_device, chunks, extra):
    # tables on both sides of 16, 32, 75 and 256 chunks, beside short ones and an empty one
    rng = np.random.default_rng(chunks)
    rows, per_table = [150_000, 9, 700, 2_000_000], [chunks * TILE + extra, 3 * TILE, 0, 17 * TILE]
    lens = np.concatenate([_lens(rng, 300, n) for n in per_table])
    idx = np.concatenate([np.minimum(rng.zipf(1.3, n) * 2_654_435_761 % h, h - 1) for h, n in zip(rows, per_table)])
    _check(gpu_device, rows, 300, lens, idx, "chunks")


@pytest.mark.parametrize("rows,batch,n", [(10_000_000, 65536, 2_000_001), (70_000, 70_001, 2_000_000), (60_000, 300, 1_000_000),
                                          (200, 65536, 200_003), (256, 70_001, 200_000)])   # payloads of 16 and 32 bits
def test_one_tall_table_is_sorted_by_digits(gpu_device, rows, batch, n):
    rng = np.random.default_rng(rows)
    idx = np.minimum(rng.zipf(1.2, n) * 2_654_435_761 % rows, rows - 1)
    _check(gpu_device, [rows], batch, _lens(rng, batch, n), idx, "digits")


def test_more_tables_than_the_partition_takes(gpu_device):
    rng = np.random.default_rng(5)
    T, batch = 4100, 9
    rows = rng.integers(1, 3000, T)
    lens = rng.integers(0, 7, T * batch)
    lens.reshape(T, batch)[rng.choice(T, 500, replace=False)] = 0
    t = np.repeat(np.arange(T), lens.reshape(T, batch).sum(1))
    _check(gpu_device, rows, batch, lens, (rng.random(t.size) * rows[t]).astype(np.int64), "many tables")


@pytest.mark.parametrize("T,batch,mean", [(4100, 5, 3.0), (1, 2000, 1800.0)])
def test_a_step_whose_lookups_are_sorted_by_digits(gpu_device, T, batch, mean):
    import tbe_testlib as tl
    from paper_2104_05158_amd import workloads as wl
    rng = np.random.default_rng(T)
    spec = wl.custom(rng.integers(50, 2000, T), rng.choice([4, 8], T), 0, batch, mean, index_dist="zipf", name="digits")
    b = wl.make_batch(spec, "cpu", seed=1)
    tl.full_parity_step(spec, b.indices.numpy(), b.offsets.numpy(), wl.make_weights(spec, "cpu", seed=2).numpy(),
                        wl.make_grad(spec, "cpu", seed=3).numpy(), gpu_device, what=f"{T} tables")
