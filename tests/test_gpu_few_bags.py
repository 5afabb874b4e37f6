"""GPU parity of the forward pass with one bag per wavefront (calls of few bags, or of wide rows) on both sides of every
border of the rule that chooses it.  Bag lengths lie around every step of the kernel: 1, 2, 4 and 8 rows for each of
the 64 / LPR lane groups, and the blocks of 64 indices.  Tolerance: the suite's for the forward pass (tbe_testlib)."""
import numpy as np
import pytest

import tbe_testlib as tl
from oracle import tbe_oracle as orc
from paper_2104_05158_amd import tbe
from paper_2104_05158_amd import workloads as wl

pytestmark = pytest.mark.gpu

LENGTHS = sorted({0} | {k * 2 ** g + d for g in range(7) for k in (1, 2, 4, 8) for d in (-1, 0, 1)} | {1000})
LIMIT = 32768     # bags


def _forward_matches(device, dims, batch, lens, dtype, layout, seed):
    """lens: [tables, batch]"""
    rng = np.random.default_rng(seed)
    rows = [int(r) for r in rng.integers(1, 3000, size=len(dims))]
    spec = wl.custom(rows, dims, dtype, batch, 1.0, name="few-bags")
    idx = np.concatenate([rng.integers(0, r, size=int(l.sum())) for r, l in zip(rows, lens)]).astype(np.int32)
    off = np.concatenate([[0], np.cumsum(lens.ravel())]).astype(np.int64)
    w = wl.make_weights(spec, "cpu", seed=seed).numpy()
    ref, scale = orc.forward(spec.rows, spec.dims, dtype, w, idx, off, batch, want_absref=True)
    import torch
    op = tl.make_op(spec, device, max_indices=max(idx.size, 1), weights=torch.from_numpy(w).to(device), layout=layout)
    d_idx = torch.from_numpy(idx if idx.size else np.zeros(1, np.int32)).to(device)
    got = op.forward(d_idx, torch.from_numpy(off).to(device), batch, num_indices=idx.size).cpu().numpy()
    if layout == tbe.TBE_LAYOUT_TABLE_MAJOR:
        got = tl.from_table_major(got.ravel(), batch, dims)
    print(f"dims={dims} batch={batch} N={idx.size} dtype={dtype} layout={layout}", flush=True)
    tl.assert_forward_close(got, ref, scale, f"{len(dims)} tables x {batch}")


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("dtype", [0, 1])
def test_lengths_around_every_step(gpu_device, dtype, layout):
    dims = [4, 8, 12, 36, 64, 128, 200, 256, 384, 512]
    rng = np.random.default_rng(3)
    lens = np.stack([rng.permutation(LENGTHS) for _ in dims])
    _forward_matches(gpu_device, dims, len(LENGTHS), lens, dtype, layout, seed=50 + dtype)
    # rows of up to 256 elements only: another lane mapping for either storage type
    _forward_matches(gpu_device, [d for d in dims if d <= 256], len(LENGTHS), lens[:8], dtype, layout, seed=52 + dtype)
    _forward_matches(gpu_device, [8, 64, 512], len(LENGTHS), lens[:3], dtype, layout, seed=54 + dtype)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("batch", [1, 8192 // 2 - 1, 8192 // 2, LIMIT // 2 - 1, LIMIT // 2])
@pytest.mark.parametrize("mean", [2.0, 5.0, 8.0])
def test_numbers_of_bags_around_the_limits(gpu_device, batch, dtype, mean):
    lens = np.random.default_rng(batch).poisson(mean, size=(2, batch))
    _forward_matches(gpu_device, [32, 4], batch, lens, dtype, 0, seed=60)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("length", [15, 16])
def test_many_bags_of_wide_rows(gpu_device, dtype, length):
    # rows that fill the wavefront: one bag per wavefront from 16 lookups a bag, whatever the number of bags
    _forward_matches(gpu_device, [260], LIMIT + 5, np.full((1, LIMIT + 5), length), dtype, 0, seed=62)


def test_all_bags_empty(gpu_device):
    _forward_matches(gpu_device, [16, 128], 5, np.zeros((2, 5), np.int64), 0, 0, seed=61)


def test_more_bags_of_wide_rows_than_one_bag_per_wavefront_can_launch(gpu_device):
    # 2^26 bags would be 2^32 threads; 16 lookups a bag, 1.07 G in all, output in 16 bits
    import torch
    batch, length, rows, dim = 1 << 26, 16, 1009, 132
    if torch.cuda.mem_get_info()[0] < 96 << 30:
        pytest.skip("needs about 60 GB of free device memory")
    w = wl.make_weights(wl.custom([rows], [dim], 0, 1, 1.0), "cpu", seed=9)
    op = tbe.TableBatchedEmbeddingBags([rows], [dim], 0, batch, batch * length, device=gpu_device,
                                       weights=w.to(gpu_device), output_dtype=tbe.TBE_DTYPE_FP16)
    idx = (torch.arange(batch * length, dtype=torch.int32, device=gpu_device) % rows)
    off = torch.arange(0, batch * length + 1, length, dtype=torch.int64, device=gpu_device)
    out = op.forward(idx, off, batch)
    bags = np.concatenate([np.arange(100), batch // 2 + np.arange(100), batch - 1 - np.arange(100)])
    got = out[torch.from_numpy(bags).to(gpu_device)].float().cpu().numpy()
    ref = w.numpy().reshape(rows, dim)[(bags[:, None] * length + np.arange(length)) % rows].astype(np.float64).sum(1)
    op.close()
    # fp32 sum of 16 terms, rounded once to fp16 (spacing 2^-24 below its normal range)
    assert np.all(np.abs(got - ref) <= 2.0 ** -11 * np.abs(ref) + 2.0 ** -24 + 16 * 2.0 ** -24 * 0.16)
