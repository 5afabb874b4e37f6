"""GPU test of the input kernels at the sizes where their launch sequence changes: prefix sums of one workgroup, of
tiles that add up what lies before them, of tiles that read totals, of scanned totals; lengths on both sides of
the border between 32-bit and 64-bit wavefront sums; permutes whose blocks find their starts themselves (few large
blocks, also with empty and very uneven ones) and those that get them from a launch of their own; bucketize over
tiles and shard counts on both sides of its tables' sizes.  Bit-exact against the oracle or numpy."""
import numpy as np
import pytest
import torch

from oracle import inputs_oracle as io
from paper_2104_05158_amd import tbe
from test_gpu_inputs import _gpu_bucketize, _gpu_lengths_to_offsets, _gpu_permute

pytestmark = pytest.mark.gpu

TILE = 4096


@pytest.mark.parametrize("n", [8 * TILE - 1, 8 * TILE, 8 * TILE + 1, 9 * TILE + 7, 3072 * TILE, 3072 * TILE + 1, 4096 * TILE, 4096 * TILE + 1])
def test_prefix_sums_around_every_launch_border(gpu_device, n):
    lens = np.random.default_rng(n).integers(0, 60, n).astype(np.int32)
    got = _gpu_lengths_to_offsets(lens, gpu_device)
    assert np.array_equal(got, np.concatenate([[0], np.cumsum(lens, dtype=np.int64)]))


@pytest.mark.parametrize("top", [(1 << 23) - 1, 1 << 23, (1 << 31) - 1])
@pytest.mark.parametrize("n", [70, 3 * TILE + 5, 11 * TILE])
def test_prefix_sums_of_large_lengths(gpu_device, n, top):
    lens = np.random.default_rng(n).integers(0, 2, n).astype(np.int64) * top
    got = _gpu_lengths_to_offsets(lens.astype(np.int32), gpu_device)
    assert np.array_equal(got, np.concatenate([[0], np.cumsum(lens)]))


@pytest.mark.parametrize("W,T,B,kind", [(16, 16, 64, "uneven"), (16, 16, 64, "even"), (16, 17, 64, "even"), (2, 3, 4096, "even"),
                                        (5, 7, 333, "uneven"), (1, 256, 9, "uneven"),
                                        # one workgroup for the starts, and a prefix sum of sizes (of lengths for one bag a block)
                                        (32, 32, 5, "even"), (25, 41, 2, "uneven"), (25, 41, 3, "even"), (60, 70, 4, "uneven"),
                                        (41, 25, 1, "even"), (60, 70, 1, "uneven")])
def test_permute_starts(gpu_device, W, T, B, kind):
    rng = np.random.default_rng(W * T)
    n = W * T * B
    lens = np.full(n, 40, np.int32)
    if kind == "uneven":       # nearly everything in a few blocks, most blocks empty
        lens[:] = 0
        for r in rng.choice(W * T, 3, replace=False):
            lens[r * B:(r + 1) * B] = rng.integers(0, 2 * 40 * W * T, B)
    idx = rng.integers(0, 1 << 30, int(lens.sum())).astype(np.int32)
    ref = io.permute_wtb_to_twb(W, T, B, lens, idx)
    got = _gpu_permute(W, T, B, torch.from_numpy(lens).to(gpu_device), torch.from_numpy(idx).to(gpu_device), gpu_device)
    for g, r, name in zip(got, ref, ("lengths", "offsets", "indices")):
        assert np.array_equal(g, r), name


@pytest.mark.parametrize("W", [1, 2, 3, 8, 9, 33, 128, 129, 257, 1024])
def test_bucketize_divisors_and_remainders(gpu_device, W):
    """Shard sizes around powers of two up to 2^31, rows next to every shard border, bags that end off every tile."""
    rng = np.random.default_rng(W)
    blk = [1, 2, 3, 4, 5, 255, 256, 257, 65535, 65537, (1 << 20) + 1, (1 << 21) - 1, (1 << 31) // W]
    rows = np.array([min(b * W, (1 << 31) - 1) - k for b in blk for k in (0, 1) if b * W - k > 0], np.int64)
    T, B = len(rows), 261
    blks = (rows + W - 1) // W
    lens = rng.integers(0, 14, (T, B))
    lens[:, rng.choice(B, 20, replace=False)] = 0
    lens[0, 3] = 2048 * 2 + 1
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    per = lens.sum(1)
    idx = []
    for t in range(T):
        r = rng.integers(0, W, per[t]) * blks[t] + rng.integers(-1, 2, per[t])      # shard borders
        free = rng.integers(0, rows[t], per[t])
        idx.append(np.clip(np.where(rng.random(per[t]) < 0.5, r, free), 0, rows[t] - 1))
    idx = np.concatenate(idx).astype(np.int32)
    ref = io.bucketize_rowwise(rows, B, W, idx, offsets)
    got = _gpu_bucketize(rows, B, W, torch.from_numpy(idx).to(gpu_device), torch.from_numpy(offsets).to(gpu_device), gpu_device)
    for g, r, name in zip(got, ref, ("lengths", "offsets", "indices")):
        assert np.array_equal(g, r[:len(g)]), name
