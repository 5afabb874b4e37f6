"""GPU parity of the two ways long runs are cut: by position while the largest gradient block of a table
(batch x dim x bytes) fits 4 MiB, by bag window and as dense rows beyond.  Run lengths lie on both sides of every
border: the threshold (128 by position, 512 by window, 1024 dense), whole pieces, and the length from which
pieces grow (128 x 256 lookups).  Tolerances are the suite's (tbe_testlib)."""
import numpy as np
import pytest

import tbe_testlib as tl
from paper_2104_05158_amd import workloads as wl
from test_gpu_run_classes import _explicit_case

pytestmark = pytest.mark.gpu

CASES = {
    # name: (batch, dims, run lengths of every table)
    "by_position": (53, [4, 64, 512], [127, 128, 129, 255, 256, 257, 385, 3000, 1, 1, 2]),
    "by_position_long_pieces": (700, [64, 8], [128 * 256 - 1, 128 * 256, 128 * 256 + 1, 70000, 5]),
    "block_of_exactly_4_MiB": (2048, [512, 4], [129, 511, 513, 1024, 1025, 5000] + [1] * 70),
    "block_beyond_4_MiB": (2200, [512, 4, 64, 128], [129, 511, 512, 513, 600, 1023, 1024, 1025, 3000, 5000] + [1] * 70),
}


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("case", sorted(CASES))
def test_long_runs_on_both_sides_of_every_border(gpu_device, case, dtype):
    batch, dims, lens = CASES[case]
    spec, idx, off = _explicit_case(dims, [np.array(lens) for _ in dims], batch=batch, seed=41 + dtype, dtype=dtype)
    w = wl.make_weights(spec, "cpu", seed=42).numpy()
    g = wl.make_grad(spec, "cpu", seed=43).numpy()
    m0 = np.random.default_rng(44).uniform(0, 1, spec.total_rows).astype(np.float32)
    print(f"{case}: N={idx.size} dtype={dtype}", flush=True)
    tl.full_parity_step(spec, idx, off, w, g, gpu_device, lr=0.03, m0=m0, what=case)


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("bad", [False, True])
def test_runs_by_position_beside_dense_ones(gpu_device, layout, bad):
    """A call of 4 M lookups whose gradient block fits 4 MiB: runs of 513 .. 1024 lookups are cut by position, longer ones
    summed as dense rows; a bag that holds one row 300 times (more than a count's byte) takes its table's dense runs
    to the plain sum."""
    rng = np.random.default_rng(7)
    batch, dims = 1100, [8, 64]
    lens = [np.concatenate([rng.integers(500, 1100, 900), rng.integers(1025, 6000, 500), [1, 2, 128, 129, 512, 513, 1024, 1025],
                            rng.integers(1, 300, 400), [20_000]]) for _ in dims]
    spec, idx, off = _explicit_case(dims, lens, batch=batch, seed=51, dtype=0)
    assert idx.size >= 4_000_000 and batch * max(dims) * 4 <= 4 << 20
    if bad:
        hot = int(np.argmax(np.bincount(idx[:off[batch]])))
        at = int(off[5])
        where = np.flatnonzero(idx[:off[batch]] == hot)[:300]
        idx[where], idx[at:at + 300] = idx[at:at + 300].copy(), hot
        assert off[6] - off[5] >= 300
    w = wl.make_weights(spec, "cpu", seed=52).numpy()
    g = wl.make_grad(spec, "cpu", seed=53).numpy()
    print(f"N={idx.size} layout={layout} bad={bad}", flush=True)
    tl.full_parity_step(spec, idx, off, w, g, gpu_device, lr=0.03, what="position and dense", layout=layout)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("n", [(1 << 19) - 37, 1 << 19, (1 << 19) + 1])
def test_long_runs_found_by_position_and_listed(gpu_device, n, dtype):
    """Calls on both sides of the size from which long runs are listed instead of found by position: runs that start at every
    place of the positions of a partial row, one behind the other and with short ones between, some of more than 256 pieces."""
    rng = np.random.default_rng(n)
    lens = [np.concatenate([rng.integers(120, 400, 500), [33_000, 40_000, 1, 64, 63, 129, 192, 193], rng.integers(1, 200, 300)]) for _ in range(2)]
    lens[0] = np.concatenate([lens[0], [1] * 3])
    rest = n - sum(int(x.sum()) for x in lens)
    lens[1] = np.concatenate([lens[1], [rest // 2, rest - rest // 2]])
    spec, idx, off = _explicit_case([128, 36], lens, batch=900, seed=55 + dtype, dtype=dtype)
    assert idx.size == n
    w = wl.make_weights(spec, "cpu", seed=56).numpy()
    g = wl.make_grad(spec, "cpu", seed=57).numpy()
    print(f"N={n} dtype={dtype}", flush=True)
    tl.full_parity_step(spec, idx, off, w, g, gpu_device, lr=0.03, what="found and listed")
