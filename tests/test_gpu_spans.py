"""GPU parity of the update kernel's spans of 16, 32, 64 and 128 sorted positions: which one a call takes depends on its
lookups and on the width of its rows.  Runs that end on, before and behind the end of a span and of the payloads staged
with it, runs that cover whole spans, and a ragged last span.  Tolerances are the suite's (tbe_testlib)."""
import numpy as np
import pytest

import tbe_testlib as tl
from paper_2104_05158_amd import workloads as wl
from test_gpu_run_classes import _explicit_case

pytestmark = pytest.mark.gpu

LENS = [1, 2, 14, 1, 15, 16, 17, 1, 31, 32, 33, 48, 49, 63, 64, 65, 80, 96, 127, 128, 129, 200, 511, 512, 513, 640]


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("span, dims, copies", [(16, [8], 4), (16, [512, 64, 4], 3), (32, [8], 25), (64, [8], 45), (64, [8, 8], 30),
                                                (128, [8, 4], 56)])
def test_runs_around_the_ends_of_spans(gpu_device, span, dims, copies, dtype):
    lens = [np.concatenate([LENS] * copies + [[1] * (7 + t)]) for t in range(len(dims))]
    spec, idx, off = _explicit_case(dims, lens, batch=701, seed=61 + dtype, dtype=dtype)
    lanes = sum((d + 7) // 8 for d in dims) / len(dims)
    assert span == next((s for s in (16, 32, 64) if idx.size <= s * 4096 * lanes), 128)
    w = wl.make_weights(spec, "cpu", seed=62).numpy()
    g = wl.make_grad(spec, "cpu", seed=63).numpy()
    print(f"span {span}: N={idx.size} dims={dims} dtype={dtype}", flush=True)
    tl.full_parity_step(spec, idx, off, w, g, gpu_device, lr=0.03, what="spans")
