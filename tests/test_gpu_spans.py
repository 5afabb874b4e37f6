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


SMALL = {
    # name: (dims, run lengths of every table): calls whose long runs the update kernel's own workgroups sum, or just do not
    "around_the_threshold": ([64], [127, 128, 129, 130, 131, 1, 1, 2, 255, 256, 257, 600]),
    "most_lookups_64": ([64], [4096 - 129, 129]),
    "one_more_64": ([64], [4096 - 129, 130]),
    "most_lookups_512": ([512], [383, 129]),
    "one_more_512": ([512], [383, 130]),
    "several_tables": ([8, 36, 128], [129, 1, 300, 128, 40]),
    "narrow_rows": ([4], [8192 - 129 * 9] + [129] * 9),
}


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("case", sorted(SMALL))
def test_long_runs_of_small_calls(gpu_device, case, dtype, layout):
    dims, lens = SMALL[case]
    spec, idx, off = _explicit_case(dims, [np.array(lens) for _ in dims], batch=67, seed=71 + dtype, dtype=dtype)
    w = wl.make_weights(spec, "cpu", seed=72).numpy()
    g = wl.make_grad(spec, "cpu", seed=73).numpy()
    m0 = np.random.default_rng(74).uniform(0, 1, spec.total_rows).astype(np.float32)
    print(f"{case}: N={idx.size} dtype={dtype} layout={layout}", flush=True)
    tl.full_parity_step(spec, idx, off, w, g, gpu_device, lr=0.03, m0=m0, what=case, layout=layout)


def test_small_long_runs_with_other_optimizers_and_repeated_updates(gpu_device):
    import torch

    import test_gpu_optimizers as tgo
    from paper_2104_05158_amd import tbe

    spec, idx, off = _explicit_case([64, 12], [np.array([129, 700, 1, 2, 128])] * 2, batch=31, seed=81, dtype=0)
    for optimizer in (tbe.TBE_OPT_ADAGRAD, tbe.TBE_OPT_ADAM):
        tgo._run(spec, optimizer, tbe.TBE_DTYPE_FP32, gpu_device, steps=2, seed=82, batch=(idx, off))
    # two updates after one sort leave what two whole steps leave
    w = wl.make_weights(spec, "cpu", seed=83).to(gpu_device)
    d_idx, d_off = torch.from_numpy(idx).to(gpu_device), torch.from_numpy(off).to(gpu_device)
    d_g = wl.make_grad(spec, "cpu", seed=84).to(gpu_device)
    a, b = (tl.make_op(spec, gpu_device, max_indices=idx.size, weights=w.clone()) for _ in range(2))
    a.backward_sort(d_idx, d_off, spec.batch)
    for _ in range(2):
        a.backward_update_rowwise_adagrad(d_g, 0.05, 1e-8)
        b.backward_rowwise_adagrad(d_idx, d_off, spec.batch, d_g, 0.05, 1e-8)
    assert torch.equal(a.weights, b.weights) and torch.equal(a.state, b.state)
    a.close()
    b.close()
