"""GPU test of the long runs that the update kernel finds by position and finishes itself: whichever wavefront sums the last piece
of a run, the result is the same bits, update after update of one sort and from batch to batch, and it is the sum of
the run's gradient rows (a float64 sum; error bound n * 2^-24 of the sum of magnitudes for a sum of n terms in any order)."""
import numpy as np
import pytest
import torch

from paper_2104_05158_amd import tbe
from paper_2104_05158_amd import workloads as wl
from test_gpu_run_classes import _explicit_case

pytestmark = pytest.mark.gpu

STEPS = {
    tbe.TBE_OPT_ROWWISE_ADAGRAD: lambda op, g: op.backward_update_rowwise_adagrad(g, 0.01, 1e-8),
    tbe.TBE_OPT_ADAGRAD: lambda op, g: op.backward_update_adagrad(g, 0.01, 1e-8),
    tbe.TBE_OPT_ADAM: lambda op, g: op.backward_update_adam(g, 0.01, 0.9, 0.999, 1e-8, 1),
}


@pytest.mark.parametrize("opt", sorted(STEPS))
@pytest.mark.parametrize("dims,batch", [([128, 36], 900), ([512, 4, 64], 300)])
def test_every_update_gives_the_same_bits(gpu_device, opt, dims, batch):
    rng = np.random.default_rng(batch)
    lens = [np.concatenate([[129, 40_000, 255, 256, 257], rng.integers(120, 700, 120), rng.integers(1, 60, 300)]) for _ in dims]
    spec, idx, off = _explicit_case(dims, lens, batch=batch, seed=3, dtype=0)
    other = np.full_like(idx, 1)                         # a second batch: one run a table, other places
    w0 = wl.make_weights(spec, "cpu", seed=4)
    g = wl.make_grad(spec, "cpu", seed=5)
    print(f"N={idx.size} dims={dims} opt={opt}", flush=True)
    op = tbe.TableBatchedEmbeddingBags(spec.rows, spec.dims, 0, batch, idx.size, device=gpu_device, weights=w0.to(gpu_device), optimizer=opt)
    d_idx, d_off, d_g = (torch.from_numpy(x).to(gpu_device) for x in (idx, off, g.numpy()))
    d_w0, d_other = w0.to(gpu_device).reshape(-1), torch.from_numpy(other).to(gpu_device)
    first = None
    for again in range(8):
        if again == 4:                                   # (fresh counts after another batch)
            op.backward_sort(d_other, d_off, batch)
            STEPS[opt](op, d_g)
        if again in (0, 4):
            op.backward_sort(d_idx, d_off, batch)
        op.weights.reshape(-1).copy_(d_w0)
        op.state.zero_()
        STEPS[opt](op, d_g)
        got = (op.weights.cpu().numpy().copy(), op.state.cpu().numpy().copy())
        first = first or got
        assert np.array_equal(got[0], first[0]) and np.array_equal(got[1], first[1]), again
    if opt == tbe.TBE_OPT_ROWWISE_ADAGRAD:               # the moment is the mean square of the aggregated gradient
        base, col = 0, 0
        bag = np.repeat(np.arange(off.size - 1), np.diff(off))
        for t, (h, d) in enumerate(zip(spec.rows, spec.dims)):
            mine = (bag // batch) == t
            rows, b = idx[mine], bag[mine] % batch
            block = g.numpy()[:, col:col + d].astype(np.float64)
            G, A = np.zeros((h, d)), np.zeros((h, d))
            np.add.at(G, rows, block[b])
            np.add.at(A, rows, np.abs(block[b]))
            n = np.bincount(rows, minlength=h)
            err = np.minimum(n, 300)[:, None] * 2.0 ** -24 * A      # (sums of 128 .. 300 rows, of whose sums at most 300 again)
            bound = (2 * np.abs(G) * 2 * err + (2 * err) ** 2).mean(1) + 1e-6 * (G ** 2).mean(1) + 1e-12
            assert (np.abs(first[1].reshape(-1)[base:base + h] - (G ** 2).mean(1)) <= bound).all(), t
            base, col = base + h, col + d
    op.close()
