"""GPU parity of the forward pass on both sides of the table size up to which rows are addressed by 32-bit offsets, and
of what an offset past the table or a mixed-precision addition could get wrong: bags that end inside a step, subnormal
values, Inf and NaN next to other bags' rows.

Oracle: the same gathers and sums in float64 by torch.  Tolerance: fp16 tables hold values of 2^-24 k, |k| < 2^10 here, so
sums of up to 70 of them are exact in fp32; fp32 sums of at most 70 terms are within 70 * 2^-24 of the sum of magnitudes."""
import numpy as np
import pytest
import torch

import tbe_testlib as tl
from paper_2104_05158_amd import workloads as wl

pytestmark = pytest.mark.gpu

LIMIT = 0xffff0000     # bytes
LENGTHS = [0, 1, 3, 4, 5, 15, 16, 17, 31, 33, 63, 64, 65, 70]


def _forward(device, rows, dims, dtype, w, idx, lens):
    spec = wl.custom(rows, dims, dtype, lens.shape[1], 1.0, name="offsets")
    op = tl.make_op(spec, device, max_indices=idx.numel(), weights=w)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens.ravel())])).to(device)
    return op.forward(idx.to(torch.int32), off, lens.shape[1], num_indices=idx.numel())


@pytest.mark.parametrize("batch", [600, 40000])              # one bag per wavefront, one per lane group
@pytest.mark.parametrize("dtype,dim", [(0, 256), (0, 512), (1, 128)])
@pytest.mark.parametrize("beyond", [False, True])
def test_tables_around_the_offset_limit(gpu_device, beyond, dtype, dim, batch):
    esz = 4 if dtype == 0 else 2
    rows = [LIMIT // (dim * esz) + (1 if beyond else 0), 1000]
    tdt = torch.float32 if dtype == 0 else torch.float16
    g = torch.Generator(device=gpu_device).manual_seed(7)
    w = torch.empty(sum(rows) * dim, dtype=tdt, device=gpu_device)
    # only the rows that are looked up are filled: both ends of the tables
    ids = [torch.cat([torch.arange(500), torch.arange(r - 500, r)]).to(gpu_device) for r in rows]
    w.zero_()
    for t, i in enumerate(ids):
        v = torch.randint(-1023, 1024, (i.numel(), dim), generator=g, device=gpu_device).to(torch.float32) * 2.0 ** -24
        w.view(-1, dim)[i + (rows[0] if t else 0)] = v.to(tdt)
    lens = np.resize(np.array(LENGTHS), (2, batch)) if batch == 600 else np.resize(np.array([0, 1, 3, 5, 2]), (2, batch))
    picks = [i[torch.randint(0, i.numel(), (int(l.sum()),), generator=g, device=gpu_device)] for i, l in zip(ids, lens)]
    print(f"rows={rows} dim={dim} dtype={dtype} batch={batch}", flush=True)
    out = _forward(gpu_device, rows, [dim, dim], dtype, w, torch.cat(picks), lens)
    for t in range(2):
        bag = torch.repeat_interleave(torch.arange(batch, device=gpu_device), torch.from_numpy(lens[t]).to(gpu_device))
        x = w.view(-1, dim)[picks[t] + (rows[0] if t else 0)].double()
        ref = torch.zeros(batch, dim, dtype=torch.float64, device=gpu_device).index_add_(0, bag, x)
        mag = torch.zeros_like(ref).index_add_(0, bag, x.abs())
        err = (out[:, t * dim:(t + 1) * dim].double() - ref).abs()
        assert bool((err <= 70 * 2.0 ** -24 * mag * (dtype == 0)).all())


@pytest.mark.parametrize("batch", [600, 40000])
@pytest.mark.parametrize("dim", [16, 36, 128, 512])
def test_non_finite_rows_reach_their_own_bags_only(gpu_device, dim, batch):
    rng = np.random.default_rng(5)
    rows = 300
    for dtype, tdt in ((0, torch.float32), (1, torch.float16)):
        w = torch.from_numpy(rng.integers(-1023, 1024, size=(rows, dim)) * 2.0 ** -24).to(tdt)
        w[rows - 1], w[rows - 2] = float("inf"), float("nan")
        lens = rng.integers(0, 8, size=(1, batch))
        idx = rng.integers(0, rows, size=int(lens.sum()))
        out = _forward(gpu_device, [rows], [dim], dtype, w.ravel().to(gpu_device), torch.from_numpy(idx).to(gpu_device), lens).cpu()
        bag = np.repeat(np.arange(batch), lens[0])
        ref = torch.zeros(batch, dim, dtype=torch.float64).index_add_(0, torch.from_numpy(bag), w.double()[torch.from_numpy(idx)])
        assert torch.equal(torch.isnan(out), torch.isnan(ref)) and torch.equal(torch.isinf(out), torch.isinf(ref))
        assert torch.equal(torch.nan_to_num(out, 0, 0, 0), torch.nan_to_num(ref, 0, 0, 0).float())
