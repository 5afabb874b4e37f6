"""GPU parity of the update's sums of rows that take the whole wavefront (more than 256 columns), six or eight of them in flight:
runs of every length around the steps, the 64 payloads a wavefront holds, the pieces, and runs of more pieces than it holds, beside
narrow tables, for every gradient type and layout.  The oracle gets the values the library reads; tolerances are the suite's."""
import numpy as np
import pytest
import torch

import tbe_testlib as tl
from paper_2104_05158_amd import tbe
from paper_2104_05158_amd import workloads as wl
from test_gpu_run_classes import _explicit_case

pytestmark = pytest.mark.gpu
GRADS = {"fp32": (tbe.TBE_DTYPE_FP32, torch.float32), "fp16": (tbe.TBE_DTYPE_FP16, torch.float16), "bf16": (tbe.TBE_DTYPE_BF16, torch.bfloat16)}


@pytest.mark.parametrize("grad", sorted(GRADS))
@pytest.mark.parametrize("dtype,layout", [(0, 0), (1, 0), (0, 1)])
def test_runs_around_the_steps_of_wide_rows(gpu_device, dtype, layout, grad):
    dims = [260, 512, 64, 384]
    lens = [np.array(list(range(1, 21)) + [47, 48, 49, 53, 54, 55, 59, 60, 61, 62, 63, 64, 65, 66, 69, 70, 71, 72, 73, 126, 127, 128, 129, 130, 191, 192,
                     193, 255, 256, 257, 385, 1000, 1537, 9000] + [1] * 40) for _ in dims]
    spec, idx, off = _explicit_case(dims, lens, batch=211, seed=61 + dtype, dtype=dtype)
    print(f"N={idx.size} dtype={dtype} layout={layout} {grad}", flush=True)
    w0 = wl.make_weights(spec, "cpu", seed=62).numpy()
    m0 = np.random.default_rng(63).uniform(0, 1, spec.total_rows).astype(np.float32)
    code, kind = GRADS[grad]
    g = wl.make_grad(spec, "cpu", seed=64).to(kind)
    ref = tl.oracle_step(spec, idx, off, w0, m0, g.float().numpy(), 0.03, 1e-8)
    op = tbe.TableBatchedEmbeddingBags(spec.rows, spec.dims, dtype, spec.batch, idx.size, device=gpu_device,
                                       weights=torch.from_numpy(w0.copy()).to(gpu_device), grad_dtype=code, layout=layout)
    op.state.copy_(torch.from_numpy(m0))
    g = torch.from_numpy(tl.to_table_major(g.float().numpy(), spec.dims)).to(kind) if layout else g
    op.backward_rowwise_adagrad(torch.from_numpy(idx).to(gpu_device), torch.from_numpy(off).to(gpu_device), spec.batch, g.to(gpu_device), 0.03, 1e-8)
    tl.assert_update_close(spec, ref, w0, m0, op.weights.cpu().numpy(), op.state.cpu().numpy(), 0.03, 1e-8, grad)
    op.close()
