"""The row kernels (embedding + norm, split sums + residual + norm, RoPE + append) at their
edges, through whole bf16 steps against the oracle: row counts around the 64 from which rows
are dealt to the XCDs in blocks of 8, row lengths that leave threads without columns, norm
gains and embeddings that are not 16-byte aligned (read element by element).

The unaligned models hold the same numbers as the aligned ones, so every output must be the
same, bit for bit."""
import numpy as np
import pytest
import torch

import wisp_inputs as wi
from gpu_harness import Workload, check_written, gpu_model, log, run_gpu
from oracle import fixtures as fx

pytestmark = pytest.mark.gpu


def _unaligned(t):
    buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    buf[1:].copy_(t.reshape(-1))
    return buf[1:]


@pytest.mark.parametrize("d_model", [256, 288])
@pytest.mark.parametrize("rows", [63, 64, 65, 130])
def test_steps_around_the_row_blocks(rows, d_model):
    shape = wi.ModelShape(f"rows-{d_model}", 2, d_model, 4, 2, 64, 512, 1024, "bf16", 10000.0)
    gamma, left = [], rows
    while left > 0:                                  # requests of up to 17 rows, the last shorter
        gamma.append(min(left, 17) - 1)
        left -= gamma[-1] + 1
    ctx = [(13 * k) % 40 + 1 for k in range(len(gamma))]
    mix = wi.custom_mix(shape, ctx, gamma, kv_source="prefill", name=f"rows{rows}", t_draft=1.0, sigma=0.5)
    log(f"rows {rows} d_model {d_model}")
    wl = Workload(mix, fx.host_model(shape))
    gm = gpu_model(shape)
    acc, out, logits, pools = run_gpu(gm, wl)
    d = np.abs(logits - wl.logits_ref)
    log(f"  max-abs logits error {d.max():.3e}")
    assert d.max() <= 2e-2                           # the bar of the small bf16 model's other steps
    check_written(pools, wl.pools_ref, wl.pools0, wl.pt, mix.ctx_len, mix.rows, shape.head_dim, True,
                  pools_ref32=wl.pools_ref32)
    keep = []
    for name in ("attn_norm", "mlp_norm"):
        for l, layer in enumerate(gm.layers):
            keep.append(_unaligned(layer[name]))
            gm._arrs[name][l] = keep[-1].data_ptr()
    keep += [_unaligned(gm.embed), _unaligned(gm.final_norm)]
    gm.c.embed, gm.c.final_norm = keep[-2].data_ptr(), keep[-1].data_ptr()
    again = run_gpu(gm, wl)
    for x, y in zip((acc, out, logits), again[:3]):
        np.testing.assert_array_equal(x, y)
