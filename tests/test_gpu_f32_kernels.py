"""The fp32 path's projections (16-column tiles of 16, 32 or 64 rows) and attention (a
workgroup per row and head) at their edges, against the oracle: row counts around the tile
heights, a vocabulary that is no multiple of 16, head widths that leave idle threads, contexts
that end inside an octet or a page, and weights and pages that are only 4-byte aligned."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2601_11652_amd as W
import wisp_inputs as wi
from gpu_harness import Workload, check_written, gpu_model, pools_to_dev, run_gpu, to_dev
from oracle import fixtures as fx

pytestmark = pytest.mark.gpu

V301 = wi.ModelShape("f32-v301", 2, 96, 4, 2, 32, 160, 301, "f32", 10000.0)
HD96 = wi.ModelShape("f32-hd96-wave", 1, 192, 2, 1, 96, 64, 96, "f32", 10000.0)


def _mix(shape, rows):
    gamma = [16] * (rows // 17) + ([rows % 17 - 1] if rows % 17 else [])
    ctx = np.random.default_rng(rows).integers(0, 300, size=len(gamma)).astype(np.int32)
    return wi.custom_mix(shape, ctx, np.array(gamma, np.int32), kv_source="prefill", name=f"f32-{rows}")


def _check(shape, mix, wl, logits, pools):
    err = np.abs(logits - wl.logits_ref).max(axis=1) / np.abs(wl.logits_ref).max(axis=1)
    assert err.max() <= 1e-4
    check_written(pools, wl.pools_ref, wl.pools0, wl.pt, mix.ctx_len, mix.rows, shape.head_dim, False)


@pytest.mark.parametrize("shape", [V301, HD96], ids=lambda s: s.name)
@pytest.mark.parametrize("rows", [1, 16, 17, 32, 33, 64, 65, 130])
def test_row_and_column_edges(shape, rows):
    mix = _mix(shape, rows)
    wl = Workload(mix, fx.host_model(shape))
    _, _, logits, pools = run_gpu(gpu_model(shape), wl)
    _check(shape, mix, wl, logits, pools)


def test_operands_that_are_only_4_byte_aligned():
    mix = _mix(V301, 40)
    wl = Workload(mix, fx.host_model(V301))
    gm = gpu_model(V301)

    def shifted(t):
        b = torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")
        b[1:].copy_(t.reshape(-1))
        return b

    keep = [shifted(gm.lm_head)] + [shifted(l["w_down"]) for l in gm.layers]
    gm.c.lm_head = keep[0][1:].data_ptr()
    downs = (ctypes.c_void_p * 2)(*[t[1:].data_ptr() for t in keep[1:]])
    gm.c.w_down = ctypes.cast(downs, ctypes.POINTER(ctypes.c_void_p))
    _, _, logits, pools = run_gpu(gm, wl)
    _check(V301, mix, wl, logits, pools)
    # the attention alone on shifted pages
    model = W.GpuModel.shape_only(V301)
    desc = W.BatchDesc(mix.ctx_len, mix.gamma, to_dev(wl.pt), 1.0, mix.req_id)
    q = torch.randn(mix.M, V301.n_q_heads, V301.head_dim, device="cuda")
    outs = []
    k, v = pools_to_dev(wl.pools_ref, V301.head_dim)
    for kv in (W.KVPool(k[:1], v[:1]), W.KVPool(*[shifted(x[:1])[1:].view(x[:1].shape) for x in (k, v)])):
        out = torch.full_like(q, float("nan"))
        ws = W.workspace(W.wisp_workspace_size(model, desc))
        W.wisp_attention(model, kv, desc, q, out, ws)
        W.wisp_check(ws)
        outs.append(out.cpu())
    assert torch.isfinite(outs[0]).all() and torch.equal(outs[0], outs[1])
