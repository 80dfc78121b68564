"""One request of the longest prompt with 64 query heads per kv head: more than 65536 row
groups of 32 rows.  The first and the last rows against plain torch in fp32 (the last ones
belong to the groups past 65536), the others for having been written at all.  Tolerance as in
the general attention test."""
import numpy as np
import pytest
import torch

import paper_2601_11652_amd as W
import wisp_inputs as wi
from gpu_harness import log, to_dev

pytestmark = pytest.mark.gpu


def test_more_than_65536_row_groups():
    n_q, hd, gamma = 64, 64, W.GAMMA_MAX
    T = W.PREFILL_MAX + gamma + 1
    rng = np.random.default_rng(5)
    n_blocks = (T + 15) // 16 + 2
    r = lambda a: ((a.view(np.uint32) + 0x7FFF + ((a.view(np.uint32) >> 16) & 1)) >> 16).astype(np.uint16)
    k, v = (r(rng.standard_normal((n_blocks, 1, 16, hd), np.float32)) for _ in range(2))
    perm = rng.permutation(n_blocks)[:(T + 15) // 16].astype(np.int32)
    shape = wi.ModelShape("attn", 1, 256, n_q, 1, hd, 256, 256, "bf16", 1e4)
    model = W.GpuModel.shape_only(shape)
    kv = W.KVPool(to_dev(wi.pages_from_slots(k, "k")[None]), to_dev(wi.pages_from_slots(v, "v")[None]))
    desc = W.BatchDesc([0], [gamma], to_dev(perm[None]), 1.0, prefill_len=[W.PREFILL_MAX])
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    q = torch.randn(T, n_q, hd, device="cuda", generator=g).to(torch.bfloat16)
    out = torch.full_like(q, float("nan"))
    plan = W.attention_plan(model, desc)
    log(f"{T} rows, {plan['rows']} per group, {plan['items'][:, 2].max() + 1} groups, {len(plan['items'])} items")
    ws = W.workspace(W.wisp_workspace_size(model, desc))
    W.wisp_attention(model, kv, desc, q, out, ws)
    W.wisp_check(ws)
    assert torch.isfinite(out).all()
    K, V = (to_dev(a[perm].reshape(-1, hd)).float()[:T] for a in (k, v))
    for rows in (range(0, 24), range(T - 24, T)):
        for j in rows:
            s = (q[j].float() @ K[:j + 1].t().contiguous()) / 8.0
            want = torch.softmax(s, -1) @ V[:j + 1]
            err = (out[j].float() - want).abs()
            assert err.max() < 2.5e-2 and err.mean() < 3e-3, (j, float(err.max()))
