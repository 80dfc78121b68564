"""wisp_verify_noalloc (the entry point for callers that cannot allocate) against
wisp_verify through the C ABI: two calls in a row on one GPU, the second with a smaller
batch, on the fp32 and the bf16 model.  Same kernels and plan, so the outputs (logits,
accept lengths, emitted tokens) and the KV written into the pools must be identical to
the workspace path's, bit for bit; a token id out of range is reported through the
caller's fault word and not through later clean calls.  A batch whose attention partials alone
would pass the static scratch runs with fewer of them: the same results within rounding."""
import numpy as np
import pytest
import torch

import paper_2601_11652_amd as W
import wisp_inputs as wi
from oracle import fixtures as fx
from gpu_harness import Workload, check_decisions_on_gpu_logits, gpu_model, log, pools_to_dev, to_dev

pytestmark = pytest.mark.gpu

MINI_BF16 = wi.ModelShape("mini-bf16-gqa", 2, 256, 8, 2, 64, 512, 1024, "bf16", 10000.0)


def _run_both(gm, wl):
    mix = wl.mix
    hd = mix.shape.head_dim
    desc = W.BatchDesc(mix.ctx_len, mix.gamma, to_dev(wl.pt), wl.T, mix.req_id)
    tokens = to_dev(wl.tokens)
    q = to_dev(wl.q) if wl.q.shape[0] else torch.zeros(1, dtype=torch.float32, device="cuda")
    outs = []
    for path in ("workspace", "noalloc"):
        kv = W.KVPool(*pools_to_dev(wl.pools0, hd))
        acc = torch.full((mix.B,), -7, dtype=torch.int32, device="cuda")
        out = torch.full((mix.M,), -7, dtype=torch.int32, device="cuda")
        logits = torch.full((mix.M, mix.shape.vocab), float("nan"), dtype=torch.float32, device="cuda")
        if path == "workspace":
            ws = W.workspace(W.wisp_workspace_size(gm.c, desc))
            W.wisp_verify(gm.c, kv, desc, tokens, q, wl.seed, acc, out, logits, ws)
            W.wisp_check(ws)
        else:
            fault = torch.zeros(1, dtype=torch.int32, device="cuda")
            W.wisp_verify_noalloc(gm.c, kv, desc, tokens, q, wl.seed, acc, out, logits, fault)
            torch.cuda.synchronize()
            assert int(fault.item()) == 0
        torch.cuda.synchronize()
        outs.append((acc.cpu().numpy(), out.cpu().numpy(), logits.cpu().numpy(), kv.k.cpu(), kv.v.cpu()))
    return outs


@pytest.mark.parametrize("shape", [wi.TINY, MINI_BF16], ids=["fp32", "bf16"])
def test_noalloc_matches_the_workspace_path_twice(shape):
    gm = gpu_model(shape)
    model = fx.host_model(shape)
    # a batch, then a smaller one: the shared scratch keeps the first call's contents
    for name, ctx, gamma in (("first", [37, 0, 90, 15, 120, 3], [4, 16, 2, 0, 7, 1]), ("second", [50, 8], [3, 1])):
        mix = wi.custom_mix(shape, ctx, gamma, kv_source="prefill", name=f"noalloc-{name}", t_draft=1.0, sigma=0.5)
        log(f"{shape.name} {name}: ctx={ctx} gamma={gamma} (M = {mix.M})")
        (a1, o1, l1, k1, v1), (a2, o2, l2, k2, v2) = _run_both(gm, Workload(mix, model))
        np.testing.assert_array_equal(a1, a2)
        np.testing.assert_array_equal(o1, o2)
        np.testing.assert_array_equal(l1, l2)
        assert torch.equal(k1, k2) and torch.equal(v1, v2)


def test_noalloc_reports_faults_in_the_callers_word():
    shape = wi.TINY
    mix = wi.custom_mix(shape, [20, 40], [2, 3], name="noalloc-fault")
    pt_np, nb = wi.page_table(mix)
    gm = gpu_model(shape)
    kv = W.KVPool.zeros(shape.n_layers, nb, shape.n_kv_heads, shape.head_dim, torch.float32)
    desc = W.BatchDesc(mix.ctx_len, mix.gamma, to_dev(pt_np), 1.0)
    q = torch.full((int(mix.gamma.sum()), shape.vocab), 1.0 / shape.vocab, device="cuda")
    acc = torch.empty(mix.B, dtype=torch.int32, device="cuda")
    out = torch.empty(mix.M, dtype=torch.int32, device="cuda")
    logits = torch.empty(mix.M, shape.vocab, device="cuda")
    bad = torch.zeros(mix.M, dtype=torch.int32, device="cuda")
    bad[2] = shape.vocab
    good = torch.zeros(mix.M, dtype=torch.int32, device="cuda")
    fault = torch.zeros(1, dtype=torch.int32, device="cuda")
    W.wisp_verify_noalloc(gm.c, kv, desc, bad, q, 1, acc, out, logits, fault)
    W.wisp_verify_noalloc(gm.c, kv, desc, good, q, 2, acc, out, logits, fault)
    torch.cuda.synchronize()
    assert int(fault.item()) == 1            # the token-id bit, kept across the clean call
    fault.zero_()
    W.wisp_verify_noalloc(gm.c, kv, desc, good, q, 3, acc, out, logits, fault)
    torch.cuda.synchronize()
    assert int(fault.item()) == 0


@pytest.mark.parametrize("n_kv,hd,ctx", [(4, 128, 500), (8, 64, 2000)], ids=["whole groups", "longer items"])
def test_noalloc_with_fewer_attention_partials(n_kv, hd, ctx):
    """120 requests of 17 rows: the workspace of wisp_verify passes the static scratch, through
    its partials; noalloc cuts the contexts into fewer parts (or none).  Logits within the
    stated bf16 bound of wisp_verify's, 2e-2 max-abs, K/V within two bf16 roundings of values of
    that size, decisions as the oracle takes them on the same logits."""
    shape = wi.ModelShape(f"noalloc-{n_kv}", 1, 512, 32, n_kv, hd, 512, 1024, "bf16", 10000.0)
    B, gamma = 120, 16
    mix = wi.custom_mix(shape, [ctx + 3 * k for k in range(B)], [gamma] * B, name="noalloc-big")
    pt, nb = wi.page_table(mix)
    gm = gpu_model(shape)
    desc = W.BatchDesc(mix.ctx_len, mix.gamma, to_dev(pt), 1.0, mix.req_id)
    need = W.wisp_workspace_size(gm.c, desc)
    log(f"{shape.name}: workspace {need >> 20} MiB")
    assert need > 128 << 20
    g = torch.Generator(device="cuda")
    g.manual_seed(17)
    pool = lambda: torch.randn(1, nb, n_kv, 16 * hd, device="cuda", generator=g).to(torch.bfloat16)
    k0, v0 = pool(), pool()
    q = torch.softmax(2.5 * torch.randn(B * gamma, shape.vocab, device="cuda", generator=g), -1)
    tokens = torch.randint(0, shape.vocab, (mix.M,), device="cuda", dtype=torch.int32, generator=g)
    res = []
    for noalloc in (False, True, True):
        kv = W.KVPool(k0.clone(), v0.clone())
        acc = torch.full((B,), -7, dtype=torch.int32, device="cuda")
        out = torch.full((mix.M,), -7, dtype=torch.int32, device="cuda")
        logits = torch.full((mix.M, shape.vocab), float("nan"), device="cuda")
        if noalloc:
            fault = torch.zeros(1, dtype=torch.int32, device="cuda")
            W.wisp_verify_noalloc(gm.c, kv, desc, tokens, q, 5, acc, out, logits, fault)
            assert int(fault.item()) == 0
        else:
            ws = W.workspace(need)
            W.wisp_verify(gm.c, kv, desc, tokens, q, 5, acc, out, logits, ws)
            W.wisp_check(ws)
        res.append((logits, kv.k, kv.v, acc, out))
    d = (res[1][0] - res[0][0]).abs().max().item()
    log(f"  logits differ by at most {d:.3e}")
    assert d <= 2e-2
    for a, b in zip(res[0][1:3], res[1][1:3]):
        assert ((a.float() - b.float()).abs() <= 2 * 2.0 ** -8 * a.float().abs().max()).all()
    for a, b in zip(res[1], res[2]):
        assert torch.equal(a, b)
    n = [x.cpu().numpy() for x in (res[1][3], res[1][4], res[1][0], tokens, q)]
    check_decisions_on_gpu_logits(n[0], n[1], n[2], n[3], n[4], mix.gamma, 1.0, 5, req_id=mix.req_id)
