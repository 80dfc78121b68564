"""bf16 attention where one wave runs several work items, against the oracle.

Beyond 16 page pairs per wave the plan cuts the pairs of all row groups into equal shares per
wave (groups of 32, 48 or 64 query rows), below it gives every item a wave, so the cases sit where a share begins, ends or changes its operands: shares
longer than the 64 pages whose block ids a wave holds at once, groups of one and two pairs
(the next group's descriptor and query rows are then not ahead), row groups with one row left,
a context that ends inside a page, prompts (32-row groups whose keys end at their own last
row), and query rows that are not 16-byte aligned (read through registers).  Tolerance as in
the general attention test: K, V and q are bf16 on both sides, the softmax weights and the
output are rounded to bf16, |error| <= ~2^-8 max|V|.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2601_11652_amd as W
import wisp_inputs as wi
from gpu_harness import log, to_dev

pytestmark = pytest.mark.gpu


def _run(ctx, gamma, prefill, n_q, n_kv, hd, seed, offset=0):
    rng = np.random.default_rng(seed)
    ctx, gamma, prefill = (np.asarray(a, np.int32) for a in (ctx, gamma, prefill))
    rows = prefill + gamma + 1
    need = (ctx + rows + 15) // 16
    n_blocks = int(min(need.sum(), 700)) + 3            # requests may share pages: only read here
    pt = np.full((len(ctx), int(need.max()) + 1), -1, np.int32)
    for i, n in enumerate(need):
        pt[i, :n] = rng.integers(0, n_blocks, n)
    r = lambda a: ((a.view(np.uint32) + 0x7FFF + ((a.view(np.uint32) >> 16) & 1)) >> 16).astype(np.uint16)
    k, v = (r(rng.standard_normal((n_blocks, n_kv, 16, hd), np.float32)) for _ in range(2))
    q = r(rng.standard_normal((int(rows.sum()), n_q, hd), np.float32))
    shape = wi.ModelShape("attn", 1, 256, n_q, n_kv, hd, 256, 256, "bf16", 1e4)
    model = W.GpuModel.shape_only(shape)
    kv = W.KVPool(to_dev(wi.pages_from_slots(k, "k")[None]), to_dev(wi.pages_from_slots(v, "v")[None]))
    desc = W.BatchDesc(ctx, gamma, to_dev(pt), 1.0, **({"prefill_len": prefill} if prefill.any() else {}))
    ws = W.workspace(W.wisp_workspace_size(model, desc))
    buf = torch.zeros(q.size + offset, dtype=torch.int16, device="cuda")
    dq = buf[offset:].view(torch.bfloat16).view(q.shape)
    dq.copy_(torch.from_numpy(q.view(np.int16)).view(torch.bfloat16))
    out = torch.zeros(q.shape, dtype=torch.bfloat16, device="cuda")
    W.wisp_attention(model, kv, desc, dq, out, ws)
    W.wisp_check(ws)
    f = lambda a: (a.astype(np.uint32) << 16).view(np.float32)
    got = f(out.cpu().view(torch.int16).numpy().view(np.uint16)).astype(np.float64)
    want = oracle.paged_attention(f(q).astype(np.float64), k.reshape(n_blocks, n_kv, 16 * hd),
                                  v.reshape(n_blocks, n_kv, 16 * hd), pt, ctx, rows, n_kv, True)
    err = np.abs(got - want)
    log(f"  max {err.max():.2e} mean {err.mean():.2e}")
    assert err.max() < 2.5e-2, err.max()
    assert err.mean() < 3e-3, err.mean()
    # every output row depends on its own query rows only: in place gives the same bytes
    W.wisp_attention(model, kv, desc, dq, dq, ws)
    W.wisp_check(ws)
    assert torch.equal(dq.view(torch.int16), out.view(torch.int16))


def _spread(n, lo, hi, seed):
    return np.exp(np.random.default_rng(seed).uniform(np.log(lo), np.log(hi), n)).astype(int).tolist()


@pytest.mark.parametrize("name,ctx,gamma,prefill,n_q,n_kv,hd", [
    ("32 rows, shares of several windows", _spread(26, 14000, 31000, 1), [k % 17 for k in range(26)], [0] * 26, 16, 8, 64),
    ("48 rows", _spread(20, 2000, 9000, 2), [11, 3, 10, 0] * 5, [0] * 20, 32, 8, 128),
    ("64 rows and one more", _spread(20, 2000, 9000, 3), [15, 16, 12, 7, 0] * 4, [0] * 20, 16, 4, 64),
    ("64 rows, 128 columns", _spread(12, 3000, 9000, 4), [15, 16, 14, 13] * 3, [0] * 12, 32, 8, 128),
    ("groups of one to four pairs between long ones", [15000 if k % 20 == 7 else k % 120 for k in range(240)],
     [k % 8 for k in range(240)], [0] * 240, 32, 8, 128),
    ("groups of one pair between long ones", [21000 + k if k % 16 == 3 else k % 24 for k in range(200)],
     [k % 7 for k in range(200)], [0] * 200, 16, 8, 64),
    ("one item per wave, more items than wave slots", [k % 90 for k in range(300)], [k % 8 for k in range(300)], [0] * 300, 32, 8, 128),
    ("one item per wave, two waves per SIMD", _spread(48, 700, 3000, 5), [k % 8 for k in range(48)], [0] * 48, 32, 8, 128),
    ("prompts in shares", [16, 9000, 3], [1, 0, 2], [2100, 300, 1999], 32, 8, 128),
    ("prompts", [0, 37, 500, 16], [3, 0, 5, 1], [600, 257, 0, 70], 32, 8, 128),
    ("prompts, 64 columns", [5, 0, 900], [2, 4, 8], [333, 512, 0], 16, 2, 64),
])
def test_attention_shares_match_oracle(name, ctx, gamma, prefill, n_q, n_kv, hd):
    log(f"attention shares: {name}")
    _run(ctx, gamma, prefill, n_q, n_kv, hd, seed=len(ctx) + n_q)


@pytest.mark.parametrize("ctx,gamma", [([40, 700, 3], [2, 7, 0]), ([k % 60 for k in range(200)], [k % 5 for k in range(200)])])
@pytest.mark.parametrize("offset", [0, 4])
def test_attention_query_alignment(ctx, gamma, offset):
    log(f"attention of {len(ctx)} requests, q {2 * offset} bytes past an aligned address")
    _run(ctx, gamma, [0] * len(ctx), 32, 8, 128, seed=7, offset=offset)
