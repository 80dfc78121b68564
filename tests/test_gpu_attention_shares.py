"""bf16 attention over its work list, against the oracle.

The plan gives every item a wave or cuts the pairs of all row groups (of 32, 48 or 64 query
rows) into equal shares per wave, so the cases sit where a share begins, ends or changes its
operands: shares longer than the 64 pages whose block ids a wave holds at once, groups of one
and two pairs between long ones for each row count and head width (the next group's descriptor
and query rows are then not ahead), row groups with one row left, a context that ends inside a
page, prompts (32-row groups whose keys end at their own last row, dispatched in turn), and
query rows that are not 16-byte aligned (read through registers).  Every case states the rows
per group and whether waves run shares, and checks that the plan of 256 compute units does so.
Tolerance as in the general attention test: K, V and q are bf16 on both sides, the softmax
weights and the output are rounded to bf16, |error| <= ~2^-8 max|V|.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2601_11652_amd as W
import wisp_inputs as wi
from gpu_harness import log, to_dev

pytestmark = pytest.mark.gpu


def _run(ctx, gamma, prefill, n_q, n_kv, hd, seed, offset=0, plan=None):
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
    if plan and torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert _plan(ctx, gamma, prefill, n_q, n_kv, hd) == plan
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


def _plan(ctx, gamma, prefill, n_q, n_kv, hd):
    """(rows per group, whether waves run shares) of the plan."""
    model = W.GpuModel.shape_only(wi.ModelShape("attn", 1, 256, n_q, n_kv, hd, 256, 256, "bf16", 1e4))
    p = W.attention_plan(model, W.BatchDesc(ctx, gamma, None, 1.0, None, prefill if np.any(prefill) else None))
    return p["rows"], p["shares"]


def _mixed(n, lo, hi, seed, every=8):
    """Contexts of one or two pairs, every eighth a long one."""
    long = _spread(n, lo, hi, seed)
    return [long[k] if k % every == every - 1 else (7 * k) % 41 for k in range(n)]


CASES = [
    ("shares of several windows, 32 rows", _spread(40, 6000, 16000, 1), [k % 17 for k in range(40)], [0] * 40, 8, 8, 64, (32, True)),
    ("shares of several windows, up to 34 rows", _spread(26, 14000, 31000, 1), [k % 17 for k in range(26)], [0] * 26, 16, 8, 64, (32, True)),
    ("shares of several windows, 48 rows", _spread(26, 14000, 31000, 13), [16] * 26, [0] * 26, 16, 8, 64, (48, True)),
    ("32 rows, groups of one and two pairs", _mixed(400, 6000, 9000, 6), [k % 8 for k in range(400)], [0] * 400, 32, 8, 128, (32, True)),
    ("48 rows, groups of one and two pairs", _mixed(200, 4000, 9000, 7), [8 + k % 4 for k in range(200)], [0] * 200, 32, 8, 128, (48, True)),
    ("64 rows, groups of one and two pairs", _mixed(200, 4000, 9000, 8), [12 + k % 4 for k in range(200)], [0] * 200, 32, 8, 128, (64, True)),
    ("48 rows and 64 columns, groups of one and two pairs", _mixed(320, 5000, 9000, 9), [8 + k % 4 for k in range(320)], [0] * 320, 32, 8, 64, (48, True)),
    ("64 rows and 64 columns, groups of one and two pairs", _mixed(320, 4000, 9000, 10), [12 + k % 4 for k in range(320)], [0] * 320, 16, 4, 64, (64, True)),
    ("64 rows and one more", _spread(40, 3000, 6000, 11), [15, 16, 15, 12, 7] * 8, [0] * 40, 32, 8, 128, (64, True)),
    ("one item per wave, 48 rows", _spread(20, 2000, 9000, 2), [11, 3, 10, 0] * 5, [0] * 20, 32, 8, 128, (48, False)),
    ("one item per wave, 64 columns", _spread(20, 2000, 9000, 3), [15, 16, 12, 7, 0] * 4, [0] * 20, 16, 4, 64, (32, False)),
    ("one item per wave, 64 rows", _spread(12, 3000, 9000, 4), [15, 16, 14, 13] * 3, [0] * 12, 32, 8, 128, (64, False)),
    ("groups of one to four pairs between long ones", [15000 if k % 20 == 7 else k % 120 for k in range(240)],
     [k % 8 for k in range(240)], [0] * 240, 32, 8, 128, (32, True)),
    ("groups of one pair between long ones", [21000 + k if k % 16 == 3 else k % 24 for k in range(200)],
     [k % 7 for k in range(200)], [0] * 200, 16, 8, 64, (32, True)),
    ("one item per wave, more items than wave slots", [k % 90 for k in range(300)], [k % 8 for k in range(300)], [0] * 300, 32, 8, 128, (32, False)),
    ("one item per wave, two waves per SIMD", _spread(48, 700, 3000, 5), [k % 8 for k in range(48)], [0] * 48, 32, 8, 128, (32, False)),
    ("keys shared by row groups, 64 columns", _spread(64, 1000, 3000, 12), [15, 16] * 32, [0] * 64, 32, 4, 64, (48, False)),
    ("prompts in turn", [16, 9000, 3], [1, 0, 2], [2100, 300, 1999], 32, 8, 128, (32, False)),
    ("prompts", [0, 37, 500, 16], [3, 0, 5, 1], [600, 257, 0, 70], 32, 8, 128, (32, False)),
    ("prompts, 64 columns", [5, 0, 900], [2, 4, 8], [333, 512, 0], 16, 2, 64, (32, False)),
]


@pytest.mark.parametrize("name,ctx,gamma,prefill,n_q,n_kv,hd,plan", CASES, ids=[c[0] for c in CASES])
def test_attention_shares_match_oracle(name, ctx, gamma, prefill, n_q, n_kv, hd, plan):
    log(f"attention: {name}")
    _run(ctx, gamma, prefill, n_q, n_kv, hd, seed=len(ctx) + n_q, plan=plan)


@pytest.mark.parametrize("ctx,gamma", [([40, 700, 3], [2, 7, 0]), ([k % 60 for k in range(200)], [k % 5 for k in range(200)])])
@pytest.mark.parametrize("offset", [0, 4])
def test_attention_query_alignment(ctx, gamma, offset):
    log(f"attention of {len(ctx)} requests, q {2 * offset} bytes past an aligned address")
    _run(ctx, gamma, [0] * len(ctx), 32, 8, 128, seed=7, offset=offset)
