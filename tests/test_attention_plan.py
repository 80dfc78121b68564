"""The attention work list on the CPU (wisp_attention_plan): whatever the batch, every row
group's keys are covered once and in order, the waves' runs of items are contiguous, and the
figures agree with the items."""
import numpy as np
import pytest

import paper_2601_11652_amd as W
from test_abi import W as _built  # noqa: F401  (builds the library if it is not there)

FAKE = 0x1000


@pytest.fixture(autouse=True)
def _library(_built):  # noqa: F811
    pass


def model(n_q, n_kv, hd, **kw):
    m = W.wisp_model(1, 256, n_q, n_kv, hd, 256, 256, 1e-5, 1e4, W.WISP_BF16, FAKE, FAKE, FAKE)
    for k, v in kw.items():
        setattr(m, k, v)
    return m


def check(n_q, n_kv, hd, ctx, gamma, prefill=None):
    ctx, gamma = np.asarray(ctx, np.int64), np.asarray(gamma, np.int64)
    pre = np.zeros_like(ctx) if prefill is None else np.asarray(prefill, np.int64)
    desc = W.BatchDesc(ctx, gamma, None, 1.0, None, pre if pre.any() else None)
    p = W.attention_plan(model(n_q, n_kv, hd), desc)
    it, G, R = p["items"].astype(np.int64), n_q // n_kv, p["rows"]
    assert R in (32, 48, 64)
    # the row groups in order, and the last key each may see
    rows = (pre + gamma + 1) * G
    want = [(i, h, g, int(ctx[i] + (min(rows[i], (g + 1) * R) - 1) // G + 1))
            for i in range(len(ctx)) for h in range(n_kv) for g in range(-(-int(rows[i]) // R))]
    starts = np.flatnonzero(it[:, 3] == 0)
    assert len(starts) == len(want)
    np.testing.assert_array_equal(it[starts][:, :3], np.array(want)[:, :3])
    ends = np.append(starts[1:], len(it))
    np.testing.assert_array_equal(it[ends - 1, 4], np.array(want)[:, 3])
    same = np.ones(len(it), bool)
    same[starts] = False                        # items that go on with the group of the one before
    k = np.flatnonzero(same)
    np.testing.assert_array_equal(it[k, :3], it[k - 1, :3])
    np.testing.assert_array_equal(it[k, 3], it[k - 1, 4])
    assert (it[:, 3] % 32 == 0).all() and (it[:, 3] < it[:, 4]).all()
    n = ends - starts
    np.testing.assert_array_equal(it[:, 5], np.repeat(n, n) == 1)
    assert p["combined"] == (n > 1).sum() and p["most"] == n.max()
    # waves: every item in one, runs of neighbours, none past the last wave
    w = it[:, 6]
    assert w[0] >= 0 and (np.diff(w) >= 0).all() and w[-1] < p["waves"]
    if not p["shares"]:
        np.testing.assert_array_equal(w, np.arange(len(it)))
    return p


@pytest.mark.parametrize("n_q,n_kv,hd", [(32, 8, 128), (64, 8, 128), (16, 16, 128), (32, 2, 128), (16, 8, 64), (6, 3, 64),
                                         (64, 1, 64)])
def test_every_key_is_covered_once(n_q, n_kv, hd):
    rng = np.random.default_rng(n_q + n_kv)
    for _ in range(60):
        B = int(np.exp(rng.uniform(0, np.log(200))))
        hi = int(np.exp(rng.uniform(0, np.log(30000))))
        pre = np.where(rng.random(B) < rng.choice([0, 0.2]), rng.integers(1, 700, B), 0)
        check(n_q, n_kv, hd, rng.integers(0, hi + 1, B), rng.integers(0, 17, B), pre)


def test_one_request_of_more_than_65536_row_groups():
    """The longest prompt with 64 query heads per kv head has 65570 groups of 32 rows."""
    p = check(64, 1, 64, [0], [W.GAMMA_MAX], [W.PREFILL_MAX])
    assert p["items"][:, 2].max() == -(-(W.PREFILL_MAX + W.GAMMA_MAX + 1) * 64 // p["rows"]) - 1
    check(128, 2, 64, [5, 3], [W.GAMMA_MAX, 2], [W.PREFILL_MAX, 40])


@pytest.mark.parametrize("n_q,n_kv,hd,ctx,gamma,prefill,rows,shares", [
    # latency: a few requests take 32-row items whatever their heads, and one wave per item
    (64, 8, 128, [500, 900, 2000, 4000], [2, 8, 5, 1], None, 32, False),
    (32, 2, 128, [1200], [8], None, 32, False),
    (64, 8, 64, [2000, 8000], [8, 8], None, 32, False),
    # and up to 8 of them per group where more would have many partials
    (32, 8, 128, [600 + 190 * k for k in range(8)], [1 + k for k in range(8)], None, 32, False),
    # long contexts of few requests: more items per group than one round of the combine
    (32, 8, 128, [30000], [8], None, 32, False),
    # prompts: 32-row items, dispatched in turn
    (64, 8, 128, [0, 0], [2, 2], [4000, 4000], 32, False),
    (32, 8, 128, [500, 0], [5, 5], [0, 2048], 32, False),
    # many requests: shares of 48 or 64 rows; at head_dim 64 items where row groups share keys
    (32, 8, 128, [1000 + 27 * k for k in range(256)], [k % 9 for k in range(256)], None, 48, True),
    (64, 8, 128, [1000 + 27 * k for k in range(256)], [k % 8 for k in range(256)], None, 64, True),
    (64, 8, 64, [1000 + 27 * k for k in range(256)], [k % 8 for k in range(256)], None, 48, False),
])
def test_choices(n_q, n_kv, hd, ctx, gamma, prefill, rows, shares):
    p = check(n_q, n_kv, hd, ctx, gamma, prefill)
    assert (p["rows"], p["shares"]) == (rows, shares), (p["rows"], p["shares"], p["waves"])
    if len(ctx) == 1 and ctx[0] == 30000:
        assert p["most"] > 8 and p["waves"] <= 1024
    if len(ctx) == 8:
        assert p["most"] <= 8, p["most"]


def test_gpu_cases_take_the_plan_they_are_written_for():
    """The cases of the attention's GPU tests name rows per group and shares."""
    import test_gpu_attention_shares as t
    for name, ctx, gamma, prefill, n_q, n_kv, hd, plan in t.CASES:
        assert t._plan(ctx, gamma, prefill, n_q, n_kv, hd) == plan, name
    assert {(p, c[6]) for *c, p in t.CASES} >= {((r, True), h) for r in (32, 48, 64) for h in (64, 128)}
