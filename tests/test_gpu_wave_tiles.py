"""The one-wave-per-SIMD projection tiles (65 rows and more) at the edges of their row tiles,
column tiles and K ranges, against the oracle.

Shapes: K of 3 chunks of 32 columns (fewer than the LDS stages), 5, 7 and 10 (odd and even
counts), and 33 with K split (odd ranges, a last range of 3); 448 and 1056 output columns
leave the last 128- and 256-column tiles partly filled.  Rows: the last of one tile height
and the first of the next (128 / 192 / 256 / 384 rows), and several row tiles of either
height beyond.  Gate/up runs split (SwiGLU kernel) and whole (epilogue).  Logits within the
stated bf16 bound, 2e-2 max-abs; written K/V, untouched slots and decisions as in the other
parity tests.
"""
import numpy as np
import pytest

import wisp_inputs as wi
from oracle import fixtures as fx
from gpu_harness import Workload, check_decisions_on_gpu_logits, check_written, gpu_model, log, run_gpu

pytestmark = pytest.mark.gpu

K3 = wi.ModelShape("wave-k3", 2, 96, 3, 1, 64, 160, 1056, "bf16", 10000.0)
K5 = wi.ModelShape("wave-k5", 2, 160, 5, 1, 64, 224, 1056, "bf16", 10000.0)
K33 = wi.ModelShape("wave-k33", 1, 1056, 4, 2, 64, 352, 2080, "bf16", 10000.0)
WIDE = wi.ModelShape("wave-wide", 1, 160, 2, 1, 64, 28672, 1056, "bf16", 10000.0)   # gate/up fills a round

CASES = [(K3, 65), (K3, 257), (K3, 577), (K5, 96), (K5, 128), (K5, 129), (K5, 192), (K5, 193), (K5, 256), (K5, 257),
         (K5, 384), (K5, 385), (K5, 577), (K5, 1025), (K33, 70), (K33, 161), (K33, 250), (K33, 300), (K33, 449),
         (WIDE, 67), (WIDE, 150), (WIDE, 225), (WIDE, 400)]


@pytest.mark.parametrize("shape,rows", CASES, ids=[f"{s.name}-{m}" for s, m in CASES])
def test_wave_tiles_match_the_oracle(shape, rows):
    gamma = [16] * (rows // 17)
    if rows % 17:
        gamma.append(rows % 17 - 1)
    r = np.random.default_rng(rows)
    ctx = r.integers(0, 40, size=len(gamma)).astype(np.int32)
    mix = wi.custom_mix(shape, ctx, np.array(gamma, np.int32), kv_source="prefill", name=f"wave-{rows}", t_draft=1.0,
                        sigma=0.5)
    assert mix.M == rows
    wl = Workload(mix, fx.host_model(shape))
    acc, out, logits, pools = run_gpu(gpu_model(shape), wl)
    d = np.abs(logits - wl.logits_ref)
    log(f"{shape.name}: {rows} rows, logits max-abs error {d.max():.3e}")
    assert d.max() <= 2e-2
    check_written(pools, wl.pools_ref, wl.pools0, wl.pt, mix.ctx_len, mix.rows, shape.head_dim, True,
                  pools_ref32=wl.pools_ref32)
    check_decisions_on_gpu_logits(acc, out, logits, wl.tokens, wl.q, mix.gamma, 1.0, wl.seed, req_id=mix.req_id)
