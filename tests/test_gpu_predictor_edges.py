"""The draft statistics at the edges of their 8192-entry chunks (lanes and whole waves without
entries, the last entry alone in a chunk) on both load paths, and the predictor MLP with 1, 2
and 4 feature rows per workgroup, with the tolerances of the other predictor tests."""
import numpy as np
import pytest
import torch

import paper_2601_11652_amd as W
from oracle.predictor import draft_stats, reject_mlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,ld", [(2, 4), (255, 256), (1025, 1028), (8191, 8192), (8192, 8192), (8193, 8196),
                                  (8193, 8193), (16390, 16390), (24577, 24580)])
def test_draft_stats_chunk_edges(V, ld):
    x = (np.random.default_rng(V).standard_normal((3, V)) * 2.5).astype(np.float32)
    x[1, V - 1] = x[1].max() + 1.0            # the largest in the last entry
    x[2] -= 40.0
    dev = torch.full((3, ld), 1e30, device="cuda")
    dev[:, :V] = torch.from_numpy(x).cuda()
    stats = torch.empty(3, 4, device="cuda")
    W.wisp_draft_stats(dev, V, 0.9, stats)
    got, ref = stats.cpu().numpy().astype(np.float64), draft_stats(x, 0.9)
    np.testing.assert_allclose(got[:, [0, 3]], ref[:, [0, 3]], rtol=1e-5)
    np.testing.assert_allclose(got[:, 1], ref[:, 1], atol=1e-5)
    np.testing.assert_allclose(got[:, 2], ref[:, 2], rtol=1e-5, atol=1e-7)


@pytest.mark.parametrize("n_in,rows", [(1, 256), (8, 511), (8, 513), (5, 1027)])
def test_reject_mlp_rows_per_workgroup(n_in, rows):
    rng = np.random.default_rng(n_in + rows)
    p = {"mean": rng.standard_normal(n_in), "inv_std": rng.uniform(0.5, 2, n_in),
         "w1": rng.standard_normal((512, n_in)) * 0.5, "b1": rng.standard_normal(512) * 0.1,
         "w2": rng.standard_normal((128, 512)) / 16, "b2": rng.standard_normal(128) * 0.1,
         "w3": rng.standard_normal((64, 128)) / 8, "b3": rng.standard_normal(64) * 0.1,
         "w4": rng.standard_normal(64) / 4, "b4": 0.3}
    p = {k: (float(v) if k == "b4" else v.astype(np.float32)) for k, v in p.items()}
    f = rng.standard_normal((rows, n_in)).astype(np.float32)
    mlp = W.RejectMLP({k: (v if k == "b4" else torch.from_numpy(v).cuda()) for k, v in p.items()})
    out = torch.full((rows + 3,), -7.0, device="cuda")
    W.wisp_reject_predict(mlp, torch.from_numpy(f).cuda(), out[:rows])
    got = out.cpu().numpy()
    ref = reject_mlp({k: np.float64(v) if k == "b4" else v.astype(np.float64) for k, v in p.items()}, f)
    assert np.abs(got[:rows] - ref).max() <= 1e-5 and (got[rows:] == -7.0).all()
