"""The acceptance at the edges of its vocabulary chunks (8192 entries per workgroup of the
pass over the logits, 2048 of the race) and of its load widths, against the oracle: one
chunk and one more entry, vocabularies that are no multiple of 4, logits that are only
4-byte aligned, 17 rows (gamma 16), a chunk whose logits are all -inf (a masked vocabulary
tail) and greedy decoding with its argmax in the last entry.  Bit-exact except where the
oracle flags a near-tie."""
import numpy as np
import pytest
import torch

import oracle
import paper_2601_11652_amd as W
from gpu_harness import compare_decisions
from test_gpu_sampler import _batch

pytestmark = pytest.mark.gpu


def _accept(gamma, logits, toks, q, T, seed, shift):
    B, (M, V) = gamma.shape[0], logits.shape
    desc = W.BatchDesc(np.zeros(B, np.int32), gamma, None, T)
    ws = W.workspace(W.wisp_accept_workspace_size(desc, V))
    buf = torch.empty(M * V + 4, device="cuda")
    dl = buf[shift:shift + M * V].view(M, V)
    dl.copy_(torch.from_numpy(logits))
    acc = torch.full((B,), -7, dtype=torch.int32, device="cuda")
    out = torch.full((M,), -7, dtype=torch.int32, device="cuda")
    W.wisp_accept(desc, V, dl, torch.from_numpy(toks).cuda(), torch.from_numpy(q).cuda(), seed, acc, out, ws)
    W.wisp_check(ws)
    return acc.cpu().numpy(), out.cpu().numpy()


@pytest.mark.parametrize("T", [1.0, 0.7, 0.0])
@pytest.mark.parametrize("V,shift", [(2047, 0), (2048, 0), (2049, 0), (8192, 1), (8193, 0), (16388, 0), (65540, 0)])
def test_chunk_edges(V, shift, T):
    gamma, logits, toks, q = _batch(12, V, 16, seed=V + 3, gmin=12)
    if V > 16384:
        logits[:, 8192:16384] = -np.inf          # a whole chunk masked
        q[:, 8192:16384] = 0.0
    if T == 0.0:
        logits[:, V - 1] = logits[:, :V - 1].max(axis=1) + 1.0
        toks[1::2] = V - 1
    toks = np.where((toks >= 8192) & (toks < 16384) & (V > 16384), 5, toks).astype(np.int32)
    acc, out = _accept(gamma, logits, toks, q, T, 0xC0FFEE + V, shift)
    ref = oracle.accept(logits, toks, q, gamma, T, 0xC0FFEE + V)
    _, mism, unflagged = compare_decisions(acc, out, ref, gamma, toks, 1e-3, 1e-5)
    assert not unflagged and mism == 0
