"""Scores and votes with keys whose logits are -inf, where blocks of 32 keys consist of nothing else: the first block of a run or tile
of keys, a later one (the first that a wave sees when waves share the last groups of rows of a long question), a whole tile; and question
keys among them, at a question whose own keys have a kernel of their own.

Reference: softmax in float64 on the CPU.  Tolerance 1e-4 of the largest score, as for the other workloads."""
import numpy as np
import pytest
import torch

import a3_synth as synth
from paper_2511_17560_amd import api
from gpu_util import max_abs_rel

pytestmark = pytest.mark.gpu


def _share(w, q, k, hkv, causal):
    """[hkv, T]: weight that each context row receives from the question rows, per KV head."""
    out, group = np.zeros((hkv, w.total_tokens)), q.shape[1] // hkv
    n, nq = int(w.ctx_len[0]), int(w.q_lens[0])
    for g in range(hkv):
        logit = torch.einsum("jhd,td->jht", q[:, g * group:(g + 1) * group], k[:n + (nq if causal else 0), g]) / 128 ** 0.5
        if causal:
            late = torch.arange(nq)[None, :] > torch.arange(nq)[:, None]
            logit[:, :, n:].masked_fill_(late[:, None, :], -torch.inf)
        out[g, :n] = torch.softmax(logit, -1)[:, :, :n].sum((0, 1)).numpy()
    return out


@pytest.mark.parametrize("keys", [(32, 64), (0, 32), (64, 160), (0, 256), (500, 840), (0, 600), (1490, 1510)])
@pytest.mark.parametrize("dtype,hq,hkv,nq", [("bf16", 8, 2, 20), ("bf16", 8, 2, 64), ("bf16", 8, 2, 70), ("bf16", 8, 2, 90), ("bf16", 8, 2, 112), ("bf16", 7, 1, 64),
                                             ("bf16", 4, 2, 270), ("f32", 8, 2, 20)])
def test_blocks_of_keys_with_infinite_logits(dtype, hq, hkv, nq, keys):
    w = synth.custom(synth.ModelShape("inf", dtype, 32, hq, hkv, 128, 1e4), [[1500]], [nq], ratio=(15, 100))
    g = torch.Generator().manual_seed(nq + keys[0])
    q, k = torch.randn(nq, hq, 128, generator=g), torch.randn(w.total_tokens, hkv, 128, generator=g)
    q[:, :, 0], k[:, :, 0] = 2.0, 0.0
    k[keys[0]:keys[1], :, 0] = -torch.inf
    q, k = q.to(api.torch_dtype(dtype)), k.to(api.torch_dtype(dtype))
    lay = api.Layout.from_workload(w)
    votes = torch.zeros((hkv, w.total_tokens), dtype=torch.float32, device="cuda")
    scores, literal, ws = torch.zeros(w.total_tokens, device="cuda"), torch.zeros(w.total_tokens, device="cuda"), lay.workspace(0)
    api.a3_window_votes(lay, q.cuda(), k.cuda(), votes, ws)
    api.a3_question_scores_causal(lay, q.cuda(), k.cuda(), literal, ws)
    api.a3_question_scores(lay, q.cuda(), k.cuda(), scores, ws)
    want, plain = _share(w, q.double(), k.double(), hkv, True), _share(w, q.double(), k.double(), hkv, False).sum(0)
    for got, ref in ((votes, want), (literal[None], want.sum(0)[None]), (scores[None], plain[None])):
        assert max_abs_rel(got.double().cpu().numpy()[:, :1500], ref[:, :1500]) <= 1e-4
