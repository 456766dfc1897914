"""The question keys' share of the literal denominator at the question lengths where its run of the first scoring pass can
go wrong: the edges of a 32-key block, of a 64-key slot, of the 256 rows a KV head has in the one kernel and of the rounds of
256 rows in the other (one or two groups of 64 left over are shared between waves, three leave one wave out), of the 256 keys of a
tile (beyond them a kernel of its own forms the share), questions of different lengths in one batch, and query groups that do not
divide a row block.

Tolerance 1e-4 of the largest vote, as for the other workloads; the question keys are scaled so that leaving their share
out, or counting it twice, moves every vote by far more."""
import numpy as np
import pytest
import torch

import a3_synth as synth
from oracle import evict_oracle as ev
from paper_2511_17560_amd import api
from gpu_util import max_abs_rel, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,q_lens", [
    (1, 1, [1]), (1, 1, [32]), (1, 1, [33]), (1, 1, [64, 65]), (1, 1, [255]), (1, 1, [256, 3, 129]), (1, 1, [257, 5]),
    (8, 2, [31, 64]), (8, 2, [65]), (8, 2, [96, 5]), (8, 2, [200, 129, 64]), (4, 1, [256, 33]), (4, 1, [257]), (7, 1, [36, 1, 33]), (14, 2, [37, 20]), (6, 2, [85, 2]),
    (4, 1, [112]), (14, 2, [64, 57]), (8, 2, [112, 70, 90])])
def test_votes_at_the_question_lengths(hq, hkv, q_lens):
    shape = synth.ModelShape("votes", "bf16", 32, hq, hkv, 128, 1e4)
    ctx = [700, 64, 1333][:len(q_lens)]
    w = synth.custom(shape, [[c] for c in ctx], q_lens, ratio=(15, 100))
    rng = np.random.default_rng(sum(q_lens) + hq)
    k = rng.standard_normal((w.total_tokens, hkv, 128))
    q = rng.standard_normal((w.total_q, hq, 128))
    k[w.question_rows()] = 2.0 * k[w.question_rows()] + 0.9 * q.mean(axis=1)[:, None, :]
    k, q = synth.round_to_storage(k, "bf16"), synth.round_to_storage(q, "bf16")
    kw = dict(seg_start=w.seg_start, ctx_len=w.ctx_len, q_len=w.q_lens)
    scale = 1.0 / np.sqrt(128.0)
    want = ev.kv_head_votes(ev.window_votes(q, k, sm_scale=scale, **kw), hkv)
    lit = ev.question_scores_causal(q, k, sm_scale=scale, **kw)
    lay = api.Layout.from_workload(w)
    votes = torch.zeros((hkv, w.total_tokens), dtype=torch.float32, device="cuda")
    scores = torch.zeros(w.total_tokens, dtype=torch.float32, device="cuda")
    dq, dk, ws = to_dev(q, "bf16"), to_dev(k, "bf16"), lay.workspace(0)
    api.a3_window_votes(lay, dq, dk, votes, ws)
    api.a3_question_scores_causal(lay, dq, dk, scores, ws)
    torch.cuda.synchronize()
    for r in range(w.n_req):
        rows = w.ctx_rows(r)
        assert max_abs_rel(to_host(votes)[:, rows], want[:, rows]) <= 1e-4
        assert max_abs_rel(to_host(scores)[rows], lit[rows]) <= 1e-4
