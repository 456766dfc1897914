"""Window votes and the literal denominator where the question keys' share is merged by the second scoring pass (up to 32
runs of keys) and where the small kernel in front of it does that (more): one KV head, so a run is 256 keys.

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


@pytest.mark.parametrize("ctx", [[1], [255], [8191], [8192], [8193], [8192, 1, 300], [8193, 257]])
@pytest.mark.parametrize("nq", [1, 17])
def test_votes_at_the_run_counts(ctx, nq):
    shape = synth.ModelShape("votes", "bf16", 32, 4, 1, 128, 1e4)
    w = synth.custom(shape, [[c] for c in ctx], [nq] * len(ctx), ratio=(15, 100))
    rng = np.random.default_rng(sum(ctx) + nq)
    k = rng.standard_normal((w.total_tokens, 1, 128))
    q = rng.standard_normal((w.total_q, 4, 128))
    k[w.question_rows()] = 2.0 * k[w.question_rows()] + 0.9 * q.mean(axis=1)[:, None, :]
    k, q = synth.round_to_storage(k, "bf16"), synth.round_to_storage(q, "bf16")
    kw = dict(seg_start=w.seg_start, ctx_len=w.ctx_len, q_len=w.q_lens)
    scale = 1.0 / np.sqrt(128.0)
    want = ev.kv_head_votes(ev.window_votes(q, k, sm_scale=scale, **kw), 1)
    lit = ev.question_scores_causal(q, k, sm_scale=scale, **kw)
    lay = api.Layout.from_workload(w)
    votes = torch.zeros((1, w.total_tokens), dtype=torch.float32, device="cuda")
    scores = torch.zeros(w.total_tokens, dtype=torch.float32, device="cuda")
    dq, dk, ws = to_dev(q, "bf16"), to_dev(k, "bf16"), lay.workspace(0)
    api.a3_window_votes(lay, dq, dk, votes, ws)
    api.a3_question_scores_causal(lay, dq, dk, scores, ws)
    torch.cuda.synchronize()
    for r in range(w.n_req):
        rows = w.ctx_rows(r)
        assert max_abs_rel(to_host(votes)[:, rows], want[:, rows]) <= 1e-4
        assert max_abs_rel(to_host(scores)[rows], lit[rows]) <= 1e-4
