"""Scores of a question whose query rows take more than 4 GiB: all of its tokens but the last have their weight on one context key, the
last one has it on another.  Both are sums of weights of 1 (the next key's is exp(-39)): 1e-5 for the sum of 2^24 of them in fp32."""
import pytest
import torch

import a3_synth as synth
from paper_2511_17560_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hkv", [1, 2])
def test_question_rows_behind_4_gib(hkv):
    hq, n, nq = 16, 64, (1 << 20) + 1
    w = synth.custom(synth.ModelShape("long", "bf16", 64, hq, hkv, 128, 1e4), [[n]], [nq])
    lay = api.Layout.from_workload(w)
    q = torch.zeros((nq, hq, 128), dtype=torch.bfloat16, device="cuda")
    k = torch.zeros((w.total_tokens, hkv, 128), dtype=torch.bfloat16, device="cuda")
    assert q.numel() * 2 > 1 << 32
    q[:-1, :, 0], q[-1, :, 1] = 16.0, 16.0
    k[3, :, 0], k[5, :, 1] = 28.0, 28.0
    scores = torch.zeros(w.total_tokens, device="cuda")
    api.a3_question_scores(lay, q, k, scores, lay.workspace(0))
    got = scores[:n].double().cpu()
    want = torch.zeros(n, dtype=torch.float64)
    want[3], want[5] = hq * (nq - 1), hq
    assert float((got - want).abs().max()) <= 1e-5 * hq * nq and abs(float(got[5]) - hq) <= 1e-5 * hq
