"""Scores and votes whose sums of powers leave the range that the first scoring pass takes as it comes, at every way their partials are
merged: over the waves, by two threads a row or one in the second pass (up to 64 and 32 tiles of 256 keys), by the kernel before it; in all tiles,
in some, in rows of one chunk of 128 and not of another.  Tolerance as in test_gpu_scores_ranges.py."""
import pytest
import torch

import a3_synth as synth
from paper_2511_17560_amd import api
from gpu_util import max_abs_rel
from test_gpu_scores_infinite import _share

pytestmark = pytest.mark.gpu

KEYS = {"high": lambda t: torch.full(t.shape, 250.0), "low": lambda t: torch.full(t.shape, -250.0), "some tiles": lambda t: -250.0 * (t // 256 % 3 == 0),
        "one key": lambda t: 250.0 * (t == 777)}
ROWS = {"all": lambda j: torch.ones(j.shape), "one": lambda j: 1.0 * (j == 1), "last": lambda j: 1.0 * (j + 1 == len(j))}


@pytest.mark.parametrize("keys", KEYS)
@pytest.mark.parametrize("rows", ROWS)
@pytest.mark.parametrize("hq,hkv,n,nq", [(4, 2, 800, 33), (7, 1, 800, 40), (4, 1, 9000, 64), (4, 1, 7000, 100), (2, 1, 16800, 16), (4, 1, 2000, 160), (2, 1, 900, 150)])
def test_far_logits(hq, hkv, n, nq, rows, keys):
    w = synth.custom(synth.ModelShape("far", "bf16", 32, hq, hkv, 128, 1e4), [[n]], [nq])
    g = torch.Generator().manual_seed(n + nq)
    q, k = torch.randn(nq, hq, 128, generator=g), torch.randn(w.total_tokens, hkv, 128, generator=g)
    q[:, :, 0] = 16.0 * ROWS[rows](torch.arange(nq))[:, None]
    k[:, :, 0] = (KEYS[keys](torch.arange(w.total_tokens)) * 128 ** 0.5 / 16.0)[:, None]
    q, k = q.bfloat16(), k.bfloat16()
    lay = api.Layout.from_workload(w)
    votes = torch.zeros((hkv, w.total_tokens), dtype=torch.float32, device="cuda")
    scores, ws = torch.zeros(w.total_tokens, device="cuda"), lay.workspace(0).fill_(0xAB)
    api.a3_window_votes(lay, q.cuda(), k.cuda(), votes, ws)
    api.a3_question_scores(lay, q.cuda(), k.cuda(), scores, ws)
    want, plain = _share(w, q.double(), k.double(), hkv, True), _share(w, q.double(), k.double(), hkv, False).sum(0)
    assert max_abs_rel(votes.double().cpu().numpy()[:, :n], want[:, :n]) <= 1e-4
    assert max_abs_rel(scores.double().cpu().numpy()[:n], plain[:n]) <= 1e-4
