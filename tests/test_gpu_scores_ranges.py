"""The bf16 scoring passes where their paths change: rows per KV head around one, two and four chunks of 128 and around what the second pass
merges itself (256 rows, 512), tiles of 256 keys around 32 and 64, question keys around one, two, four and eight waves of 32; and logits
so large, so small or so far apart that plain fp32 sums of their powers leave the range that is taken as it comes.

Reference: softmax in float64 on the CPU.  Tolerance 1e-4 of the largest score, as for the other workloads: a logit of 250 (360 as a power of
two) is rounded to 2^-16 in the sum of its products and again as an exponent, in both passes: 4 x 2^-16 x ln 2 = 4e-5."""
import numpy as np
import pytest
import torch

import a3_synth as synth
from paper_2511_17560_amd import api
from gpu_util import max_abs_rel
from test_gpu_scores_infinite import _share

pytestmark = pytest.mark.gpu


def _check(hq, hkv, n, nq, shift=None, seed=0):
    w = synth.custom(synth.ModelShape("ranges", "bf16", 32, hq, hkv, 128, 1e4), [[n]], [nq], ratio=(15, 100))
    g = torch.Generator().manual_seed(n + nq + seed)
    q, k = torch.randn(nq, hq, 128, generator=g), torch.randn(w.total_tokens, hkv, 128, generator=g)
    if shift is not None:                                     # a logit of shift[t] at every key, beside the others
        q[:, :, 0], k[:, :, 0] = 16.0, (shift(torch.arange(w.total_tokens)) * 128 ** 0.5 / 16.0)[:, None]
    q, k = q.bfloat16(), k.bfloat16()
    lay = api.Layout.from_workload(w)
    votes = torch.zeros((hkv, w.total_tokens), dtype=torch.float32, device="cuda")
    scores, ws = torch.zeros(w.total_tokens, device="cuda"), lay.workspace(0).fill_(0xAB)
    api.a3_window_votes(lay, q.cuda(), k.cuda(), votes, ws)
    api.a3_question_scores(lay, q.cuda(), k.cuda(), scores, ws)
    want, plain = _share(w, q.double(), k.double(), hkv, True), _share(w, q.double(), k.double(), hkv, False).sum(0)
    assert max_abs_rel(votes.double().cpu().numpy()[:, :n], want[:, :n]) <= 1e-4
    assert max_abs_rel(scores.double().cpu().numpy()[:n], plain[:n]) <= 1e-4


@pytest.mark.parametrize("hq,nq", [(1, 1), (1, 15), (1, 32), (1, 33), (2, 64), (1, 129), (4, 64), (1, 256), (1, 257), (2, 129), (4, 128), (3, 171), (4, 129), (5, 129)])
def test_rows_and_question_keys(hq, nq):
    _check(hq, 1, 700, nq)


@pytest.mark.parametrize("n", [1, 31, 32, 255, 256, 257, 32 * 256, 32 * 256 + 1, 64 * 256, 64 * 256 + 1])
@pytest.mark.parametrize("hq,nq", [(2, 16), (4, 65)])
def test_keys_around_tiles(n, hq, nq):
    _check(hq, 1, n, nq)


@pytest.mark.parametrize("hq,hkv,nq", [(8, 2, 20), (4, 1, 70), (4, 1, 130)])
@pytest.mark.parametrize("shift", [
    lambda t: torch.full(t.shape, 250.0), lambda t: torch.full(t.shape, -250.0), lambda t: 250.0 - 0.25 * (t % 2000), lambda t: -250.0 + 250.0 * (t // 32 % 2),
    lambda t: 90.0 * (t == 777) - 60.0, lambda t: -250.0 * (t // 256 % 3)], ids=["high", "low", "falling", "by waves", "one", "by tiles"])
def test_logits_outside_the_plain_range(hq, hkv, nq, shift):
    _check(hq, hkv, 1500, nq, shift)
