"""bf16 scores, votes and realigned keys where a tile takes 32 keys more: contexts around the workgroup counts where that begins and ends (256 and
512 tiles over the KV heads), row counts around one chunk of 128, one and a half and two, last tiles that end before, inside and with those keys, requests shorter than the
longest and without a question token, in place and apart, with ordinary logits and with ones outside the range of plain sums.

Reference: softmax in float64.  Tolerance as in test_gpu_scores_ranges.py; realigned keys bit for bit those of a3_rope_realign, and their scores those of a3_question_scores."""
import pytest
import torch

import a3_synth as synth
from paper_2511_17560_amd import api

pytestmark = pytest.mark.gpu


def _want(w, q, k, hkv, causal):
    out, group, at = torch.zeros((hkv, w.total_tokens), dtype=torch.float64, device="cuda"), q.shape[1] // hkv, 0
    for r in range(w.n_req):
        s, n, nq = int(w.seg_start[r]), int(w.ctx_len[r]), int(w.q_lens[r])
        late = torch.arange(nq, device="cuda")[None, :] > torch.arange(nq, device="cuda")[:, None]
        for h in range(q.shape[1] if nq else 0):
            logit = q[at:at + nq, h].double() @ k[s:s + n + (nq if causal else 0), h // group].double().T.contiguous() / 128 ** 0.5
            if causal:
                logit[:, n:].masked_fill_(late, -torch.inf)
            out[h // group, s:s + n] += torch.softmax(logit, -1)[:, :n].sum(0)
        at += nq
    return out


def _check(hq, hkv, ctx, q_lens, far, half=False):
    shape = synth.ModelShape("tiles", "bf16", 64, hq, hkv, 128, 1e4, synth.ROPE_HALF if half else synth.ROPE_INTERLEAVED)
    w = synth.custom(shape, [[n // 3, n - n // 3] if n > 2 else [n] for n in ctx], q_lens)
    lay = api.Layout.from_workload(w)
    g = torch.Generator(device="cuda").manual_seed(sum(ctx))
    q, cat = (torch.randn(n, h, 128, generator=g, device="cuda") for n, h in ((w.total_q, hq), (w.total_tokens, hkv)))
    if far:                                                    # (coordinates that turn slowest: all but constant over the positions)
        d = 63 if half else 126
        q[:, :, d], cat[:, :, d] = 16.0, (torch.arange(w.total_tokens, device="cuda") // 32 % 3 * 60.0)[:, None]
    q, cat = q.bfloat16(), cat.bfloat16()
    k, votes = cat.clone(), torch.zeros((hkv, w.total_tokens), device="cuda")
    scores, ws = torch.zeros(w.total_tokens, device="cuda"), lay.workspace(0).fill_(0xAB)
    api.a3_rope_realign(lay, cat, k)
    api.a3_window_votes(lay, q, k, votes, ws)
    apart = torch.zeros_like(scores)
    api.a3_question_scores(lay, q, k, apart, ws)
    ctx_rows = torch.cat([torch.arange(int(s), int(s) + int(n), device="cuda") for s, n in zip(w.seg_start, w.ctx_len)])
    want, plain = _want(w, q, k, hkv, True)[:, ctx_rows], _want(w, q, k, hkv, False).sum(0)[ctx_rows]
    assert float((votes[:, ctx_rows] - want).abs().max()) <= 1e-4 * float(want.abs().max())
    for in_place in (False, True):
        stale = cat.clone()
        out = stale if in_place else cat.clone()
        api.a3_realign_scores(lay, q, stale, out, scores, ws)
        assert torch.equal(out, k) and torch.equal(scores[ctx_rows], apart[ctx_rows])
        assert float((scores[ctx_rows] - plain).abs().max()) <= 1e-4 * float(plain.abs().max())


@pytest.mark.parametrize("far", [False, True])
@pytest.mark.parametrize("hq,hkv,n,nq", [(48, 48, 1535, 3), (48, 48, 1408, 3), (48, 48, 1407, 3), (52, 52, 1344, 3), (52, 52, 1152, 3), (51, 51, 1326, 200), (32, 32, 2112, 9),
                                         (64, 32, 2111, 64), (64, 32, 2304, 64), (96, 32, 2305, 85), (64, 16, 4224, 32), (64, 16, 4223, 33), (64, 16, 4320, 64), (64, 16, 4320, 65),
                                         (16, 1, 67600, 16), (32, 8, 16640, 32), (32, 8, 16640, 33), (32, 8, 16639, 64), (64, 16, 4112, 64), (64, 16, 4096, 64), (32, 8, 16640, 48), (32, 8, 16672, 49), (32, 8, 16640, 64), (16, 4, 33300, 64)])
def test_around_the_lines(hq, hkv, n, nq, far):
    _check(hq, hkv, [n], [nq], far)


@pytest.mark.parametrize("far", [False, True])
@pytest.mark.parametrize("hkv,ctx,q_lens", [(16, [1080, 300, 31, 860], [7, 0, 1, 3]), (16, [1085, 256, 287, 288], [64, 1, 33, 2]), (16, [1100, 1, 257, 577], [50, 64, 5, 64]),
                                            (4, [4225, 289, 4096, 1], [64, 33, 0, 40]), (4, [300, 4319, 288, 4033], [3, 1, 7, 2])])
def test_ragged_batches(hkv, ctx, q_lens, far):
    _check(4 * hkv, hkv, ctx, q_lens, far, half=True)
