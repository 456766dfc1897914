"""The attention where its plan is large, and what its softmax divides by.

References in float64 on the CPU.  Tolerance of an output as in test_gpu_parity.py: |a - b| <= 2^-8 |b| + 2^-8 max |V|, the stored
rounding of the output and the bf16 rounding of the weights in front of the product, each 2^-9, with a factor of two in hand.
"""
import numpy as np
import pytest
import torch

import a3_synth as synth
from paper_2511_17560_amd import api
from gpu_util import idev

pytestmark = pytest.mark.gpu


def _inputs(hq, hkv, chunks, q_lens, ratio, seed):
    w = synth.custom(synth.ModelShape("plan", "bf16", 64, hq, hkv, 128, 10000.0), chunks, q_lens, ratio=ratio)
    g = torch.Generator().manual_seed(seed)
    act = []
    for r in range(w.n_req):
        rows = w.ctx_rows(r)
        k_r = int(w.sel_start[r + 1] - w.sel_start[r])
        picked = torch.randperm(len(rows), generator=g)[:k_r].sort().values.numpy() + rows[0] if len(rows) else np.zeros(0, int)
        act += [picked, np.arange(w.seg_start[r] + w.ctx_len[r], w.seg_start[r + 1])]
    act = np.concatenate(act).astype(np.int32)
    draw = lambda *s: torch.randn(*s, generator=g).bfloat16()
    return w, act, draw(len(act), hq, 128), draw(w.total_tokens, hkv, 128), draw(w.total_tokens, hkv, 128)


def _check(w, act, q, k, v, out, pick):
    got, kd, vd = out.double().cpu(), k.double(), v.double()
    group = q.shape[1] // k.shape[1]
    vmax = float(vd.abs().max())
    req = w.token_requests()
    for i in pick:
        t, s = int(act[i]), int(w.seg_start[req[act[i]]])
        for h in range(q.shape[1]):
            p = torch.softmax(kd[s:t + 1, h // group] @ q[i, h].double() / 128 ** 0.5, 0)
            want = p @ vd[s:t + 1, h // group]
            assert bool(((got[i, h] - want).abs() <= 2.0 ** -8 * want.abs() + 2.0 ** -8 * vmax).all()), (i, t, h)


@pytest.mark.parametrize("wgs", [-1, 1, 40])
def test_weights_sum_to_one(wgs, tuning):
    """Numerator and denominator carry the same weights, each rounded to bf16 once and summed in fp32: where every value is 1
    every output is exactly 1, whole tiles and merged ones.  (Divided by the sum of the unrounded weights, rows of few keys are
    off by up to 2^-9 and most of them round to another number.)"""
    tuning("attn_wgs", wgs)
    w, act, q, k, v = _inputs(8, 2, [[900, 100], [40]], [17, 5], (30, 100), 14)
    lay = api.Layout.from_workload(w)
    out = torch.zeros((len(act), 8, 128), dtype=torch.bfloat16, device="cuda")
    api.a3_fused_attention(lay, (2 * q).cuda(), idev(act), len(act), k.cuda(), torch.ones_like(v).cuda(), out, lay.workspace(len(act)))
    assert bool((out == 1).all())
