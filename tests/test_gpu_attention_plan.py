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


def test_more_items_than_the_table_holds(tuning):
    """One workgroup per KV head and 21 and 24 row tiles: a workgroup looks its first 16 items up at its start and every later
    one in the middle of its stream of loads."""
    for chunks, q_lens, ratio in (([[1400, 1170]], [33], (50, 100)), ([[600], [37, 500], [9]], [200, 70, 31], (100, 100))):
        w, act, q, k, v = _inputs(8, 2, chunks, q_lens, ratio, 11)
        assert len(act) * 4 > 20 * 256
        lay = api.Layout.from_workload(w)
        dq, dk, dv, ws = q.cuda(), k.cuda(), v.cuda(), lay.workspace(len(act))
        outs = []
        for wgs in (-1, 1):
            tuning("attn_wgs", wgs)
            out = torch.zeros_like(dq)
            api.a3_fused_attention(lay, dq, idev(act), len(act), dk, dv, out, lay.workspace(len(act)))
            _check(w, act, q, k, v, out, list(range(0, len(act), 29)) + [len(act) - 1])
            outs.append(out.double().cpu())
        # with one share nothing is cut and merged: apart only by the rounding of the weights and of the output
        assert float((outs[0] - outs[1]).abs().max()) <= 2.0 ** -7 * float(v.double().abs().max())


def test_plan_too_large_for_lds_many_requests():
    """The plan's small arrays are looked up in the workspace when they do not fit 6144 integers of LDS: 1100 requests."""
    rng = np.random.default_rng(3)
    lens = [[int(n)] for n in rng.integers(1, 9, 1100)]
    w, act, q, k, v = _inputs(4, 2, lens, rng.integers(1, 4, 1100).tolist(), (50, 100), 12)
    assert 3 * (w.n_req + 1) + 3 * w.n_req > 6144
    lay = api.Layout.from_workload(w)
    out = torch.zeros((len(act), 4, 128), dtype=torch.bfloat16, device="cuda")
    api.a3_fused_attention(lay, q.cuda(), idev(act), len(act), k.cuda(), v.cuda(), out, lay.workspace(len(act)))
    _check(w, act, q, k, v, out, range(0, len(act), 3))


def test_plan_too_large_for_lds_long_request():
    """... and all 33008 rows of one request at 16 heads per KV head, by the plan kernel and by the selecting kernel."""
    w, act, q, k, v = _inputs(16, 1, [[33000]], [8], (100, 100), 13)
    n = len(act)
    assert n == w.total_tokens and 3 * (n * 16 // 256) > 6144
    lay = api.Layout.from_workload(w)
    dq, dk, dv = q.cuda(), k.cuda(), v.cuda()
    one, two = torch.zeros_like(dq), torch.zeros_like(dq)
    ws = lay.workspace(n)
    api.a3_fused_attention(lay, dq, idev(act), n, dk, dv, one, ws)
    _check(w, act, q, k, v, one, [0, 1, 15, 16, 17, 63, 64, 5000, 20001, n - 9, n - 1])
    ws.fill_(0xAB)
    scores = torch.rand(n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    rows = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    api.a3_topk_select_plan(lay, scores, idev(w.sel_start), w.total_k, rows, n, rows, ws)
    api.a3_fused_attention_planned(lay, dq, rows, n, dk, dv, two, ws)
    assert np.array_equal(rows.cpu().numpy(), act) and torch.equal(one, two)


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
