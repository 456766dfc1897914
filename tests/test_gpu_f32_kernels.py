"""The fp32 kernels at the edges of their tiles: head dims 64 and 128, 1 to 16 query heads per KV head (3, 5 and 7 leave
rows of a 16-row tile empty), reductions of 32 elements up to several chunks per wave, contexts around 16, 64 and 128
keys, batches whose 16-row tiles span several requests.

Tolerance 1e-5 of the largest element: fp32 sums of up to 1088 products, each 2^-24 of a term, in another order than the
oracle's; scores 2e-5 element by element, as in test_gpu_parity.py.
"""
import numpy as np
import pytest
import torch

import a3_synth as synth
from oracle import workload as wl
from paper_2511_17560_amd import api
from gpu_util import idev, max_abs_rel, max_elem_rel, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,d,hidden,chunks,q_lens", [
    (1, 1, 64, 32, [[1]], [1]),
    (3, 1, 64, 96, [[15], [16], [17]], [1, 2, 3]),
    (5, 1, 128, 160, [[63, 2]], [17]),
    (16, 1, 64, 64, [[127], [129]], [5, 1]),
    (14, 2, 128, 288, [[40, 25], [1], [64]], [9, 1, 16]),
    (8, 8, 64, 1088, [[300, 212]], [33]),
])
@pytest.mark.parametrize("half", [False, True])
def test_f32_steps(hq, hkv, d, hidden, chunks, q_lens, half):
    shape = synth.ModelShape("f32", "f32", hidden, hq, hkv, d, 10000.0, synth.ROPE_HALF if half else synth.ROPE_INTERLEAVED)
    w = synth.custom(shape, chunks, q_lens, ratio=(40, 100), seed=hq * 1000 + hidden)
    b = wl.build(w)
    res, t = wl.run_oracle(b), b["t"]
    lay = api.Layout.from_workload(w)
    dev = lambda x: to_dev(x, "f32")
    x, wq, wk, wv = dev(t.x_cur), dev(t.wq), dev(t.wk), dev(t.wv)
    act = res["act_idx"]
    n = len(act)
    q = torch.zeros((n, hq, d), device="cuda")
    k = torch.zeros((n, hkv, d), device="cuda")
    v = torch.zeros_like(k)
    api.a3_selected_qkv_proj(lay, x, idev(act), n, wq, wk, wv, q_out=q, k_out=k, v_out=v)
    assert max_abs_rel(to_host(q), res["q_act"]) <= 1e-5
    assert max_abs_rel(to_host(k), res["k_fused"][act]) <= 1e-5 and max_abs_rel(to_host(v), res["v_fused"][act]) <= 1e-5
    scores = torch.zeros(w.total_tokens, device="cuda")
    ws = lay.workspace(n)
    api.a3_question_scores(lay, dev(res["q_question"]), dev(res["k_realigned"]), scores, ws)
    got = scores.cpu().numpy().astype(np.float64)
    for r in range(w.n_req):
        rows = w.ctx_rows(r)
        assert max_elem_rel(got[rows], res["scores"][rows]) <= 2e-5
    assert np.all(np.isneginf(got[w.question_rows()]))
    out = torch.zeros((n, hq, d), device="cuda")
    api.a3_fused_attention(lay, dev(res["q_act"]), idev(act), n, dev(res["k_fused"]), dev(res["v_fused"]), out, ws)
    assert max_abs_rel(to_host(out), res["out"]) <= 1e-5


@pytest.mark.parametrize("hq,hkv,d", [(1, 1, 64), (4, 2, 128), (7, 1, 64), (16, 1, 128)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_f32_attention_keeps_rows_it_may_not_see_out(hq, hkv, d, bad):
    """K and V rows that hold no finite value reach the rows that see them and no other: the rows of a 16-row tile share the
    products, in the block of 16 keys their limit lies in, in later blocks and in blocks of other waves."""
    n_ctx, lens = 300, 20
    shape = synth.ModelShape("f32", "f32", 32, hq, hkv, d, 10000.0)
    w = synth.custom(shape, [[n_ctx], [40]], [lens, 3])
    lay = api.Layout.from_workload(w)
    rng = np.random.default_rng(hq + d)
    k, v = (rng.standard_normal((w.total_tokens, hkv, d)).astype(np.float32) for _ in range(2))
    second = int(w.seg_start[1])
    act = np.array([0, 3, 15, 16, 40, 41, 43, 150, 299, 300, 305, 319, second, second + 7, second + 42], np.int32)
    hidden = np.array([42, 160, 303, second + 8])
    q = rng.standard_normal((len(act), hq, d)).astype(np.float32)
    kb, vb = k.copy(), v.copy()
    kb[hidden], vb[hidden] = bad, bad
    out = torch.zeros((len(act), hq, d), device="cuda")
    api.a3_fused_attention(lay, torch.from_numpy(q).cuda(), idev(act), len(act), torch.from_numpy(kb).cuda(), torch.from_numpy(vb).cuda(),
                           out, lay.workspace(len(act)))
    got = out.double().cpu().numpy()
    for i, t in enumerate(act):
        s = 0 if t < second else second
        if ((hidden >= s) & (hidden <= t)).any():
            assert not np.isfinite(got[i]).any()
            continue
        for h in range(hq):
            g = h // (hq // hkv)
            l = k[s:t + 1, g].astype(np.float64) @ q[i, h].astype(np.float64) / np.sqrt(d)
            p = np.exp(l - l.max())
            want = p @ v[s:t + 1, g].astype(np.float64) / p.sum()
            assert np.abs(got[i, h] - want).max() <= 1e-5 * np.abs(v).max()
