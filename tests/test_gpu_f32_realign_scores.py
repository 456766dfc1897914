"""fp32: position recovery inside the first scoring pass (its keys against a3_rope_realign bit for bit, also in place), the row statistics
merged by the second pass or by a kernel in front of it (32 and 33 tiles of 64 keys, 1024 and 1026 rows per KV head), and the row list made
by the kernel that selects.  Scores against a float64 softmax of the realigned keys, 2e-5 element by element as in test_gpu_parity.py."""
import numpy as np
import pytest
import torch

import a3_synth as synth
from paper_2511_17560_amd import api
from gpu_util import idev, max_elem_rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,d,half,chunks,q_lens", [
    (4, 2, 64, False, [[63, 2]], [5]), (4, 2, 64, True, [[64], [1, 16]], [16, 1]), (7, 1, 128, False, [[65], [130, 7]], [3, 9]),
    (4, 2, 128, True, [[31, 33, 1]], [17]), (1, 1, 64, False, [[1500, 548]], [3]), (1, 1, 64, True, [[1500, 549]], [3]),
    (2, 1, 64, False, [[100]], [512]), (2, 1, 64, False, [[100]], [513])])
def test_f32_realign_scores(hq, hkv, d, half, chunks, q_lens):
    shape = synth.ModelShape("f32r", "f32", 32, hq, hkv, d, 1e4, synth.ROPE_HALF if half else synth.ROPE_INTERLEAVED)
    w = synth.custom(shape, chunks, q_lens, ratio=(20, 100))
    lay = api.Layout.from_workload(w)
    g = torch.Generator().manual_seed(d + w.total_tokens)
    q, k = torch.randn(w.total_q, hq, d, generator=g), torch.randn(w.total_tokens, hkv, d, generator=g)
    dq, ws = q.cuda(), lay.workspace(0)
    apart = k.cuda()
    api.a3_rope_realign(lay, k.cuda(), apart)
    want = np.full(w.total_tokens, -np.inf)
    at = 0
    for r in range(w.n_req):
        rows, nq = w.ctx_rows(r), int(w.q_lens[r])
        kr = apart.double().cpu()[rows]
        p = torch.softmax(torch.einsum("jhd,tgd->jhgt", q[at:at + nq].double(), kr) / d ** 0.5, -1)
        want[rows] = sum(p[:, h, h // (hq // hkv)].sum(0) for h in range(hq)).numpy()
        at += nq
    for in_place in (False, True):
        cat = k.cuda()
        out = cat if in_place else k.cuda()
        scores = torch.zeros(w.total_tokens, device="cuda")
        api.a3_realign_scores(lay, dq, cat, out, scores, ws)
        assert torch.equal(out, apart)
        got = scores.double().cpu().numpy()
        assert np.array_equal(np.isneginf(got), np.isneginf(want))
        for r in range(w.n_req):
            assert max_elem_rel(got[w.ctx_rows(r)], want[w.ctx_rows(r)]) <= 2e-5
    if w.n_req == 1:
        n_sel, n_ctx = int(w.sel_start[-1]), int(w.ctx_len[0])
        keep = np.sort(np.argsort(-scores.cpu().numpy()[:n_ctx], kind="stable")[:n_sel])
        rows = np.concatenate([keep, np.arange(n_ctx, w.total_tokens)])
        for aside in (False, True):
            act = torch.full((len(rows) + 1,), -7, dtype=torch.int32, device="cuda")
            sel = torch.full((n_sel,), -7, dtype=torch.int32, device="cuda") if aside else act
            api.a3_topk_select_plan(lay, scores, idev(w.sel_start), n_sel, sel, len(rows), act, ws)
            assert np.array_equal(act.cpu().numpy(), np.concatenate([rows, [-7]])) and np.array_equal(sel.cpu().numpy()[:n_sel], keep)
