"""The attention's work layout of one request, read from the workspace, against the rule worked out in Python: tiles of 256 packed rows laid
end to end (a start-up cost and one unit per 64 keys each), cut into equal shares; an item per share and tile it reaches into.  One wave
makes it up to 512 tiles and 64 shares, more go through the general layout: both sides of the lines, behind the selection and from the
plan kernel; and the copy of each share's first item, at the end of the workspace, that the attention kernel starts from (up to 64 shares).
Whole numbers: exact."""
import numpy as np
import pytest
import torch

import a3_synth as synth
from paper_2511_17560_amd import api
from gpu_util import idev

pytestmark = pytest.mark.gpu

COST, TM, TK, MIN_STEPS = 4, 256, 64, 4


def _plan(act, group, shares):
    """(items, first item of each share, (first item, items) of each tile)"""
    rows = len(act) * group
    tiles = -(-rows // TM)
    kv = [int(act[min(((t + 1) * TM - 1) // group, len(act) - 1)]) + 1 for t in range(tiles)]
    steps = [-(-k // TK) for k in kv]
    pre = np.concatenate([[0], np.cumsum([s + COST for s in steps])])
    total = int(pre[-1])
    p = max(1, min(-(-(total - tiles * COST) // MIN_STEPS), shares))
    items, starts = [], []
    for q in range(p):
        beg, end = q * total // p, (q + 1) * total // p
        starts.append(len(items))
        for t in range(tiles):
            at, nxt = int(pre[t]) + COST, int(pre[t + 1])
            if beg < nxt and end > at:
                b, e = max(beg - at, 0), min(end, nxt) - at
                items.append((b * TK, min(kv[t], e * TK), kv[t], t * TM, rows, 0, 0, int(b == 0 and end >= nxt)))
    of_tile = [[i for i, x in enumerate(items) if x[3] == t * TM] for t in range(tiles)]
    return np.array(items), np.array(starts + [len(items)]), np.array([[x[0], len(x)] for x in of_tile])


@pytest.mark.parametrize("group,n,ctx,shares", [(4, 1, 40, 32), (4, 63, 200, 64), (1, 255, 300, 7), (4, 330, 2000, 32), (7, 800, 3000, 64), (7, 800, 3000, 37),
                                                (4, 500, 767, 64), (4, 500, 768, 64), (16, 300, 900, 1),
                                                (4, 1, 40, -1), (4, 63, 200, -1), (1, 255, 300, -1), (1, 257, 300, 1), (4, 330, 2000, -1),
                                                (7, 800, 3000, -1), (4, 64 * 64, 4500, 64), (4, 64 * 64 + 1, 4500, 63), (16, 512 * 16 - 1, 8400, -1),
                                                (16, 512 * 16, 8400, 64), (16, 512 * 16 + 1, 8400, 64), (4, 700, 6000, 65), (4, 500, 767, -1), (4, 500, 768, -1)])
def test_plan_of_one_request(group, n, ctx, shares, tuning):
    if shares > 0:
        tuning("attn_wgs", shares)
    tuning("attn_item_cost", COST)
    wgs = shares if shares > 0 else 256
    w = synth.custom(synth.ModelShape("plan1", "bf16", 64, group, 1, 128, 1e4), [[ctx]], [1], ratio=(n - 1, ctx))
    rng = np.random.default_rng(n)
    act = np.concatenate([np.sort(rng.permutation(ctx)[:n - 1]), [ctx]]).astype(np.int32)
    lay = api.Layout.from_workload(w)
    items, starts, of_tile = _plan(act, group, wgs)
    max_tiles = -(-n * group // TM) + 1
    max_items = max_tiles + wgs
    # 32-bit words of the arrays, in order: the plan, the partial results of cut tiles, the first items
    sizes = [4, 2, 2, 4 * max_tiles, 2 * max_tiles, max_tiles + 1, 8 * max_items, wgs + 1, max_items * TM * 128, max_items * TM * 2, 8 * wgs if wgs <= 64 else 0]

    def check(ws):
        torch.cuda.synchronize()
        words, at, arrays = ws.cpu().numpy().view(np.int32), 0, []
        for size in sizes:
            arrays.append(words[at // 4:at // 4 + size])
            at = (at + 4 * size + 255) // 256 * 256
        assert at <= 4 * len(words)
        counters, a_lo, _, tile_a, tile_b, _, got, wg_start, _, _, first = arrays
        assert counters.tolist() == [len(of_tile), len(items), len(starts) - 1, wgs] and a_lo.tolist() == [0, n]
        assert np.array_equal(got[:8 * len(items)].reshape(-1, 8), items)
        assert np.array_equal(wg_start[:len(starts)], starts)
        for q in range(len(starts) - 1):
            assert starts[q] == starts[q + 1] or wgs > 64 or np.array_equal(first[8 * q:8 * q + 8], items[starts[q]])
        assert np.array_equal(tile_b[:2 * len(of_tile)].reshape(-1, 2), of_tile)
        assert np.array_equal(tile_a[:4 * len(of_tile)].reshape(-1, 4)[:, 1], TM * np.arange(len(of_tile)))

    ws = lay.workspace(n).fill_(0xAB)
    api.a3_attention_plan(lay, idev(act), n, ws)
    check(ws)
    if n > 1:                                                 # the same rows, selected: into the list itself and beside it
        scores = torch.zeros(w.total_tokens, device="cuda")
        scores[torch.from_numpy(act[:-1]).cuda().long()] = torch.rand(n - 1, device="cuda") + 1.0
        for aside in (False, True):
            rows = torch.full((n,), -1, dtype=torch.int32, device="cuda")
            sel = torch.full((n,), -1, dtype=torch.int32, device="cuda") if aside else rows
            ws.fill_(0xAB)
            api.a3_topk_select_plan(lay, scores, idev([0, n - 1]), n - 1, sel, n, rows, ws)
            check(ws)
            assert np.array_equal(rows.cpu().numpy(), act) and np.array_equal(sel.cpu().numpy()[:n - 1], act[:-1])
