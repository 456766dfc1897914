"""The attention kernel's stream of items, and the exponent reference of its softmax.  References and tolerance as in
test_gpu_attention_plan.py."""
import numpy as np
import pytest
import torch

from paper_2511_17560_amd import api
from gpu_util import idev
from test_gpu_attention_plan import _check, _inputs

pytestmark = pytest.mark.gpu


def _attend(w, act, q, k, v):
    lay = api.Layout.from_workload(w)
    out = torch.zeros((len(act),) + tuple(q.shape[1:]), dtype=torch.bfloat16, device="cuda")
    api.a3_fused_attention(lay, q.cuda(), idev(act), len(act), k.cuda(), v.cuda(), out, lay.workspace(len(act)))
    return out


@pytest.mark.parametrize("hq,hkv", [(8, 2), (2, 2), (14, 2)])
def test_many_short_items_in_one_workgroup(hq, hkv, tuning):
    """One workgroup per KV head over 90 requests of 1 to 150 keys: more items than the ring of looked-up ones holds, most of
    one step, so that the stream of loads runs three items ahead, and requests that end anywhere in a tile of keys."""
    rng = np.random.default_rng(5)
    lens = [[int(n)] for n in rng.integers(1, 150, 90)]
    w, act, q, k, v = _inputs(hq, hkv, lens, rng.integers(1, 9, 90).tolist(), (40, 100), 15)
    tuning("attn_wgs", 1)
    _check(w, act, q, k, v, _attend(w, act, q, k, v), range(0, len(act), 7))


def test_items_of_a_few_tiles_in_one_workgroup(tuning):
    """Items of two to seven tiles of keys, one behind the other: V of the tile behind a change of item is requested two tiles
    before it and has no other wait than the one in front of the next item's rows."""
    rng = np.random.default_rng(6)
    lens = [[int(n)] for n in rng.integers(66, 420, 40)]
    w, act, q, k, v = _inputs(8, 2, lens, rng.integers(1, 9, 40).tolist(), (30, 100), 18)
    v *= torch.exp2((torch.arange(w.total_tokens) // 64 % 5).float())[:, None, None].bfloat16()      # another size from tile to tile
    tuning("attn_wgs", 1)
    _check(w, act, q, k, v, _attend(w, act, q, k, v), range(0, len(act), 5))


def test_growing_logits_move_the_reference():
    """The exponent reference only moves when a weight reaches 2 against it: logits that grow by a few powers of two from tile to
    tile of keys, that jump far at one key, that fall steeply, and single large ones."""
    w, act, q, k, v = _inputs(8, 2, [[3000]], [20], (10, 100), 16)
    t = torch.arange(w.total_tokens)
    for logit in (t / 64 * 0.4, 60.0 * (t >= 1500), 80.0 - t / 64 * 3.0, 50.0 * (t % 700 == 350)):
        kk, qq = k.clone(), q.clone()
        qq[:, :, 0] = 8.0
        kk[:, :, 0] = (logit * 128 ** 0.5 / 8.0).bfloat16()[:, None]
        _check(w, act, qq, kk, v, _attend(w, act, qq, kk, v), list(range(0, len(act), 17)) + [len(act) - 1])


@pytest.mark.parametrize("wgs", [-1, 1, 7])
@pytest.mark.parametrize("logit", [-1.0, -100.0, "up"])
@pytest.mark.parametrize("pattern", ["first 64", "first 100", "first 128", "every other tile", "three tiles of four"])
def test_keys_with_infinite_logits_before_small_ones(pattern, logit, wgs, tuning):
    """A row whose first tiles of keys, of the request or of a share of it, have weight 0 altogether (logits of -inf): the exponent
    reference is that of the first finite logit, also of one that is small or far below zero."""
    tuning("attn_wgs", wgs)
    w, act, q, k, v = _inputs(8, 2, [[1500]], [20], (30, 100), 19)
    t = torch.arange(w.total_tokens)
    none = {"first 64": t < 64, "first 100": t < 100, "first 128": t < 128, "every other tile": t // 64 % 2 == 0,
            "three tiles of four": t // 64 % 4 < 3}[pattern]
    want = torch.where(t % 400 < 300, -1.0, 3.0) if logit == "up" else torch.full(t.shape, logit)
    qq, kk = 0.1 * q, k.clone()
    qq[:, :, 0] = 8.0
    kk[:, :, 0] = torch.where(none, -torch.inf, want * 128 ** 0.5 / 8.0).bfloat16()[:, None]
    seen = [i for i in range(len(act)) if bool((~none[:int(act[i]) + 1]).any())]
    _check(w, act, qq, kk, v, _attend(w, act, qq, kk, v), seen[::23] + seen[-1:])


def test_rows_behind_the_last_visible_key_stay_out():
    """Keys and values behind the last one that a tile of rows sees are not multiplied: not finite there, finite outputs."""
    w, _, _, k, v = _inputs(8, 2, [[700]], [3], (0, 100), 17)
    rows = np.array([130, 131, 333], dtype=np.int32)
    q = torch.randn(3, 8, 128, generator=torch.Generator().manual_seed(1)).bfloat16()
    kk, vv = k.clone(), v.clone()
    kk[334:], vv[334:] = float("nan"), float("inf")
    _check(w, rows, q, k[:334], v[:334], _attend(w, rows, q, kk, vv), range(3))
