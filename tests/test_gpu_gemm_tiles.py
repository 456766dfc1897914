"""The matrix-core GEMM of the projection and of H(.) in every tile it has, at row counts around the tile edges, reduction
lengths of one slab up to more than the LDS ring holds, and with the reduction split; against float64 products on the CPU.

Tolerance: one bf16 rounding of the stored value, 2^-9 of it, plus the fp32 accumulation of K products of bf16 values, which
for the sums here stays under 2^-16 of the largest element; checked as |a - b| <= 2^-8 |b| + 2^-12 max |b|.  H(.) rounds five
times in a row (two residual rows, a norm, the activation, a norm): 2e-2 of the largest element, as in test_gpu_stack.py.
"""
import numpy as np
import pytest
import torch

import a3_synth as synth
from paper_2511_17560_amd import api
from gpu_util import idev

pytestmark = pytest.mark.gpu


def _layout(hidden, hq, hkv, ctx, half=False):
    shape = synth.ModelShape("tile", "bf16", hidden, hq, hkv, 128, 10000.0, synth.ROPE_HALF if half else synth.ROPE_INTERLEAVED)
    return api.Layout.from_workload(synth.custom(shape, [[ctx - 1]], [1]))


@pytest.mark.parametrize("tile", [2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("n,hidden,hq,hkv", [(1, 64, 1, 1), (63, 128, 3, 1), (65, 192, 2, 1), (257, 448, 7, 1), (300, 1088, 4, 2)])
def test_projection_in_every_tile(tile, n, hidden, hq, hkv, tuning):
    """Gathered rows in any order, odd head counts (a two-head tile with one head), K alone, both rotary layouts; rows that
    are not asked for stay as they were."""
    tuning("proj_ntw", tile)
    T = 400
    g = torch.Generator().manual_seed(n)
    x = torch.randn(T, hidden, generator=g).bfloat16()
    w = (torch.randn((hq + 2 * hkv) * 128, hidden, generator=g) * 0.05).bfloat16()
    rows = torch.randperm(T, generator=g)[:n].int()
    for half in (False, True):
        lay = _layout(hidden, hq, hkv, T, half)
        y = (x.double()[rows.long()] @ w.double().T).view(n, hq + 2 * hkv, 128)
        th = 10000.0 ** (-torch.arange(64, dtype=torch.float64) / 64)
        c, s = torch.cos(rows[:, None] * th)[:, None], torch.sin(rows[:, None] * th)[:, None]
        a, b = (y[..., :64], y[..., 64:]) if half else (y[..., 0::2], y[..., 1::2])
        u, v = a * c - b * s, a * s + b * c
        turned = torch.cat([u, v], -1) if half else torch.stack([u, v], -1).flatten(-2)
        want = torch.cat([turned[:, :hq + hkv], y[:, hq + hkv:]], 1)
        wd = [t.contiguous().cuda() for t in w.split([hq * 128, hkv * 128, hkv * 128])]
        q = torch.zeros((n, hq, 128), dtype=torch.bfloat16, device="cuda")
        k = torch.full((T, hkv, 128), 7.0, dtype=torch.bfloat16, device="cuda")
        vv = torch.full((T, hkv, 128), 7.0, dtype=torch.bfloat16, device="cuda")
        api.a3_selected_qkv_proj_scatter(lay, x.cuda(), idev(rows), n, *wd, q_out=q, k_fused=k, v_fused=vv)
        k_only = torch.zeros((n, hkv, 128), dtype=torch.bfloat16, device="cuda")
        api.a3_selected_qkv_proj(lay, x.cuda(), idev(rows), n, None, wd[1], None, k_out=k_only)
        at = rows.long().cuda()
        for got, ref in ((q, want[:, :hq]), (k[at], want[:, hq:hq + hkv]), (vv[at], want[:, hq + hkv:]), (k_only, want[:, hq:hq + hkv])):
            d = (got.double().cpu() - ref).abs()
            assert bool((d <= 2.0 ** -8 * ref.abs() + 2.0 ** -12 * ref.abs().max()).all()), float(d.max())
        rest = np.setdiff1d(np.arange(T), rows.numpy())
        assert bool((k[rest] == 7).all()) and bool((vv[rest] == 7).all())


@pytest.mark.parametrize("tile", [None, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("n,hidden,ffn,heads", [(1, 128, 64, 1), (65, 128, 832, 2), (129, 256, 4160, 3), (257, 384, 1024, 5),
                                                (1, 1024, 4096, 16), (66, 256, 4160, 16), (33, 384, 1984, 15)])
def test_block_tail_in_every_tile_and_split(tile, n, hidden, ffn, heads, tuning):
    """With no tile asked for, the reductions of 1920 elements and more are split eight ways here: both residual products' in the
    last three shapes, the second's in 129 x 256 x 4160 (65 slabs and 30: also into unequal shares); where the workspace only
    holds the intermediate rows, one workgroup forms all shares.  The result is the same bits in any workspace that is accepted.
    With a tile asked for nothing is split."""
    if tile is not None:
        tuning("gemm_tb", tile)
    T, eps = 300, 1e-5
    lay = _layout(hidden, heads, 1, T)
    g = torch.Generator().manual_seed(n + ffn)
    mk = lambda *s, std=1.0: (torch.randn(*s, generator=g) * std).bfloat16()
    o, r0 = mk(n, heads, 128), mk(T, hidden)
    wo, wg, wu, wd = mk(hidden, heads * 128, std=0.05), mk(ffn, hidden, std=0.05), mk(ffn, hidden, std=0.05), mk(hidden, ffn, std=0.02)
    g1, g2 = 1 + mk(hidden, std=0.1), 1 + mk(hidden, std=0.1)
    rows = torch.randperm(T, generator=g)[:n].sort().values.int()
    at = rows.long()
    norm = lambda t, w: t / torch.sqrt((t * t).mean(-1, keepdim=True) + eps) * w.double()
    r1 = r0.double()[at] + o.double().view(n, -1) @ wo.double().T
    n1 = norm(r1, g1)
    r2 = r1 + (torch.nn.functional.silu(n1 @ wg.double().T) * (n1 @ wu.double().T)) @ wd.double().T
    want = norm(r2, g2)
    dev = [t.cuda() for t in (wo, g1, wg, wu, wd, g2)]
    small = ((n * hidden * 2 + 255) // 256 + (n * ffn * 2 + 255) // 256) * 256 + 256
    need = api.a3_block_tail_ws_bytes(lay, ffn, n)
    assert (need > small) == (max(ffn, heads * 128) >= 1920)
    results = []
    for size in (need, small, (need + small) // 2, need + (1 << 20)):
        resid, nxt = r0.cuda(), torch.full((T, hidden), 5.0, dtype=torch.bfloat16, device="cuda")
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        api.a3_block_tail(lay, o.cuda(), idev(rows), n, *dev, eps, resid, nxt, ws)
        got_r, got_n = resid.double().cpu(), nxt.double().cpu()
        results.append((got_r, got_n))
        assert torch.equal(got_r, results[0][0]) and torch.equal(got_n, results[0][1])
        assert float((got_r[at] - r2).abs().max() / r2.abs().max()) <= 2e-2
        assert float((got_n[at] - want).abs().max() / want.abs().max()) <= 2e-2
        rest = np.setdiff1d(np.arange(T), rows.numpy())
        assert torch.equal(got_r[rest], r0.double()[rest]) and bool((got_n[rest] == 5).all())


@pytest.mark.parametrize("n,hidden,ffn", [(1200, 2048, 8192), (1400, 3072, 14336), (600, 8192, 14336)])
def test_block_tail_same_bits_with_and_without_room(n, hidden, ffn, tuning):
    """The larger tiles in which one workgroup forms all shares of a split reduction (128 x 128, 128 x 192, 256 x 128; the shapes
    above reach the smallest): bit for bit what the split product and its sum give, both within 2e-2 of the unsplit product."""
    lay = _layout(hidden, 8, 1, n + 1)
    g = torch.Generator(device="cuda").manual_seed(n)
    mk = lambda *s, std=1.0: (torch.randn(*s, device="cuda", generator=g) * std).bfloat16()
    o, r0 = mk(n, 8, 128), mk(n + 1, hidden)
    lw = (mk(hidden, 1024, std=0.05), 1 + mk(hidden, std=0.1), mk(ffn, hidden, std=0.02), mk(ffn, hidden, std=0.02),
          mk(hidden, ffn, std=0.02), 1 + mk(hidden, std=0.1))
    small = ((n * hidden * 2 + 255) // 256 + (n * ffn * 2 + 255) // 256) * 256 + 256
    need = api.a3_block_tail_ws_bytes(lay, ffn, n)
    assert need > small

    def run(size):
        resid, nxt = r0.clone(), torch.zeros_like(r0)
        api.a3_block_tail(lay, o, None, n, *lw, 1e-5, resid, nxt, torch.empty(size, dtype=torch.uint8, device="cuda"))
        return resid, nxt

    split, summed = run(need), run(small)
    tuning("gemm_tb", 4)
    unsplit = run(small)
    for a, b, c in zip(split, summed, unsplit):
        assert torch.equal(a, b)
        assert float((a.double() - c.double()).abs().max() / c.double().abs().max()) <= 2e-2
