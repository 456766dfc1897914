"""fp32 projection at reductions shorter than the workgroup's four waves share (32 elements are two chunks of 16: two waves have none) and a
little longer, rows on both sides of a block's two halves of 16, both rotary layouts, listed rows to compact outputs and scattered into
the caches.  Against the float64 oracle; 1e-5 of the largest element, as for the other fp32 steps."""
import numpy as np
import pytest
import torch

import a3_synth as synth
from oracle import a3_oracle as ora
from paper_2511_17560_amd import api
from gpu_util import idev, max_abs_rel, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scatter", [False, True])
@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("n", [1, 16, 17, 32, 33, 70])
@pytest.mark.parametrize("hidden,hq,hkv,d", [(32, 2, 1, 64), (32, 3, 3, 128), (64, 2, 2, 64), (96, 4, 2, 128)])
def test_f32_projection(hidden, hq, hkv, d, n, half, scatter):
    w = synth.custom(synth.ModelShape("proj", "f32", hidden, hq, hkv, d, 1e4, synth.ROPE_HALF if half else synth.ROPE_INTERLEAVED), [[60, 21]], [9])
    rng = np.random.default_rng(hidden + n)
    x, wq, wk, wv = (rng.standard_normal(s).astype(np.float32) for s in ((w.total_tokens, hidden), (hq * d, hidden), (hkv * d, hidden), (hkv * d, hidden)))
    rows = np.sort(rng.permutation(w.total_tokens)[:n])
    want = ora.selected_qkv_proj(x, rows, w.token_positions()[rows], wq, wk, wv, hq, hkv, d, 1e4, w.shape.rope_layout, "f32")
    lay, dev = api.Layout.from_workload(w), lambda a: torch.from_numpy(a).cuda()
    q = torch.zeros((n, hq, d), device="cuda")
    k, v = (torch.zeros((w.total_tokens if scatter else n, hkv, d), device="cuda") for _ in range(2))
    if scatter:
        api.a3_selected_qkv_proj_scatter(lay, dev(x), idev(rows), n, dev(wq), dev(wk), dev(wv), q_out=q, k_fused=k, v_fused=v)
        at = torch.from_numpy(rows).cuda()
        others = torch.ones(w.total_tokens, dtype=torch.bool, device="cuda")
        others[at] = False
        assert not bool(k[others].any() or v[others].any())
        k, v = k[at], v[at]
    else:
        api.a3_selected_qkv_proj(lay, dev(x), idev(rows), n, dev(wq), dev(wk), dev(wv), q_out=q, k_out=k, v_out=v)
    for got, ref in zip((q, k, v), want):
        assert max_abs_rel(to_host(got), ref) <= 1e-5
