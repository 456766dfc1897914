"""Compaction of the retained rows at the edges of a workgroup's share (8 or 16 rows of one head), for both lengths of a head's row:
bytes equal to a gather, nothing written past the last row."""
import pytest
import torch

import a3_synth as synth
from paper_2511_17560_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("hkv", [1, 3])
@pytest.mark.parametrize("total_keep", [1, 7, 8, 9, 16, 17, 130])
def test_compact(dtype, d, hkv, total_keep):
    w = synth.custom(synth.ModelShape("compact", dtype, 64, hkv, hkv, d, 1e4, synth.ROPE_HALF), [[100, 27]], [3])
    lay = api.Layout.from_workload(w)
    g = torch.Generator().manual_seed(total_keep)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    k, v = (torch.randn(w.total_tokens, hkv, d, generator=g).to(dt) for _ in range(2))
    keep = torch.stack([torch.sort(torch.randperm(w.total_tokens, generator=g)[:total_keep])[0] for _ in range(hkv)])
    k_out, v_out = (torch.full((total_keep + 1, hkv, d), 7.0, dtype=dt, device="cuda") for _ in range(2))
    api.a3_evict_compact(lay, k.cuda(), v.cuda(), keep.int().cuda(), total_keep, k_out, v_out)
    heads = torch.arange(hkv)
    for out, src in ((k_out.cpu(), k), (v_out.cpu(), v)):
        assert torch.equal(out[:total_keep], src[keep.T, heads]) and bool((out[total_keep:] == 7).all())
