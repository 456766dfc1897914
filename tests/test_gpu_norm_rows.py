"""a3_rms_norm at the widths where the number of vectors a lane keeps changes (2, 4, 8, 16 of them, or a row
read twice), and one vector past each.

Tolerance: fp32 1e-5; bf16 one rounding of the stored value (2^-8 of it, 2^-7 of the largest with the fp32 sum's share).
"""
import numpy as np
import pytest
import torch

from oracle import stack_oracle as st
import a3_synth as synth
from paper_2511_17560_amd import api
from gpu_util import max_abs_rel, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,edge", [("bf16", 512 * n) for n in (2, 4, 8, 16)] + [("f32", 256 * n) for n in (2, 4, 8, 16)])
@pytest.mark.parametrize("past", [-32, 0, 32])
def test_rms_norm_at_the_edges_of_the_widths(dtype, edge, past):
    h, n = edge + past, 7                                        # 7 rows: the last workgroup has a wave without one
    rng = np.random.default_rng(h)
    lay = api.Layout.from_workload(synth.custom(synth.ModelShape("n", dtype, h, 2, 1, 128 if dtype == "bf16" else 64, 1e4), [[n - 1]], [1]))
    x = synth.round_to_storage(rng.standard_normal((n, h)).astype(np.float32) * 3.0, dtype)
    g = synth.round_to_storage(1 + 0.2 * rng.standard_normal(h).astype(np.float32), dtype)
    want = st.rms_norm(x.astype(np.float64), g.astype(np.float64), 1e-5)
    xd, gd = to_dev(x, dtype), to_dev(g, dtype)
    out = torch.full((n + 1, h), 7.0, dtype=xd.dtype, device="cuda")
    api.a3_rms_norm(lay, xd, None, n, gd, 1e-5, out[:n])
    torch.cuda.synchronize()
    assert max_abs_rel(to_host(out)[:n], want) <= (1e-5 if dtype == "f32" else 2.0 ** -7)
    assert bool((out[n] == 7.0).all())
