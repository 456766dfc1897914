"""Codes of the quantiser where its remainder test has to hand over to the division: rounding ties, quotients a unit away
from one, scales too small or too large for a float reciprocal, infinities and NaN.  Whole numbers: exact."""
import numpy as np
import pytest
import torch

import a3_synth as synth
from oracle import q8_oracle as q8
from paper_2511_17560_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("heads", [1, 3, 8])
@pytest.mark.parametrize("d", [64, 128])
def test_codes(dtype, heads, d):
    if dtype == "bf16" and d == 64:
        pytest.skip("bf16 layouts have 128 coordinates per head")
    rng = np.random.default_rng(d + heads)
    shape = synth.ModelShape("q8", dtype, 32, heads, heads, d, 1e4)
    w = synth.custom(shape, [[45]], [2], ratio=(10, 100))
    T = w.total_tokens
    x = rng.standard_normal((T, heads, d)) * np.exp2(rng.integers(-20, 20, (T, heads, 1)))
    for t in range(8):                                        # ties at scales 2^-4 .. 2^3
        x[t] = (rng.integers(-127, 127, (heads, d)) + 0.5) * 2.0 ** (t - 4)
        x[t, :, 0] = 127.0 * 2.0 ** (t - 4)
    x = x.astype(np.float32)
    for t in range(8, 16):                                    # one unit of the last place beside a tie
        x[t] = np.nextafter(((rng.integers(-126, 126, (heads, d)) + 0.5) * 0.0625).astype(np.float32),
                            np.float32(np.inf if t % 2 else -np.inf))
        x[t, :, 0] = 127.0 * 0.0625
    for t, e in enumerate([-148, -140, -126, -118, -100, 100, 110, 120]):
        x[16 + t] = np.ldexp(rng.standard_normal((heads, d)), e).astype(np.float32)
    x[24] = 0.0
    td = torch.from_numpy(x).to(api.torch_dtype(dtype))
    x = td.float().numpy()
    qx, sx = q8.quantize_q8(x)
    special = x.copy()                                        # rows with infinities and NaN: what the float64 quotient gives
    special[30, :, 3] = np.inf
    special[31, :, 5] = np.nan
    special[32] = np.nan
    qs, ss = qx.copy(), sx.copy()
    qs[30], ss[30] = 0, np.inf
    qs[30, :, 3] = -127                                       # inf / inf is no number; those take the lowest code
    rest = special[31].copy()
    rest[:, 5] = 0
    qs[31], ss[31] = (v[0] for v in q8.quantize_q8(rest[None]))
    qs[31, :, 5] = -127
    qs[32], ss[32] = 0, 0
    lay = api.Layout.from_workload(w)
    rec = torch.full((T, api.a3_q8_row_bytes(lay)), 99, dtype=torch.uint8, device="cuda")
    api.a3_quantize_q8(lay, td.cuda(), torch.from_numpy(special).to(td.dtype).cuda(), rec)
    got = rec.cpu().numpy()
    n = heads * d
    f = lambda a: np.ascontiguousarray(a, dtype="<f4").view(np.uint8).reshape(T, -1)
    want = np.concatenate([qx.reshape(T, n).view(np.uint8), qs.reshape(T, n).view(np.uint8), f(sx), f(ss)], axis=1)
    assert np.array_equal(got, want), np.argwhere(got != want)[:5]
