"""fp32 scores where the row statistics change hands between the second pass and the kernel in front of it: 8, 16 and 32 tiles of 64 keys,
256 and 768 workgroups (tiles x KV heads), 128, 256 and 1024 rows per KV head.  Against a float64 softmax, 2e-5 element by element as in
test_gpu_parity.py."""
import numpy as np
import pytest
import torch

import a3_synth as synth
from paper_2511_17560_amd import api
from gpu_util import max_elem_rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n,hkv,rows", [(512, 33, 1024), (513, 2, 1024), (513, 33, 128), (512, 2, 1025), (1024, 16, 129), (1024, 17, 128), (1024, 17, 129),
                                        (1024, 48, 128), (1024, 49, 128), (1025, 8, 256), (1025, 8, 257), (2048, 8, 256), (2048, 9, 16), (2049, 2, 16)])
def test_f32_scores(n, hkv, rows, d):
    w = synth.custom(synth.ModelShape("merge", "f32", 32, hkv, hkv, d, 1e4), [[n]], [rows])
    g = torch.Generator(device="cuda").manual_seed(n + rows)
    q, k = torch.randn(rows, hkv, d, generator=g, device="cuda"), torch.randn(w.total_tokens, hkv, d, generator=g, device="cuda")
    lay = api.Layout.from_workload(w)
    scores, ws = torch.zeros(w.total_tokens, device="cuda"), lay.workspace(0)
    api.a3_question_scores(lay, q, k, scores, ws)
    want = torch.zeros(n, dtype=torch.float64, device="cuda")
    for h in range(hkv):
        want += torch.softmax(q[:, h].double() @ k[:n, h].double().T.contiguous() / d ** 0.5, -1).sum(0)
    got = scores.double().cpu().numpy()
    assert max_elem_rel(got[:n], want.cpu().numpy()) <= 2e-5 and np.all(np.isneginf(got[n:]))
