"""GPU parity of the layer-stack entry points (a3_rms_norm, a3_block_tail) and of the whole A^3 schedule
over a small stack (paper_2511_17560_amd.stack.fuse_stack) against the stack oracle.

Tolerances (max |a-b| / max |b| per tensor unless stated):
  RMSNorm                      fp32 1e-5; bf16 one rounding of the stored value (2^-7)
  H(.) (a3_block_tail)         fp32 2e-5; bf16 2e-2 (five stored tensors in a row, each rounded once, and
                               K up to 14336 products per sum), mean |a-b| <= 2e-3 of the scale
  stack                        fp32 1e-4; bf16 2e-2 after four blocks, mean |a-b| <= 4e-3 of the scale.  A block
                               stores five bf16 tensors in a row, each within 2^-8 of its value: were the twenty
                               roundings of four blocks all to line up, 20 * 2^-9 = 4e-2; they are independent,
                               their sum has a deviation of sqrt(20) * 2^-9 / sqrt(3) = 5e-3 of the element, and the
                               bar stands at four of those deviations
  selection                    a row picked on one side only has an oracle score within 1e-3 of the k-th largest
"""
import numpy as np
import pytest
import torch

from oracle import a3_oracle as ora
from oracle import stack_oracle as st
import a3_synth as synth
from paper_2511_17560_amd import api, stack
from gpu_util import idev, max_abs_rel, to_dev, to_host

pytestmark = pytest.mark.gpu

F64 = np.float64


def _layout(shape, T):
    """A one-request layout with T rows; the stack entry points only read sizes from it."""
    w = synth.custom(shape, [[T - 1]], [1])
    return api.Layout.from_workload(w)


def _mean_rel(got, want):
    return float(np.abs(got - want).mean()) / float(np.abs(want).max())


@pytest.mark.parametrize("dtype,h,T,n", [("f32", 96, 50, 17), ("bf16", 256, 300, 123), ("bf16", 4096, 700, 700),
                                          ("f32", 512, 9, 9)])
def test_rms_norm(dtype, h, T, n):
    rng = np.random.default_rng(7)
    shape = synth.ModelShape("n", dtype, h, 2, 1, 128 if dtype == "bf16" else 64, 1e4)
    lay = _layout(shape, T)
    x = synth.round_to_storage(rng.standard_normal((T, h)).astype(np.float32) * 3.0, dtype)
    g = synth.round_to_storage(1 + 0.2 * rng.standard_normal(h).astype(np.float32), dtype)
    idx = np.sort(rng.choice(T, size=n, replace=False)).astype(np.int32)
    eps = 1e-5
    want = st.rms_norm(x.astype(F64)[idx], g.astype(F64), eps)
    xd, gd = to_dev(x, dtype), to_dev(g, dtype)
    out = torch.full_like(xd, 7.0)
    api.a3_rms_norm(lay, xd, idev(idx) if n < T else None, n, gd, eps, out)
    torch.cuda.synchronize()
    got = to_host(out)
    assert max_abs_rel(got[idx], want) <= (1e-5 if dtype == "f32" else 2.0 ** -7)
    rest = np.setdiff1d(np.arange(T), idx)
    assert np.all(got[rest] == 7.0)
    # in place
    api.a3_rms_norm(lay, xd, idev(idx) if n < T else None, n, gd, eps, xd)
    torch.cuda.synchronize()
    assert np.array_equal(to_host(xd)[idx], got[idx])


TAIL_CASES = {
    # name: (dtype, hidden, Hq, head_dim, ffn, T, n_act)
    "f32-tiny": ("f32", 512, 8, 64, 1024, 300, 77),
    "f32-odd": ("f32", 96, 3, 64, 80, 40, 40),
    "bf16-small": ("bf16", 1024, 8, 128, 1536, 700, 333),
    "bf16-ragged-tiles": ("bf16", 384, 3, 128, 448, 500, 261),      # last feature tiles half empty
    "bf16-one-row": ("bf16", 256, 2, 128, 512, 10, 1),
    "bf16-llama": ("bf16", 4096, 32, 128, 14336, 2000, 450),
    "bf16-all-rows": ("bf16", 512, 4, 128, 1024, 640, 640),          # act_idx NULL
    "bf16-short-k": ("bf16", 128, 1, 128, 64, 400, 390),             # reductions of one and two 64-element slabs
}


@pytest.mark.parametrize("case", ["bf16-small", "bf16-ragged-tiles", "bf16-llama"])
@pytest.mark.parametrize("tb", ["2", "3", "4", "5", "6", "7"])
def test_block_tail_other_gemm_loops(case, tb, tuning):
    """The GEMMs of H(.) with every tile forced (the library picks one per GEMM), their reductions not split."""
    tuning("gemm_tb", tb)
    test_block_tail(case)


@pytest.mark.parametrize("case", list(TAIL_CASES))
def test_block_tail(case):
    dtype, h, Hq, d, f, T, n = TAIL_CASES[case]
    rng = np.random.default_rng(sum(map(ord, case)))
    shape = synth.ModelShape(case, dtype, h, Hq, 8 if Hq % 8 == 0 else 1, d, 1e4, ffn=f)
    lay = _layout(shape, T)
    r2s = lambda a: synth.round_to_storage(np.asarray(a, dtype=np.float32), dtype)
    nrm = lambda *s: rng.standard_normal(s).astype(np.float32)
    lw = dict(wo=r2s(nrm(h, Hq * d) * 0.02), g_post=r2s(1 + 0.1 * nrm(h)), w_gate=r2s(nrm(f, h) * 0.03),
              w_up=r2s(nrm(f, h) * 0.03), w_down=r2s(nrm(h, f) * 0.02))
    g_next = r2s(1 + 0.1 * nrm(h))
    attn = r2s(nrm(n, Hq, d))
    resid = r2s(nrm(T, h))
    idx = np.sort(rng.choice(T, size=n, replace=False)).astype(np.int32)
    eps = 1e-5
    want = st.block_tail(attn.astype(F64), resid.astype(F64)[idx], {k: v.astype(F64) for k, v in lw.items()},
                         g_next.astype(F64), eps, dtype)
    dev = {k: to_dev(v, dtype) for k, v in lw.items()}
    resid_d, hid_d = to_dev(resid, dtype), torch.full((T, h), 5.0, dtype=api.torch_dtype(dtype), device="cuda")
    ws = torch.empty(api.a3_block_tail_ws_bytes(lay, f, n), dtype=torch.uint8, device="cuda")
    api.a3_block_tail(lay, to_dev(attn, dtype), idev(idx) if n < T else None, n, dev["wo"], dev["g_post"],
                      dev["w_gate"], dev["w_up"], dev["w_down"], to_dev(g_next, dtype), eps, resid_d, hid_d, ws)
    torch.cuda.synchronize()
    got_r, got_x = to_host(resid_d), to_host(hid_d)
    tol, mtol = (2e-5, 2e-6) if dtype == "f32" else (2e-2, 2e-3)
    assert max_abs_rel(got_r[idx], want["resid"]) <= tol
    assert max_abs_rel(got_x[idx], want["hidden_next"]) <= tol
    assert _mean_rel(got_r[idx], want["resid"]) <= mtol and _mean_rel(got_x[idx], want["hidden_next"]) <= mtol
    # the MLP branch alone (what the second residual added), so that a slip there cannot hide behind r1
    assert max_abs_rel(got_r[idx] - want["resid_mid"], want["resid"] - want["resid_mid"]) <= (1e-4 if dtype == "f32" else 6e-2)
    rest = np.setdiff1d(np.arange(T), idx)
    assert np.array_equal(got_r[rest], resid.astype(F64)[rest]) and np.all(got_x[rest] == 5.0)
    # too small a workspace is an error, not a launch
    with pytest.raises(api.A3Error):
        api.a3_block_tail(lay, to_dev(attn, dtype), None, n, dev["wo"], dev["g_post"], dev["w_gate"], dev["w_up"],
                          dev["w_down"], to_dev(g_next, dtype), eps, resid_d, hid_d, ws[:256])


@pytest.mark.parametrize("n", [1702, 16448])
def test_block_tail_full_size_sampled_rows(n):
    """The Llama-3-8B shape at the 16K configuration's row counts (the 1702 active rows of a fused layer; all
    16448 rows of block 0), in the launch configuration the benchmark times.  H(.) treats rows independently,
    so the oracle is run on 96 sampled rows (first and last rows of the list included)."""
    dtype, h, Hq, d, f, T = "bf16", 4096, 32, 128, 14336, 16448
    rng = np.random.default_rng(1234 + n)
    shape = synth.ModelShape("llama", dtype, h, Hq, 8, d, 5e5, ffn=f)
    lay = _layout(shape, T)
    r2s = lambda a: synth.round_to_storage(a, dtype)
    nrm = lambda *s: rng.standard_normal(s, dtype=np.float32)
    lw = dict(wo=r2s(nrm(h, Hq * d) * np.float32(0.02)), g_post=r2s(1 + np.float32(0.1) * nrm(h)),
              w_gate=r2s(nrm(f, h) * np.float32(0.03)), w_up=r2s(nrm(f, h) * np.float32(0.03)),
              w_down=r2s(nrm(h, f) * np.float32(0.02)))
    g_next = r2s(1 + np.float32(0.1) * nrm(h))
    attn, resid = r2s(nrm(n, Hq * d)), r2s(nrm(T, h))
    idx = np.sort(rng.choice(T, size=n, replace=False)).astype(np.int32)
    pick = np.unique(np.concatenate([[0, n - 1], rng.choice(n, size=94, replace=False)]))
    want = st.block_tail(attn[pick].astype(F64), resid[idx[pick]].astype(F64), {k: v.astype(F64) for k, v in lw.items()},
                         g_next.astype(F64), 1e-5, dtype)
    dev = {k: to_dev(v, dtype) for k, v in lw.items()}
    resid_d, hid_d = to_dev(resid, dtype), torch.full((T, h), 5.0, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(api.a3_block_tail_ws_bytes(lay, f, n), dtype=torch.uint8, device="cuda")
    api.a3_block_tail(lay, to_dev(attn, dtype), idev(idx) if n < T else None, n, dev["wo"], dev["g_post"],
                      dev["w_gate"], dev["w_up"], dev["w_down"], to_dev(g_next, dtype), 1e-5, resid_d, hid_d, ws)
    torch.cuda.synchronize()
    rows = torch.as_tensor(idx[pick].astype(np.int64), device="cuda")
    got_r, got_x = to_host(resid_d[rows]), to_host(hid_d[rows])
    assert max_abs_rel(got_r, want["resid"]) <= 2e-2 and _mean_rel(got_r, want["resid"]) <= 2e-3
    assert max_abs_rel(got_x, want["hidden_next"]) <= 2e-2 and _mean_rel(got_x, want["hidden_next"]) <= 2e-3
    assert max_abs_rel(got_r - want["resid_mid"], want["resid"] - want["resid_mid"]) <= 6e-2
    # rows outside the list are untouched (checked on the device: no 270 MB round trip)
    mask = torch.ones(T, dtype=torch.bool, device="cuda")
    mask[torch.as_tensor(idx.astype(np.int64), device="cuda")] = False
    assert bool((hid_d[mask] == 5.0).all()) and bool((resid_d[mask] == to_dev(resid, dtype)[mask]).all())


STACK_CASES = {
    "tiny-f32": (synth.ModelShape("tiny-stack", "f32", 128, 4, 2, 64, 10000.0, synth.ROPE_HALF, ffn=192),
                 [[60, 41, 77]], [9], (20, 100), 3),
    "batched-f32": (synth.ModelShape("tiny-stack", "f32", 128, 4, 2, 64, 10000.0, synth.ROPE_INTERLEAVED, ffn=192),
                    [[30, 45], [64]], [5, 7], (30, 100), 4),
    "small-bf16": (synth.ModelShape("small-stack", "bf16", 256, 4, 2, 128, 500000.0, synth.ROPE_HALF, ffn=512),
                   [[100, 37, 300, 65]], [19], (15, 100), 4),
    "batched-bf16": (synth.ModelShape("small-stack", "bf16", 256, 8, 2, 128, 500000.0, synth.ROPE_HALF, ffn=384),
                     [[130, 70], [33], [257, 64, 90]], [5, 33, 12], (20, 100), 3),
    # seven query heads on one KV head, a feed-forward width that is no multiple of a tile, one-token chunks
    "g7-bf16": (synth.ModelShape("g7-stack", "bf16", 256, 7, 1, 128, 1000000.0, synth.ROPE_INTERLEAVED, ffn=320),
                [[90, 1, 120, 2], [50]], [11, 30], (25, 100), 3),
    # the two ends of the ratio: everything recomputed (the schedule is then the plain prefill), nothing but the question
    "all-rows-bf16": (synth.ModelShape("small-stack", "bf16", 256, 4, 2, 128, 500000.0, synth.ROPE_HALF, ffn=512),
                      [[70, 45], [80]], [9, 4], (100, 100), 3),
    "question-only-f32": (synth.ModelShape("tiny-stack", "f32", 128, 4, 2, 64, 10000.0, synth.ROPE_HALF, ffn=192),
                          [[60, 41], [33]], [9, 14], (0, 100), 3),
}


@pytest.mark.parametrize("case", list(STACK_CASES))
def test_fuse_stack(case):
    """Block 0 on every row, selection at layer 1 on the true keys, rows [Re, Q] afterwards, on caches
    that a chunk-wise prefill of the same stack produced (oracle, CPU).  The selection must equal the
    oracle's up to near-ties; the oracle is then run on the GPU's selection and every layer's attention
    output, the residual stream and the final hidden states are compared on the active rows."""
    shape, chunk_lens, q_lens, ratio, n_layers = STACK_CASES[case]
    dt = shape.dtype
    w = synth.custom(shape, chunk_lens, q_lens, ratio=ratio, seed=77)
    sw = synth.draw_stack_weights(w, n_layers)
    # wider query/key weights than the draw's 0.02: at these small widths the logits would otherwise be
    # nearly flat and every score a near-tie
    for lw in sw["layers"]:
        for k in ("wq", "wk"):
            lw[k] = synth.round_to_storage(lw[k] * np.float32(5.0), dt)
    layers64 = [{k: v.astype(F64) for k, v in lw.items()} for lw in sw["layers"]]
    sh = dict(n_q_heads=shape.n_q_heads, n_kv_heads=shape.n_kv_heads, head_dim=shape.head_dim, base=shape.rope_base,
              layout=shape.rope_layout, sm_scale=1.0 / np.sqrt(shape.head_dim), eps=shape.rms_eps)
    idx = dict(seg_start=w.seg_start, ctx_len=w.ctx_len, q_len=w.q_lens, chunk_start=w.chunk_start,
               chunk_len=w.chunk_len, chunk_delta=w.chunk_delta, sel_start=w.sel_start, positions=w.token_positions())
    r0 = sw["resid0"].astype(F64)
    g_final = sw["g_final"].astype(F64)
    k_cat, v_cat = st.precompute_stack_caches(r0, w.chunk_start, w.chunk_len, layers64, g_final, sh, dt)
    want = st.fuse_stack(r0, k_cat, v_cat, layers64, g_final, sh, storage=dt, **idx)

    lay = api.Layout.from_workload(w)
    dev_layers = [{k: to_dev(v, dt) for k, v in lw.items()} for lw in sw["layers"]]
    resid = to_dev(sw["resid0"], dt)
    got = stack.fuse_stack(lay, shape, dev_layers, to_dev(sw["g_final"], dt), resid, [to_dev(k, dt) for k in k_cat],
                           [to_dev(v, dt) for v in v_cat], w.sel_start, w.question_rows(), keep=True)
    torch.cuda.synchronize()
    got_act = got["act_idx"].cpu().numpy()
    assert np.all(np.diff(got_act) > 0) and got["n_act"] == len(want["act_idx"])
    flips = set(got_act.tolist()) ^ set(want["act_idx"].tolist())
    for r in range(w.n_req):
        k_r = int(w.sel_start[r + 1] - w.sel_start[r])
        rows = w.ctx_rows(r)
        if k_r == 0 or k_r == len(rows):
            continue
        kth = np.sort(want["scores"][rows])[::-1][k_r - 1]
        for row in flips:
            if rows[0] <= row <= rows[-1]:
                assert abs(want["scores"][row] - kth) <= 1e-3 * abs(kth), (row, want["scores"][row], kth)
    assert len(flips) <= max(2, len(got_act) // 25)
    sc_tol = 1e-4 if dt == "f32" else 2e-2
    ctx = np.concatenate([w.ctx_rows(r) for r in range(w.n_req)])
    assert max_abs_rel(to_host(got["scores"])[ctx], want["scores"][ctx]) <= sc_tol
    if flips:   # same selection on both sides from here on
        want = st.fuse_stack(r0, k_cat, v_cat, layers64, g_final, sh, storage=dt,
                             forced_sel_idx=got["sel_idx"].cpu().numpy(), **idx)
    tol, mtol = (1e-4, 1e-5) if dt == "f32" else (2e-2, 4e-3)
    for l in range(n_layers):
        g_out = to_host(got["per_layer"][l]["out"])
        assert max_abs_rel(g_out, want["per_layer"][l]["out"]) <= tol, l
        if l >= 1:
            assert max_abs_rel(to_host(got["per_layer"][l]["k"])[got_act], want["per_layer"][l]["k"][got_act]) <= tol, l
    g_res, g_hid = to_host(got["resid"])[got_act], to_host(got["hidden"])[got_act]
    assert max_abs_rel(g_res, want["resid"]) <= tol and _mean_rel(g_res, want["resid"]) <= mtol
    assert max_abs_rel(g_hid, want["hidden"]) <= tol and _mean_rel(g_hid, want["hidden"]) <= mtol


@pytest.mark.parametrize("case", ["tiny-f32", "batched-bf16"])
def test_prefill_stack(case):
    """Every block on every row against the oracle's full prefill; and, on one chunk alone, Eq. 1: the
    chunk's per-layer K/V at chunk-local positions."""
    shape, chunk_lens, q_lens, ratio, n_layers = STACK_CASES[case]
    dt = shape.dtype
    w = synth.custom(shape, chunk_lens, q_lens, ratio=ratio, seed=78)
    sw = synth.draw_stack_weights(w, n_layers)
    for lw in sw["layers"]:
        for k in ("wq", "wk"):
            lw[k] = synth.round_to_storage(lw[k] * np.float32(5.0), dt)
    layers64 = [{k: v.astype(F64) for k, v in lw.items()} for lw in sw["layers"]]
    sh = dict(n_q_heads=shape.n_q_heads, n_kv_heads=shape.n_kv_heads, head_dim=shape.head_dim, base=shape.rope_base,
              layout=shape.rope_layout, sm_scale=1.0 / np.sqrt(shape.head_dim), eps=shape.rms_eps)
    want = st.full_prefill_stack(sw["resid0"].astype(F64), w.token_positions(), w.seg_start, layers64,
                                 sw["g_final"].astype(F64), sh, dt)
    lay = api.Layout.from_workload(w)
    dev_layers = [{k: to_dev(v, dt) for k, v in lw.items()} for lw in sw["layers"]]
    got = stack.prefill_stack(lay, shape, dev_layers, to_dev(sw["g_final"], dt), to_dev(sw["resid0"], dt), keep_kv=True)
    torch.cuda.synchronize()
    tol, mtol = (1e-4, 1e-5) if dt == "f32" else (2e-2, 4e-3)
    for l in range(n_layers):
        assert max_abs_rel(to_host(got["k"][l]), want["k"][l]) <= tol, l
        assert max_abs_rel(to_host(got["v"][l]), want["v"][l]) <= tol, l
    assert max_abs_rel(to_host(got["hidden"]), want["hidden"]) <= tol
    assert _mean_rel(to_host(got["hidden"]), want["hidden"]) <= mtol
    # one chunk on its own (the second of the first request)
    s0, n = int(w.chunk_start[1]), int(w.chunk_len[1])
    w1 = synth.custom(shape, [[n - 1]], [1])
    lay1 = api.Layout.from_workload(w1)
    alone = stack.prefill_stack(lay1, shape, dev_layers, to_dev(sw["g_final"], dt),
                                to_dev(sw["resid0"][s0:s0 + n], dt), keep_kv=True)
    torch.cuda.synchronize()
    k_cat, v_cat = st.precompute_stack_caches(sw["resid0"].astype(F64), w.chunk_start, w.chunk_len, layers64,
                                              sw["g_final"].astype(F64), sh, dt)
    for l in range(n_layers):
        assert max_abs_rel(to_host(alone["k"][l]), k_cat[l][s0:s0 + n]) <= tol, l
        assert max_abs_rel(to_host(alone["v"][l]), v_cat[l][s0:s0 + n]) <= tol, l


def test_chunk_cache_load_and_streamed_stack():
    """a3_chunk_cache_load puts every chunk block at its packed rows (bit-exact, other rows untouched), and
    the schedule run on caches streamed from pinned host memory layer by layer gives bit for bit what it
    gives on resident caches."""
    from paper_2511_17560_amd import loader
    shape, chunk_lens, q_lens, ratio, n_layers = STACK_CASES["batched-bf16"]
    n_layers = 6
    dt = shape.dtype
    w = synth.custom(shape, chunk_lens, q_lens, ratio=ratio, seed=79)
    sw = synth.draw_stack_weights(w, n_layers)
    for lw in sw["layers"]:
        for k in ("wq", "wk"):
            lw[k] = synth.round_to_storage(lw[k] * np.float32(5.0), dt)
    lay = api.Layout.from_workload(w)
    rng = np.random.default_rng(3)
    T = w.total_tokens
    tdt = api.torch_dtype(dt)
    caches_k = [None, None] + [synth.round_to_storage(rng.standard_normal((T, shape.n_kv_heads, shape.head_dim), dtype=np.float32), dt)
                               for _ in range(n_layers - 2)]
    caches_v = [None, None] + [synth.round_to_storage(rng.standard_normal((T, shape.n_kv_heads, shape.head_dim), dtype=np.float32), dt)
                               for _ in range(n_layers - 2)]
    pin = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(tdt).pin_memory()
    host_k = [None if ck is None else [pin(ck[s:s + n]) for s, n in zip(w.chunk_start, w.chunk_len)] for ck in caches_k]
    host_v = [None if cv is None else [pin(cv[s:s + n]) for s, n in zip(w.chunk_start, w.chunk_len)] for cv in caches_v]
    # the copy itself
    k_dev = torch.full((T, shape.n_kv_heads, shape.head_dim), 9.0, dtype=tdt, device="cuda")
    v_dev = torch.full_like(k_dev, 9.0)
    api.a3_chunk_cache_load(lay, w.chunk_start, w.chunk_len, host_k[2], host_v[2], k_dev, v_dev)
    torch.cuda.synchronize()
    ctx = np.concatenate([w.ctx_rows(r) for r in range(w.n_req)])
    assert np.array_equal(to_host(k_dev)[ctx], caches_k[2][ctx].astype(F64)) and np.array_equal(to_host(v_dev)[ctx], caches_v[2][ctx].astype(F64))
    assert np.all(to_host(k_dev)[w.question_rows()] == 9.0)
    with pytest.raises(api.A3Error):
        api.a3_chunk_cache_load(lay, [T - 3], [10], [host_k[2][0]], [host_v[2][0]], k_dev, v_dev)   # runs past the last row
    # the schedule, resident against streamed
    dev_layers = [{k: to_dev(v, dt) for k, v in lw.items()} for lw in sw["layers"]]
    g_final = to_dev(sw["g_final"], dt)

    def resident():
        kc = [None if c is None else to_dev(np.where(np.isin(np.arange(T), ctx)[:, None, None], c, 0), dt) for c in caches_k]
        vc = [None if c is None else to_dev(np.where(np.isin(np.arange(T), ctx)[:, None, None], c, 0), dt) for c in caches_v]
        return stack.fuse_stack(lay, shape, dev_layers, g_final, to_dev(sw["resid0"], dt), kc, vc, w.sel_start,
                                w.question_rows())

    a = resident()
    cs = loader.ChunkCacheStream(lay, shape, w.chunk_start, w.chunk_len, host_k, host_v, depth=2)
    b = stack.fuse_stack(lay, shape, dev_layers, g_final, to_dev(sw["resid0"], dt), None, None, w.sel_start,
                         w.question_rows(), cache_stream=cs)
    torch.cuda.synchronize()
    assert torch.equal(a["act_idx"], b["act_idx"])
    rows = a["act_idx"].long()
    assert torch.equal(a["hidden"][rows], b["hidden"][rows]) and torch.equal(a["resid"][rows], b["resid"][rows])


def test_fuse_stack_llama_shape_16k_layer_by_layer():
    """The schedule at full size: Llama-3-8B's block shape, one request of 32 chunks of 512 tokens and a 64-token
    question, r = 10 %, three blocks (block 0 on every row, layer 1 with the selection, one fused layer on a
    drawn chunk cache), in the launch configuration the benchmark times.  The float64 oracle cannot run this
    stack whole in test time, so every step is checked on its own: the oracle gets the inputs the GPU had at that
    step (the kept hidden states, caches and residual stream) and computes the step for sampled rows (the
    first and last of the list always among them); each comparison is then one step deep and carries the
    per-step bar (bf16: 2e-2 of the tensor's largest value).  The selection is compared as a set, up to near-ties."""
    shape = synth.ModelShape("llama-3-8b-block", "bf16", 4096, 32, 8, 128, 500000.0, synth.ROPE_HALF, ffn=14336)
    dt, n_layers, tol = "bf16", 3, 2e-2
    w = synth.custom(shape, [[512] * 32], [64], ratio=(10, 100), seed=91)
    T, Hkv, d = w.total_tokens, shape.n_kv_heads, shape.head_dim
    sw = synth.draw_stack_weights(w, n_layers)
    rng = np.random.default_rng(92)
    cache_k = synth.round_to_storage(rng.standard_normal((T, Hkv, d), dtype=np.float32), dt)
    cache_v = synth.round_to_storage(rng.standard_normal((T, Hkv, d), dtype=np.float32), dt)
    lay = api.Layout.from_workload(w)
    dev_layers = [{k: to_dev(v, dt) for k, v in lw.items()} for lw in sw["layers"]]
    got = stack.fuse_stack(lay, shape, dev_layers, to_dev(sw["g_final"], dt), to_dev(sw["resid0"], dt),
                           [None, None, to_dev(cache_k, dt)], [None, None, to_dev(cache_v, dt)], w.sel_start,
                           w.question_rows(), keep=True)
    torch.cuda.synchronize()
    kept = [{k: to_host(v) for k, v in pl.items()} for pl in got["per_layer"]]
    act = got["act_idx"].cpu().numpy().astype(np.int64)
    n_act = len(act)
    q_rows = np.asarray(w.question_rows(), dtype=np.int64)
    assert n_act == int(w.sel_start[-1]) + len(q_rows) and np.all(np.diff(act) > 0)
    del dev_layers
    torch.cuda.empty_cache()

    pos = np.asarray(w.token_positions())
    proj = dict(n_q_heads=shape.n_q_heads, n_kv_heads=Hkv, head_dim=d, base=shape.rope_base,
                layout=shape.rope_layout, storage=dt)
    scale, eps = 1.0 / np.sqrt(d), shape.rms_eps
    l64 = lambda l: {k: v.astype(F64) for k, v in sw["layers"][l].items()}
    close = lambda a, b: max_abs_rel(np.asarray(a, dtype=F64), b) <= tol

    # ---- block 0 on sampled rows of the whole input ------------------------------------------------------
    lw = l64(0)
    rows = np.unique(np.concatenate([[0, 511, 512, T - 65, T - 64, T - 1], rng.choice(T, size=42, replace=False)]))
    r0 = sw["resid0"].astype(F64)
    x0 = ora.store(st.rms_norm(r0[rows], lw["g_in"], eps), dt)
    q, k, v = ora.selected_qkv_proj(x0, np.arange(len(rows)), pos[rows], lw["wq"], lw["wk"], lw["wv"], **proj)
    assert close(kept[0]["k"][rows], k) and close(kept[0]["v"][rows], v)
    o = ora.fused_attention(q, rows, kept[0]["k"], kept[0]["v"], w.seg_start, scale, dt)
    assert close(kept[0]["out"][rows], o)
    t = st.block_tail(kept[0]["out"][rows].astype(F64), r0[rows], lw, sw["layers"][1]["g_in"].astype(F64), eps, dt)
    assert close(kept[0]["resid"][rows], t["resid"]) and close(kept[0]["x_next"][rows], t["hidden_next"])

    # ---- layer 1: true keys, scores, selection, attention of the rows [Re, Q] ------------------------------------
    lw = l64(1)
    x1 = kept[0]["x_next"].astype(F64)
    _, k, v = ora.selected_qkv_proj(x1, rows, pos[rows], lw["wq"], lw["wk"], lw["wv"], **proj)
    assert close(kept[1]["k"][rows], k) and close(kept[1]["v"][rows], v)
    qq, _, _ = ora.selected_qkv_proj(x1, q_rows, pos[q_rows], lw["wq"], lw["wk"], lw["wv"], **proj)
    scores = ora.question_scores(qq, kept[1]["k"], w.seg_start, w.ctx_len, w.q_lens, scale)
    ctx = w.ctx_rows(0)
    assert max_abs_rel(to_host(got["scores"])[ctx], scores[ctx]) <= tol
    want_sel = ora.topk_select(scores, w.seg_start, w.ctx_len, w.sel_start)
    flips = set(got["sel_idx"].cpu().numpy().tolist()) ^ set(want_sel.tolist())
    kth = np.sort(scores[ctx])[::-1][int(w.sel_start[1]) - 1]
    assert len(flips) <= n_act // 25 and all(abs(scores[r] - kth) <= 1e-2 * abs(kth) for r in flips)
    pick = np.unique(np.concatenate([[0, n_act - 65, n_act - 64, n_act - 1], rng.choice(n_act, size=44, replace=False)]))
    q, _, _ = ora.selected_qkv_proj(x1, act[pick], pos[act[pick]], lw["wq"], lw["wk"], lw["wv"], **proj)
    o = ora.fused_attention(q, act[pick], kept[1]["k"], kept[1]["v"], w.seg_start, scale, dt)
    assert close(kept[1]["out"][pick], o)
    t = st.block_tail(kept[1]["out"][pick].astype(F64), kept[0]["resid"][act[pick]].astype(F64), lw,
                      sw["layers"][2]["g_in"].astype(F64), eps, dt)
    assert close(kept[1]["resid"][pick], t["resid"]) and close(kept[1]["x_next"][pick], t["hidden_next"])

    # ---- layer 2: Eq. 2 on the drawn cache, Eq. 5 on the rows [Re, Q] --------------------------------------------
    lw = l64(2)
    k_re = ora.rope_realign(cache_k, w.chunk_start, w.chunk_len, w.chunk_delta, shape.rope_base, shape.rope_layout, dt)
    rest = np.setdiff1d(np.arange(T), act)
    assert close(kept[2]["k"][rest], k_re[rest]) and np.array_equal(kept[2]["v"][rest], cache_v[rest])
    x2 = kept[1]["x_next"][pick].astype(F64)
    q, k, v = ora.selected_qkv_proj(x2, np.arange(len(pick)), pos[act[pick]], lw["wq"], lw["wk"], lw["wv"], **proj)
    assert close(kept[2]["k"][act[pick]], k) and close(kept[2]["v"][act[pick]], v)
    o = ora.fused_attention(q, act[pick], kept[2]["k"], kept[2]["v"], w.seg_start, scale, dt)
    assert close(kept[2]["out"][pick], o)
    t = st.block_tail(kept[2]["out"][pick].astype(F64), kept[1]["resid"][pick].astype(F64), lw,
                      sw["g_final"].astype(F64), eps, dt)
    assert close(kept[2]["resid"][pick], t["resid"]) and close(kept[2]["x_next"][pick], t["hidden_next"])
    assert np.array_equal(to_host(got["resid"])[act[pick]], kept[2]["resid"][pick])
    assert np.array_equal(to_host(got["hidden"])[act[pick]], kept[2]["x_next"][pick])
