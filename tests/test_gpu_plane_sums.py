"""Products split over K whose partial planes the next kernel adds up: every consumer of such planes (convolution, gated
norm, residual norm, q/k norm + RoPE, SwiGLU) in every instance that can meet more than one plane, against the float64
oracle.  A product of few tiles is split once each part keeps four 64-wide k-tiles (K >= 512): here K is 1024 and more,
and the planes are 2 to 8.  A plane left out, added twice or read at a wrong stride is an error of the order of the result."""
import numpy as np
import pytest

import oracle.hspec_oracle as O
from gpu_util import assert_close, dev, empty, host
from paper_2609_24197_amd import hspec, inputs as I

pytestmark = pytest.mark.gpu


def _cfg(**kw):
    base = dict(name="planes", B=3, k=16, d_model=1024, H=16, P=64, N=16, G=1, chunk=16, Hq=8, Hkv=2, D=128, r=64,
                lengths="uniform:0:90")
    base.update(kw)
    return I.StepConfig(**base)


MAMBA = {
    "conv4_few_tokens": _cfg(H=8, G=2),
    "conv4_many_tokens": _cfg(B=64, d_model=4096, H=12, N=128),     # four tokens per thread from 512 workgroups
    "conv3": _cfg(conv_w=3, H=8, G=2),
    "conv4_odd_heads": _cfg(H=5, k=7),                              # rows of in_proj not 16-byte aligned
    "norm_of_4608": _cfg(B=1, k=5, H=72),                           # gated-norm groups of 4097 to 8192 channels
    "rows_14": _cfg(B=2, k=7, H=8),
    "rows_112": _cfg(B=7, H=8),
    "rows_160": _cfg(B=10, H=8),
}


@pytest.mark.parametrize("name", sorted(MAMBA))
def test_mamba_planes(name):
    cfg = MAMBA[name]
    W = I.make_weights(cfg, 1)
    x = I.make_inputs(cfg, seed=1)
    d = dev(dict(h_last=x["h_last"], u=x["block_emb"]))
    ws = hspec.workspace(hspec.mamba_block_scan_workspace(cfg))
    out = empty((cfg.B, cfg.k, cfg.d_model))
    hspec.mamba_block_scan(cfg, dev(W), d["h_last"], d["u"], out, ws)
    S0, _ = O.state_init(x["h_last"], W["W_r"], W["W_dS"], cfg.H, cfg.P, cfg.N)
    assert_close(host(out), O.mamba_mixer(O.f64(x["block_emb"]), S0, W, cfg), name)


ATTN = {
    "fused_list": _cfg(),
    "d64": _cfg(B=2, k=7, Hq=4, D=64),
    "rows_112_causal": _cfg(B=7, block_causal=True),
    "list_of_its_own": _cfg(B=520, k=1, d_model=2048, Hq=2, Hkv=2, D=64, lengths="uniform:0:40"),
    "segments_of_64": _cfg(B=2, k=7, Hq=2, Hkv=1, D=64),            # a product per segment: no planes left
}


@pytest.mark.parametrize("name", sorted(ATTN))
def test_attn_planes(name):
    cfg = ATTN[name]
    W = I.make_weights(cfg, 2)
    x = I.make_inputs(cfg, seed=2)
    xin = I.normal("attn_x", (cfg.B, cfg.k, cfg.d_model), 1.0, 2, cfg.dtype)
    d = dev(dict(x, xin=xin))
    maxL = int(max(x["ctx_lens"]))
    ws = hspec.workspace(hspec.target_kv_block_attn_workspace(cfg, x["page_table"].shape[1], x["num_pages"], maxL))
    out = empty((cfg.B, cfg.k, cfg.d_model))
    hspec.target_kv_block_attn(cfg, dev(W), d["xin"], d, out, ws, maxL)
    assert hspec.read_status(ws) == 0
    assert_close(host(out), O.attention_layer(O.f64(xin), W, x, cfg), name)


STEP = {   # the residual (bf16 block embeddings) and the planes of out_proj in one norm: rows of one, two and more pieces
    "row_1024": _cfg(),
    "row_4608": _cfg(d_model=4608, precise_io=True),
    "row_8256": _cfg(B=2, k=4, d_model=8256, H=32, Hq=4, Hkv=1, precise_io=True),
    "row_1024_precise": _cfg(B=7, precise_io=True),
    "gated_norm_of_8448": _cfg(B=5, k=13, d_model=3072, H=132, Hq=4, Hkv=1, precise_io=True),   # past 8192: two passes
}


@pytest.mark.parametrize("name", sorted(STEP))
def test_step_planes(name):
    cfg = STEP[name]
    W = I.make_weights(cfg, 3)
    x = I.make_inputs(cfg, seed=3)
    maxL = int(max(x["ctx_lens"]))
    ws = hspec.workspace(hspec.draft_step_workspace(cfg, x["page_table"].shape[1], x["num_pages"], maxL))
    out = empty((cfg.B, cfg.k, cfg.d_model))
    hspec.draft_step(cfg, dev(W), dev(x), out, ws, maxL)
    assert hspec.read_status(ws) == 0
    assert_close(host(out), O.draft_step(W, x, cfg), name)


@pytest.mark.parametrize("B,k,ff", [(2, 7, 1024), (3, 16, 1032), (7, 16, 1024), (10, 16, 768)])
def test_drafter_planes(B, k, ff):
    """Every product of the drafter split, but for the MLP of ff = 1032, which does not fill tiles: the planes go to SwiGLU, to
    the norm with the fp32 residual, to the convolution and to RoPE, from hi/lo rows, 14 to 160 of them."""
    cfg = _cfg(B=B, k=k, ff=ff, H=16, n_fuse=2)
    shared, L = I.make_drafter_weights(cfg, seed=4)
    x = I.make_drafter_inputs(cfg, seed=4, n_caches=3)
    X = dev({n: v for n, v in x.items() if n != "caches"})
    X["caches"] = [dev(c) for c in x["caches"]]
    layers = [{n: (hspec.to_device(v) if isinstance(v, np.ndarray) else v) for n, v in W.items()} for W in L]
    maxL = int(x["ctx_lens"].max())
    ws = hspec.workspace(hspec.drafter_forward_workspace(cfg, x["page_table"].shape[1], x["num_pages"], maxL))
    out = empty((B, k, cfg.d_model))
    hspec.drafter_forward(cfg, dev(shared), layers, X, out, ws, maxL)
    assert hspec.read_status(ws) == 0
    assert_close(host(out), O.drafter_forward(L, shared, x, x["caches"], cfg), f"{B} x {k}, ff {ff}")


@pytest.mark.parametrize("B,k,layers,Hkv,D,dm", [
    (1, 8, 10, 2, 128, 2048),     # a group of eight layers and a short one, both split
    (3, 16, 9, 1, 128, 1024),     # 48 rows, one tile of 128 columns a segment
    (7, 16, 2, 2, 64, 1024),      # 112 rows
    (1, 7, 3, 1, 64, 1024),       # segments of 64 rows: a product per segment, no planes
    (20, 16, 3, 4, 128, 512),     # 320 rows, unsplit
])
def test_inject_planes(B, k, layers, Hkv, D, dm):
    """Row segments under hi/lo A, and the cache append's sum of planes, to the rounding of the cache: bf16 (2^-8 of the value)
    and 1e-4 of the fp32 sums and hi/lo planes.  (With one bf16 plane of the fused rows the error is about 1e-3.)"""
    cfg = I.StepConfig(name="i", B=B, k=k, d_model=dm, H=2, P=64, N=16, G=1, chunk=16, Hq=Hkv, Hkv=Hkv, D=D,
                       lengths="uniform:0:40", n_fuse=2)
    L = I.make_lengths(cfg, 1)
    pt, pages = I.make_page_table(cfg, L + k, 1)
    W = I.make_inject_weights(cfg, 5, layers)
    h = I.normal("h", (B, k, cfg.d_h), 1.0, 5, "bf16")
    zero = np.zeros((pages, cfg.page_size, Hkv, D), np.uint16)
    caches = [dict(k_cache=zero, v_cache=zero) for _ in range(layers)]
    d = dict(W_fc=hspec.to_device(W["W_fc"]), layers=[dev(w) for w in W["layers"]])
    dc = [dev(dict(k_cache=zero.copy(), v_cache=zero.copy())) for _ in range(layers)]
    ws = hspec.workspace(hspec.kv_inject_workspace(cfg, pt.shape[1], pages))
    hspec.kv_inject(cfg, d, hspec.to_device(h), dc, hspec.to_device(pt), hspec.to_device(L), ws)
    assert hspec.read_status(ws) == 0
    ref = O.kv_inject(h, W["W_fc"], W["layers"], caches, pt, L, cfg)
    for l in range(layers):
        for name in ("k_cache", "v_cache"):
            got = I.bf16_bits_to_f32(host(dc[l][name])).astype(np.float64)
            want = np.asarray(ref[l][name], np.float64)
            assert (np.abs(got - want) <= 2.0 ** -8 * np.abs(want) + 1e-4).all(), (l, name)


@pytest.mark.parametrize("B,k,H", [(1, 16, 16), (3, 16, 16), (7, 16, 8), (10, 16, 16)])
def test_hi_lo_rows(B, k, H):
    """out_proj with hi/lo rows (32-, 64- and 128-row tiles).  What is left is the scan's S0 and C in fp16: each is off by at most
    2^-11 of itself, 2^-11 / sqrt(3) in the mean square, and the two together by less than 2^-11 of the output (2.3e-4 to
    2.6e-4 measured).  With the lo plane of the rows missing it is 2^-8 / sqrt(3) of bf16 and more: 1.7e-3 measured."""
    cfg = _cfg(B=B, k=k, H=H, precise_io=True)
    W = I.make_weights(cfg, 6)
    x = I.make_inputs(cfg, seed=6)
    d = dev(dict(h_last=x["h_last"], u=x["block_emb"]))
    ws = hspec.workspace(hspec.mamba_block_scan_workspace(cfg))
    out = empty((B, k, cfg.d_model))
    hspec.mamba_block_scan(cfg, dev(W), d["h_last"], d["u"], out, ws)
    S0, _ = O.state_init(x["h_last"], W["W_r"], W["W_dS"], cfg.H, cfg.P, cfg.N)
    ref = O.mamba_mixer(O.f64(x["block_emb"]), S0, W, cfg)
    assert_close(host(out), ref, "out", rel_l2=2.0 ** -11)
