"""KV injection over layer groups: one layer, more than one group of eight, row segments that do and do not
fill column tiles, few and many rows, both storages; unmapped positions and bad pages are flagged and
skipped, every other slot keeps its value."""
import numpy as np
import pytest

import oracle.hspec_oracle as O
from gpu_util import dev, host
from paper_2609_24197_amd import hspec, inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,k,layers,Hkv,D,dm,dtype", [
    (1, 1, 1, 1, 64, 64, "bf16"), (3, 5, 9, 2, 64, 128, "bf16"), (2, 16, 3, 1, 128, 192, "bf16"),
    (20, 16, 8, 2, 128, 256, "bf16"), (4, 4, 10, 3, 64, 72, "bf16"), (2, 3, 9, 1, 64, 64, "f32"),
])
def test_inject_groups(B, k, layers, Hkv, D, dm, dtype):
    cfg = I.StepConfig(name="i", B=B, k=k, d_model=dm, H=2, P=64, N=16, G=1, chunk=16, Hq=Hkv, Hkv=Hkv, D=D, dtype=dtype,
                       lengths="uniform:0:40", n_fuse=2)
    L = I.make_lengths(cfg, 1)
    pt, pages = I.make_page_table(cfg, L + k, 1, extra_pages=2)
    W = I.make_inject_weights(cfg, 1, layers)
    h = I.normal("h", (B, k, cfg.d_h), 1.0, 1, dtype)
    shape = (pages, cfg.page_size, Hkv, D)
    caches = [dict(k_cache=I.normal(f"k{i}", shape, 1.0, 1, dtype), v_cache=I.normal(f"v{i}", shape, 1.0, 1, dtype))
              for i in range(layers)]
    d = dict(W_fc=hspec.to_device(W["W_fc"]), layers=[dev(w) for w in W["layers"]])
    dc = [dev(c) for c in caches]
    ws = hspec.workspace(hspec.kv_inject_workspace(cfg, pt.shape[1], pages))
    hspec.kv_inject(cfg, d, hspec.to_device(h), dc, hspec.to_device(pt), hspec.to_device(L), ws)
    assert hspec.read_status(ws) == 0
    ref = O.kv_inject(h, W["W_fc"], W["layers"], caches, pt, L, cfg)
    written = {int(pt[b, (L[b] + i) // 16]) * 16 + (int(L[b]) + i) % 16 for b in range(B) for i in range(k)}
    rest = np.array([s for s in range(pages * 16) if s not in written])
    f = (lambda a: np.asarray(a, np.float64)) if dtype == "f32" else (lambda a: I.bf16_bits_to_f32(a).astype(np.float64))
    for l in range(layers):
        for name in ("k_cache", "v_cache"):
            got, old = f(host(dc[l][name])), f(caches[l][name])
            want = np.asarray(ref[l][name], np.float64)
            # bf16: the result's own rounding (2^-9 of it) and the operands' hi/lo planes; fp32: the planes
            tol = (2.0 ** -8 if dtype == "bf16" else 2e-4) * np.maximum(1.0, np.abs(want))
            assert (np.abs(got - want) <= tol).all(), (l, name)
            assert np.array_equal(got.reshape(pages * 16, -1)[rest], old.reshape(pages * 16, -1)[rest])


def test_inject_flags_and_skips():
    cfg = I.StepConfig(name="i", B=3, k=4, d_model=64, H=2, P=64, N=16, G=1, chunk=16, Hq=1, Hkv=1, D=64,
                       lengths="list:3,14,30")
    L = np.array([3, 14, 30], np.int32)
    pt = np.array([[0, 1], [2, 9], [3, 4]], np.int32)      # request 1 runs into a page outside the pool,
    pages = 5                                              # request 2 past the table
    W = I.make_inject_weights(cfg, 2, 2)
    caches = [dict(k_cache=I.normal(f"k{i}", (pages, 16, 1, 64), 1.0, 2, "bf16"),
                   v_cache=I.normal(f"v{i}", (pages, 16, 1, 64), 1.0, 2, "bf16")) for i in range(2)]
    d = dict(W_fc=hspec.to_device(W["W_fc"]), layers=[dev(w) for w in W["layers"]])
    dc = [dev(c) for c in caches]
    ws = hspec.workspace(hspec.kv_inject_workspace(cfg, 2, pages))
    h = I.normal("h", (3, 4, cfg.d_h), 1.0, 2, "bf16")
    hspec.kv_inject(cfg, d, hspec.to_device(h), dc, hspec.to_device(pt), hspec.to_device(L), ws)
    assert hspec.read_status(ws) == hspec.DEV_BAD_PAGE | hspec.DEV_BAD_CTX_LEN
    written = {3, 4, 5, 6, 2 * 16 + 14, 2 * 16 + 15, 4 * 16 + 14, 4 * 16 + 15}
    for l in range(2):
        changed = (host(dc[l]["k_cache"]).reshape(80, -1) != caches[l]["k_cache"].reshape(80, -1)).any(1)
        assert set(np.nonzero(changed)[0]) == written


@pytest.mark.parametrize("length", [2**31 - 1, 2**31 - 3, 32, 29, -1, -2**31])
def test_inject_length_past_the_table(length):
    """A length whose new positions lie past a table of 32 positions, up to the largest int32 (where length + i has no
    int32): flagged, and only the mapped positions written."""
    cfg = I.StepConfig(name="i", B=1, k=4, d_model=64, H=2, P=64, N=16, G=1, chunk=16, Hq=1, Hkv=1, D=64, lengths="list:3")
    pt, pages = np.array([[2, 1]], np.int32), 3
    W = I.make_inject_weights(cfg, 2, 1)
    cache = dict(k_cache=I.normal("k", (pages, 16, 1, 64), 1.0, 2, "bf16"), v_cache=I.normal("v", (pages, 16, 1, 64), 1.0, 2, "bf16"))
    d = dict(W_fc=hspec.to_device(W["W_fc"]), layers=[dev(w) for w in W["layers"]])
    dc = dev(cache)
    ws = hspec.workspace(hspec.kv_inject_workspace(cfg, 2, pages))
    h = I.normal("h", (1, 4, cfg.d_h), 1.0, 2, "bf16")
    hspec.kv_inject(cfg, d, hspec.to_device(h), [dc], hspec.to_device(pt), hspec.to_device(np.array([length], np.int32)), ws)
    assert hspec.read_status(ws) == hspec.DEV_BAD_CTX_LEN
    changed = (host(dc["k_cache"]).reshape(48, -1) != cache["k_cache"].reshape(48, -1)).any(1)
    assert set(np.nonzero(changed)[0]) == ({16 + 13, 16 + 14, 16 + 15} if length == 29 else set())


@pytest.mark.parametrize("share", ["layers", "k_and_v", "interleaved"])
@pytest.mark.parametrize("layers,Hkv,D", [(2, 1, 64), (3, 3, 64), (8, 2, 128), (9, 5, 128)])
def test_inject_caches_that_share_memory(share, layers, Hkv, D):
    """Caches that share memory are written in the order of the layers, k before v: one cache for all layers keeps the
    last layer's rows, one tensor for k and v keeps v, and pools that overlap without a common slot keep all."""
    import torch
    B, k = 3, 5
    cfg = I.StepConfig(name="i", B=B, k=k, d_model=64, H=2, P=64, N=16, G=1, chunk=16, Hq=Hkv, Hkv=Hkv, D=D,
                       lengths="list:3,14,30")
    L = I.make_lengths(cfg, 1)
    pt, pages = I.make_page_table(cfg, L + k, 1)
    W = I.make_inject_weights(cfg, 3, layers)
    d = dict(W_fc=hspec.to_device(W["W_fc"]), layers=[dev(w) for w in W["layers"]])
    h = hspec.to_device(I.normal("h", (B, k, cfg.d_h), 1.0, 3, "bf16"))
    lens = hspec.to_device(L)

    def inject(caches, table, npages):
        ws = hspec.workspace(hspec.kv_inject_workspace(cfg, table.shape[1], npages))
        hspec.kv_inject(cfg, d, h, caches, hspec.to_device(table), lens, ws)
        assert hspec.read_status(ws) == 0

    zeros = lambda n: torch.zeros(n, 16, Hkv, D, dtype=torch.bfloat16, device="cuda")  # noqa: E731
    own = [dict(k_cache=zeros(pages), v_cache=zeros(pages)) for _ in range(layers)]
    inject(own, pt, pages)
    if share == "layers":
        one = dict(k_cache=zeros(pages), v_cache=zeros(pages))
        inject([one] * layers, pt, pages)
        assert torch.equal(one["k_cache"], own[-1]["k_cache"]) and torch.equal(one["v_cache"], own[-1]["v_cache"])
    elif share == "k_and_v":
        ts = [zeros(pages) for _ in range(layers)]
        inject([dict(k_cache=t, v_cache=t) for t in ts], pt, pages)
        assert all(torch.equal(t, c["v_cache"]) for t, c in zip(ts, own))
    else:                       # page p of cache i is page p * n + i of one pool (the tail keeps the ranges inside it)
        n = 2 * layers
        pool = zeros(2 * pages * n)
        view = [pool[i:i + pages * n] for i in range(n)]
        inject([dict(k_cache=view[2 * l], v_cache=view[2 * l + 1]) for l in range(layers)], pt * n, pages * n)
        for l in range(layers):
            assert torch.equal(pool[2 * l:pages * n:n], own[l]["k_cache"])
            assert torch.equal(pool[2 * l + 1:pages * n:n], own[l]["v_cache"])
