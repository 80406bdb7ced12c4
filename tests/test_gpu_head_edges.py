"""The rank-256 Markov step at the edges of its tiles: requests that do not fill a block of 16 or a tile
of 64, vocabularies that do not fill a workgroup's 128 columns, forced positions (one launch), ties, NaN
scores, and no write outside the logits."""
import pytest

from paper_2609_24197_amd import hspec, inputs as I

pytestmark = pytest.mark.gpu


def _run(B, k, V, mode, seed=0):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed + B * 31 + V)
    cfg = I.StepConfig(name="h", B=B, k=k, d_model=64, H=2, P=64, N=16, G=1, chunk=16, Hq=4, Hkv=1, D=64, lengths="fixed:1")
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    W = dict(norm_f_w=1 + 0.1 * r(64), W_lm=(r(V, 64) / 8).bfloat16(), E_M=r(V, 256).bfloat16(),
             U_M=(r(V, 256) / 16).bfloat16())
    x = dict(hidden=r(B, k, 64), prev=torch.randint(0, V, (B,), generator=g, device="cuda", dtype=torch.int32))
    forced = torch.randint(0, V, (B, k), generator=g, device="cuda", dtype=torch.int32) if mode == "forced" else None
    gumbel = -torch.log(-torch.log(torch.rand(B, k, V, generator=g, device="cuda").clamp(1e-6, 1 - 1e-6))) \
        if mode == "gumbel" else None
    hc = hspec.head_cfg(cfg, V, 256, 0.7)
    ws = hspec.workspace(hspec.draft_head_workspace(hc))
    tok = torch.full((B, k), -1, dtype=torch.int32, device="cuda")
    n = B * k * V
    buf = torch.full((n + 64,), float("nan"), device="cuda")
    logits = buf[:n].view(B, k, V)
    hspec.draft_head(hc, W, x["hidden"], x["prev"], tok, ws, logits=logits, gumbel=gumbel, forced=forced)
    assert hspec.read_status(ws) == 0
    assert torch.isnan(buf[n:]).all()
    tok2 = torch.full((B, k), -1, dtype=torch.int32, device="cuda")   # without the logits output
    hspec.draft_head(hc, W, x["hidden"], x["prev"], tok2, ws, gumbel=gumbel, forced=forced)
    assert torch.equal(tok, tok2)
    return W, x, forced, gumbel, tok, logits


@pytest.mark.parametrize("mode", ["greedy", "gumbel", "forced"])
@pytest.mark.parametrize("B,k,V", [(1, 1, 1), (1, 3, 129), (15, 2, 128), (17, 3, 1000), (64, 2, 384), (65, 2, 260),
                                   (130, 3, 97)])
def test_markov_edges(B, k, V, mode):
    import torch
    W, x, forced, gumbel, tok, logits = _run(B, k, V, mode)
    h = x["hidden"].double()
    hn = h / torch.sqrt((h * h).mean(-1, keepdim=True) + 1e-6) * W["norm_f_w"].double()
    follow = forced if forced is not None else tok        # the chain the device followed
    prev = torch.cat([x["prev"][:, None], follow[:, :-1]], 1).long()
    ref = hn @ W["W_lm"].double().t().contiguous() + W["E_M"][prev].double() @ W["U_M"].double().t().contiguous()
    # the normalised hidden state enters as one bf16 plane: 2^-9 of each of 64 terms of size ~ 1 / 8
    assert (logits.double() - ref).abs().max() < 2e-2
    score = logits / 0.7 + gumbel if gumbel is not None else logits
    best = score.max(-1).values
    got = score.gather(-1, tok.long()[..., None])[..., 0]
    assert torch.all(got >= best - 1e-5)                  # (the noise is added in another rounding)
    if gumbel is None:
        assert torch.equal(tok.long(), (logits == best[..., None]).int().argmax(-1))   # lowest column of a tie


def test_markov_ties_and_nan():
    import torch
    B, k, V = 5, 2, 300
    cfg = I.StepConfig(name="h", B=B, k=k, d_model=64, H=2, P=64, N=16, G=1, chunk=16, Hq=4, Hkv=1, D=64, lengths="fixed:1")
    W = dict(norm_f_w=torch.ones(64, device="cuda"), W_lm=torch.zeros(V, 64, device="cuda").bfloat16(),
             E_M=torch.zeros(V, 256, device="cuda").bfloat16(), U_M=torch.zeros(V, 256, device="cuda").bfloat16())
    hc = hspec.head_cfg(cfg, V, 256)
    ws = hspec.workspace(hspec.draft_head_workspace(hc))
    tok = torch.full((B, k), -1, dtype=torch.int32, device="cuda")
    prev = torch.zeros(B, dtype=torch.int32, device="cuda")
    hidden = torch.ones(B, k, 64, device="cuda")
    hspec.draft_head(hc, W, hidden, prev, tok, ws)
    assert (tok == 0).all() and hspec.read_status(ws) == 0
    W["W_lm"][7] = float("nan")                            # a NaN score counts as -inf and is flagged
    W["W_lm"][200] = 1.0
    hspec.draft_head(hc, W, hidden, prev, tok, ws)
    assert (tok == 200).all() and hspec.read_status(ws) == hspec.DEV_NONFINITE
