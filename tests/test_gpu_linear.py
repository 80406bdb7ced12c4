"""Streamed products (row-major bf16 W): tile edges, remainders, K splits and segments against
float64.  The products are exact in fp32 (8 x 8 significant bits), so only the fp32 sums differ:
K additions in any order are within K 2^-24 of the sum of magnitudes."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [
    (1, 4, 64), (7, 129, 64), (16, 128, 4096), (31, 260, 192), (32, 6144, 256), (33, 127, 320), (63, 1028, 4160),
    (64, 512, 2048), (65, 130, 128), (112, 4096, 1024), (127, 6320, 4096), (128, 4096, 12288), (129, 388, 448),
    (217, 6144, 512), (255, 4100, 1088), (256, 4096, 4096), (257, 260, 4096), (512, 4096, 3072), (1000, 4096, 256),
    (1024, 4224, 64),
])
@pytest.mark.parametrize("residual", [False, True])
def test_streamed_product(M, N, K, residual):
    import torch
    from paper_2609_24197_amd import hspec
    g = torch.Generator(device="cuda").manual_seed(M * 7 + N)
    A = torch.randn(M, K, generator=g, device="cuda").bfloat16()
    W = torch.randn(N, K, generator=g, device="cuda").bfloat16()
    R = torch.randn(M, N, generator=g, device="cuda") if residual else None
    out = torch.full((M, N), float("nan"), device="cuda")
    ws = hspec.workspace(hspec.linear_workspace(hspec.BF16, M, N, K))
    ref = A.double() @ W.double().t().contiguous()
    mag = A.double().abs() @ W.double().abs().t().contiguous()
    if residual:
        ref, mag = ref + R.double(), mag + R.double().abs()
    hspec.linear(hspec.BF16, A, W, out, ws, R=R)
    first = out.clone()
    assert ((out.double() - ref).abs() <= (K + 1) * 2.0 ** -24 * mag + 1e-30).all()
    out.fill_(float("nan"))
    hspec.linear(hspec.BF16, A, W, out, ws, R=R)
    assert torch.equal(out, first)   # one order of sums
