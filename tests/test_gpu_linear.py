"""Streamed products (row-major bf16 W, one plane of A), the paths beside them and fp32 operands: tile edges, remainders
and K splits against float64 (row segments and hi/lo A are in test_gpu_plane_sums.py).  The products of bf16 operands are
exact in fp32 (8 x 8 significant bits), so only the fp32 sums differ: K additions in any order are within K 2^-24 of the sum
of magnitudes."""
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


@pytest.mark.parametrize("M,N,K", [
    (1, 65536, 64), (16, 65412, 256), (17, 65540, 320), (64, 131073, 64), (64, 131076, 512), (65, 65536, 256), (96, 66000, 64),
    (128, 131072, 256), (128, 131072, 320),
])
@pytest.mark.parametrize("residual", [False, True])
def test_many_columns_short_k(M, N, K, residual):
    """Both sides of the line between the streamed tiles and the weight-streaming kernel."""
    import torch
    from paper_2609_24197_amd import hspec
    g = torch.Generator(device="cuda").manual_seed(M * 5 + N)
    A = torch.randn(M, K, generator=g, device="cuda").bfloat16()
    W = torch.randn(N, K, generator=g, device="cuda").bfloat16()
    R = torch.randn(M, N, generator=g, device="cuda") if residual else None
    guard = torch.full((M * N + 64,), float("nan"), device="cuda")
    out = guard[:M * N].view(M, N)
    ws = hspec.workspace(hspec.linear_workspace(hspec.BF16, M, N, K))
    hspec.linear(hspec.BF16, A, W, out, ws, R=R)
    ref = A.double() @ W.double().t().contiguous()
    mag = A.double().abs() @ W.double().abs().t().contiguous()
    if residual:
        ref, mag = ref + R.double(), mag + R.double().abs()
    assert ((out.double() - ref).abs() <= (K + 1) * 2.0 ** -24 * mag + 1e-30).all()
    assert guard[M * N:].isnan().all()


@pytest.mark.parametrize("M,N,K", [
    # a handful of tiles of 256 rows and more, every one split over K: whole and scalar fix-up, ragged M and N
    (256, 96, 640), (300, 98, 1024), (1000, 40, 512), (512, 256, 1536),
    # K that is no multiple of 64 (from 129 rows)
    (129, 130, 96), (300, 258, 1056), (200, 2049, 160), (513, 1028, 32),
    # more than one round of tiles: 256-row tiles with the last 8 split (ragged M and N; scalar fix-up), 128-row tiles
    (800, 16768, 1024), (800, 16766, 1024), (800, 16768, 992), (256, 33000, 256),
])
@pytest.mark.parametrize("residual", [False, True])
def test_large_tiles(M, N, K, residual):
    """The large tiles: whole tiles, tiles split over K with their fix-up, ragged edges."""
    import torch
    from paper_2609_24197_amd import hspec
    g = torch.Generator(device="cuda").manual_seed(M * 3 + N + K)
    A = torch.randn(M, K, generator=g, device="cuda").bfloat16()
    W = torch.randn(N, K, generator=g, device="cuda").bfloat16()
    R = torch.randn(M, N, generator=g, device="cuda") if residual else None
    guard = torch.full((M * N + 64,), float("nan"), device="cuda")
    out = guard[:M * N].view(M, N)
    ws = hspec.workspace(hspec.linear_workspace(hspec.BF16, M, N, K))
    hspec.linear(hspec.BF16, A, W, out, ws, R=R)
    ref = A.double() @ W.double().t().contiguous()
    mag = A.double().abs() @ W.double().abs().t().contiguous()
    if residual:
        ref, mag = ref + R.double(), mag + R.double().abs()
    assert ((out.double() - ref).abs() <= (K + 1) * 2.0 ** -24 * mag + 1e-30).all()
    assert guard[M * N:].isnan().all()


@pytest.mark.parametrize("M,N,K", [(3, 33, 64), (20, 300, 128), (60, 127, 192), (130, 698, 640), (352, 698, 640), (520, 1030, 256),
                                   (16, 256, 4096), (300, 130, 2048)])
def test_streamed_product_over_its_residual(M, N, K):
    """C in the memory of R, products of one part and of several: every result reads its own residual before it is
    stored; nothing past C is written."""
    import torch
    from paper_2609_24197_amd import hspec
    g = torch.Generator(device="cuda").manual_seed(M + N)
    A = torch.randn(M, K, generator=g, device="cuda").bfloat16()
    W = torch.randn(N, K, generator=g, device="cuda").bfloat16()
    R = torch.randn(M, N, generator=g, device="cuda")
    ws = hspec.workspace(hspec.linear_workspace(hspec.BF16, M, N, K))
    ref = torch.empty(M, N, device="cuda")
    hspec.linear(hspec.BF16, A, W, ref, ws, R=R)
    guard = torch.full((M * N + 64,), float("nan"), device="cuda")
    out = guard[:M * N].view(M, N)
    out.copy_(R)
    hspec.linear(hspec.BF16, A, W, out, ws, R=out)
    assert torch.equal(out, ref)
    assert guard[M * N:].isnan().all()
    exact = A.double() @ W.double().t().contiguous() + R.double()
    mag = A.double().abs() @ W.double().abs().t().contiguous() + R.double().abs()
    assert ((ref.double() - exact).abs() <= (K + 1) * 2.0 ** -24 * mag + 1e-30).all()


@pytest.mark.parametrize("M,N,K", [
    (1, 8, 8), (3, 15, 40), (16, 16, 256), (17, 40, 264), (32, 272, 1000), (33, 33, 2048), (64, 1030, 520),
    (65, 260, 72), (129, 130, 1000), (260, 300, 64),
])
def test_fp32_product(M, N, K):
    """fp32 operands read in place, split into hi/lo planes on chip: each element keeps all but 2^-18 of itself,
    the lo x lo term (2^-18) is left out, and 3 K terms are added in fp32."""
    import torch
    from paper_2609_24197_amd import hspec
    g = torch.Generator(device="cuda").manual_seed(M * 11 + N)
    A = torch.randn(M, K, generator=g, device="cuda")
    W = torch.randn(N, K, generator=g, device="cuda")
    R = torch.randn(M, N, generator=g, device="cuda")
    guard = torch.full((M * N + 64,), float("nan"), device="cuda")
    out = guard[:M * N].view(M, N)
    ws = hspec.workspace(hspec.linear_workspace(hspec.F32, M, N, K))
    ref = A.double() @ W.double().t().contiguous() + R.double()
    mag = A.double().abs() @ W.double().abs().t().contiguous() + R.double().abs()
    hspec.linear(hspec.F32, A, W, out, ws, R=R)
    assert ((out.double() - ref).abs() <= (3 * 2.0 ** -18 + (3 * K + 1) * 2.0 ** -24) * mag).all()
    assert guard[M * N:].isnan().all()


@pytest.mark.parametrize("M,N,K", [
    # several groups of 64 rows of 16-column tiles, up to the last that still takes them
    (65, 16, 2048), (127, 40, 264), (220, 64, 520), (400, 2040, 72), (1000, 33, 1032), (3000, 17, 40),
    # one column tile more: 128 x 128 tiles; up to 128 rows: 128 x 256; up to 64 rows with two k-steps: 64 x 256
    (400, 2049, 72), (300, 2890, 264), (100, 7300, 136), (40, 131100, 64),
])
@pytest.mark.parametrize("residual", [False, True])
def test_fp32_product_of_many_rows(M, N, K, residual):
    """The bound of test_fp32_product on both sides of the line between the 16-column tiles and the large ones."""
    import torch
    from paper_2609_24197_amd import hspec
    g = torch.Generator(device="cuda").manual_seed(M * 13 + N)
    A = torch.randn(M, K, generator=g, device="cuda")
    W = torch.randn(N, K, generator=g, device="cuda")
    R = torch.randn(M, N, generator=g, device="cuda") if residual else None
    guard = torch.full((M * N + 64,), float("nan"), device="cuda")
    out = guard[:M * N].view(M, N)
    ws = hspec.workspace(hspec.linear_workspace(hspec.F32, M, N, K))
    hspec.linear(hspec.F32, A, W, out, ws, R=R)
    ref = A.double() @ W.double().t().contiguous()
    mag = A.double().abs() @ W.double().abs().t().contiguous()
    if residual:
        ref, mag = ref + R.double(), mag + R.double().abs()
    assert ((out.double() - ref).abs() <= (3 * 2.0 ** -18 + (3 * K + 1) * 2.0 ** -24) * mag).all()
    assert guard[M * N:].isnan().all()


@pytest.mark.parametrize("M,K", [(5, 40), (64, 64), (100, 128), (300, 264)])
@pytest.mark.parametrize("over", ["A", "W"])
def test_fp32_product_over_an_operand(M, K, over):
    """C in the memory of A (N == K) or of W (M == N == K): the result of the call with a C of its own."""
    import torch
    from paper_2609_24197_amd import hspec
    N = K
    M = M if over == "A" else K
    g = torch.Generator(device="cuda").manual_seed(M + K)
    A = torch.randn(M, K, generator=g, device="cuda")
    W = torch.randn(N, K, generator=g, device="cuda")
    ws = hspec.workspace(hspec.linear_workspace(hspec.F32, M, N, K))
    ref = torch.empty(M, N, device="cuda")
    hspec.linear(hspec.F32, A, W, ref, ws)
    hspec.linear(hspec.F32, A, W, A if over == "A" else W, ws)
    assert torch.equal(A if over == "A" else W, ref)
