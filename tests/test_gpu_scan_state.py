"""The scan over several chunks, or with a final state, at the edges of its work split: heads that
do not fill a workgroup of four, every state size, ragged last chunks, no initial state, hi/lo
storage, a final-state buffer that is not 16-byte aligned.  Operands enter the products exactly
(bf16) or as hi/lo planes (16 significant bits each product), sums are fp32: 2e-5 of the result."""
import numpy as np
import pytest

import oracle.hspec_oracle as O
from gpu_util import dev, host
from paper_2609_24197_amd import hspec, inputs as I

pytestmark = pytest.mark.gpu

CASES = [   # B, T, H, N, G, chunk, dtype, with S0
    (1, 17, 1, 128, 1, 16, "bf16", True),
    (3, 40, 3, 128, 3, 16, "bf16", True),
    (1, 33, 5, 64, 1, 16, "f32", True),
    (2, 16, 6, 16, 2, 16, "bf16", False),
    (1, 20, 7, 32, 1, 7, "f32", False),
    (5, 3, 2, 128, 1, 1, "f32", True),
    (2, 31, 12, 16, 4, 16, "f32", True),
    (1, 1, 4, 64, 1, 16, "bf16", True),
]


@pytest.mark.parametrize("case", CASES, ids=[str(c) for c in CASES])
@pytest.mark.parametrize("shift", [0, 1])
def test_scan_state(case, shift):
    import torch
    B, T, H, N, G, chunk, dtype, with_s0 = case
    s = I.make_scan_inputs(B, T, H, 64, N, G, seed=T + H, dtype=dtype, s0=with_s0)
    d = dev({k: v for k, v in s.items() if v is not None})
    code = hspec.F32 if dtype == "f32" else hspec.BF16
    ws = hspec.workspace(hspec.ssd_scan_workspace(B, T, H, 64, N, G, code))
    ny = B * T * H * 64
    ybuf = torch.full((ny + 16 * H * 64,), float("nan"), device="cuda")   # (room for a whole chunk past the end)
    y = ybuf[:ny].view(B, T, H, 64)
    n = B * H * 64 * N
    buf = torch.full((n + 8,), float("nan"), device="cuda")
    S = buf[shift:shift + n].view(B, H, 64, N)
    hspec.ssd_scan(B, T, H, 64, N, G, chunk, code, d["x"], d["dt"], d["A"], d["Bm"], d["Cm"], d["Dskip"],
                   d.get("S0"), y, S, ws)
    yr, Sr = O.ssd_sequential(s["x"], s["dt"], s["A"], s["Bm"], s["Cm"], s["Dskip"], s["S0"])
    for got, ref in ((host(y), yr), (host(S), Sr)):
        assert np.abs(got - ref).max() <= 2e-5 * max(1.0, np.abs(ref).max())
    assert torch.isnan(ybuf[ny:]).all()
    rest = host(buf)
    assert np.isnan(rest[:shift]).all() and np.isnan(rest[shift + n:]).all()   # nothing written outside
