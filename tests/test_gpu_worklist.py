"""Work list of the KV sweep at the edges of its request counts: several lanes per request and one,
remainders of four (the requests are read four at a time), more than one pass of the workgroup, and past
the ranked range.  Ragged lengths with ties and empty contexts, against the oracle."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from gpu_util import assert_close  # noqa: E402
from paper_2609_24197_amd import inputs as I  # noqa: E402
from test_gpu_primitives import _ref_attn, _run_attn, _small_attn_cfg  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("split", [0, 64])
@pytest.mark.parametrize("B", [1, 3, 5, 64, 129, 255, 257, 514, 4097])
def test_requests(B, split):
    lens = [(37 * i * i + 11 * i) % (290 if B < 600 else 70) if i % 3 else 150 for i in range(B)]
    cfg = _small_attn_cfg(B=B, k=2, Hq=2, Hkv=1, D=64, lengths="list:" + ",".join(map(str, lens)))
    x = I.make_attn_inputs(cfg, seed=B)
    o, st = _run_attn(cfg, x, split=split)
    assert st == 0
    assert_close(o, _ref_attn(cfg, x), f"{B} requests, split {split}")
