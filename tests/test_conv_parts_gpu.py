"""The conv backward where its blocks and its weight-gradient sum change: channel counts
around a block of 256 (64 groups of 4), token counts around a run of 16 and a block of 64,
and numbers of parts around the 4 groups and the 8-deep sum of one group.

Tolerances, against max(|element|, rms of the tensor): a term is accurate to about 2e-6 (the
fast exponential and reciprocal of the sigmoid, four products), and a weight gradient is an
fp32 sum of at most 64 x 33 such terms in chains of at most 16 + 4 + 66, so at most 1e-5
of the sum of magnitudes, which is within 10 of the scale for sums of mixed sign of this
length: 1e-4.  dx in bf16 is rounded to 2^-9 of itself: 2^-8.
"""
import numpy as np
import pytest

import kla_inputs as K
from kla_testutil import rel_err, to_np, to_torch
from oracle import block as OB

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,C", [
    (1, 1, 8), (1, 19, 248), (3, 64, 256), (2, 65, 264), (1, 257, 520), (5, 79, 16), (33, 18, 40), (8, 131, 8)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_conv_backward_edges(B, T, C, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_10743_amd as kla
    g = np.random.default_rng(B + T + C)
    x, du = (K.quantise(g.standard_normal((B, T, C)), dtype) for _ in range(2))
    w = g.standard_normal((C, 4)).astype(np.float32).astype(np.float64)
    bias = g.standard_normal(C).astype(np.float32).astype(np.float64)
    dev = lambda a: torch.tensor(a, dtype=torch.float32, device="cuda:0")
    dx, dw, db = kla.kla_conv_silu_backward(to_torch(x, dtype, "cuda:0"), dev(w), dev(bias), to_torch(du, dtype, "cuda:0"))
    rx, rw, rb = OB.conv_silu_backward(x, w, bias, du)
    assert rel_err(to_np(dx), rx, 1.0) <= (2.0 ** -8 if dtype == "bf16" else 1e-4)
    assert rel_err(to_np(dw), rw, 1.0) <= 1e-4
    assert rel_err(to_np(db), rb, 1.0) <= 1e-4
