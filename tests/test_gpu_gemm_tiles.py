"""The large-K product on each of its tile sizes (64 with K split, 64, 128, 256)
with remainders in rows, channels and K (a last stage of 32, an odd number of
64-wide steps), every epilogue, and GELU over its range."""
import math

import numpy as np
import pytest

from oracle import numerics as NU
from oracle import ops as O
from paper_2609_30379_amd import synth

from .gpu_util import check, dev, host

pytestmark = pytest.mark.gpu

SIZES = [
    (1, 384, 8), (65, 416, 72), (64, 3072, 768),     # 64-wide tiles, K split between two wave sets
    (513, 416, 1544),                                # 64-wide
    (1700, 416, 2312),                               # 128-wide
    (4000, 448, 2312),                               # 256-wide
]


@pytest.mark.parametrize("epi", ["none", "gelu", "residual"])
@pytest.mark.parametrize("R,K,N", SIZES)
def test_gemm_tiles(R, K, N, epi):
    import torch
    from paper_2609_30379_amd import binding as B
    x = synth.normal(1, "x", (R, K), 1.0, "bf16")
    w = synth.normal(2, "w", (N, K), 0.5 / math.sqrt(K), "bf16")
    b = synth.normal(3, "b", (N,), 0.1)
    g, be = synth.normal(4, "g", (K,), 0.1, loc=1.0), synth.normal(5, "be", (K,), 0.1)
    res = synth.normal(6, "r", (R, N), 1.0, "bf16") if epi == "residual" else None
    y = torch.full((R, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    B.nt_layernorm_linear(dev(x, "bf16"), dev(w, "bf16"), dev(b, "f32"), y, ln=(dev(g, "f32"), dev(be, "f32")),
                          epilogue=epi, residual=None if res is None else dev(res, "bf16"))
    # the rows enter the product rounded to bf16
    xn = NU.round_bf16(NU.layernorm(x, g, be))
    p = O.layernorm_linear(xn, w, b, epilogue=epi, residual=res)
    check(host(y), p, "bf16", f"product {R}x{K}->{N} {epi}")


@pytest.mark.parametrize("R", [64, 704])
def test_gelu_over_its_range(R):
    """y = GELU(x) through an identity product, against x erfc(-x / sqrt 2) / 2:
    one bf16 rounding (2^-9 of the value) plus fp32 errors far below it;
    infinities and NaN that a bias brings in: GELU is inf, 0 and NaN there.
    64 rows run on the small-row kernel; 704 rows are 44 x 6 of its blocks, more
    than the CUs, and run on the large-K product."""
    import torch
    from paper_2609_30379_amd import binding as B
    K = 384
    x = np.concatenate([np.linspace(-12, 12, R * K - 2), [0.0, -0.0]])
    x = synth.snap_bf16(x.astype(np.float32)).reshape(-1, K)
    y = torch.empty(x.shape, dtype=torch.bfloat16, device="cuda")
    B.nt_layernorm_linear(dev(x, "bf16"), dev(np.eye(K), "bf16"), None, y, epilogue="gelu")
    got, ref = host(y), 0.5 * x * np.vectorize(math.erfc)(-x / math.sqrt(2))
    # 2^-8: half an ulp is at most 2^-8 of the smaller end of a binade
    assert np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-30)
    b = np.zeros(K)
    b[:3] = [np.inf, np.nan, -np.inf]
    B.nt_layernorm_linear(dev(np.zeros_like(x), "bf16"), dev(np.eye(K), "bf16"), dev(b, "f32"), y, epilogue="gelu")
    got = host(y)
    assert np.all(np.isposinf(got[:, 0])) and np.all(np.isnan(got[:, 1])) and np.all(got[:, 2:] == 0)
