"""Pair attention on batches of many samples: the persistent forward kernel finds
its rows among more than one step of samples, empty ones between them."""
import numpy as np
import pytest

from oracle import ops as O
from paper_2609_30379_amd import synth

from .gpu_util import check, dev, host

pytestmark = pytest.mark.gpu

D = 32


def _lengths(batch, most, seed):
    """Lengths 0 .. most, a third of them empty, the first and the last among them."""
    rng = np.random.default_rng(seed)
    L = rng.integers(1, most + 1, batch) * (rng.random(batch) < 0.67)
    L[0] = L[-1] = 0
    return [int(n) for n in L]


@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("L", [
    [5, 0, 0, 0], [0, 0, 0, 7, 0], [1] * 40,              # fewer rows than workgroups
    [222, 218, 216, 40, 213, 208, 0, 209, 208],
    _lengths(63, 70, 1), _lengths(64, 70, 2), _lengths(65, 70, 3), _lengths(200, 40, 4) + [256, 0, 300],
    _lengths(4097, 9, 5),                                 # more than 64 x 64 samples
], ids=lambda L: f"{len(L)} samples")
def test_forward_many_samples(axis, L):
    import torch
    from paper_2609_30379_amd import binding as B
    H = 2
    R, c = sum(n * n for n in L), H * D
    x = synth.normal(3, "qkv", (R, 3 * c), 1.0, "bf16")
    x[:, 2 * c:] *= 0.5
    bias = synth.normal(4, "bias", (R, H), 1.0, "bf16")
    xd = dev(x, "bf16")
    out = torch.full((R, c), float("nan"), dtype=torch.bfloat16, device="cuda")
    B.nt_pair_row_attention(B.NestedLayout(L), axis, H, D, xd[:, :c], xd[:, c:2 * c], xd[:, 2 * c:], out,
                            bias=dev(np.ascontiguousarray(bias.T), "bf16"), bias_layout="heads")
    ref = O.pair_row_attention(x[:, :c], x[:, c:2 * c], x[:, 2 * c:], bias, L, H, D, axis=axis)
    check(host(out), ref, "bf16", f"attention axis {axis}, {len(L)} samples of up to {max(L)}")
