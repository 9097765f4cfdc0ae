"""Pair attention on batches of many samples: the persistent forward kernel finds
its rows among more than one step of samples, empty ones between them, and
launches of more than 2^32 threads: the backward of one long and very many short
samples, attention over the tokens of very many."""
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


@pytest.mark.parametrize("images", [True, False])
def test_backward_one_long_and_many_short_samples(images):
    """512 and 360000 samples of one element, 12 heads: 4.3 million workgroups of
    16 waves, more than one row of a grid holds.  A sample of one element has
    weight 1, so dv = dout and the other gradients are 0; the long sample's are
    those of a batch of its own, to the bit."""
    import torch
    from paper_2609_30379_amd import binding as B
    H, n, many = 12, 512, 360000
    c, R = H * D, n * n + many
    g = torch.Generator(device="cuda").manual_seed(1)
    normal = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)     # noqa: E731
    qkv, dout, bias = normal(R, 3 * c), normal(R, c), normal(R, H)

    def run(L, rows):
        lay = B.NestedLayout(L)
        nbytes = B.attention_backward_workspace_bytes(lay, 0, H, D) if images else 8 * H * rows
        x, dqkv = qkv[:rows], torch.full((rows, 3 * c), float("nan"), dtype=torch.bfloat16, device="cuda")
        dbias = torch.full((rows, H), float("nan"), device="cuda")
        B.nt_pair_row_attention_backward(lay, 0, H, D, x[:, :c], x[:, c:2 * c], x[:, 2 * c:], dout[:rows], dqkv[:, :c],
                                         dqkv[:, c:2 * c], dqkv[:, 2 * c:], bias=bias[:rows], dbias=dbias,
                                         workspace=B.workspace_tensor(nbytes))
        return dqkv, dbias

    dqkv, dbias = run([n] + [1] * many, R)
    alone, alone_bias = run([n], n * n)
    assert torch.equal(dqkv[:n * n], alone) and torch.equal(dbias[:n * n], alone_bias)
    short = dqkv[n * n:]
    assert torch.equal(short[:, 2 * c:], dout[n * n:])
    # dS = P (dP - D) with D = P dP / P: equal up to the last bit of dP, |dP| < 64
    assert float(short[:, :2 * c].abs().max()) < 1e-3 and float(dbias[n * n:].abs().max()) < 1e-4


@pytest.mark.parametrize("axis", [2, 3])
def test_single_attention_of_very_many_samples(axis):
    """720000 samples of one token, 12 heads: 8.64 million workgroups of 8 waves.
    A sample of one token has weight 1, so o = v."""
    import torch
    from paper_2609_30379_amd import binding as B
    H, many = 12, 720000
    c = H * D
    qkv = torch.randn(many, 3 * c, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda").to(torch.bfloat16)
    out = torch.full((many, c), float("nan"), dtype=torch.bfloat16, device="cuda")
    B.nt_pair_row_attention(B.NestedLayout([1] * many), axis, H, D, qkv[:, :c], qkv[:, c:2 * c], qkv[:, 2 * c:], out)
    assert torch.equal(out, qkv[:, 2 * c:])
