"""Pair attention on batches with samples longer than 512: the row kernel's
8- and 16-wave instances at the edges of their LDS (640, 641, 1024 keys) and of
a 64-key chunk, shorter samples of the same batch on the persistent kernel, with
and without bias and gate, masked keys, and a call without room for the bias
image."""
import numpy as np
import pytest

from oracle import ops as O
from paper_2609_30379_amd import synth

from .gpu_util import check, dev, host

pytestmark = pytest.mark.gpu

D = 32


def _run(L, H, axis, bias=True, gate=False, masked=False, image=True, scale=None):
    import torch
    from paper_2609_30379_amd import binding as B
    lay = B.NestedLayout(L)
    R, c = sum(n * n for n in L), H * D
    x = synth.normal(3, "qkvg", (R, 4 * c), 1.0, "bf16")
    x[:, 2 * c:3 * c] *= 0.5
    bv = synth.normal(4, "bias", (R, H), 1.0, "bf16") if bias else None
    if masked:                                 # whole leading chunks of keys, then single keys; never the last key
        o = 0
        for n in L:
            b = bv[o:o + n * n].reshape(n, n, H)
            k = slice(0, n - 1)
            m = np.zeros((n, n), bool)
            m[:, :min(130, n - 1)] = True
            m[:, k] |= np.random.default_rng(n).random((n, n - 1)) < 0.2
            b[(m if axis == 0 else m.T)] = -np.inf
            o += n * n
    xd = dev(x, "bf16")
    out = torch.full((R, c), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = None if image else torch.empty(16, dtype=torch.uint8, device="cuda")
    call = lambda: B.nt_pair_row_attention(lay, axis, H, D, xd[:, :c], xd[:, c:2 * c], xd[:, 2 * c:3 * c], out,  # noqa: E731
                                           bias=dev(np.ascontiguousarray(bv.T), "bf16") if bias else None,
                                           bias_layout="heads", workspace=ws, gate=xd[:, 3 * c:] if gate else None, scale=scale)
    call()
    first = host(out)
    call()
    assert np.array_equal(host(out), first)
    ref = O.pair_row_attention(x[:, :c], x[:, c:2 * c], x[:, 2 * c:3 * c], bv, L, H, D, axis=axis, scale=scale,
                               gate=x[:, 3 * c:] if gate else None)
    check(first, ref, "bf16", f"long pair attention axis {axis} {L} H={H} bias {bias} gate {gate} masked {masked} image {image}")


@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("L,H,kw", [
    ([513, 0, 40, 300], 3, {}),
    ([577, 16], 1, dict(gate=True)),           # one key past a chunk
    ([640, 40], 1, dict(masked=True)),
    ([641, 1], 1, dict(gate=True)),            # the 16-wave instance
    ([530, 65], 1, dict(bias=False)),
    ([520, 33], 1, dict(image=False)),
    ([514, 20], 1, dict(scale=0.0)),           # the bias image cannot be divided by these scales
    ([514, 20], 1, dict(scale=-0.2, gate=True)),
    ([514, 20], 1, dict(scale=0.0, bias=False)),
])
def test_long_pair_attention(axis, L, H, kw):
    _run(L, H, axis, **kw)


def test_longest_pair_attention():
    _run([1024], 1, 0)
