"""Pair attention backward on every instance and edge of its tiles: the 4-, 8-
and 16-wave row kernels (longest sample up to 128, up to the LDS of two
workgroups per CU, beyond), tile and 32-row step remainders, both axes, and a
workspace with and without room for the bias images."""
import numpy as np
import pytest

from oracle import grads as G
from paper_2609_30379_amd import synth

from .gpu_util import dev, host
from .test_gpu_backward import check_grad

pytestmark = pytest.mark.gpu

D = 32
CASES = [
    ([1, 15, 16, 17], 3),              # single tiles and one key past a tile
    ([31, 32, 33, 0, 64, 65], 2),      # 32-row steps and 64-key blocks
    ([127, 128], 1),                   # the 4-wave instance at its limit
    ([129, 5, 161], 2),                # the 8-wave instance
    ([330], 1),                        # the 16-wave instance
    ([512, 1], 1),                     # its longest sample: most LDS, eight row chunks
]


@pytest.mark.parametrize("images", [True, False])
@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("L,H", CASES)
def test_attention_backward_paths(axis, L, H, images):
    import torch
    from paper_2609_30379_amd import binding as B
    lay = B.NestedLayout(L)
    R, c = sum(n * n for n in L), H * D
    qkv = synth.normal(5, "q", (R, 3 * c), 1.0, "bf16")
    bias = synth.normal(6, "b", (R, H), 1.0, "bf16")
    dout = synth.normal(7, "d", (R, c), 1.0, "bf16")
    qd, bd = dev(qkv, "bf16"), dev(bias, "bf16")
    # the smallest accepted workspace holds the softmax statistics alone
    nbytes = B.attention_backward_workspace_bytes(lay, axis, H, D) if images else 8 * H * R
    dqkv = torch.full((R, 3 * c), float("nan"), dtype=torch.bfloat16, device="cuda")
    dbias = torch.full((R, H), float("nan"), device="cuda")
    outs = []
    for _ in range(2):
        B.nt_pair_row_attention_backward(lay, axis, H, D, qd[:, :c], qd[:, c:2 * c], qd[:, 2 * c:], dev(dout, "bf16"),
                                         dqkv[:, :c], dqkv[:, c:2 * c], dqkv[:, 2 * c:], bias=bd, dbias=dbias,
                                         workspace=B.workspace_tensor(nbytes))
        outs.append((dqkv.clone(), dbias.clone()))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
    rq, rk, rv, rb = G.pair_row_attention_backward(qkv[:, :c], qkv[:, c:2 * c], qkv[:, 2 * c:], bias, dout, L, H, D,
                                                   axis=axis)
    what = f"attention backward axis {axis} L={L} H={H} images {images}"
    got = host(dqkv)
    check_grad(got[:, :c], rq, what + " dq")
    check_grad(got[:, c:2 * c], rk, what + " dk")
    check_grad(got[:, 2 * c:], rv, what + " dv")
    # fp32 throughout: sums of N terms of order max |dB|, 2^-24 each, and the
    # native exponential's 2^-22: far inside 1e-5 of the largest gradient
    err = np.max(np.abs(host(dbias) - rb)) / np.max(np.abs(rb))
    assert err <= 1e-5, f"{what} dbias: {err:.3g}"
