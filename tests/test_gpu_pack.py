"""Re-tiling of packed triangle operands: channel counts on the whole-line kernel
(multiples of 64) and on the general one, lengths at the edges of a 16 x 32 tile,
operands as column slices; checked through the contraction, which reads every
position of the planes."""
import numpy as np
import pytest

from oracle import ops as O
from paper_2609_30379_amd import synth

from .gpu_util import check, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("direction", [0, 1])
@pytest.mark.parametrize("C", [32, 64, 96, 192])
def test_packed_operands(C, direction):
    import torch
    from paper_2609_30379_amd import binding as B
    L = [1, 15, 16, 0, 17, 31, 32, 33, 47]
    R = sum(n * n for n in L)
    lay = B.NestedLayout(L)
    ab = synth.normal(1, "ab", (R, 2 * C), 0.3, "bf16")
    wide = torch.full((R, 2 * C + 16), float("nan"), dtype=torch.bfloat16, device="cuda")
    wide[:, 8:8 + 2 * C] = dev(ab, "bf16")
    z = torch.zeros((R, C), dtype=torch.bfloat16, device="cuda")
    B.nt_triangle_mul(lay, direction, wide[:, 8:8 + C], wide[:, 8 + C:8 + 2 * C], z)
    ref = O.triangle_mul(ab[:, :C], ab[:, C:], L, "incoming" if direction else "outgoing")
    check(host(z), ref, "bf16", f"packed triangle C={C} direction {direction}")


def test_contraction_of_very_many_channels():
    """2560000 channels of one sample: more than 2^32 threads.  Planes of ones
    contract to N, exactly."""
    import torch
    from paper_2609_30379_amd import binding as B
    C, n = 2560000, 2
    plane = torch.ones((C, 512), dtype=torch.bfloat16, device="cuda")
    z = torch.zeros((n * n, C), dtype=torch.bfloat16, device="cuda")
    B.nt_triangle_mul(B.NestedLayout([n]), 0, plane, plane, z, operands="pair_tiled")
    assert bool((z == n).all())
