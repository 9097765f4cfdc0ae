"""Pair attention where the bias leaves the ordinary range: finite masks from
-1e9 to the lowest bf16 value on whole leading chunks of keys and on whole rows,
and -inf on leading chunks, for samples on each side of 256 and of 512 keys (axes
0 and 1) and for single attention (axis 3)."""
import functools

import numpy as np
import pytest

from oracle import ops as O
from paper_2609_30379_amd import synth

from .gpu_util import check, dev, host

pytestmark = pytest.mark.gpu

D = 32
LOWEST = -3.3895313892515355e38                # the lowest finite bf16 value
MASKS = [-1e9, -1e12, -1e15, -1e20, -1e30, -1e32, -5e37, -1e38, -2e38, LOWEST, -np.inf]


def _call(L, H, axis, x, bv, scale=None, gate=False):
    import torch
    from paper_2609_30379_amd import binding as B
    c = H * D
    xd = dev(x, "bf16")
    out = torch.full((x.shape[0], c), float("nan"), dtype=torch.bfloat16, device="cuda")
    B.nt_pair_row_attention(B.NestedLayout(L), axis, H, D, xd[:, :c], xd[:, c:2 * c], xd[:, 2 * c:3 * c], out,
                            bias=None if bv is None else dev(np.ascontiguousarray(bv.T), "bf16"), bias_layout="heads",
                            scale=scale, gate=xd[:, 3 * c:] if gate else None)
    return host(out)


def _reference(L, H, axis, x, bv, scale=None, gate=False):
    c = H * D
    if axis == 3:
        return O.single_attention_pair_bias(x[:, :c], x[:, c:2 * c], x[:, 2 * c:3 * c], bv, L, H, D, scale=scale)
    return O.pair_row_attention(x[:, :c], x[:, c:2 * c], x[:, 2 * c:3 * c], bv, L, H, D, axis=axis, scale=scale,
                                gate=x[:, 3 * c:] if gate else None)


def _inputs(L, H, axis):
    rows = sum(L) if axis == 3 else sum(n * n for n in L)
    x = synth.normal(3, "qkvg", (rows, 4 * H * D), 1.0, "bf16")
    x[:, 2 * H * D:3 * H * D] *= 0.5
    return x, synth.normal(4, "bias", (sum(n * n for n in L), H), 1.0, "bf16")


def _masks(L, axis):
    """Cells under the mask: `lead` the first 130 keys (never the last key),
    `whole` every key of each fifth query; `rows` the packed rows of those
    queries."""
    lead, whole, rows = [], [], []
    for n in L:
        q = np.arange(n) % 5 == 4
        m, w = np.zeros((n, n), bool), np.zeros((n, n), bool)      # [query, key]
        m[~q, :min(130, n - 1)] = True
        w[q] = True
        lead.append((m.T if axis == 1 else m).ravel())
        whole.append((w.T if axis == 1 else w).ravel())
        if axis == 3:
            rows.append(q)
        else:                                  # cell of (pair row, query): the query is the column on axis 0
            rows.append((np.tile(q, n) if axis == 0 else np.repeat(q, n)))
    return np.concatenate(lead), np.concatenate(whole), np.concatenate(rows)


@functools.lru_cache(maxsize=1)
def _masked_reference(L, H, axis, whole_rows):
    x, bv = _inputs(L, H, axis)
    lead, whole, rows = _masks(L, axis)
    bv = bv.copy()
    bv[lead] = -np.inf
    if whole_rows:                             # equal masks of 1e9 and more absorb the score: the mean of the values
        bv[whole] = 0.0
        x = x.copy()
        x[rows, :H * D] = 0.0
    return _reference(list(L), H, axis, x, bv)


@pytest.mark.parametrize("L,H,axis", [
    ((200,), 2, 0), ((200,), 2, 1),
    ((300, 140), 1, 0), ((300, 140), 1, 1),
    ((514, 200, 33), 1, 0), ((514, 200, 33), 1, 1),
    ((641, 257), 1, 0),
    ((140, 300), 2, 3),
])
def test_masked_chunks(L, H, axis):
    x, bv = _inputs(L, H, axis)
    lead, whole, _ = _masks(L, axis)
    for value in MASKS:
        finite = np.isfinite(value)
        b = bv.copy()
        b[lead] = value
        if finite:
            b[whole] = value
        check(_call(list(L), H, axis, x, b), _masked_reference(L, H, axis, bool(finite)), "bf16",
              f"masked attention axis {axis} {L} mask {value:g}")
