"""What a user of the packed pair-state library has it do, as measurable cases.

Every case goes through the public entry points: the runners of
`paper_2609_30379_amd.blocks` (a pair block, the four-block stack, the token
encoder layer, the training step of the single-pair-single program) and, for
single layers, the C-ABI calls of `paper_2609_30379_amd.binding` in the order a
model calls them.  Sizes are those of the repository's workloads
(`paper_2609_30379_amd.synth`) and of the length ranges they are drawn from;
lengths are ragged and mostly odd.

Kinds
  pair_block        pair block or stack (PairRun): forward, fp32 or bf16
  attention_layer   triangle attention: LayerNorm + q|k|v(|gate)|bias projection,
                    row or column attention, output projection + residual
  triangle_layer    gated triangle multiplication: operand and gate projections,
                    contraction, gated residual
  single_attention  attention over single tokens with bias from the pair state
  attention_train   pair attention forward and backward on one training step
  triangle_train    triangle contraction forward and backward on packed operands
  mechanism         training step: forward, diagnostic loss, every gradient
  encoder           pre-LayerNorm encoder layer on packed tokens
"""
from __future__ import annotations

import dataclasses
import math

import numpy as np
import torch

from paper_2609_30379_amd import binding as B
from paper_2609_30379_amd import blocks, synth

BF16, F32, F64 = torch.bfloat16, torch.float32, torch.float64
BLOCK_STEPS = "bcast,lin,att_row,tri_out,trans,single"
STACK_STEPS = "bcast,tri_out,tri_in,att_row,att_col,trans,single"
TINY_STEPS = "bcast,lin,att_row,tri_out,single"


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # One block of a small fp32 model: few rows, a dozen launches, so
        # latency and launch count are what a user sees.
        dict(name="block_tiny_f32", kind="pair_block", dtype="f32", c_s=32, c_z=16, heads=2, hidden=64, blocks=1,
             steps=TINY_STEPS, batch=4, dist="uniform", lo=4, hi=16, median=0.0, sigma=0.0, length_seed=0),
        # One block over a bucketed (near-uniform) batch.
        dict(name="block_b8_n208_224", kind="pair_block", dtype="bf16", c_s=384, c_z=128, heads=4, hidden=512, blocks=1,
             steps=BLOCK_STEPS, batch=8, dist="uniform", lo=208, hi=224, median=0.0, sigma=0.0, length_seed=0),
        # The four-block stack on a ragged batch: the headline inference call.
        dict(name="stack4_b16_lognormal192", kind="pair_block", dtype="bf16", c_s=384, c_z=128, heads=4, hidden=512,
             blocks=4, steps=STACK_STEPS, batch=16, dist="lognormal", lo=16, hi=768, median=192.0, sigma=0.6,
             length_seed=0),
        # Gated column attention on a batch of the same distribution that has
        # samples longer than 512, as more than half of such batches do.
        dict(name="att_col_gated_b16_to_586", kind="attention_layer", axis=1, gated=True, batch=16, dist="lognormal",
             lo=16, hi=768, median=192.0, sigma=0.6, length_seed=17),
        # Row attention of one mid-size sample: interactive inference.
        dict(name="att_row_b1_n193", kind="attention_layer", axis=0, gated=False, batch=1, dist="uniform", lo=193,
             hi=193, median=0.0, sigma=0.0, length_seed=0),
        # Gated triangle multiplication of the gated stack.
        dict(name="tri_out_gated_b16", kind="triangle_layer", direction=0, batch=16, dist="lognormal", lo=16, hi=768,
             median=192.0, sigma=0.6, length_seed=0),
        # The single track's attention with pair bias, 12 heads of 32.
        dict(name="single_att_b8_n32_512", kind="single_attention", batch=8, dist="uniform", lo=32, hi=512, median=0.0,
             sigma=0.0, length_seed=1),
        # Training: pair attention forward + backward on the square pair lengths.
        dict(name="att_row_train_b8_n66_317", kind="attention_train", axis=0, batch=8, dist="uniform", lo=66, hi=317,
             median=0.0, sigma=0.0, length_seed=2),
        # Training: triangle contraction forward + backward, incoming.
        dict(name="tri_in_train_b8_n66_317", kind="triangle_train", direction=1, batch=8, dist="uniform", lo=66,
             hi=317, median=0.0, sigma=0.0, length_seed=2),
        # Training step of the single-pair-single program, non-leading layout
        # (three feature vectors per packed position).
        dict(name="mechanism_s3_b8_n40_182", kind="mechanism", rect=False, s_axis=3, batch=8, dist="uniform", lo=40,
             hi=182, col_lo=0, col_hi=0, median=0.0, sigma=0.0, length_seed=4),
        # Encoder layer over a full token batch (bulk scoring) ...
        dict(name="encoder_b64_lognormal230", kind="encoder", batch=64, dist="lognormal", lo=16, hi=512, median=230.0,
             sigma=0.5, length_seed=0),
        # ... and over a few requests (serving).
        dict(name="encoder_b4_lognormal230", kind="encoder", batch=4, dist="lognormal", lo=16, hi=512, median=230.0,
             sigma=0.5, length_seed=0),
    ]


def _loguniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_lengths(rng, n_lo, n_hi, batch_hi, cells_hi):
    """Batch geometry with samples between n_lo and n_hi and at most cells_hi pair cells."""
    batch = _loguniform(rng, 1, batch_hi)
    hi = _loguniform(rng, max(n_lo, 24), n_hi)
    hi = min(hi, int(math.sqrt(cells_hi)))
    lo = rng.choice([max(n_lo, hi // 6), max(n_lo, hi - hi // 12), max(n_lo, hi // 2)])
    batch = max(1, min(batch, cells_hi // (hi * hi)))
    return dict(batch=batch, dist="uniform", lo=int(lo), hi=int(hi), median=0.0, sigma=0.0,
                length_seed=rng.randrange(1 << 20))


def _draw_lognormal(rng, batch_hi, median, sigma, lo, hi, cells_hi):
    """A batch of the ragged distribution; the seed is advanced until it fits."""
    c = dict(batch=_loguniform(rng, 1, batch_hi), dist="lognormal", lo=lo, hi=hi, median=median, sigma=sigma,
             length_seed=rng.randrange(1 << 20))
    while sum(int(n) ** 2 for n in _lengths(c)) > cells_hi:
        c["length_seed"] += 1
    return c


def draw(rng):
    kind = rng.choice(["pair_block", "pair_block", "attention_layer", "attention_layer", "triangle_layer",
                       "single_attention", "attention_train", "triangle_train", "mechanism", "encoder", "encoder"])
    c = dict(kind=kind)
    if kind == "pair_block":
        what = rng.choice(["f32", "block", "block", "stack"])
        if what == "f32":
            c.update(dtype="f32", c_s=32, c_z=16, heads=2, hidden=64, blocks=1, steps=TINY_STEPS)
            c.update(_draw_lengths(rng, 4, 24, 8, 2000))
        else:
            cz = rng.choice([64, 128, 128, 128])
            c.update(dtype="bf16", c_s=384, c_z=cz, heads=cz // 32, hidden=4 * cz)
            c.update(dict(blocks=1, steps=BLOCK_STEPS) if what == "block"
                     else dict(blocks=rng.randint(1, 3), steps=STACK_STEPS))
            c.update(_draw_lengths(rng, 32, 512, 8, 650000))
    elif kind == "attention_layer":
        c.update(axis=rng.randrange(2), gated=rng.random() < 0.5)
        c.update(_draw_lognormal(rng, 16, 192.0, 0.6, 16, 768, 1200000) if rng.random() < 0.5
                 else _draw_lengths(rng, 16, 512, 8, 900000))
    elif kind == "triangle_layer":
        c.update(direction=rng.randrange(2))
        c.update(_draw_lognormal(rng, 16, 192.0, 0.6, 16, 768, 900000) if rng.random() < 0.5
                 else _draw_lengths(rng, 16, 512, 8, 900000))
    elif kind == "single_attention":
        c.update(_draw_lengths(rng, 16, 512, 8, 900000))
    elif kind in ("attention_train", "triangle_train"):
        c.update(dict(axis=rng.randrange(2)) if kind == "attention_train" else dict(direction=rng.randrange(2)))
        c.update(_draw_lengths(rng, 32, 317, 8, 400000))
    elif kind == "mechanism":
        what = rng.choice(["square", "rect", "nonleading"])
        lo, hi = {"square": (66, 317), "rect": (66, 307), "nonleading": (40, 182)}[what]
        c.update(rect=what == "rect", s_axis=3 if what == "nonleading" else 1, col_lo=66 if what == "rect" else 0,
                 col_hi=309 if what == "rect" else 0)
        c.update(batch=_loguniform(rng, 1, 8), dist="uniform", lo=lo, hi=hi, median=0.0, sigma=0.0,
                 length_seed=rng.randrange(1 << 20))
    else:
        c.update(batch=_loguniform(rng, 1, 56), dist="lognormal", lo=16, hi=512, median=230.0, sigma=0.5,
                 length_seed=rng.randrange(1 << 20))
    return c


# ------------------------------------------------------------------ geometry
def _dist(case):
    if case["dist"] == "uniform":
        return ("uniform", case["lo"], case["hi"])
    return ("lognormal", case["median"], case["sigma"], case["lo"], case["hi"])


def _lengths(case):
    w = synth.Workload("lengths", "pair", case["batch"], _dist(case), case["length_seed"], "bf16")
    return [int(n) for n in synth.lengths_for(w)]


def _workload(case, seed):
    """The runner's workload description of a case, its values drawn from `seed`."""
    kind, L = case["kind"], _lengths(case)
    if kind == "pair_block":
        return synth.Workload("case", "pair", case["batch"], _dist(case), seed, case["dtype"], c_s=case["c_s"],
                              c_z=case["c_z"], heads=case["heads"], head_dim=case["c_z"] // case["heads"],
                              hidden=case["hidden"], blocks=case["blocks"], transition="trans" in case["steps"],
                              tri_incoming="tri_in" in case["steps"], col_attention="att_col" in case["steps"],
                              gains=synth._pair_gains(max(L), blocks=case["blocks"]),
                              steps=tuple(case["steps"].split(",")))
    if kind == "mechanism":
        return synth.Workload("case", "mechanism", case["batch"], _dist(case), seed, "bf16", c_s=384, c_z=128,
                              hidden=512, gains=synth.mechanism_gains(), s_axis=case["s_axis"],
                              col_dist=("uniform", case["col_lo"], case["col_hi"]) if case["rect"] else ())
    return synth.Workload("case", "tokens", case["batch"], _dist(case), seed, "bf16", c_s=768, heads=12, head_dim=64,
                          hidden=3072, gains={"qkv": 0.5, "o": 0.5, "ffn1": 0.5, "ffn2": 0.5})


def _cols(case):
    if not case["rect"]:
        return None
    w = _workload(case, case["length_seed"])
    return [int(m) for m in synth.cols_for(dataclasses.replace(w, seed=case["length_seed"]))]


# -------------------------------------------------------------------- inputs
class _Values:
    """Seeded device tensors: activations, weights [out, in] and vectors of a layer."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(int(seed) & 0x7FFFFFFF)

    def normal(self, *shape, std=1.0, mean=0.0, dtype=BF16):
        return torch.empty(shape, dtype=F32, device="cuda").normal_(mean, std, generator=self.g).to(dtype)

    def linear(self, n_out, n_in, gain):
        return self.normal(n_out, n_in, std=gain / math.sqrt(n_in)), self.normal(n_out, std=0.1 * gain, dtype=F32)

    def ln(self, c):
        return self.normal(c, std=0.1, mean=1.0, dtype=F32), self.normal(c, std=0.1, dtype=F32)


def _empty(*shape, dtype=BF16):
    return torch.empty(shape, dtype=dtype, device="cuda")


def _round8(n):
    return max(8, (n + 7) // 8 * 8)


def prepare(case, seed):
    kind = case["kind"]
    st = {"kind": kind, "case": case}
    L = _lengths(case)
    if kind == "pair_block":
        st["run"] = blocks.PairRun(_workload(case, seed), lengths=L)
        return st
    if kind == "encoder":
        st["run"] = blocks.TokenRun(_workload(case, seed), lengths=L)
        return st
    if kind == "mechanism":
        st["run"] = blocks.MechanismRun(_workload(case, seed), lengths=L, cols=_cols(case))
        return st

    v = _Values(seed)
    C, H, d = 128, 4, 32
    lay = B.NestedLayout(L)
    R, T = lay.sum_n2, lay.sum_n
    st.update(layout=lay, lengths=L)
    if kind == "attention_layer":
        st["z"] = v.normal(R, C, std=0.6)
        st["ln"] = v.ln(C)
        (wq, bq), (wb, bb) = v.linear(3 * C, C, 0.5), v.linear(H, C, 0.6)
        st["w"], st["b"] = torch.cat([wq, wb]).contiguous(), torch.cat([bq, bb]).contiguous()
        st["wg"], st["bg"] = v.linear(C, C, 1.0) if case["gated"] else (None, None)
        st["wo"], st["bo"] = v.linear(C, C, 0.5)
        st.update(qkv=_empty(R, 3 * C), bias=_empty(H, _round8(R)), o=_empty(R, C), out=_empty(R, C),
                  g=_empty(R, C) if case["gated"] else None,
                  ws=B.workspace_tensor(B.attention_workspace_bytes(lay, case["axis"], H, d)))
    elif kind == "triangle_layer":
        st["z"] = v.normal(R, C, std=0.6)
        st["ln"], st["ln_t"] = v.ln(C), v.ln(C)
        gp = 4.0 * math.sqrt(0.3 / max(L))
        parts = [v.linear(C, C, gp), v.linear(C, C, 1.0), v.linear(C, C, gp), v.linear(C, C, 1.0)]
        st["w"] = torch.cat([w for w, _ in parts]).contiguous()
        st["b"] = torch.cat([b for _, b in parts]).contiguous()
        st["wg"], st["bg"] = v.linear(C, C, 1.0)
        st["wo"], st["bo"] = v.linear(C, C, 0.5)
        st.update(ab=_empty(2 * C, _round8(lay.sum_pad)), g=_empty(R, C), t=_empty(R, C), out=_empty(R, C))
    elif kind == "single_attention":
        Cs, Hs = 384, 12
        st["s"] = v.normal(T, Cs)
        st["ln"] = v.ln(Cs)
        st["w"], st["b"] = v.linear(3 * Cs, Cs, 0.7)
        st["wo"], st["bo"] = v.linear(Cs, Cs, 0.5)
        st["bias"] = v.normal(Hs, _round8(R), std=0.6)
        st.update(qkv=_empty(T, 3 * Cs), o=_empty(T, Cs), out=_empty(T, Cs),
                  ws_proj=B.workspace_tensor(B.layernorm_linear_workspace_bytes(T, Cs, 3 * Cs)),
                  ws=B.workspace_tensor(B.attention_workspace_bytes(lay, 3, Hs, d)))
    elif kind == "attention_train":
        st.update(qkv=v.normal(R, 3 * C, std=0.6), bias=v.normal(H, _round8(R), std=0.6), do=v.normal(R, C, std=0.1),
                  o=_empty(R, C), dqkv=_empty(R, 3 * C), dbias=_empty(H, _round8(R), dtype=F32),
                  ws=B.workspace_tensor(B.attention_workspace_bytes(lay, case["axis"], H, d)),
                  ws_bwd=B.workspace_tensor(B.attention_backward_workspace_bytes(lay, case["axis"], H, d)))
        st["dbias"].zero_()
    elif kind == "triangle_train":
        st.update(ab=v.normal(R, 2 * C, std=(0.3 / max(L)) ** 0.25), z0=v.normal(R, C, std=0.6),
                  dt=v.normal(R, C, std=0.1), z=_empty(R, C), dab=_empty(R, 2 * C),
                  ws=B.workspace_tensor(B.triangle_workspace_bytes(lay, C)))
    else:
        raise ValueError(kind)
    return st


# ----------------------------------------------------------------------- run
def _grad_keys(r):
    """The weight gradients a step writes (square pairs: u and v as one stacked projection)."""
    return [k for k in r.grads if r.sep or k.split(".")[0] not in ("u", "v")]


def run(st):
    kind, case = st["kind"], st["case"]
    if kind == "pair_block":
        s, z = st["run"].step()
        return {"s": s, "z": z}
    if kind == "encoder":
        x, pooled = st["run"].step()
        return {"x": x, "pooled": pooled}
    if kind == "mechanism":
        r = st["run"]
        loss_s, loss_p, xt, pt = r.step()
        out = {"loss_s": loss_s, "loss_p": loss_p, "xt": xt, "pt": pt, "dx": r.dx}
        if r.rect:
            out["dy"] = r.dy
        out.update({"d_" + k: r.grads[k] for k in _grad_keys(r)})
        return out

    lay, C, H, d = st["layout"], 128, 4, 32
    if kind == "attention_layer":
        z, qkv, o = st["z"], st["qkv"], st["o"]
        B.nt_layernorm_linear(z, st["w"], st["b"], qkv, ln=st["ln"], n_tail=H, y_tail=st["bias"], layout=lay)
        if case["gated"]:
            B.nt_layernorm_linear(z, st["wg"], st["bg"], st["g"], ln=st["ln"], layout=lay)
        B.nt_pair_row_attention(lay, case["axis"], H, d, qkv[:, :C], qkv[:, C:2 * C], qkv[:, 2 * C:], o,
                                bias=st["bias"], bias_layout="heads", workspace=st["ws"], gate=st["g"])
        return B.nt_layernorm_linear(o, st["wo"], st["bo"], st["out"], epilogue="residual", residual=z, layout=lay,
                                     residual_layout=lay)
    if kind == "triangle_layer":
        tiled = ("pair_tiled", "pair_tiled_t")[case["direction"]]
        z, ab, t = st["z"], st["ab"], st["t"]
        B.nt_layernorm_linear(z, st["w"], st["b"], None, ln=st["ln"], epilogue="sigmoid_glu", hidden=C, n_tail=2 * C,
                              y_tail=ab, tail_layout=tiled, layout=lay, c_out=2 * C)
        B.nt_layernorm_linear(z, st["wg"], st["bg"], st["g"], ln=st["ln"], layout=lay)
        B.nt_triangle_mul_gated(lay, case["direction"], ab[:C], ab[C:], t, operands=tiled)
        return B.nt_layernorm_linear(t, st["wo"], st["bo"], st["out"], ln=st["ln_t"], epilogue="gated_residual",
                                     residual=z, gate=st["g"], layout=lay, residual_layout=lay)
    if kind == "single_attention":
        Cs, s, qkv, o = 384, st["s"], st["qkv"], st["o"]
        B.nt_layernorm_linear(s, st["w"], st["b"], qkv, ln=st["ln"], layout=lay, level="singles",
                              workspace=st["ws_proj"])
        B.nt_pair_row_attention(lay, 3, 12, d, qkv[:, :Cs], qkv[:, Cs:2 * Cs], qkv[:, 2 * Cs:], o, bias=st["bias"],
                                bias_layout="heads", workspace=st["ws"])
        return B.nt_layernorm_linear(o, st["wo"], st["bo"], st["out"], epilogue="residual", residual=s, layout=lay,
                                     level="singles")
    if kind == "attention_train":
        qkv, dqkv, R = st["qkv"], st["dqkv"], lay.sum_n2
        q, k, v = qkv[:, :C], qkv[:, C:2 * C], qkv[:, 2 * C:]
        B.nt_pair_row_attention(lay, case["axis"], H, d, q, k, v, st["o"], bias=st["bias"], bias_layout="heads",
                                workspace=st["ws"])
        B.nt_pair_row_attention_backward(lay, case["axis"], H, d, q, k, v, st["do"], dqkv[:, :C], dqkv[:, C:2 * C],
                                         dqkv[:, 2 * C:], bias=st["bias"], dbias=st["dbias"], bias_layout="heads",
                                         workspace=st["ws_bwd"])
        return {"o": st["o"], "dqkv": dqkv, "dbias": st["dbias"][:, :R]}
    a, b = st["ab"][:, :C], st["ab"][:, C:]
    z, dab = st["z"], st["dab"]
    z.copy_(st["z0"])
    B.nt_triangle_mul(lay, case["direction"], a, b, z, workspace=st["ws"])
    dab.zero_()
    B.nt_triangle_mul_backward(lay, case["direction"], a, b, st["dt"], dab[:, :C], dab[:, C:], workspace=st["ws"])
    return {"z": z, "dab": dab}


# ---------------------------------------------------------------------- work
def work(case):
    """Inputs read once and outputs written once (weights included), and the
    multiply-adds of the products, of one pass."""
    kind, L = case["kind"], _lengths(case)
    S, R, N3 = sum(L), sum(n * n for n in L), sum(n ** 3 for n in L)
    C, H, d = 128, 4, 32
    if kind == "pair_block":
        C, Cs, F, e = case["c_z"], case["c_s"], case["hidden"], 4 if case["dtype"] == "f32" else 2
        steps = case["steps"].split(",")
        weights = {"bcast": 2 * C * Cs, "lin": C * C, "att": 4 * C * C + case["heads"] * C, "tri": 2 * C * C,
                   "trans": 3 * C * F, "single": C * Cs}
        flops = {"bcast": 4 * S * C * Cs + R * C, "lin": 2 * R * C * C,
                 "att": 2 * R * C * (4 * C + case["heads"]) + 4 * C * N3, "tri": 4 * R * C * C + 2 * C * N3,
                 "trans": 6 * R * C * F, "single": R * C + 2 * S * C * Cs}
        nb, nf = 0, 0
        for b in range(case["blocks"]):
            for t in steps:
                if t == "lin" and b:
                    continue
                nb += weights[t.split("_")[0]] * e
                nf += flops[t.split("_")[0]]
        return {"bytes": nb + (2 * S * Cs + R * C) * e, "flops": nf}
    if kind == "encoder":
        c, F = 768, 3072
        return {"bytes": 2 * (2 * S * c + 4 * c * c + 2 * c * F) + 4 * len(L) * c,
                "flops": 2 * S * c * (4 * c + 2 * F) + 4 * c * R}
    if kind == "mechanism":
        Cx, Cp, F, Sx = 384, 128, 512, case["s_axis"]
        M = _cols(case)
        cells = (R if M is None else sum(n * m for n, m in zip(L, M))) * Sx
        rows, cols = S * Sx, (S if M is None else sum(M)) * Sx
        nin = rows * Cx + (0 if M is None else cols * Cx)
        # forward and backward of the projections, the transition and the
        # single update (the backward has twice the forward's products, and
        # recomputes the gate and up products it does not store)
        flops = 6 * (rows + cols) * Cx * Cp + 18 * cells * Cp * F + 6 * rows * Cp * Cx
        weights = 2 * Cx * Cp + 3 * Cp * F + Cp * Cx
        return {"bytes": 2 * nin + 4 * nin + 2 * rows * Cx + 2 * cells * Cp + 6 * weights, "flops": flops}
    if kind == "attention_layer":
        cols = 4 * C + H + (C if case["gated"] else 0)
        return {"bytes": 4 * R * C + 2 * cols * C, "flops": 2 * R * C * cols + 4 * H * d * N3}
    if kind == "triangle_layer":
        return {"bytes": 4 * R * C + 12 * C * C, "flops": 12 * R * C * C + 2 * C * N3}
    if kind == "single_attention":
        return {"bytes": 4 * S * 384 + 2 * 12 * R + 8 * 384 * 384, "flops": 8 * S * 384 * 384 + 4 * 384 * R}
    if kind == "attention_train":
        # q, k, v, do, bias in; o, dq, dk, dv, dbias out; two products forward, five backward
        return {"bytes": 2 * R * (8 * C + H) + 4 * R * H, "flops": 14 * H * d * N3}
    return {"bytes": 2 * R * 7 * C, "flops": 6 * C * N3}


# ----------------------------------------------------------------- tolerance
# About four times the largest error seen against exact(): fp32 sums in another
# order, or one bf16 rounding of each stored tensor on the way (2^-9 relative
# each), which travels through the steps that follow it.
_TOLERANCE = {
    "attention_layer": {"rel": 0.007, "max": 0.02},
    "triangle_layer": {"rel": 0.01, "max": 0.065},
    "single_attention": {"rel": 0.007, "max": 0.02},
    "attention_train": {"rel": 0.011, "max": 0.12},
    "triangle_train": {"rel": 0.007, "max": 0.016},
    "mechanism": {"rel": 0.012, "max": 0.075},
    "encoder": {"rel": 0.01, "max": 0.05},
}


def tolerance(case):
    if case["kind"] != "pair_block":
        return dict(_TOLERANCE[case["kind"]])
    if case["dtype"] == "f32":
        return {"rel": 1e-6, "max": 5e-6}
    return {"rel": 0.018, "max": 0.1} if case["blocks"] == 1 else {"rel": 0.028, "max": 0.25}


# --------------------------------------------------------------------- exact
def _f64(t):
    if isinstance(t, np.ndarray):
        t = torch.from_numpy(np.ascontiguousarray(t))
    return t.to(device="cuda", dtype=F64)


def _norm(x, ln):
    return torch.nn.functional.layer_norm(x, (x.shape[-1],), _f64(ln[0]), _f64(ln[1]), 1e-5)


def _linear(x, w, b):
    return x @ _f64(w).T + _f64(b)


def _swiglu(x, w, b, w2, b2):
    g, u = _linear(x, w, b).chunk(2, -1)
    return _linear(torch.nn.functional.silu(g) * u, w2, b2)


def _cells(L):
    o = 0
    for n in L:
        yield n, slice(o, o + n * n)
        o += n * n


def _rows(L):
    o = 0
    for n in L:
        yield n, slice(o, o + n)
        o += n


def _pair_attention(q, k, v, bias, H):
    """Row attention of one sample: q, k, v [N, N, H*d], bias [N, N, H]."""
    n, d = q.shape[0], q.shape[2] // H
    beta = bias.permute(2, 0, 1)
    out = []
    step = max(1, (1 << 26) // max(1, H * n * n))
    for r in range(0, n, step):
        qr, kr, vr = (t[r:r + step].reshape(-1, n, H, d).transpose(1, 2) for t in (q, k, v))
        p = torch.softmax(qr @ kr.transpose(2, 3) / math.sqrt(d) + beta, -1)
        out.append((p @ vr).transpose(1, 2).reshape(-1, n, H * d))
    return torch.cat(out)


def _attention_op(q, k, v, bias, L, H, axis):
    out = []
    for n, c in _cells(L):
        t = [x[c].reshape(n, n, -1) for x in (q, k, v, bias)]
        if axis == 1:
            t = [x.transpose(0, 1) for x in t]
        o = _pair_attention(*t, H)
        out.append((o.transpose(0, 1) if axis == 1 else o).reshape(n * n, -1))
    return torch.cat(out)


def _triangle_op(a, b, L, direction):
    out = []
    for n, c in _cells(L):
        x, y = (t[c].reshape(n, n, -1).permute(2, 0, 1) for t in (a, b))
        t = x.transpose(1, 2) @ y if direction else x @ y.transpose(1, 2)
        out.append(t.permute(1, 2, 0).reshape(n * n, -1))
    return torch.cat(out)


def _broadcast_op(u, v, L, M):
    return torch.cat([(u[r][:, None] + v[c][None]).reshape(n * m, *u.shape[1:])
                      for (n, r), (m, c) in zip(_rows(L), _rows(M))])


def _column_mean(z, L, M):
    out, o = [], 0
    for n, m in zip(L, M):
        out.append(z[o:o + n * m].reshape(n, m, *z.shape[1:]).mean(1))
        o += n * m
    return torch.cat(out)


def _exact_pair_block(case, r):
    L, C, H = r.lengths, case["c_z"], case["heads"]
    s, z = _f64(r.s_init), None
    for b, p in enumerate(r.params):
        for t in case["steps"].split(","):
            if t == "bcast":
                uv = _linear(s, p["uv.w"], p["uv.b"])
                add = _broadcast_op(uv[:, :C], uv[:, C:], L, L)
                z = add if z is None else z + add
            elif t == "lin" and b == 0:
                z = _linear(_norm(z, (p["lin.ln_g"], p["lin.ln_b"])), p["lin.w"], p["lin.b"])
            elif t.startswith("att_"):
                y = _linear(_norm(z, (p[t + ".ln_g"], p[t + ".ln_b"])), p[t + ".w"], p[t + ".b"])
                o = _attention_op(y[:, :C], y[:, C:2 * C], y[:, 2 * C:3 * C], y[:, 3 * C:], L, H, int(t == "att_col"))
                z = z + _linear(o, p[t + ".wo"], p[t + ".bo"])
            elif t.startswith("tri_"):
                y = _linear(_norm(z, (p[t + ".ln_g"], p[t + ".ln_b"])), p[t + ".w"], p[t + ".b"])
                z = z + _triangle_op(y[:, :C], y[:, C:], L, int(t == "tri_in"))
            elif t == "trans":
                z = z + _swiglu(_norm(z, (p["trans.ln_g"], p["trans.ln_b"])), p["trans.w"], p["trans.b"],
                                p["trans.w2"], p["trans.b2"])
            elif t == "single":
                s = s + _linear(_column_mean(z, L, L), p["single.w"], p["single.b"])
    return {"s": s, "z": z}


def _exact_encoder(r):
    p, L, H = r.params, r.lengths, 12
    x = _f64(r.x_init)
    c = x.shape[1]
    y = _linear(_norm(x, (p["ln1_g"], p["ln1_b"])), p["qkv.w"], p["qkv.b"])
    o = []
    for n, t in _rows(L):
        q, k, v = (m.reshape(n, H, c // H).transpose(0, 1) for m in y[t].split(c, -1))
        o.append((torch.softmax(q @ k.transpose(1, 2) / math.sqrt(c // H), -1) @ v).transpose(0, 1).reshape(n, c))
    x = x + _linear(torch.cat(o), p["o.w"], p["o.b"])
    h = _linear(_norm(x, (p["ln2_g"], p["ln2_b"])), p["ffn1.w"], p["ffn1.b"])
    x = x + _linear(torch.nn.functional.gelu(h), p["ffn2.w"], p["ffn2.b"])
    return {"x": x, "pooled": torch.stack([x[t].mean(0) for _, t in _rows(L)])}


def _exact_mechanism(case, r):
    L, Sx = r.lengths, case["s_axis"]
    M = r.cols if r.rect else L
    p = {k: _f64(t).requires_grad_() for k, t in r.params.items()}
    x = _f64(r.x_init).reshape(-1, Sx, 384).requires_grad_()
    y = _f64(r.y_init).reshape(-1, 1, 384).requires_grad_() if r.rect else x
    lin = lambda t, n: t @ p[n + ".w"].T + p[n + ".b"]                       # noqa: E731
    P = _broadcast_op(lin(x, "u"), lin(y, "v"), L, M)
    xn = torch.nn.functional.layer_norm(P, (128,), p["trans.ln_g"], p["trans.ln_b"], 1e-5)
    g, u = (xn @ p["trans.w"].T + p["trans.b"]).chunk(2, -1)
    Pt = P + (torch.nn.functional.silu(g) * u) @ p["trans.w2"].T + p["trans.b2"]
    xt = x + lin(_column_mean(Pt, L, M), "g")
    n = len(L)
    loss_s, loss_p, o = [], [], 0
    for i, (rows, t) in enumerate(_rows(L)):
        loss_s.append((1.0 + i / n) * (xt[t] ** 2).sum() / (Sx * 384 * sum(L)))
        loss_p.append((1.5 - i / (2.0 * n)) * (Pt[o:o + rows * M[i]] ** 2).sum() / (Sx * 128 * Pt.shape[0]))
        o += rows * M[i]
    loss_s, loss_p = torch.stack(loss_s), torch.stack(loss_p)
    (loss_s.sum() + loss_p.sum()).backward()
    out = {"loss_s": loss_s.detach(), "loss_p": loss_p.detach(), "xt": xt.detach().reshape(-1, Sx * 384),
           "pt": Pt.detach().reshape(-1, Sx * 128), "dx": x.grad.reshape(-1, Sx * 384)}
    if r.rect:
        out["dy"] = y.grad.reshape(-1, 384)
    for k in _grad_keys(r):
        out["d_" + k] = torch.cat([p["u" + k[2:]].grad, p["v" + k[2:]].grad]) if k.startswith("uv.") else p[k].grad
    return out


def exact(case, seed):
    st = prepare(case, seed)                      # for its inputs alone
    kind = case["kind"]
    if kind == "pair_block":
        return _exact_pair_block(case, st["run"])
    if kind == "encoder":
        return _exact_encoder(st["run"])
    if kind == "mechanism":
        return _exact_mechanism(case, st["run"])
    L, C, H = st["lengths"], 128, 4
    if kind == "attention_layer":
        z = _f64(st["z"])
        y = _linear(_norm(z, st["ln"]), st["w"], st["b"])
        o = _attention_op(y[:, :C], y[:, C:2 * C], y[:, 2 * C:3 * C], y[:, 3 * C:], L, H, case["axis"])
        if case["gated"]:
            o = o * torch.sigmoid(_linear(_norm(z, st["ln"]), st["wg"], st["bg"]))
        return z + _linear(o, st["wo"], st["bo"])
    if kind == "triangle_layer":
        z = _f64(st["z"])
        x = _norm(z, st["ln"])
        ap, ag, bp, bg = _linear(x, st["w"], st["b"]).chunk(4, -1)
        t = _triangle_op(torch.sigmoid(ag) * ap, torch.sigmoid(bg) * bp, L, case["direction"])
        g = torch.sigmoid(_linear(x, st["wg"], st["bg"]))
        return z + g * _linear(_norm(t, st["ln_t"]), st["wo"], st["bo"])
    if kind == "single_attention":
        s = _f64(st["s"])
        y = _linear(_norm(s, st["ln"]), st["w"], st["b"])
        o = []
        for (n, t), (_, c) in zip(_rows(L), _cells(L)):
            q, k, v = (m.reshape(n, 12, 32).transpose(0, 1) for m in y[t].split(384, -1))
            beta = _f64(st["bias"][:, c]).reshape(12, n, n)
            o.append((torch.softmax(q @ k.transpose(1, 2) / math.sqrt(32) + beta, -1) @ v).transpose(0, 1)
                     .reshape(n, 384))
        return s + _linear(torch.cat(o), st["wo"], st["bo"])
    if kind == "attention_train":
        R = sum(n * n for n in L)
        qkv, bias = _f64(st["qkv"]).requires_grad_(), _f64(st["bias"][:, :R]).T.contiguous().requires_grad_()
        dout = _f64(st["do"])
        o = torch.empty_like(dout)
        for n, c in _cells(L):                    # one sample's graph at a time
            os_ = _attention_op(qkv[c, :C], qkv[c, C:2 * C], qkv[c, 2 * C:], bias[c], [n], H, case["axis"])
            o[c] = os_.detach()
            os_.backward(dout[c])
        return {"o": o, "dqkv": qkv.grad, "dbias": bias.grad.T.contiguous()}
    a, b = (_f64(t).requires_grad_() for t in (st["ab"][:, :C], st["ab"][:, C:]))
    t = _triangle_op(a, b, L, case["direction"])
    t.backward(_f64(st["dt"]))
    return {"z": _f64(st["z0"]) + t.detach(), "dab": torch.cat([a.grad, b.grad], 1)}
