"""The oracle with matrix operands rounded to BF16 (test helper).

BF16 mode rounds the operands of every matrix product of the network, in the
forward and in the adjoint, and accumulates in FP32; everything else (first
embedding layer, gates, softmax, layer norm, descriptor, the type part of the
first fitting layer) stays FP32.  This evaluates the same in FP64 with only
that rounding, which leaves of a BF16 force error what FP32 noise does to
values at a rounding boundary.
"""

from __future__ import annotations

import numpy as np
import torch

from oracle import dpa1_oracle as orc


def to_bf16(x: torch.Tensor) -> torch.Tensor:
    return x.float().bfloat16().double()


def rounded_energies(rounding):
    """A stand-in for the oracle's atomic_energies with rounding(operand) in its products."""

    class Product(torch.autograd.Function):
        @staticmethod
        def forward(ctx, a, b):
            a, b = rounding(a), rounding(b)
            ctx.save_for_backward(a, b)
            return a @ b

        @staticmethod
        def backward(ctx, g):
            a, b = ctx.saved_tensors
            g = rounding(g)
            return (g @ b.transpose(-1, -2),
                    a.transpose(-1, -2) @ g if ctx.needs_input_grad[1] else None)

    mm = Product.apply

    def layer(x, W, b, fixed=0.0, residual=True):
        y = torch.tanh(mm(x, W) + b + fixed)
        fin, fout = W.shape
        if residual and fout in (fin, 2 * fin):
            y = y + (x if fout == fin else torch.cat([x, x], dim=-1))
        return y

    def energies(model, d, mask, nnei, tc, tn, rcut, sel):
        t = model.t
        B, n, _ = d.shape
        temb = t["type_embedding"]
        r = torch.sqrt((d * d).sum(-1))
        sw = orc.switch(r, model.rcut_smth, rcut) * mask
        s, rhat = sw / r, d / r[..., None]
        Rt = torch.cat([s[..., None], s[..., None] * rhat], dim=-1)
        x = torch.cat([s[..., None], temb[tn], temb[tc][:, None, :].expand(B, n, -1)], dim=-1)
        G = torch.tanh(x @ t["emb0.W"] + t["emb0.b"])
        for l in range(1, len(model.emb)):
            G = layer(G, t[f"emb{l}.W"], t[f"emb{l}.b"])
        S, D = model.attn_shift, model.attn_dim
        ww = sw[:, :, None] * sw[:, None, :]
        cos = rhat @ rhat.transpose(1, 2)
        keys = mask[:, None, :].expand(B, n, n)
        pad = (sel - nnei).to(d.dtype)
        for a in range(model.n_attn):
            W = torch.cat([t[f"attn{a}.W{c}"] for c in "qkv"], dim=1)
            b = torch.cat([t[f"attn{a}.b{c}"] for c in "qkv"])
            q, k, v = (mm(G, W) + b).split(D, dim=-1)
            lam = (mm(q, k.transpose(1, 2).contiguous()) / np.sqrt(D) + S) * ww - S
            lam = torch.where(keys, lam, torch.full_like(lam, -np.inf))
            mx = torch.clamp(lam.amax(dim=-1), min=-S)
            ex = torch.exp(lam - mx[..., None])
            p = ex / (ex.sum(-1) + pad[:, None] * torch.exp(-S - mx))[..., None]
            y = mm(mm(p * ww * cos, v), t[f"attn{a}.Wo"]) + t[f"attn{a}.bo"]
            G = G + orc._layer_norm(y, t[f"attn{a}.ln_gamma"], t[f"attn{a}.ln_beta"], model.ln_eps)
        T = Rt.transpose(1, 2) @ G / sel
        z = (T.transpose(1, 2) @ T[:, :, :model.axis]).reshape(B, -1)
        W = t["fit0.W"]
        z = layer(z, W[:z.shape[1]], t["fit0.b"], temb[tc] @ W[z.shape[1]:], residual=False)
        for l in range(1, len(model.fit)):
            z = layer(z, t[f"fit{l}.W"], t[f"fit{l}.b"])
        return z @ t["w_out"] + t["b_out"][0] + t["energy_bias"][tc]

    return energies


def compute(monkeypatch, model, coords, types, box, n, rcut, sel, rounding=to_bf16):
    """The oracle's compute with rounded operands."""
    with monkeypatch.context() as m:
        m.setattr(orc, "atomic_energies", rounded_energies(rounding))
        return orc.compute(model, coords, types, box, n, 0, rcut, sel)
