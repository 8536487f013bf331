"""How many bits the adjoint's two-term f16 operands keep.

Force errors against the FP64 oracle, relative to the forces' root mean square
and averaged likewise.  The whole model in FP32 (torch, logits included) is off
by 1.1e-6 to 6.4e-6 on these systems; products whose lower terms are
dropped, or whose operands are rounded to f16, by 2.5e-4 and more.  The bound is
three times the former.

Weights whose scales are far apart: a feature that is zero leaves its rows of
W_QKV free, 2^28 above the others' here (a scale for the whole matrix would
leave those 11 bits, 2.1e-4 and more in the forces).
"""

import numpy as np
import pytest

from clusters import compact_cluster
from oracle import dpa1_oracle as orc
from paper_2604_07276_amd import synth

pytestmark = pytest.mark.gpu

RC, SEL = 6.0, 120
F_REL = 2e-5


def system(name):
    kind, atoms = name[0], int(name[1:])
    if kind == "c":
        return compact_cluster(atoms, atoms - 1)
    s = synth.open_cluster(atoms, {9: 4.0, 41: 4.0, 150: 9.0}[atoms], 5, seed=atoms)
    return s.coords, s.types


def dead_feature(t, m=17, e=28):
    """Feature m of the attention layers' inputs is zero, its weights there 2^e of the others'."""
    for name in ("emb2.W", "emb2.b", "attn0.ln_gamma", "attn0.ln_beta"):
        t[name][..., m] = 0.0
    for a in (0, 1):
        for q in "qkv":
            t[f"attn{a}.W{q}"][m] *= 2.0 ** e


def check(shape, weights, name, tmp_path):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_07276_amd import binding
    p = str(tmp_path / "w.bin")
    synth.write_weights(p, shape, weights)
    x, types = system(name)
    m = binding.Model(p, RC, SEL)
    try:
        _, F, _, _ = m.compute(x, types, None, len(x), 0)
    finally:
        m.close()
    r = orc.compute(orc.load_model(p), x, types, None, len(x), 0, RC, SEL).forces
    err = np.sqrt(np.mean((F - r) ** 2) / np.mean(r ** 2))
    print(f"relative force error {err:.1e}", flush=True)
    assert err <= F_REL


@pytest.mark.parametrize("name", ["o9", "o41", "o150", "c17", "c34", "c66", "c98", "c121"])
@pytest.mark.parametrize("width", [97, 100, 104, 112])
def test_split_operands_keep_fp32(width, name, tmp_path):
    print(f"case: split operands, width {width}, system {name}", flush=True)
    shape = synth.ModelShape(emb=(25, 50, width))
    check(shape, synth.draw_weights(shape, 2), name, tmp_path)


@pytest.mark.parametrize("name", ["o41", "c34", "c98"])
@pytest.mark.parametrize("width", [97, 104, 105])
def test_rows_of_other_scales(width, name, tmp_path):
    print(f"case: a dead feature, width {width}, system {name}", flush=True)
    shape = synth.ModelShape(emb=(25, 50, width))
    t = synth.draw_weights(shape, 2)
    dead_feature(t)
    check(shape, t, name, tmp_path)


def scaled_channel(t, what, f=17, e=30):
    """Channel f of the attention layers: one factor 2^-e of itself (or zero), the other 2^e."""
    for a in (0, 1):
        low, high = {"vo": (("Wv", "bv"), ("Wo",)), "ov": (("Wo",), ("Wv", "bv")),
                     "qk": (("Wq", "bq"), ("Wk", "bk")), "kq": (("Wk", "bk"), ("Wq", "bq"))}[what[:2]]
        for names, factor in ((low, 0.0 if what.endswith("0") else 2.0 ** -e), (high, 2.0 ** e)):
            for n in names:
                w = t[f"attn{a}.{n}"]
                w[(f,) if n == "Wo" else (..., f)] *= factor


@pytest.mark.parametrize("name", ["o41", "c34", "c98"])
@pytest.mark.parametrize("what", ["vo", "ov", "qk", "kq", "vo0", "ov0", "qk0", "kq0"])
def test_channels_of_other_scales(what, name, tmp_path):
    """V and W_O (or Q and K) trade a factor of 2^30 in one channel: the function is the same."""
    print(f"case: channel scales {what}, system {name}", flush=True)
    shape = synth.ModelShape()
    t = synth.draw_weights(shape, 2)
    scaled_channel(t, what)
    check(shape, t, name, tmp_path)


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("e", [-120, -100, -62, -31, 31, 62, 120])
def test_energy_unit(e, precision, tmp_path):
    """Forces and virial are linear in w_out: in another energy unit (an eV is about 2^-62 joules)
    they are the same times a power of two, to the bit."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_07276_amd import binding
    print(f"case: energy unit 2^{e}, {precision}", flush=True)
    x, types = system("o41")
    shape = synth.ModelShape()
    p = str(tmp_path / "w.bin")
    got = []
    for k in (0, e):
        t = synth.draw_weights(shape, 2)
        t["w_out"] = t["w_out"] * 2.0 ** k
        t["b_out"] = t["b_out"] * 2.0 ** k
        t["energy_bias"] = t["energy_bias"] * 2.0 ** k
        synth.write_weights(p, shape, t)
        m = binding.Model(p, RC, SEL)
        try:
            if precision == "bf16":
                m.set_precision(binding.PREC_BF16)
            _, F, V, _ = m.compute(x, types, None, len(x), 0)
            got.append((F * 2.0 ** -k, V * 2.0 ** -k))
        finally:
            m.close()
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
