"""Adjoint products on two-term f16 operands, at the edges of their shapes.

The adjoint of the attention core takes its operands the same way, in classes
of up to 32, 64, 96 and 128 neighbours (the 96 class two centres to a
workgroup): compact clusters in which every atom is every other one's
neighbour put all centres at the edges of the classes.

The adjoints of the attention projections run on split operands for embedding
widths of 97 to 112: one to four real features in the last 16-wide chunk
(97, 100), a fuller last chunk (104) and the widest one, whose QKV adjoint
does not fit the resident kernel and stays on FP32 operands (112).  Forces are
compared with the FP64 oracle at the bounds of the FP32 parity tests, for a
periodic box and for open clusters whose pair counts leave ragged row tiles
(one pair, a few, more than one tile).
"""

import numpy as np
import pytest

from oracle import dpa1_oracle as orc
from paper_2604_07276_amd import synth

pytestmark = pytest.mark.gpu

RC, SEL = 6.0, 120
E_TOL, F_TOL = 1e-6, 1e-4  # eV per atom, eV/A: the FP32 parity bounds


@pytest.mark.parametrize("width", [97, 100, 104, 112])
@pytest.mark.parametrize("atoms", [2, 9, 41, 192])
def test_split_adjoints_match_oracle(width, atoms, tmp_path):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_07276_amd import binding
    print(f"case: split adjoints, width {width}, {atoms} atoms", flush=True)
    p = str(tmp_path / "w.bin")
    synth.make_weights(p, seed=5, shape=synth.ModelShape(emb=(25, 50, width)))
    s = synth.parity_system(2) if atoms == 192 else synth.open_cluster(atoms, 4.0, 5, seed=atoms)
    m = binding.Model(p, RC, SEL)
    try:
        E, F, _, _ = m.compute(s.coords, s.types, s.box, atoms, 0)
    finally:
        m.close()
    r = orc.compute(orc.load_model(p), s.coords, s.types, s.box, atoms, 0, RC, SEL)
    assert abs(E - r.energy) <= E_TOL * atoms
    assert np.abs(F - r.forces).max() <= F_TOL


def compact_cluster(atoms, seed):
    """The grid points nearest to a grid's centre, 0.95 A apart with a little jitter: every pair
    of up to 121 atoms is within the cutoff."""
    rng = np.random.default_rng(seed)
    g = np.stack(np.meshgrid(*[np.arange(-4, 5) * 0.95] * 3, indexing="ij"), -1).reshape(-1, 3)
    x = g[np.argsort((g * g).sum(1), kind="stable")[:atoms]]
    return x + rng.uniform(-0.03, 0.03, x.shape), rng.integers(0, 5, atoms).astype(np.int32)


@pytest.mark.parametrize("neighbours", [16, 31, 32, 33, 63, 64, 65, 80, 95, 96, 97, 119, 120])
def test_split_attention_adjoint_at_class_edges(neighbours, tmp_path):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_07276_amd import binding
    print(f"case: split attention adjoint, {neighbours} neighbours", flush=True)
    p = str(tmp_path / "w.bin")
    synth.make_weights(p, seed=2)
    x, types = compact_cluster(neighbours + 1, neighbours)
    m = binding.Model(p, RC, SEL)
    try:
        E, F, _, _ = m.compute(x, types, None, len(x), 0)
        _, nn = m.debug_nlist(len(x))
        # the same centres beside a small class: other class lists, the same bits
        far = np.concatenate([x, x[:5] + 40.0])
        _, F2, _, _ = m.compute(far, np.concatenate([types, types[:5]]), None, len(far), 0)
    finally:
        m.close()
    assert (nn == neighbours).all()
    r = orc.compute(orc.load_model(p), x, types, None, len(x), 0, RC, SEL)
    # the FP32 parity bound, 1e-4 eV/A, at the 0.02 eV/A of the systems it is stated for
    rms = np.sqrt(np.mean(r.forces ** 2))
    assert abs(E - r.energy) <= E_TOL * len(x)
    assert np.abs(F - r.forces).max() <= F_TOL * max(1.0, rms / 0.02)
    assert np.array_equal(F2[:len(x)], F)
