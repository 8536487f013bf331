"""Adjoint products on two-term f16 operands, at the edges of their shapes.

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
