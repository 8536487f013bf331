"""Fitting-net products of few rows against the general ones.

Up to 1024 rows the fitting net's products take one wavefront per tile of
outputs instead of the streaming kernel's blocks, with every sum in the same
order.  Atoms of a cluster without other clusters in reach must therefore have
the same energies, bit for bit, whether the cluster is computed alone (few
rows, ragged tiles) or with enough copies of itself for the streaming kernel;
the forces, whose order of summation is by cells, agree to rounding.
"""

import numpy as np
import pytest

from paper_2604_07276_amd import synth

pytestmark = pytest.mark.gpu

RC, SEL = 6.0, 120


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("atoms", [2, 15, 17, 100])
def test_few_rows_equal_many(atoms, precision, tmp_path):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_07276_amd import binding
    print(f"case: few fitting rows, {atoms} atoms, {precision}", flush=True)
    p = str(tmp_path / "w.bin")
    synth.make_weights(p, seed=3, shape=synth.STUDENT_SHAPE)
    s = synth.open_cluster(atoms, 2.0 if atoms < 15 else 5.0, 5, seed=atoms)
    x = np.round(s.coords * 2.0 ** 20) / 2.0 ** 20  # differences are exact at every offset
    copies = 1025 // atoms + 1
    side = int(np.ceil(copies ** (1 / 3)))
    at = 32.0 * np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij"), -1).reshape(-1, 3)
    many = (at[:copies, None, :] + x).reshape(-1, 3)
    prec = binding.PREC_FP32 if precision == "fp32" else binding.PREC_BF16
    m = binding.Model(p, RC, SEL)
    try:
        m.set_precision(prec)
        _, F1, _, e1 = m.compute(x, s.types, None, atoms, 0, True)
        _, F2, _, e2 = m.compute(many, np.tile(s.types, copies), None, len(many), 0, True)
    finally:
        m.close()
    assert len(many) > 1024
    e2, F2 = e2.reshape(copies, atoms), F2.reshape(copies, atoms, 3)
    assert np.array_equal(e1, e2[0])
    assert np.abs(F1 - F2[0]).max() <= 1e-6 * max(1.0, np.abs(F1).max())
