"""BF16 attention adjoint at the edges of its classes.

Classes of up to 32, 64 and 96 neighbours put six, three and two centres into a
workgroup, in tiles of 16 taken in pairs: compact clusters in which every atom
is every other one's neighbour put all centres at the edges of tiles and
classes.  Forces are compared with the FP64 oracle at the BF16 target, and must
keep their bits beside centres of another class.
"""

import numpy as np
import pytest

from oracle import dpa1_oracle as orc
from paper_2604_07276_amd import synth

pytestmark = pytest.mark.gpu

RC, SEL = 6.0, 120
F_RMSE = 5e-3  # eV/A: the stated BF16 target


def compact_cluster(atoms, seed):
    """The grid points nearest to a grid's centre, 0.95 A apart with a little jitter: every pair
    of up to 121 atoms is within the cutoff."""
    rng = np.random.default_rng(seed)
    g = np.stack(np.meshgrid(*[np.arange(-4, 5) * 0.95] * 3, indexing="ij"), -1).reshape(-1, 3)
    x = g[np.argsort((g * g).sum(1), kind="stable")[:atoms]]
    return x + rng.uniform(-0.03, 0.03, x.shape), rng.integers(0, 5, atoms).astype(np.int32)


@pytest.mark.parametrize("neighbours", [1, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 81, 95, 96])
def test_bf16_attention_adjoint_at_class_edges(neighbours, tmp_path):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_07276_amd import binding
    print(f"case: BF16 attention adjoint, {neighbours} neighbours", flush=True)
    p = str(tmp_path / "w.bin")
    synth.make_weights(p, seed=2)
    x, types = compact_cluster(neighbours + 1, neighbours)
    m = binding.Model(p, RC, SEL)
    try:
        m.set_precision(binding.PREC_BF16)
        _, F, _, _ = m.compute(x, types, None, len(x), 0)
        _, nn = m.debug_nlist(len(x))
        far = np.concatenate([x, x[:5] + 40.0])
        _, F2, _, _ = m.compute(far, np.concatenate([types, types[:5]]), None, len(far), 0)
    finally:
        m.close()
    assert (nn == neighbours).all()
    r = orc.compute(orc.load_model(p), x, types, None, len(x), 0, RC, SEL)
    # the target at the 0.02 eV/A of the systems it is stated for
    rms = np.sqrt(np.mean(r.forces ** 2))
    assert np.sqrt(np.mean((F - r.forces) ** 2)) <= F_RMSE * max(1.0, rms / 0.02)
    assert np.array_equal(F2[:len(x)], F)
