"""Attention classes with several centres to a workgroup, all of them at work.

The forward puts up to four centres into a workgroup and the BF16 adjoint up to
six, each with wavefronts, LDS and barriers of its own; part p of a workgroup
takes the centres p grids further on in the class list.  A cluster in which
every atom is every other one's neighbour is computed alone, where only part 0
has centres, and as so many copies of itself, out of each other's reach, that
every part takes more than one.  Every copy must have the energies and forces of
the one, bit for bit.

BF16 forces are compared with the oracle on operands rounded to BF16, at 1e-2 of
their root mean square: what that rounding does to them, against which FP32
noise at the rounding's boundaries remains.
"""

import numpy as np
import pytest

import bf16_oracle
from clusters import compact_cluster
from oracle import dpa1_oracle as orc
from paper_2604_07276_amd import synth

RC, SEL = 6.0, 120
NEIGHBOURS = [16, 31, 32, 33, 63, 64, 65, 95, 96, 97, 120]


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("neighbours", NEIGHBOURS)
def test_copies_equal_one(neighbours, precision, tmp_path):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_07276_amd import binding
    n = neighbours + 1
    # centres to a workgroup: at most 6, 3, 2 and 1 in the classes of 32, 64, 96 and 128; a second
    # round of every part with the persistent grid of one workgroup per CU
    parts = 6 if neighbours <= 32 else 3 if neighbours <= 64 else 2
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    copies = (parts + 1) * cus // n + 3
    print(f"case: {copies} clusters of {neighbours} neighbours, {precision}", flush=True)
    p = str(tmp_path / "w.bin")
    synth.make_weights(p, seed=2)
    x, types = compact_cluster(n, neighbours)
    x = np.round(x * 2.0 ** 20) / 2.0 ** 20  # differences are exact at every offset
    side = int(np.ceil(copies ** (1 / 3)))
    at = 32.0 * np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij"), -1).reshape(-1, 3)
    many = (at[:copies, None, :] + x).reshape(-1, 3)
    m = binding.Model(p, RC, SEL)
    try:
        m.set_precision(binding.PREC_FP32 if precision == "fp32" else binding.PREC_BF16)
        _, F1, _, e1 = m.compute(x, types, None, n, 0, True)
        _, F, _, e = m.compute(many, np.tile(types, copies), None, len(many), 0, True)
        _, nn = m.debug_nlist(len(many))
    finally:
        m.close()
    assert (nn == neighbours).all() and len(many) > parts * cus + cus
    assert np.array_equal(e.reshape(copies, n), np.tile(e1, (copies, 1)))
    assert np.array_equal(F.reshape(copies, n, 3), np.tile(F1, (copies, 1, 1)))


@pytest.mark.gpu
@pytest.mark.parametrize("neighbours", [1, 15, 17, 48, 81] + NEIGHBOURS)
def test_bf16_forces_match_rounded_oracle(neighbours, tmp_path, monkeypatch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_07276_amd import binding
    print(f"case: BF16 forces, {neighbours} neighbours", flush=True)
    p = str(tmp_path / "w.bin")
    synth.make_weights(p, seed=2)
    x, types = compact_cluster(neighbours + 1, neighbours)
    m = binding.Model(p, RC, SEL)
    try:
        m.set_precision(binding.PREC_BF16)
        _, F, _, _ = m.compute(x, types, None, len(x), 0)
    finally:
        m.close()
    r = bf16_oracle.compute(monkeypatch, orc.load_model(p), x, types, None, len(x), RC, SEL).forces
    err = np.sqrt(np.mean((F - r) ** 2) / np.mean(r ** 2))
    print(f"relative force error {err:.1e}", flush=True)
    assert err <= 1e-2


def test_rounded_oracle_without_rounding_is_the_oracle(tmp_path, monkeypatch):
    p = str(tmp_path / "w.bin")
    synth.make_weights(p, seed=2)
    x, types = compact_cluster(12, 11)
    model = orc.load_model(p)
    a = bf16_oracle.compute(monkeypatch, model, x, types, None, 12, RC, SEL, rounding=lambda v: v)
    b = orc.compute(model, x, types, None, 12, 0, RC, SEL)
    assert np.abs(a.forces - b.forces).max() <= 1e-12 * np.abs(b.forces).max()
    assert np.abs(a.atom_energy - b.atom_energy).max() <= 1e-12
