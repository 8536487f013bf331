"""The same inputs give the same bits whatever the handle computed before.

The first fitting layer is summed in slices for up to 4095 centres; whether it
is must not depend on the size that earlier steps gave the workspace.  Sparse
systems, whose own workspace is small, are computed on a fresh handle and again
after a larger, denser system on the same handle.
"""

import numpy as np
import pytest

from paper_2604_07276_amd import synth

pytestmark = pytest.mark.gpu

RC, SEL = 6.0, 120


def dimers(atoms):
    """Pairs of atoms 2 A apart, 9 A from each other: one neighbour to an atom."""
    side = int(np.ceil((atoms / 2) ** (1 / 3)))
    at = 9.0 * np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij"), -1).reshape(-1, 3)
    x = np.repeat(at, 2, axis=0)
    x[1::2, 0] += 2.0
    x += np.random.default_rng(atoms).uniform(-0.2, 0.2, x.shape)
    return x[:atoms], np.random.default_rng(1).integers(0, 5, atoms).astype(np.int32)


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("model", ["student", "dpa1"])
@pytest.mark.parametrize("atoms", [2, 15, 1024, 1025, 1500, 4095])
def test_bits_do_not_depend_on_earlier_steps(atoms, model, precision, tmp_path):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_07276_amd import binding
    print(f"case: {atoms} sparse atoms after a larger system, {model}, {precision}", flush=True)
    p = str(tmp_path / "w.bin")
    shape = synth.STUDENT_SHAPE if model == "student" else synth.ModelShape()
    synth.make_weights(p, seed=3, shape=shape)
    if atoms == 15:
        s = synth.open_cluster(15, 5.0, 5, seed=15)
        x, types = s.coords, s.types
    else:
        x, types = dimers(atoms)
    n = max(1100, atoms + 1)
    larger = synth.lattice_system(n, (n / 0.1) ** (1 / 3), (0.64, 0.10, 0.03, 0.22, 0.01), seed=0)
    m = binding.Model(p, RC, SEL)
    try:
        m.set_precision(binding.PREC_FP32 if precision == "fp32" else binding.PREC_BF16)
        first = m.compute(x, types, None, atoms, 0, True)
        m.compute(larger.coords, larger.types, larger.box, n, 0)
        again = m.compute(x, types, None, atoms, 0, True)
    finally:
        m.close()
    assert first[0] == again[0]
    assert all(np.array_equal(a, b) for a, b in zip(first[1:], again[1:]))


def test_precision_changes_on_one_handle(tmp_path):
    """FP32 lays out no buffers that only the BF16 128 class reads; BF16 adds them when it is set,
    and both give a fresh handle's bits in any order."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_07276_amd import binding
    print("case: FP32 and BF16 in turn, 600 atoms of 94 to 119 neighbours", flush=True)
    p = str(tmp_path / "w.bin")
    synth.make_weights(p, seed=3)
    s = synth.lattice_system(600, (600 / 0.118) ** (1 / 3), (0.64, 0.10, 0.03, 0.22, 0.01), seed=0)
    want = {}
    for prec in (binding.PREC_FP32, binding.PREC_BF16):
        m = binding.Model(p, RC, SEL)
        m.set_precision(prec)
        want[prec] = m.compute(s.coords, s.types, s.box, 600, 0)
        want[prec, "bytes"] = m.memory_info()[0]
        m.close()
    assert want[binding.PREC_FP32, "bytes"] < want[binding.PREC_BF16, "bytes"]
    m = binding.Model(p, RC, SEL)
    try:
        for prec in (binding.PREC_FP32, binding.PREC_BF16, binding.PREC_FP32, binding.PREC_BF16):
            m.set_precision(prec)
            before = m.memory_info()[0]
            got = m.compute(s.coords, s.types, s.box, 600, 0)
            assert got[0] == want[prec][0]
            assert all(np.array_equal(a, b) for a, b in zip(got[1:3], want[prec][1:3]))
            assert before in (0, m.memory_info()[0])  # laid out by the call that needs it
    finally:
        m.close()
    # a budget that holds the FP32 layout without recomputation, and the BF16 one only with it
    m = binding.Model(p, RC, SEL)
    try:
        m.set_memory_budget(want[binding.PREC_FP32, "bytes"])
        got = m.compute(s.coords, s.types, s.box, 600, 0)
        assert not m.memory_info()[1] and np.array_equal(got[1], want[binding.PREC_FP32][1])
        m.set_precision(binding.PREC_BF16)
        assert m.memory_info()[1]
        got = m.compute(s.coords, s.types, s.box, 600, 0)
        assert np.array_equal(got[1], want[binding.PREC_BF16][1])
    finally:
        m.close()
