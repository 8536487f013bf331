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


def test_adjoint_of_a_refused_forward(tmp_path):
    """A forward that is refused for its memory leaves no earlier forward to differentiate (its
    pair offsets are the new system's by then), and the handle goes on with what fits."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_07276_amd import binding
    print("case: adjoint after a forward over the memory budget, 150 atoms", flush=True)
    p = str(tmp_path / "w.bin")
    synth.make_weights(p, seed=3)
    c = synth.open_cluster(150, 9.0, 5, seed=9)
    dev = torch.device("cuda:0")
    x0 = torch.tensor(c.coords, device=dev)
    x1 = 0.7 * x0  # more than twice the neighbour pairs
    t = torch.tensor(c.types, device=dev)
    e = torch.zeros(1, dtype=torch.float64, device=dev)
    g = torch.zeros((150, 3), dtype=torch.float64, device=dev)
    m = binding.Model(p, RC, SEL)
    try:
        m.forward_device(x0, t, None, 150, 0, e)
        m.backward_device(g)
        m.sync()
        want = g.clone()
        m.set_memory_budget(m.memory_info()[0])
        m.forward_device(x0, t, None, 150, 0, e)
        m.sync()
        m.forward_device(x1, t, None, 150, 0, e)
        with pytest.raises(binding.DPError) as ei:
            m.sync()
        assert ei.value.code == -8
        with pytest.raises(binding.DPError) as ei:
            m.forward_device(x1, t, None, 150, 0, e)
        assert ei.value.code == -7
        with pytest.raises(binding.DPError) as ei:
            m.backward_device(g)
        assert ei.value.code == -1
        m.set_memory_budget(0)
        m.forward_device(x0, t, None, 150, 0, e)
        m.backward_device(g)
        m.sync()
        assert torch.equal(g, want)
    finally:
        m.close()


@pytest.mark.parametrize("atoms", [192, 2000, 9000])
def test_captured_steps_of_both_precisions(atoms, tmp_path):
    """Steps captured in FP32 and, after the precision was set and without a step in between, in
    BF16 on one handle: both graphs replay in turn, on other coordinates, with an eager step's
    bits."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_07276_amd import binding
    print(f"case: captured steps, {atoms} atoms", flush=True)
    p = str(tmp_path / "w.bin")
    synth.make_weights(p, seed=3)
    s = synth.lattice_system(atoms, (atoms / 0.1) ** (1 / 3), (0.64, 0.10, 0.03, 0.22, 0.01), seed=0)
    dev = torch.device("cuda:0")
    x0 = torch.tensor(s.coords, device=dev)
    x, t = x0.clone(), torch.tensor(s.types, device=dev)

    def outputs():
        return [torch.zeros(k, dtype=torch.float64, device=dev) for k in (1, (atoms, 3), 9)]

    m, eager = binding.Model(p, RC, SEL), binding.Model(p, RC, SEL)
    try:
        got, graphs = {}, {}
        for prec in (binding.PREC_FP32, binding.PREC_BF16):
            m.set_precision(prec)
            got[prec] = outputs()
            if prec == binding.PREC_FP32:
                m.compute_device(x, t, s.box, atoms, 0, *got[prec])
                m.sync()
            torch.cuda.synchronize()
            graphs[prec] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graphs[prec]):
                m.compute_device(x, t, s.box, atoms, 0, *got[prec])
        for k in range(3):
            noise = np.random.default_rng(k).normal(0.0, 0.01, (atoms, 3))
            x.copy_(x0 + torch.tensor(noise, device=dev))
            for prec, graph in graphs.items():
                graph.replay()
                torch.cuda.synchronize()
                eager.set_precision(prec)
                want = outputs()
                eager.compute_device(x, t, s.box, atoms, 0, *want)
                eager.sync()
                assert all(torch.equal(a, b) for a, b in zip(got[prec], want))
    finally:
        m.close()
        eager.close()
