"""Systems of different neighbour counts taking turns on one handle.

The attention classes to launch are chosen from the counts of a recent step, so
the first step after a sparser (or less dense) one finds its centres in classes
that were empty.  Such a step must take about as long as the same step among
its own kind (twice as long at most: a grid left at a few workgroups takes six
times as long) and give the same bits.
"""

import numpy as np
import pytest

from paper_2604_07276_amd import synth

pytestmark = pytest.mark.gpu

RC, SEL = 6.0, 120
FRACTIONS = (0.64, 0.10, 0.03, 0.22, 0.01)


def neighbours(s):
    from scipy.spatial import cKDTree
    x = np.mod(s.coords, np.diag(s.box))
    return np.array([len(q) - 1 for q in cKDTree(x, boxsize=np.diag(s.box)).query_ball_point(x, RC)])


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("atoms", [600, 4096])
@pytest.mark.parametrize("before, after", [(0.045, 0.085), (0.085, 0.118)])
def test_step_after_a_sparser_one(before, after, atoms, precision, tmp_path):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_07276_amd import binding
    print(f"case: {atoms} atoms at {after} after {before} per cubic A, {precision}", flush=True)
    p = str(tmp_path / "w.bin")
    synth.make_weights(p, seed=2)
    systems = [synth.lattice_system(atoms, (atoms / rho) ** (1 / 3), FRACTIONS, seed=0)
               for rho in (before, after)]
    few, many = (neighbours(s) for s in systems)
    # no centre of the one is in the class of the other's bulk
    top = 32 * ((np.median(many) - 1) // 32)
    assert few.max() <= top and many.max() <= SEL
    dev = torch.device("cuda:0")
    args = [(torch.tensor(s.coords, device=dev), torch.tensor(s.types, device=dev), s.box)
            for s in systems]
    e = torch.zeros(1, dtype=torch.float64, device=dev)
    f = torch.zeros((atoms, 3), dtype=torch.float64, device=dev)
    v = torch.zeros(9, dtype=torch.float64, device=dev)
    m = binding.Model(p, RC, SEL)

    def step(k):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        start.record()
        x, t, box = args[k]
        m.compute_device(x, t, box, atoms, 0, e, f, v)
        end.record()
        m.sync()
        return start.elapsed_time(end)

    try:
        if precision == "bf16":
            m.set_precision(binding.PREC_BF16)
        step(0)  # lays the workspace out for the larger box
        with pytest.raises(binding.DPError):
            step(1)  # more pairs than the workspace holds: it grows at the next call
        step(1)
        usual, mixed = [], []
        for _ in range(5):
            step(1)
            usual.append(step(1))
            want = f.clone()
            step(0)
            step(0)
            mixed.append(step(1))
            assert torch.equal(f, want)
    finally:
        m.close()
    print(f"us: usual {1e3 * min(usual):.0f}, after the other {1e3 * min(mixed):.0f}", flush=True)
    assert min(mixed) <= 2.0 * min(usual)
