"""Binning, neighbour lists and pair offsets at the edges of their routes.

Up to 8192 atoms and 4096 cells one block bins the atoms (1024 threads, several
atoms and cells each), beyond that five launches; the pair offsets come from one
block with chunks of a multiple of four centres, which also lists the attention
classes of up to 4096 centres.  Lists are compared with the oracle's, the
energies of a repeated step (the first lays the workspace out and takes a path
of its own) with the first one's, and the two attention routes through them.
"""

import numpy as np
import pytest

from oracle import dpa1_oracle as orc
from paper_2604_07276_amd import synth

pytestmark = pytest.mark.gpu

RC, SEL = 6.0, 120


def gas(n, length, seed):
    """n atoms in a periodic cube: a jittered subset of a grid, at least 0.9 A apart."""
    rng = np.random.default_rng(seed)
    side = int(np.ceil(n ** (1 / 3)))
    step = length / side
    assert step > 1.3
    g = np.stack(np.meshgrid(*[(np.arange(side) + 0.5) * step] * 3, indexing="ij"), -1)
    x = rng.permutation(g.reshape(-1, 3))[:n] + rng.uniform(-0.2, 0.2, (n, 3))
    return x, rng.integers(0, 5, n).astype(np.int32), np.diag([length] * 3)


@pytest.mark.parametrize("n,length", [(5, 13.0), (600, 112.0), (1023, 30.0), (1025, 30.0),
                                      (4097, 46.0), (8192, 58.0), (8193, 58.0)])
def test_lists_at_route_edges(n, length, tmp_path):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_07276_amd import binding
    print(f"case: cells, {n} atoms, box {length}", flush=True)
    p = str(tmp_path / "w.bin")
    synth.make_weights(p, seed=2, shape=synth.STUDENT_SHAPE)
    x, types, box = gas(n, length, n)
    m = binding.Model(p, RC, SEL)
    try:
        first = m.compute(x, types, box, n, 0, True)
        again = m.compute(x, types, box, n, 0, True)
        nl, nn = m.debug_nlist(n)
        bad = types.copy()
        bad[n - 1] = 7
        with pytest.raises(binding.DPError):
            m.compute(x, bad, box, n, 0)
        last = m.compute(x, types, box, n, 0, True)
    finally:
        m.close()
    ref = orc.neighbor_list(x, box, RC, np.arange(n))
    for i in range(n):
        k = len(ref[i])
        assert nn[i] == k and np.array_equal(nl[i, :k], ref[i]) and np.all(nl[i, k:] == -1), i
    for a, b, c in zip(first, again, last):
        assert np.array_equal(a, b) and np.array_equal(a, c)


@pytest.mark.parametrize("n", [4096, 4097])
def test_attention_lists_at_route_edges(n, tmp_path):
    """The classes listed by the scan's block and by a launch of their own: the same bits as the
    first step, whose classes are always listed by the launch."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_07276_amd import binding
    print(f"case: attention class lists, {n} atoms", flush=True)
    p = str(tmp_path / "w.bin")
    synth.make_weights(p, seed=2, shape=synth.ModelShape())
    x, types, box = gas(n, 46.0, n)
    m = binding.Model(p, RC, SEL)
    try:
        first = m.compute(x, types, box, n, 0, True)
        for _ in range(2):
            again = m.compute(x, types, box, n, 0, True)
            for a, b in zip(first, again):
                assert np.array_equal(a, b)
    finally:
        m.close()


@pytest.mark.parametrize("shift", [0.0, 0.1])
@pytest.mark.parametrize("length,away", [(18.0, 0), (24.0, 0), (24.0, 3000)])
def test_pairs_at_the_cutoff(length, away, shift, tmp_path):
    """A 2 A lattice has pairs at exactly 6 A along the axes and the (4, 4, 2) directions: the
    periodic test without divisions must take the same ones as the oracle, also for atoms many
    boxes away and with coordinates that round."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_07276_amd import binding
    print(f"case: pairs at the cutoff, box {length}, {away} boxes away, shift {shift}", flush=True)
    p = str(tmp_path / "w.bin")
    synth.make_weights(p, seed=2, shape=synth.STUDENT_SHAPE)
    g = np.arange(0.0, length, 2.0)
    x = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3) + shift
    n = len(x)
    rng = np.random.default_rng(n)
    x = x + length * away * rng.integers(-1, 2, (n, 3))
    box = np.diag([length] * 3)
    m = binding.Model(p, RC, SEL)
    try:
        m.compute(x, rng.integers(0, 5, n).astype(np.int32), box, n, 0)
        nl, nn = m.debug_nlist(n)
    finally:
        m.close()
    ref = orc.neighbor_list(x, box, RC, np.arange(n))
    for i in range(n):
        k = len(ref[i])
        assert nn[i] == k and np.array_equal(nl[i, :k], ref[i]), i


@pytest.mark.parametrize("atoms", [1, 3])
def test_attention_free_model_without_pairs(atoms, tmp_path):
    """Atoms out of each other's reach: no pair row exists, so no pair kernel has a grid."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_07276_amd import binding
    print(f"case: no pairs, {atoms} atoms", flush=True)
    p = str(tmp_path / "w.bin")
    synth.make_weights(p, seed=2, shape=synth.STUDENT_SHAPE)
    x = np.arange(3.0 * atoms).reshape(atoms, 3) * 20.0
    types = np.arange(atoms, dtype=np.int32)
    m = binding.Model(p, RC, SEL)
    try:
        for _ in range(2):
            E, F, V, _ = m.compute(x, types, None, atoms, 0)
    finally:
        m.close()
    r = orc.compute(orc.load_model(p), x, types, None, atoms, 0, RC, SEL)
    assert abs(E - r.energy) <= 1e-6 * atoms
    assert not F.any() and not V.any()
