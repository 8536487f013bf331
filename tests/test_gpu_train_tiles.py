"""Student trainer at the edges of its row and pair tiles.

The pair passes take a centre's neighbours in tiles of 16, and the weight
gradients take atoms and pairs in steps of 64 rows and less: compact clusters
whose neighbour count is one, a tile less one, a tile, a tile and one and a
ragged few, plus an atom without neighbours.  Loss and gradient are compared
with the FP64 double-backward oracle at the bounds of the trainer's parity
tests.
"""

import numpy as np
import pytest

from oracle import dpa1_oracle as orc
from oracle import train_oracle as tro
from paper_2604_07276_amd import synth

pytestmark = pytest.mark.gpu

RC, SEL, PE, PF = 6.0, 120, 1.0, 100.0


def cluster(neighbours, seed):
    """neighbours + 1 atoms near a grid, all within the cutoff of each other (the grid points
    nearest to its centre, 0.95 A apart, with a little jitter), and one atom far away."""
    rng = np.random.default_rng(seed)
    g = np.stack(np.meshgrid(*[np.arange(-4, 5) * 0.95] * 3, indexing="ij"), -1).reshape(-1, 3)
    x = g[np.argsort((g * g).sum(1), kind="stable")[:neighbours + 1]]
    x = x + rng.uniform(-0.03, 0.03, x.shape)
    return np.vstack([x, [[40.0, 0.0, 0.0]]]), rng.integers(0, 5, neighbours + 2).astype(np.int32)


@pytest.mark.parametrize("neighbours", [1, 15, 16, 17, 63, 66])
@pytest.mark.parametrize("precision,tol", [("fp32", 1e-4), ("bf16", 5e-2)])
def test_gradient_at_tile_edges(precision, tol, neighbours, tmp_path):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_07276_amd import binding
    print(f"case: trainer tiles, {neighbours} neighbours, {precision}", flush=True)
    p = str(tmp_path / "student.bin")
    synth.make_weights(p, seed=1, shape=synth.STUDENT_SHAPE)
    x, types = cluster(neighbours, seed=neighbours)
    frames = x[None]
    rng = np.random.default_rng(31)
    e_lab, f_lab = rng.normal(0.0, 1.0, size=1), rng.normal(0.0, 0.05, size=frames.shape)
    model = orc.load_model(p)
    (L, _, _), grads = tro.loss_and_grad(model, frames, types, None, e_lab, f_lab, RC, SEL, PE,
                                         PF)
    ref = tro.flatten(model, grads)
    prec = binding.PREC_FP32 if precision == "fp32" else binding.PREC_BF16
    dev = torch.device("cuda:0")
    tr = binding.Trainer(p, RC, SEL, pref_e=PE, pref_f=PF, precision=prec)
    try:
        loss, g = tr.gradient(torch.tensor(frames, device=dev), torch.tensor(types, device=dev),
                              None, torch.tensor(e_lab, device=dev),
                              torch.tensor(f_lab, device=dev))
    finally:
        tr.close()
    assert loss[0] == pytest.approx(L, rel=1e-5 if precision == "fp32" else 2e-2)
    off = 0
    for k in tro.param_names(model):
        n = model.t[k].numel()
        a, b = g[off:off + n], ref[off:off + n]
        assert np.linalg.norm(a - b) <= tol * max(np.linalg.norm(b), 1e-30), k
        off += n
