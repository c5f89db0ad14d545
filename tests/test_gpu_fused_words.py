"""Fused generations from precomputed random numbers where their layout changes:
one to five rounds per thread, individuals that straddle rounds, padded quads,
generation counts on both sides of one launch's 64, each algorithm."""
import numpy as np
import pytest

from paper_2511_01255_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q():
    import torch
    assert torch.cuda.is_available(), "a GPU is required"
    from paper_2511_01255_amd import qpm
    qpm.lib()
    return qpm


@pytest.mark.parametrize("n,npop,parts,algo,variant", [
    (4990, 4, (5, 2), 0, 0),     # five rounds, the largest rows
    (33, 64, (1, 63, 6), 0, 1),  # 7 of 16 quads padding, one round
    (640, 30, (64, 1), 0, 0),    # 160 quads: individuals straddle rounds
    (130, 37, (65,), 1, 0),      # DE alone
    (1999, 10, (9,), 2, 0),      # grey wolf alone
], ids=lambda v: str(v).replace(" ", ""))
def test_fused_rounds_equal_oracle(q, orc, n, npop, parts, algo, variant):
    G = sum(parts)
    z = inputs.uniform_boundaries(n, 2.0)
    xo, fo, _, _ = orc.Design(z, inputs.DK1, inputs.DK2).run_algo(npop, G, 0.5, 0.9, 21, algo, inst=2,
                                                                  variant=variant, control=0)
    D = q.precompute_phases(z, inputs.DK1, inputs.DK2)
    R = q.Run(D, npop, G, seed=21, inst=2, prec=1, gwo_variant=variant, algo=algo, fused=1)
    for k in parts:
        R.advance(k)
    x, f, _, _ = R.read()
    R.destroy()
    assert np.array_equal(x.cpu().numpy(), xo)
    assert np.max(np.abs(f.cpu().numpy() - fo) / np.maximum(fo, 1e-300)) <= 1e-12
