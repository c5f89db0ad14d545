"""Fused generations in launches of one to three make their random numbers
themselves, longer ones read those of a launch before: the trajectory is the same
however the generations are split into calls."""
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


# 1 to 5 rounds of 1024 (individual, gene quad) slots per generation
@pytest.mark.parametrize("prec", [1, 0])
@pytest.mark.parametrize("algo", [0, 1, 2])
@pytest.mark.parametrize("n,npop,variant", [(5, 4, 0), (64, 8, 1), (100, 16, 0), (256, 32, 0), (191, 64, 1), (800, 15, 0),
                                            (1000, 16, 0), (300, 64, 1), (2500, 8, 0)])
def test_generations_in_any_split(q, n, npop, variant, algo, prec):
    D = q.precompute_phases(inputs.jittered_boundaries(n, 2.0, 0.2, seed=n), inputs.DK1, inputs.DK2)
    out = []
    for split in ((12,), (1, 1, 2, 3, 1, 4), (3, 3, 3, 3)):
        R = q.Run(D, npop, 12, seed=9, prec=prec, fused=1, algo=algo, gwo_variant=variant)
        for k in split:
            R.advance(k)
        x, f, L, g = R.read()
        out.append((x.cpu().numpy(), f.cpu().numpy(), L, g))
        R.destroy()
    for x, f, L, g in out[1:]:
        assert np.array_equal(x, out[0][0]) and np.array_equal(f, out[0][1]) and (L, g) == out[0][2:]
