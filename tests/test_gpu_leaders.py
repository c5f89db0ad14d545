"""The leaders of a generation where their reductions change form: one to many
groups of candidates, more than 64 and more than 256 of them, populations of
equal fitness values, and grey-wolf steps on both sides of the size up to which
they merge the candidates themselves. Every decision is the oracle's."""
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


@pytest.mark.parametrize("algo", [0, 1, 2])
@pytest.mark.parametrize("n,npop", [(40, 65), (3, 300), (1, 130), (40, 1345), (33, 5461), (33, 5500), (1025, 1500),
                                    (1025, 1501)])
def test_leaders_equal_oracle(q, orc, n, npop, algo):
    G = 3
    z = inputs.uniform_boundaries(n, 2.0)
    xo, fo, _, _ = orc.Design(z, inputs.DK1, inputs.DK2).run_algo(npop, G, 0.5, 0.9, 5, algo, inst=1, variant=0,
                                                                  control=0)
    R = q.Run(q.precompute_phases(z, inputs.DK1, inputs.DK2), npop, G, seed=5, inst=1, prec=1, algo=algo, fused=-1)
    R.advance(G)
    x, f, L, _ = R.read()
    R.destroy()
    x, f = x.cpu().numpy(), f.cpu().numpy()
    assert np.array_equal(x, xo)
    assert np.max(np.abs(f - fo) / np.maximum(fo, 1e-300)) <= 1e-12
    if algo != 0:  # the leaders of the final population: best first, lowest slot first
        assert L == list(np.lexsort((np.arange(npop), -f))[:3])
