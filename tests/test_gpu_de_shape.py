"""DE steps in the default launch shape at sizes around its changes against the
oracle."""
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


# (group, chunk) pairs on both sides of the two- and four-pass rule, the
# smallest population, partial groups, chunks and words
@pytest.mark.parametrize("n,npop", [(1, 4), (1023, 63), (1024, 1020), (1025, 1021), (4099, 961), (257, 4099)])
def test_de_default_shape_matches_oracle(q, orc, n, npop):
    x, _ = q.init_population(npop, n, seed=7)
    u, ub = q.de_step(x, n, 0.7, 0.6, seed=11, generation=5)
    uo, _ = orc.de_step(x.cpu().numpy()[:, :n], 0.7, 0.6, seed=11, g=5)
    assert np.array_equal(u.cpu().numpy()[:, :n], uo)
    want = inputs.pack_bits(np.where(uo < 0, -1, 1), ub.shape[1])
    assert np.array_equal(ub.cpu().numpy().view(np.uint32), want)
    assert not u.cpu().numpy()[:, n:].any()
