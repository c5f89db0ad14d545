"""An untuned multi-kernel run and a call score a population on one plan: the
fitness a run holds equals that of qpm_eval_fitness for the same signs and the
same population size, bit for bit. Objectives: the same here (a call on a short
design may add its words in another order, which FP64 shows at 5 to 8 words)."""
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


def _bits(x):
    import torch
    s = np.where(x.cpu().numpy() < 0, -1, 1).astype(np.int8)
    return torch.from_numpy(inputs.pack_bits(s).view(np.int32)).cuda()


# one segment up to 20 words, 2 and more words per wave, 31 to 48 and more
# segments, staged walks
@pytest.mark.parametrize("prec", [1, 0])
@pytest.mark.parametrize("n,npop", [(128, 80), (300, 70), (500, 1000), (640, 300), (641, 300), (2000, 500),
                                    (7680, 130), (12224, 86), (12472, 86), (13000, 200), (20000, 300), (30000, 130),
                                    (31000, 80), (10000, 1300), (49999, 1001), (640, 19264), (600, 38500)])
def test_run_fitness_equals_the_call(q, n, npop, prec):
    D = q.precompute_phases(inputs.jittered_boundaries(n, 2.0, 0.2, seed=n), inputs.DK1, inputs.DK2)
    R = q.Run(D, npop, 4, seed=5, prec=prec, fused=-1)
    for g in (0, 2):
        R.advance(g)
        x, f, _, _ = R.read()
        e = q.eval_fitness(D, _bits(x), npop, prec)
        assert np.array_equal(f.cpu().numpy(), e.cpu().numpy()), (n, npop, g)
    R.destroy()


@pytest.mark.parametrize("prec", [1, 0])
@pytest.mark.parametrize("kind,K", [("shg", 1), ("shg", 5), ("thg", 1), ("thg", 3)])
@pytest.mark.parametrize("n,npop", [(100, 70), (500, 300), (640, 90), (3000, 500), (9000, 300)])
def test_objective_run_equals_the_call(q, n, npop, kind, K, prec):
    z = inputs.uniform_boundaries(n, 3.0)
    periods = (6.2, 6.9, 8.1, 9.3, 11.7)
    if kind == "shg":
        dks = [(2 * np.pi / p, 0.0) for p in periods[:K]]
    else:
        dks = [(inputs.DK1, inputs.DK2), (0.30, 0.90), (0.31, 0.97)][:K]
    ds = [q.precompute_phases(z, a, b) for a, b in dks]
    O = q.Objective(ds, q.OBJ_SHG if kind == "shg" else q.OBJ_THG, beta=0.1)
    R = q.Run(O, npop, 4, seed=5, prec=prec)
    R.advance(2)
    x, f, _, _ = R.read()
    assert np.array_equal(f.cpu().numpy(), q.eval_objective(O, _bits(x), npop, prec).cpu().numpy())
    R.destroy()
