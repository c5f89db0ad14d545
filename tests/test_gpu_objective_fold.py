"""The fold of the objective's segments where its batches of designs and its
default launch shape change: 1, 4, 5 and 8 designs in runs (FP64, every decision
the oracle's), evaluations on both sides of 256 and 400 workgroups and of 48
segments, with partial groups of 16 and 64 genomes."""
import numpy as np
import pytest

from paper_2511_01255_amd import inputs

pytestmark = pytest.mark.gpu

DKS = [(inputs.DK1 * (1.0 + 0.03 * k), inputs.DK2 * (1.0 - 0.02 * k)) for k in range(8)]


@pytest.fixture(scope="module")
def q():
    import torch
    assert torch.cuda.is_available(), "a GPU is required"
    from paper_2511_01255_amd import qpm
    qpm.lib()
    return qpm


def _pair(q, orc, z, K, kind):
    gd = [q.precompute_phases(z, k1, k2) for k1, k2 in DKS[:K]]
    od = [orc.Design(z, k1, k2) for k1, k2 in DKS[:K]]
    return q.Objective(gd, kind, 0.6, 1.5), orc.Objective(od, kind, 0.6, 1.5)


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("K,npop,n,G", [(1, 65, 1300, 4), (4, 17, 1300, 4), (5, 70, 1300, 4), (8, 33, 1300, 4),
                                        (1, 66, 6200, 2), (3, 20, 6017, 2)])  # (49 and 47 segments or more)
def test_run_equals_oracle(q, orc, K, npop, n, G, kind):
    O, Oo = _pair(q, orc, inputs.uniform_boundaries(n, 2.0), K, kind)
    xo, fo, _, _ = Oo.hwsda_run(npop, G, 0.5, 0.9, 2)
    R = q.Run(O, npop, G, seed=2, prec=q.PREC_F64)
    R.advance(G)
    x, f, _, _ = R.read()
    R.destroy()
    assert np.array_equal(x.cpu().numpy(), xo)
    assert np.max(np.abs(f.cpu().numpy() - fo)) <= 1e-12 * max(1.0, np.max(np.abs(fo)))


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("n,npop,K", [(2048, 1985, 2), (2049, 2049, 3), (6400, 1990, 2), (12801, 1000, 1), (9894, 89, 1),
                                      (12000, 80, 2), (6145, 100, 3), (6144, 100, 3),
                                      (2561, 9792, 2), (2561, 9792, 5), (2561, 9793, 3), (33, 70, 8), (640, 70, 1), (640, 129, 3),
                                      (641, 70, 1), (128, 65, 8), (256, 100, 5), (257, 33, 6)])
def test_default_shape_matches_oracle(q, orc, n, npop, K, kind, prec):
    import torch
    O, Oo = _pair(q, orc, inputs.jittered_boundaries(n, 2.0, 0.3, seed=n), K, kind)
    d = inputs.random_signs(npop, n, seed=K)
    some = np.unique(np.linspace(0, npop - 1, 40).astype(int))
    bits = torch.from_numpy(inputs.pack_bits(d).view(np.int32)).cuda()
    f, G = q.eval_objective(O, bits, npop, prec, with_G=True)
    Go, fo = Oo(d[some])
    tol = 1e-12 if prec == 1 else 1e-5
    assert np.max(np.abs(G.cpu().numpy().T[some] - Go) / np.max(np.abs(Go), axis=0, keepdims=True)) <= tol
    assert np.max(np.abs(f.double().cpu().numpy()[some] - fo)) <= tol * max(1.0, np.max(np.abs(fo)))
