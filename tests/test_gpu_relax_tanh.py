"""The FP64 relaxation's tanh, seen through single-domain crystals: S = d^2 c with
d = tanh theta, where c is S at theta = 30 (d = 1). Bound: d within 0.75 ulp (the
library's tanh is 0.86 off), plus the two roundings of d (d c)."""
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


@pytest.mark.parametrize("lo,hi", [(0.0, 1.0), (0.17, 0.19), (0.35, 0.55), (1.0, 4.0), (4.0, 20.0), (18.0, 30.0)])
def test_tanh_within_three_quarters_of_an_ulp(q, lo, hi):
    import torch
    rng = np.random.default_rng(17)
    x = rng.uniform(lo, hi, 400001).astype(np.float32)
    x[0] = 30.0
    x[1::2] *= -1.0
    D = q.precompute_phases(inputs.uniform_boundaries(1, 2.0), inputs.DK1, inputs.DK2)
    _, S = q.relax_forward(D, torch.from_numpy(x[:, None]).cuda(), q.PREC_F64)[:2]
    S = S.cpu().numpy().reshape(-1, 2)
    d = np.abs(np.tanh(x.astype(np.longdouble)))
    ulp = np.spacing(d.astype(np.float64)).astype(np.longdouble) / d
    for c in range(2):
        got = S[:, c].astype(np.longdouble) / np.longdouble(S[0, c])
        assert np.max(np.abs(got / (d * d) - 1) - 1.5 * ulp) <= 2.0 ** -52


def test_tanh_of_special_values(q):
    import torch
    x = np.array([30.0, np.inf, -np.inf, 20.0, -1e30, 0.0, -0.0, 1e-40, np.nan], dtype=np.float32)
    D = q.precompute_phases(inputs.uniform_boundaries(1, 2.0), inputs.DK1, inputs.DK2)
    th = torch.from_numpy(x[:, None]).cuda()
    _, S = q.relax_forward(D, th, q.PREC_F64)[:2]
    S = S.cpu().numpy().reshape(-1, 2)
    assert np.all(S[1:5] == S[0]) and np.all(S[5:7] == 0) and np.all(np.isnan(S[8]))
    assert np.allclose(S[7], np.float64(x[7]) ** 2 * S[0], rtol=2.0 ** -51, atol=0.0)  # tanh x = x
