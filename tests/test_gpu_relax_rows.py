"""The relaxation on rows of any length and alignment, around the ends of its
chunks, segments and row groups, and its FP64 tanh."""
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


# row length less n, and the first row's offset in floats
@pytest.mark.parametrize("pad,shift", [(0, 0), (1, 0), (2, 1), (8, 3)])
@pytest.mark.parametrize("n,B", [(15, 3), (16, 64), (17, 65), (127, 63), (129, 128), (1030, 100), (4097, 67)])
@pytest.mark.parametrize("prec", [1, 0])
def test_rows_match_oracle(q, orc, n, B, pad, shift, prec):
    import torch
    z = inputs.jittered_boundaries(n, 2.0, 0.2, seed=n)
    D, O = q.precompute_phases(z, inputs.DK1, inputs.DK2), orc.Design(z, inputs.DK1, inputs.DK2)
    theta = inputs.relax_theta(B, n, seed=n)
    flat = torch.full((B * (n + pad) + shift,), float("nan"), device="cuda")
    th = flat[shift:].view(B, n + pad)
    th[:, :n] = torch.from_numpy(np.ascontiguousarray(theta, dtype=np.float32)).cuda()
    _, S, E = q.relax_forward(D, th, prec, keep_edges=True)
    So, fo, go = O.relax(np.asarray(theta, dtype=np.float32).astype(np.float64))
    Sc = S.cpu().numpy()
    Sc = Sc[:, 0] + 1j * Sc[:, 1]
    # the tolerances of the relaxation's other oracle tests
    assert np.max(np.abs(Sc - So)) <= (1e-12 if prec == 1 else 1e-5) * np.max(np.abs(So))
    gf = torch.ones(B, device="cuda")
    for edges in (E, None):
        g = q.relax_backward(D, th, S, gf, prec, edges=edges).cpu().numpy()
        scale = np.maximum(np.max(np.abs(go), axis=1, keepdims=True), 1e-300)
        assert np.max(np.abs(g[:, :n] - go) / scale) <= (1e-6 if prec == 1 else 1e-4)
        assert not g[:, n:].any()


def test_fp64_tanh(q):
    # one domain: S = c tanh(theta)^2, so S / S(1) is the square of a tanh: 2
    # ulp each for both tanh and a rounding for each product and the quotient
    import torch
    D = q.precompute_phases(np.array([0.0, 2.0]), inputs.DK1, inputs.DK2)
    rng = np.random.default_rng(3)
    t = np.concatenate([rng.uniform(-6, 6, 4000), rng.uniform(-25, 25, 500), 2.0 ** rng.uniform(-40, 0, 1500),
                        [0.0, -0.0, 20.0, 1e30, np.inf, -np.inf]]).astype(np.float32)
    th = torch.from_numpy(np.concatenate([[np.float32(40.0)], t]).reshape(-1, 1)).cuda()
    _, S = q.relax_forward(D, th, 1)
    S = S.cpu().numpy()
    want = np.tanh(t.astype(np.longdouble)) ** 2
    for c in (0, 1):
        got = S[1:, c].astype(np.longdouble) / np.longdouble(S[0, c])
        assert np.max(np.abs(got - want) / np.maximum(want, np.longdouble(1e-300))) <= 2e-15
    th[1] = float("nan")
    assert torch.isnan(q.relax_forward(D, th, 1)[1][1]).all()
