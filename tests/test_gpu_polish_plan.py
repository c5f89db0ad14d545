"""A polish compares the leaders' present signs with the projected ones, so a
projection that flips no sign replaces nothing: accepted is 0 and every gene and
fitness stays as it was, whatever launch plan the run evaluates with (its own
words per wave, a tuned shape, the fused generations' walk)."""
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


# words per wave of the run and of a three-row evaluation differ at all but 1500;
# the last rows: segmented, per-domain and fused evaluations
@pytest.mark.parametrize("prec", [1, 0])
@pytest.mark.parametrize("n,npop,opts", [
    (300, 70, {}), (300, 1000, {}), (500, 70, {}), (512, 500, {}), (500, 1000, {}), (640, 70, {}), (640, 1000, {}),
    (1500, 96, {}), (13000, 200, {}), (10000, 1300, {}), (640, 1000, {"tune": 1}), (10000, 1300, {"tune": 1}),
    (1500, 96, {"fit_kernel": "FIT_SEGMENTED"}), (640, 100, {"fit_kernel": "FIT_PER_GENOME"}),
    (256, 32, {"fused": 1}), (300, 32, {"fused": 1}), (500, 32, {"fused": 1}), (300, 32, {"fused": 1, "algo": "ALGO_GWO"}),
])
def test_polish_without_flips_changes_nothing(q, n, npop, opts, prec):
    if opts.get("fit_kernel") == "FIT_PER_GENOME" and prec == 0:
        pytest.skip("the per-domain walk of a whole genome is FP64 only")
    kw = {k: getattr(q, v) if isinstance(v, str) else v for k, v in opts.items()}
    kw.setdefault("fused", -1)
    D = q.precompute_phases(inputs.jittered_boundaries(n, 2.0, 0.2, seed=n), inputs.DK1, inputs.DK2)
    R = q.Run(D, npop, 8, seed=3, prec=prec, **kw)
    for g in range(6):
        x0, f0, _, _ = R.read()
        assert R.polish(0) == 0
        assert R.polish(3, 0.0) == 0  # (any step flips a gene that is exactly 0)
        x1, f1, _, _ = R.read()
        assert np.array_equal(x0.cpu().numpy(), x1.cpu().numpy())
        assert np.array_equal(f0.cpu().numpy(), f1.cpu().numpy())
        R.advance(1)
    R.destroy()
