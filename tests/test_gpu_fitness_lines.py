"""Both sides of the lines of the default table shape: 5000 (FP32) and 6000 (FP64)
wave words of work (64-genome groups x words), 12,000 in both; 20 words (one
launch), the number of its segments, and several genome groups per workgroup
there; the words per wave that keep the segments below 48. Tolerances are the
fitness's own (FP64 1e-12, FP32 1e-5, plain or against 1 % of the median)."""
import numpy as np
import pytest

from paper_2511_01255_amd import inputs

pytestmark = pytest.mark.gpu

TOL = {0: 1e-5, 1: 1e-12}


@pytest.fixture(scope="module")
def q():
    import torch
    assert torch.cuda.is_available(), "a GPU is required"
    from paper_2511_01255_amd import qpm
    qpm.lib()
    return qpm


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("words,npop", [
    (100, 3200), (100, 3201), (250, 1280), (250, 1281),          # work 5000 and above
    (100, 3840), (100, 3841), (3001, 128), (2999, 128),          # work 6000, two groups
    (200, 3840), (200, 3841), (240, 70), (241, 70), (383, 70), (384, 70),  # 12,000; 31 to 47 segments of 2 words
    (376, 70), (377, 70), (564, 70), (565, 70), (752, 70), (753, 70), (940, 70), (941, 70),  # 48 segments
    (1, 70), (4, 65), (8, 65), (9, 64), (16, 64), (17, 130), (20, 130), (21, 130),           # segments of one launch
    (20, 16000), (20, 16001), (20, 19200), (20, 19264), (17, 45200), (20, 38464), (12, 64100)])
def test_both_sides_match_the_segmented_kernel(q, orc, words, npop, prec):
    import torch
    n = 32 * words - 3
    z = inputs.jittered_boundaries(n, 2.0, 0.2, seed=words)
    D = q.precompute_phases(z, inputs.DK1, inputs.DK2)
    rng = np.random.default_rng(npop)
    ld = inputs.ld_for(npop)
    b = rng.integers(0, 1 << 32, (words, ld), dtype=np.uint64).astype(np.uint32)
    b[-1] &= (1 << 29) - 1  # padding bits are 0
    bits = torch.from_numpy(b.view(np.int32)).cuda()
    f = q.eval_fitness(D, bits, npop, prec).double().cpu().numpy()
    g = q.eval_fitness(D, bits, npop, 1, kernel=q.FIT_SEGMENTED).cpu().numpy()
    assert np.max(np.abs(f - g) / np.maximum(g, 1e-2 * np.median(g))) <= 2 * TOL[prec]
    some = np.unique(np.linspace(0, npop - 1, 5).astype(int))
    _, fo = orc.Design(z, inputs.DK1, inputs.DK2).fitness(inputs.unpack_bits(b[:, some], len(some), n))
    assert np.max(np.abs(f[some] - fo) / np.maximum(fo, 1e-2 * np.median(g))) <= TOL[prec]
