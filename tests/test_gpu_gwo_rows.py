"""Grey-wolf steps of large populations (four individuals per workgroup): every
gene and bit word against the oracle, leaders together in one group, at the ends
and past the last whole group; what the plain step leaves alone; a large batch
against the same designs one by one."""
import ctypes as C

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


@pytest.mark.parametrize("n,npop,lead", [(10001, 1001, (1000, 4, 999)), (2500, 4003, (8, 9, 11)), (1030, 9750, (0, 9748, 9749)),
                                         (10000, 1024, (3, 1023, 512))])
@pytest.mark.parametrize("variant", [0, 1])
def test_large_step_matches_oracle(q, orc, n, npop, lead, variant):
    import torch
    assert n * npop >= 10000000
    x, _ = q.init_population(npop, n, seed=9)
    yo = orc.gwo_step(x.cpu().numpy()[:, :n], np.array(lead), 0.8, 4, 6, inst=2, variant=variant)
    want = x.cpu().numpy().copy()
    moved = np.ones(npop, dtype=bool)
    moved[list(lead)] = False
    want[moved, :n] = yo[moved]
    words = inputs.pack_bits(np.where(want[:, :n] < 0, -1, 1), q.ld_for(npop))
    words[:, list(lead)] = 0
    y, yb = q.gwo_step(x, n, lead, 0.8, 4, 6, inst=2, variant=variant)
    assert np.array_equal(y.cpu().numpy(), want)
    assert np.array_equal(yb.cpu().numpy().view(np.uint32), words)
    # the plain step: leader rows and words, padding genes and columns untouched,
    # words at an address that is no multiple of 16 bytes
    y = torch.full_like(x, 7.0)
    store = torch.full((words.size + 1,), 0x55555555, dtype=torch.int32, device="cuda")
    b = store[1:]
    L = np.array(lead, dtype=np.int32)
    q._check(q.lib().qpm_gwo_step(C.c_void_p(x.data_ptr()), npop, n, x.shape[1], L.ctypes.data, 0.8, 4, 6, 2, variant,
                                  C.c_void_p(y.data_ptr()), C.c_void_p(b.data_ptr()), words.shape[1], q._stream(None)))
    want[:, n:] = 7.0
    want[~moved] = 7.0
    words[:, list(lead)] = 0x55555555
    words[:, npop:] = 0x55555555
    assert np.array_equal(y.cpu().numpy(), want)
    assert np.array_equal(b.cpu().numpy().view(np.uint32).reshape(words.shape), words)


def test_large_batch_equals_single_runs(q):
    npop, G = 250, 3
    zs = [inputs.uniform_boundaries(n, 2.0) for n in (20003, 13000, 9001)]
    assert sum(len(z) - 1 for z in zs) * npop >= 10000000
    B = q.precompute_phases_batched(zs, [inputs.DK1] * 3, [inputs.DK2] * 3)
    R = q.BatchRun(B, npop, G, seed=8, prec=1, tune=0)
    R.advance(G)
    for b, z in enumerate(zs):
        x, f, L = R.read(b)[:3]
        S = q.Run(q.precompute_phases(z, inputs.DK1, inputs.DK2), npop, G, seed=8, inst=b, prec=1)
        S.advance(G)
        xs, fs, Ls, _ = S.read()
        S.destroy()
        assert np.array_equal(x.cpu().numpy(), xs.cpu().numpy()) and list(L) == list(Ls)
        f, fs = f.cpu().numpy(), fs.cpu().numpy()
        assert np.max(np.abs(f - fs) / np.maximum(fs, 1e-300)) <= 1e-12
    R.destroy()
