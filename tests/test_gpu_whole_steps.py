"""Steps that write whole rows into uncleared results: every element equals that
of the plain step into cleared (DE) or copied (grey-wolf) ones, which the
oracle tests cover."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q():
    import torch
    assert torch.cuda.is_available(), "a GPU is required"
    from paper_2511_01255_amd import qpm
    qpm.lib()
    return qpm


def _p(t):
    return C.c_void_p(t.data_ptr())


# partial quads, words, chunks and row groups; row and column padding of none,
# the usual and more than a block of it
@pytest.mark.parametrize("n,npop,xpad,bpad", [(1, 4, 0, 0), (63, 64, 0, 0), (64, 65, 64, 64), (1023, 100, 4, 0),
                                              (1024, 4096, 0, 0), (1025, 1021, 1088, 64), (300, 4099, 0, 0)])
def test_whole_equals_plain(q, n, npop, xpad, bpad):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    ldx, ld, W = q.ldx_for(n) + xpad, q.ld_for(npop) + bpad, q.words(n)
    x = torch.rand(npop, ldx, generator=gen, device="cuda") * 2.0 - 1.0  # (padding too)
    L, s = q.lib(), q._stream(None)
    lead = np.array([npop - 1, 0, npop // 2], dtype=np.int32)

    def out(fill, bfill):
        return torch.full_like(x, fill), torch.full((W, ld), bfill, dtype=torch.int32, device="cuda")

    u, ub = out(0.0, 0)
    w, wb = out(float("nan"), -1)
    for fn, o, ob in ((L.qpm_de_step, u, ub), (L.qpm_de_step_whole, w, wb)):
        q._check(fn(_p(x), npop, n, ldx, 0.5, 0.9, 3, 2, 1, _p(o), _p(ob), ld, s))
    assert torch.equal(u, w) and torch.equal(ub, wb)
    for variant in (0, 1):
        y, yb = out(0.0, 0)
        y.copy_(x)
        w, wb = out(float("nan"), -1)
        for fn, o, ob in ((L.qpm_gwo_step, y, yb), (L.qpm_gwo_step_whole, w, wb)):
            q._check(fn(_p(x), npop, n, ldx, lead.ctypes.data, 1.3, 3, 2, 1, variant, _p(o), _p(ob), ld, s))
        assert torch.equal(y, w) and torch.equal(yb, wb)


# layouts that keep the cleared and copied results: a long row, a view, a leaf
# that asks for gradients
@pytest.mark.parametrize("form", ["plain", "long", "grad"])
def test_binding_forms_agree(q, form):
    import torch
    n, npop = 70, 33
    x, _ = q.init_population(npop, n, seed=5)
    ref = [q.de_step(x, n, 0.5, 0.9, 1, 2, shape=(1, 1)), q.gwo_step(x, n, [1, 2, 3], 0.7, 1, 2)]
    if form == "long":
        x = torch.cat([x, torch.zeros(npop, 64, device="cuda")], 1)
    if form == "grad":
        x = x.clone().requires_grad_()
    got = [q.de_step(x, n, 0.5, 0.9, 1, 2), q.gwo_step(x, n, [1, 2, 3], 0.7, 1, 2)]
    for (a, ab), (b, bb) in zip(ref, got):
        assert torch.equal(a[:, :n], b[:, :n]) and torch.equal(ab, bb) and not b[:, n:].any()
    assert got[1][0].requires_grad == (form == "grad")
