"""Batched evaluations on plans kept with the batch: more shapes than are kept,
growing and shrinking populations, several streams and threads at once, and a
captured graph, all against each population's own single-design evaluations."""
import threading

import numpy as np
import pytest

from paper_2511_01255_amd import inputs

pytestmark = pytest.mark.gpu

NS = [700, 33, 4099, 1]


@pytest.fixture(scope="module")
def q():
    import torch
    assert torch.cuda.is_available(), "a GPU is required"
    from paper_2511_01255_amd import qpm
    qpm.lib()
    return qpm


def _batch(q):
    zs = [inputs.uniform_boundaries(n, 2.0) for n in NS]
    return q.precompute_phases_batched(zs, [inputs.DK1] * len(NS), [inputs.DK2] * len(NS))


def _population(q, npop, seed):
    """(packed words, FP64 fitness by the per-domain kernel of the single designs)"""
    import torch
    bits, f = [], []
    for k, n in enumerate(NS):
        b = torch.from_numpy(inputs.pack_bits(inputs.random_signs(npop, n, seed=seed + k)).view(np.int32)).cuda()
        D = q.precompute_phases(inputs.uniform_boundaries(n, 2.0), inputs.DK1, inputs.DK2)
        bits.append(b)
        f.append(q.eval_fitness(D, b, npop, q.PREC_F64, kernel=q.FIT_SEGMENTED))
    return torch.cat(bits), torch.stack(f)


def _close(f, g):
    import torch
    floor = 1e-2 * g.median(dim=1, keepdim=True).values
    return bool(((f - g).abs() <= 2e-12 * torch.maximum(g, floor)).all())


def test_more_shapes_than_kept_and_any_population(q):
    B = _batch(q)
    pops = [_population(q, n, 10 * n) for n in (65, 300, 3, 129)]
    for _ in range(2):
        for bits, g in pops:
            npop = g.shape[1]
            assert _close(q.batch_eval_fitness(B, bits, npop, q.PREC_F64), g)
            for gw in (1, 2, 4):
                for wpw in (1, 2):
                    assert _close(q.batch_eval_fitness_table(B, bits, npop, q.PREC_F64, gw, wpw), g)
            for waves, wpw in ((4, 1), (8, 3), (16, 2), (4, 7), (16, 40)):
                assert _close(q.batch_eval_fitness(B, bits, npop, q.PREC_F64, waves, wpw), g)


def test_streams_threads_and_capture(q):
    import torch
    B = _batch(q)
    pops = [_population(q, n, n) for n in (70, 200, 257, 64, 130, 90)]
    bad = []

    def work(k):
        bits, g = pops[k]
        s = torch.cuda.Stream()
        torch.cuda.synchronize()
        for _ in range(20):
            with torch.cuda.stream(s):
                f = q.batch_eval_fitness(B, bits, g.shape[1], q.PREC_F64)
            s.synchronize()
            if not _close(f, g):
                bad.append(k)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(pops))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
    # a shape already evaluated can be captured
    bits, g = pops[0]
    f = torch.empty_like(g)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        q.batch_eval_fitness(B, bits, g.shape[1], q.PREC_F64, out=f)
    for _ in range(3):
        f.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert _close(f, g)
        q.batch_eval_fitness(B, pops[1][0], pops[1][1].shape[1], q.PREC_F64)
