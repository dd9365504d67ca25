"""Calls over a few ciphertexts run as two halves on two streams: the same
integers as on one stream, for every split (even, odd, a wave halved, half-
waves evened out), with and without graphs, and replayed."""
import pytest
import torch

import synth
from paper_2602_24271_amd import Context
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=[(12, 1), (15, 3)], ids=["2^12", "2^15"])
def ctx(request):
    require_gpu()
    log2_n, alpha = request.param
    c = Context.paper(log2_n, alpha=alpha)
    key = lambda s: synth.uniform_device_residues((c.dnum, 2), c.moduli_pq, c.n, s, c.device)
    c.set_relin_key(key(1))
    for i, g in enumerate(c.galois_elements()):
        c.set_galois_key(g, key(10 + i))
    yield c
    c.close()


def cts(c, n, seed):
    return synth.uniform_device_residues((n, 2), c.q, c.n, seed, c.device)


def both(c, f):
    """f() on two streams (twice, on different workspaces) equals one stream."""
    c.set_tuning(streams=1)
    want = f()
    c.set_tuning(streams=2)
    for _ in range(2):
        got = f()
        for a, b in zip(want, got):
            assert torch.equal(a, b)


@pytest.mark.parametrize("n", [2, 3, 9])
def test_few_ciphertexts(ctx, n):
    x, y = cts(ctx, n, 2), cts(ctx, n, 3)
    both(ctx, lambda: [ctx.eq_mask(x, y), ctx.eq_mask(x, y[:1]), ctx.sum_slots(x),
                       ctx.mul_relin(x, y), ctx.square_relin(x)])


@pytest.mark.parametrize("use_graph", [False, True])
@pytest.mark.parametrize("sizes,wave", [((1, 2), 32), ((7, 8), 32), ((4, 1, 6), 4), ((5, 3, 1), 6),
                                        ((1, 1, 5, 2), 3)])
def test_batched_splits(ctx, sizes, wave, use_graph):
    items = [(cts(ctx, m, 20 + i), cts(ctx, 1, 40 + i)) for i, m in enumerate(sizes)]
    both(ctx, lambda: ctx.eq_mask_batched(items, wave_ct=wave, use_graph=use_graph))
