"""The key-switch product at every chunk width it narrows to: a squaring of n
ciphertexts equals the squarings of each one alone (whose results the
full-size tests pin against the oracle), and the small ring's chunks equal
the oracle."""
import numpy as np
import pytest
import torch

import synth
from oracle import bfv
from paper_2602_24271_amd import Context
from tests.gpu_common import Setup, require_gpu

pytestmark = pytest.mark.gpu

COUNTS = (2, 3, 4, 5, 7, 11, 17)   # widths 2, 3, 4, 6, 8, 12 and two chunks of 12


@pytest.mark.parametrize("alpha", [1, 2, 3])
def test_widths_equal_single_ciphertexts(alpha):
    require_gpu()
    ctx = Context.paper(15, alpha=alpha)
    dev = ctx.device
    ctx.set_relin_key(synth.uniform_device_residues((ctx.dnum, 2), ctx.moduli_pq, ctx.n, 1, dev))
    x = synth.uniform_device_residues((max(COUNTS), 2), ctx.q, ctx.n, 2, dev)
    alone = torch.cat([ctx.square_relin(x[i:i + 1].clone()) for i in range(x.shape[0])])
    for n in COUNTS:
        assert torch.equal(ctx.square_relin(x[:n].clone()), alone[:n]), n
    ctx.close()


@pytest.mark.parametrize("n", [1, 2, 3, 9])
def test_small_ring_widths(n):
    S = Setup(6, seed=70, alpha=3)
    rng = np.random.default_rng(n)
    a = np.stack([np.stack([synth.uniform_residues(rng, S.pr.q, S.pr.n) for _ in range(2)])
                  for _ in range(n)])
    got = S.ctx.square_relin(torch.from_numpy(a).to(S.ctx.device)).cpu().numpy()
    for i in range(n):
        ct = tuple(bfv.from_limbs(a[i, k], S.pr.q) for k in range(2))
        np.testing.assert_array_equal(got[i], S.limbs(bfv.square_relin(S.pr, S.rk, ct)))
