"""The staged automorphism (90 limbs and more: a limb per workgroup, through
LDS) at every ring it is built for, against the direct one: three ciphertexts
together take the first, each one alone the second, and rotations and sums are
the same integers."""
import pytest
import torch

import synth
from paper_2602_24271_amd import Context
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("log2_n", [10, 11, 12, 13, 14, 15])
@pytest.mark.parametrize("alpha", [1, 3])
def test_staged_equals_direct(log2_n, alpha):
    require_gpu()
    c = Context.paper(log2_n, alpha=alpha)
    c.set_tuning(streams=1)
    key = lambda s: synth.uniform_device_residues((c.dnum, 2), c.moduli_pq, c.n, s, c.device)
    c.set_relin_key(key(1))
    els = c.galois_elements()
    for i, g in enumerate(els):
        c.set_galois_key(g, key(10 + i))
    n = 3
    assert n * 2 * c.L >= 90 > 2 * c.L
    x = synth.uniform_device_residues((n, 2), c.q, c.n, 2, c.device)
    one = [x[i:i + 1].clone() for i in range(n)]
    for g in (els[0], els[-2], els[-1]):   # the largest step, step 1, the swap
        assert torch.equal(c.rotate(x, g), torch.cat([c.rotate(t, g) for t in one])), g
    assert torch.equal(c.sum_slots(x), torch.cat([c.sum_slots(t) for t in one]))
    c.close()
