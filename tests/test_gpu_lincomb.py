"""The comparison's 256 x 128 linear combinations on the integer matrix cores
(rings of N >= 32; N = 16 keeps the FP64 form): the smallest rings that take
each form, against the oracle's program, and the host's byte split of every
coefficient."""
import numpy as np
import pytest
import torch

from oracle import compare
from tests.gpu_common import Setup


def test_coefficients_are_two_signed_bytes_and_127():
    """The form holds c - 127 in two signed bytes: every odd coefficient of
    p = 65537 lies in the range the context checks."""
    c = [compare.centred(x, 65537) for x in compare.lt_coefficients(65537)[1::2]]
    assert len(c) == 256 * 128
    assert min(c) - 127 >= -128 * 256 - 128 and max(c) - 127 <= 127 * 256 + 127


@pytest.mark.gpu
@pytest.mark.parametrize("log2_n,alpha,n", [(4, 3, 1), (5, 3, 2), (5, 1, 1), (6, 2, 3)])
def test_lt_against_the_oracle(log2_n, alpha, n):
    S = Setup(log2_n, seed=30 + log2_n, alpha=alpha)
    rng = np.random.default_rng(7)
    xs = [rng.integers(0, 65537, S.pr.n) for _ in range(n)]
    xs[0][:3] = [30000, 29999, 30001]
    cx = [S.enc(v, 600 + i) for i, v in enumerate(xs)]
    cy = S.enc(np.full(S.pr.n, 30000), 610)
    got = S.ctx.compare(S.to_dev(cx), S.to_dev([cy]), "lt")
    torch.cuda.synchronize()
    for i in (0, n - 1):
        np.testing.assert_array_equal(got[i].cpu().numpy(),
                                      S.limbs(compare.lt(S.pr, S.rk, cx[i], cy)))
