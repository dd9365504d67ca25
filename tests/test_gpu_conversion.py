"""The base conversions on the matrix cores for every prime count the library
is built for, at a ring smaller than a workgroup: residues whose conversion
digits are as large as they get, against the exact-integer oracle."""
import numpy as np
import pytest
import torch

import synth
from oracle import bfv, nt
from paper_2602_24271_amd import Context
from tests.gpu_common import Setup, require_gpu

pytestmark = pytest.mark.gpu

# every L, with each digit width it is built for (steps of four primes: all
# remainders of L and L + 1)
CASES = [(L, 1) for L in (2, 3, 4, 8, 12, 15, 16, 17, 20, 24)] + [(16, 2), (4, 2), (15, 3), (12, 3)]


class ChainSetup(Setup):
    def __init__(self, log2_n, L, alpha, seed):
        require_gpu()
        n = 1 << log2_n
        primes = nt.primes_congruent_one_below(1 << 49, 1 << 16, L + alpha)
        P = primes[0] if alpha == 1 else tuple(primes[:alpha])
        self.pr = bfv.Params(n, 65537, tuple(primes[alpha:]), P)
        self.sk, self.rk = bfv.keygen(self.pr, synth.key_randomness(seed, n, self.pr.moduli_pq,
                                                                     self.pr.dnum))
        self.ctx = Context(log2_n, 65537, list(self.pr.q), list(self.pr.special))
        self.ctx.set_relin_key(torch.from_numpy(self.rk.limbs(self.pr)).to(self.ctx.device))


def extreme_limbs(pr, rng):
    """int64 [2, L, N]: random residues, and coefficients with x_i = y (Q/q_i)
    mod q_i, so that the lift's residues y_i are all +-(q_i - 1)/2, or have
    every base-256 digit at an end of its range, or are 0 or +-1."""
    q = list(pr.q)
    Q = 1
    for p in q:
        Q *= p
    out = np.stack([synth.uniform_residues(rng, q, pr.n) for _ in range(2)])
    top = sum(127 << (8 * a) for a in range(6))
    ys = [lambda p: (p - 1) // 2, lambda p: -((p - 1) // 2), lambda p: top, lambda p: -top - 1,
          lambda p: top + (1 << 46), lambda p: 0, lambda p: 1, lambda p: -1]
    for c, f in enumerate(ys):
        for i, p in enumerate(q):
            out[0, i, c] = f(p) * (Q // p) % p
            out[1, i, pr.n - 1 - c] = (f(p) if i % 2 else -f(p)) * (Q // p) % p
    return out


@pytest.mark.parametrize("L,alpha", CASES)
def test_product_of_extreme_residues(L, alpha):
    S = ChainSetup(6, L, alpha, seed=100 + L)
    pr = S.pr
    rng = np.random.default_rng(L * 4 + alpha)
    a, b = extreme_limbs(pr, rng), extreme_limbs(pr, rng)[:, :, ::-1].copy()
    ca, cb = (tuple(bfv.from_limbs(v[k], pr.q) for k in range(2)) for v in (a, b))
    da, db = (torch.from_numpy(v[None]).to(S.ctx.device) for v in (a, b))
    got = S.ctx.multiply(da, db)
    np.testing.assert_array_equal(got[0].cpu().numpy(), S.limbs(bfv.multiply(pr, ca, cb)))
    sq = S.ctx.square_relin(da)
    np.testing.assert_array_equal(sq[0].cpu().numpy(), S.limbs(bfv.square_relin(pr, S.rk, ca)))
