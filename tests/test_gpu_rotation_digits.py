"""Rotations of ciphertexts whose second component has vanishing digits: the
negated coefficient's digits from the coefficient's (lower digits zero, all
zero, all at their top), read where they lie (few limbs) and staged through LDS
(90 limbs and more), against the oracle."""
import numpy as np
import pytest
import torch

import synth
from oracle import bfv, galois
from tests.gpu_common import Setup, galois_keys

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("log2_n,n_ct", [(6, 1), (6, 4), (10, 4)])
@pytest.mark.parametrize("alpha", [1, 2, 3])
def test_vanishing_digits(alpha, log2_n, n_ct):
    S = Setup(log2_n, seed=90, alpha=alpha)
    pr = S.pr
    rng = np.random.default_rng(alpha)
    a = np.stack([np.stack([synth.uniform_residues(rng, pr.q, pr.n) for _ in range(2)])
                  for _ in range(n_ct)])
    # c1 = D in every digit group: multiples of the group's first primes
    specials = []
    for j in range(pr.dnum):
        p = [int(x) for x in pr.digit_primes(j)]
        prod = [1]
        for x in p:
            prod.append(prod[-1] * x)
        specials.append([0, 1, prod[-1] - 1] + [m for b in prod[:-1] for m in (b, b * 3, prod[-1] - b)])
    for c in range(min(pr.n, len(specials[0]) * 2)):
        for j in range(pr.dnum):
            d = specials[j][c % len(specials[j])]
            for k, p in enumerate(pr.digit_primes(j)):
                a[0, 1, j * alpha + k, (5 * c + 1) % pr.n] = d % int(p)
    a[-1, 1] = 0 if n_ct > 1 else a[-1, 1]          # a trivial encryption's c1
    for i, g in enumerate([3, 2 * pr.n - 1]):
        key = galois.galois_key(pr, S.sk, g, synth.switch_randomness(300 + i, pr.n, pr.moduli_pq,
                                                                     pr.dnum))
        S.ctx.set_galois_key(g, torch.from_numpy(key.limbs(pr)).to(S.ctx.device))
        got = S.ctx.rotate(torch.from_numpy(a).to(S.ctx.device), g).cpu().numpy()
        for ct in sorted({0, n_ct - 1}):
            x = tuple(bfv.from_limbs(a[ct, k], pr.q) for k in range(2))
            np.testing.assert_array_equal(got[ct], S.limbs(galois.apply_galois(pr, key, x, g)))


@pytest.mark.parametrize("alpha", [1, 3])
def test_sum_of_a_trivial_encryption(alpha):
    S = Setup(6, seed=91, alpha=alpha)
    keys = galois_keys(S, seed=950)
    rng = np.random.default_rng(5)
    a = np.zeros((1, 2, S.pr.L, S.pr.n), dtype=np.int64)
    a[0, 0] = synth.uniform_residues(rng, S.pr.q, S.pr.n)
    got = S.ctx.sum_slots(torch.from_numpy(a).to(S.ctx.device)).cpu().numpy()
    x = tuple(bfv.from_limbs(a[0, k], S.pr.q) for k in range(2))
    np.testing.assert_array_equal(got[0], S.limbs(galois.sum_slots(S.pr, keys, x)))
