"""The key-switch product by parity on one stream, where the ciphertext counts
alone choose its width: every width in one pass, and several passes over the
key with a ragged last one, equal to each ciphertext alone."""
import pytest
import torch

import synth
from paper_2602_24271_amd import Context
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu

# ciphertexts, ks_chunk: the passes' widths and their ciphertexts
CASES = [(2, 32), (3, 32), (4, 32), (5, 32),   # 2, 3, 4, 6 wide
         (7, 32), (11, 32), (16, 32),          # 8, 12, 16 wide
         (17, 32),                             # 12 wide: 12 + 5
         (25, 32),                             # 16 wide: 16 + 9
         (33, 32),                             # 12 wide: 12 + 12 + 9
         (9, 4), (10, 4), (9, 8)]              # 3 + 3 + 3, 4 + 4 + 2, 6 + 3


@pytest.mark.parametrize("alpha", [1, 2, 3])
def test_passes_equal_single_ciphertexts(alpha):
    require_gpu()
    c = Context.paper(15, alpha=alpha)
    c.set_relin_key(synth.uniform_device_residues((c.dnum, 2), c.moduli_pq, c.n, 1, c.device))
    x = synth.uniform_device_residues((max(n for n, _ in CASES), 2), c.q, c.n, 2, c.device)
    alone = torch.cat([c.square_relin(x[i:i + 1].clone()) for i in range(x.shape[0])])
    for n, ch in CASES:
        c.set_tuning(streams=1, ks_chunk=ch)
        assert torch.equal(c.square_relin(x[:n].clone()), alone[:n]), (n, ch)
    c.close()
