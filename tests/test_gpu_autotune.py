"""The autotuner times the kernels that calls run: levels whose mod-down lifts
the result for the next (counted at that lift's site under the debug switch
that sends half of all lifts through the exact path)."""
import pytest

import synth
from paper_2602_24271_amd import Context
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu

I64_LIFT, MODDOWN_LIFT = 5, 3   # include/nshe.h, nshe_margin_sites


@pytest.mark.parametrize("alpha", [1, 3])
def test_levels_of_the_chain_are_timed(alpha):
    require_gpu()
    c = Context.paper(15, alpha=alpha)
    c.set_relin_key(synth.uniform_device_residues((c.dnum, 2), c.moduli_pq, c.n, 1, c.device))
    x = synth.uniform_device_residues((2, 2), c.q, c.n, 2, c.device)
    c.set_debug(wide_lift_window=True)
    tuned = c.autotune(x, max_wave_ct=2)
    sites = c.margin_sites()
    c.close()
    assert sites[I64_LIFT] > 0 and sites[MODDOWN_LIFT] > 0, sites
    # by coefficient parity the key-switch product is at most 16 wide
    assert not tuned["split_forward"] or tuned["ks_chunk"] <= 16
