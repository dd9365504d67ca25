"""The join's reference rows in groups: every workspace size from the smallest
on gives the same integers, equal to the sum of one-row joins (which the join
tests pin against the oracle)."""
import ctypes

import pytest
import torch

import synth
from paper_2602_24271_amd import Context, _lib
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("log2_n,alpha,n", [(6, 1, 1), (6, 3, 2), (12, 2, 3)])
def test_workspace_sizes_agree(log2_n, alpha, n):
    require_gpu()
    ctx = Context.paper(log2_n, alpha=alpha)
    lib, h, dev = ctx._lib, ctx._h, ctx.device
    uni = lambda lead, moduli, s: synth.uniform_device_residues(lead, moduli, ctx.n, s, dev)
    ctx.set_relin_key(uni((ctx.dnum, 2), ctx.moduli_pq, 1))
    for i, g in enumerate(ctx.galois_elements()):
        ctx.set_galois_key(g, uni((ctx.dnum, 2), ctx.moduli_pq, 10 + i))
    a, bk, ba = uni((n, 2), ctx.q, 2), uni((1, 2), ctx.q, 3), uni((1, 2), ctx.q, 4)
    rows = [ctx.n - 1, 0, ctx.n // 2, 5, 9]
    low = lib.nshe_join_workspace_bytes(h, n)
    wide = lib.nshe_join_workspace_wide_bytes(h, n, len(rows))
    assert wide > low

    def join(rs, size):
        ws = torch.empty(size, dtype=torch.uint8, device=dev)
        out = torch.empty_like(a)
        _lib.check(lib.nshe_join_sum(h, a.data_ptr(), bk.data_ptr(), ba.data_ptr(),
                                     (ctypes.c_int32 * len(rs))(*rs), len(rs), out.data_ptr(), n,
                                     ws.data_ptr(), size,
                                     torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        return out

    want = ctx.sum(torch.stack([join([r], low) for r in rows]))
    for size in (low, lib.nshe_join_workspace_wide_bytes(h, n, 1),
                 lib.nshe_join_workspace_wide_bytes(h, n, 2) + 8, wide):
        assert torch.equal(join(rows, max(size, low)), want), size
    assert torch.equal(ctx.join_sum(a, bk, ba, rows), want)
    ctx.close()
