"""The comparison program's products in batches: every workspace size from the
smallest on gives the integers of one ciphertext at a time in the smallest
(which the comparison tests pin against the oracle)."""
import pytest
import torch

import synth
from paper_2602_24271_amd import Context, _lib
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("log2_n,alpha,n", [(6, 3, 1), (6, 1, 3), (10, 2, 2), (12, 3, 5)])
def test_workspace_sizes_agree(log2_n, alpha, n):
    require_gpu()
    ctx = Context.paper(log2_n, alpha=alpha)
    lib, h, dev = ctx._lib, ctx._h, ctx.device
    ctx.set_relin_key(synth.uniform_device_residues((ctx.dnum, 2), ctx.moduli_pq, ctx.n, 1, dev))
    x = synth.uniform_device_residues((n, 2), ctx.q, ctx.n, 2, dev)
    y = synth.uniform_device_residues((1, 2), ctx.q, ctx.n, 3, dev)
    low = lib.nshe_compare_workspace_bytes(h, n)
    wide = lib.nshe_compare_workspace_wide_bytes(h, n)
    assert wide > low

    def lt(xs, size):
        ws = torch.empty(size, dtype=torch.uint8, device=dev)
        out = torch.empty_like(xs)
        _lib.check(lib.nshe_compare(h, xs.data_ptr(), y.data_ptr(), 1, 0, out.data_ptr(),
                                    xs.shape[0], ws.data_ptr(), size,
                                    torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        return out

    one = lib.nshe_compare_workspace_bytes(h, 1)
    want = torch.cat([lt(x[i:i + 1].clone(), one) for i in range(n)])
    for size in (low, low + 2 * ctx.workspace_bytes(n) + 8, wide, wide + 4096):
        assert torch.equal(lt(x, size), want), size
    ctx.close()
