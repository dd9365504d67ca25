"""Outputs that lie on other ciphertexts' inputs (shifted by a ciphertext, on a
broadcast operand, on another item's operand): a call reads what it was given
before it overwrites it, also where it would otherwise run in two halves."""
import pytest
import torch

import synth
from paper_2602_24271_amd import Context, _lib
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    require_gpu()
    c = Context.paper(15, alpha=3)
    key = lambda s: synth.uniform_device_residues((c.dnum, 2), c.moduli_pq, c.n, s, c.device)
    c.set_relin_key(key(1))
    for i, g in enumerate(c.galois_elements()):
        c.set_galois_key(g, key(10 + i))
    yield c
    c.close()


def cts(c, n, seed):
    return synth.uniform_device_residues((n, 2), c.q, c.n, seed, c.device)


def call(c, name, *args):
    _lib.check(getattr(c._lib, name)(c._h, *args, torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()


# where the output starts in a buffer whose ciphertexts 1..n are the first operand
SHIFTS = [0, 1, 2]


@pytest.mark.parametrize("shift", SHIFTS)
@pytest.mark.parametrize("op", ["square", "mul_a", "mul_b", "eq_x", "eq_y", "sum"])
def test_shifted_output(ctx, op, shift):
    n = 9
    buf, other = cts(ctx, n + 2, 2), cts(ctx, n, 3)
    x = buf[1:n + 1]
    want = {"square": lambda: ctx.square_relin(x.clone()),
            "mul_a": lambda: ctx.mul_relin(x.clone(), other),
            "mul_b": lambda: ctx.mul_relin(other, x.clone()),
            "eq_x": lambda: ctx.eq_mask(x.clone(), other),
            "eq_y": lambda: ctx.eq_mask(other, x.clone()),
            "sum": lambda: ctx.sum_slots(x.clone())}[op]()
    out = buf[shift:shift + n]
    ws = ctx.workspace(n)
    w = (ws.data_ptr(), ws.numel())
    p, o, r = x.data_ptr(), other.data_ptr(), out.data_ptr()
    if op == "square":
        call(ctx, "nshe_square_relin", p, r, n, *w)
    elif op == "sum":
        call(ctx, "nshe_sum_slots", p, r, n, *w)
    elif op[:3] == "mul":
        call(ctx, "nshe_mul_relin", *((p, o) if op == "mul_a" else (o, p)), r, n, *w)
    else:
        call(ctx, "nshe_eq_mask", *((p, o) if op == "eq_x" else (o, p)), r, n, 0, *w)
    assert torch.equal(out, want)


def test_broadcast_operand_in_the_output(ctx):
    n = 4
    x, buf = cts(ctx, n, 4), cts(ctx, n, 5)
    y = buf[1:2]
    want = ctx.eq_mask(x, y.clone())
    ws = ctx.workspace(n)
    call(ctx, "nshe_eq_mask", x.data_ptr(), y.data_ptr(), buf.data_ptr(), n, 1, ws.data_ptr(),
         ws.numel())
    assert torch.equal(buf, want)


@pytest.mark.parametrize("use_graph", [False, True])
def test_items_on_other_items(ctx, use_graph):
    """Item 0's output is item 1's operand, item 1's output item 0's, and item
    2 is in place: one wave reads all of them first."""
    a, b, d = cts(ctx, 2, 6), cts(ctx, 2, 7), cts(ctx, 3, 8)
    y = [cts(ctx, 1, 9 + i) for i in range(3)]
    want = [ctx.eq_mask(t.clone(), v) for t, v in zip((a, b, d), y)]
    got = ctx.eq_mask_batched([(a, y[0]), (b, y[1]), (d, y[2])], wave_ct=7, use_graph=use_graph,
                              outs=[b, a, d])
    torch.cuda.synchronize()
    for u, v in zip(got, want):
        assert torch.equal(u, v)


def test_a_later_wave_reads_what_an_earlier_one_wrote(ctx):
    """Waves of two: item 1's operand is item 0's output, a wave before."""
    a, y = cts(ctx, 2, 12), cts(ctx, 1, 13)
    m, z = torch.empty_like(a), torch.empty_like(a)
    first = ctx.eq_mask(a, y)
    want = ctx.eq_mask(first.clone(), y)   # (a clone: its depth is not tracked)
    ctx.eq_mask_batched([(a, y), (m, y)], wave_ct=2, outs=[m, z])
    torch.cuda.synchronize()
    assert torch.equal(m, first) and torch.equal(z, want)
