"""The binding's wide workspaces: taken where most of the free memory stays
free, never under capture, and the call's smallest workspace otherwise (the
device's memory stands in as numbers; no GPU)."""
import pytest
import torch

from paper_2602_24271_amd import Context

GB = 1 << 30


@pytest.fixture
def ctx(monkeypatch):
    c = Context.__new__(Context)
    c._h, c._ws, c.device = None, None, torch.device("cpu")
    state = {"free": 0, "cached": 0, "capturing": False, "limit": 1 << 60}

    def empty(n, **kw):
        if n > state["limit"]:
            raise torch.OutOfMemoryError
        return torch.zeros(1, dtype=torch.uint8).expand(n)
    monkeypatch.setattr(torch, "empty", empty)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: state["capturing"])
    monkeypatch.setattr(torch.cuda, "mem_get_info", lambda d=None: (state["free"], 288 * GB))
    monkeypatch.setattr(torch.cuda, "memory_reserved", lambda d=None: state["cached"])
    monkeypatch.setattr(torch.cuda, "memory_allocated", lambda d=None: 0)
    c.state = state
    return c


@pytest.mark.parametrize("free,cached,capturing,got", [
    (200 * GB, 0, False, 3 * GB), (17 * GB, 0, False, 3 * GB), (16 * GB, 0, False, GB),
    (4 * GB, 0, False, GB), (4 * GB, 13 * GB, False, 3 * GB), (200 * GB, 0, True, GB)])
def test_wide_leaves_the_free_memory(ctx, free, cached, capturing, got):
    ctx.state.update(free=free, cached=cached, capturing=capturing)
    assert ctx._workspace_wide(3 * GB, GB).numel() == got


def test_a_large_call_still_takes_what_little_its_batches_add(ctx):
    ctx.state.update(free=200 * GB)
    assert ctx._workspace_wide(56 * GB, 54 * GB).numel() == 56 * GB


def test_held_and_failing(ctx):
    ctx.state.update(free=200 * GB, limit=2 * GB)
    assert ctx._workspace_wide(3 * GB, GB).numel() == GB      # the allocation failed
    ctx.state.update(limit=1 << 60)
    assert ctx._workspace_wide(3 * GB, GB).numel() == 3 * GB
    ctx.state.update(free=0)
    assert ctx._workspace_wide(3 * GB, GB).numel() == 3 * GB  # held already
    assert ctx._workspace_wide(4 * GB, 2 * GB).numel() == 3 * GB
