"""The Python binding's own bookkeeping, with a stand-in for the library (no GPU needed)."""
import types

import pytest

from paper_2506_22668_amd import binding


class _Lib:
    """Counts the graphs that are alive."""

    def __init__(self):
        self.alive, self.extracted, self.explained = 0, 0, 0

    def ds_extract(self, h, target, opts, out):
        self.alive += 1
        self.extracted += 1
        out._obj.value = 4096 + self.extracted
        return 0

    def ds_cgraph_get_info(self, cg, info):
        info._obj.num_players = 5
        return 0

    def ds_cgraph_free(self, h, cg):
        assert cg.value == 4096 + self.extracted
        self.alive -= 1
        return 0

    def ds_explain_cgraph(self, h, cg, *args):
        assert cg.value == 4096 + self.extracted
        self.alive -= 1
        self.explained += 1
        return 0


def _context(empty=None, sync=None):
    import torch
    ctx = object.__new__(binding.Context)
    ctx.torch = types.SimpleNamespace(float32=torch.float32, int64=torch.int64, empty=empty or torch.empty)
    ctx.lib, ctx.device, ctx.h = _Lib(), torch.device("cpu"), None
    ctx._sync_inputs = sync or (lambda: None)
    return ctx


def test_an_explanation_takes_over_the_extracted_graph():
    ctx = _context()
    phi, es, ed, rep, rc = ctx.explain(3, 100, 1)
    assert len(phi) == len(es) == len(ed) == 5 and rc == 0
    assert (ctx.lib.alive, ctx.lib.extracted, ctx.lib.explained) == (0, 1, 1)


def test_no_memory_for_the_buffers_releases_the_extracted_graph():
    calls = []

    def empty(*a, **k):
        import torch
        calls.append(a)
        if len(calls) == 2:
            raise torch.cuda.OutOfMemoryError("no memory")
        return torch.empty(*a, **k)

    ctx = _context(empty=empty)
    with pytest.raises(RuntimeError):
        ctx.explain(3, 100, 1)
    assert (ctx.lib.alive, ctx.lib.extracted, ctx.lib.explained) == (0, 1, 0)


@pytest.mark.parametrize("args", [("x", 100, 1), (3, "many", 1), (3, 100, None)])
def test_arguments_are_converted_before_a_graph_is_extracted(args):
    ctx = _context()
    with pytest.raises((TypeError, ValueError)):
        ctx.explain(*args)
    assert (ctx.lib.alive, ctx.lib.extracted, ctx.lib.explained) == (0, 0, 0)
