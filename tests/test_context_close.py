"""Closing a context from Python, without a GPU: which stream it waits for."""
import torch

from paper_2403_08063_amd import solver


def test_close_waits_for_the_contexts_own_stream(monkeypatch):
    calls = []

    class Stream:
        def __init__(self, name):
            self.name = name

        def synchronize(self):
            calls.append(self.name)

    class Lib:
        def mg_destroy(self, ctx):
            calls.append("destroy")

    monkeypatch.setattr(solver, "lib", Lib)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: Stream("current"))
    mg = object.__new__(solver.Multigrid)
    mg.stream, mg.device, mg._ctx = Stream("own"), torch.device("cuda:0"), object()
    mg.close()
    mg.close()
    assert calls == ["own", "destroy"]
