"""A captured run outlives the names of its solver and of its loss buffer."""
import gc
import weakref

import numpy as np
import pytest
import torch

import tr_inputs as ti
from gpu_util import DEV, flat_paper, rounded, say, to_dev, unfold
from oracle import tr

pytestmark = pytest.mark.gpu

from paper_2303_16492_amd import _lib as L  # noqa: E402
from paper_2303_16492_amd import api  # noqa: E402
from paper_2303_16492_amd.driver import TRSolver  # noqa: E402


def _solver(prec, scaled=True, m_H=0, seed=3):
    dtype = torch.float64 if prec == "f64" else torch.float32
    I, R = [30, 25, 28], [3, 4, 3]
    X = rounded(tr.full_tensor(ti.gaussian_cores(1, 3, I, R)), dtype)
    cores = [to_dev(unfold(rounded(c, dtype)), dtype) for c in ti.gaussian_cores(2, 3, I, R, scale=0.5)]
    return TRSolver(cores, to_dev(flat_paper(X), dtype), I, R, 200, scaled=scaled, prec=prec, m_H=m_H, seed=seed,
                    rule=api.step_rule("fixed", alpha=0.5 if scaled else 0.05))


@pytest.mark.parametrize("scaled", [False, True])
def test_graph_keeps_what_it_replays_into(scaled, monkeypatch):
    ref = _solver("f32", scaled)
    ref.run(7)
    torch.cuda.synchronize()
    sol = _solver("f32", scaled)
    losses = torch.zeros(3, dtype=torch.float64, device=DEV)
    say("graph lifetime, scaled", scaled)
    g = sol.capture(3, losses)
    cores, alive, buf = sol.cores, weakref.ref(sol), weakref.ref(losses)
    del sol, losses
    gc.collect()
    junk = [torch.full((1 << 18,), float("nan"), device=DEV) for _ in range(8)]   # takes freed blocks, if any are
    g.replay()
    g.replay()
    torch.cuda.synchronize()
    assert alive() is not None and buf() is not None
    assert all(torch.equal(a, b) for a, b in zip(cores, ref.cores))
    assert np.all(np.isfinite(buf().cpu().numpy()))
    del junk
    # dropped: the graph first, then the events and buffers
    order = []
    gone = L.HipEvent.__del__
    monkeypatch.setattr(L.HipEvent, "__del__", lambda self: (order.append("event"), gone(self)))
    reset = type(g).reset
    monkeypatch.setattr(type(g), "reset", lambda self: (order.append("graph"), reset(self)), raising=False)
    del g
    gc.collect()
    assert alive() is None and buf() is None
    assert order == ["graph"] + ["event"] * (3 if scaled else 0)


@pytest.mark.parametrize("prec,m_H", [("f32", 0), ("f32", 150), ("f64", 0), ("f64", 150), ("bf16", 0), ("f16", 0)])
def test_captured_run_stays_on_one_stream(prec, m_H):
    """Nothing of it is captured on the solver's second stream; the steps are those
    of the eager run on two."""
    ref = _solver(prec, m_H=m_H)
    assert ref.opts is not None
    ref.run(7)   # eager: two streams
    torch.cuda.synchronize()
    sol = _solver(prec, m_H=m_H)
    say("captured run", prec, m_H)
    sol.run(1)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        sol.run(3)
        with torch.cuda.stream(sol.aux):
            joined = torch.cuda.is_current_stream_capturing()
    assert not joined
    g.replay()
    g.replay()
    torch.cuda.synchronize()
    assert sol.t == 7 and all(torch.equal(a, b) for a, b in zip(sol.cores, ref.cores))
