"""Whole steps where the workspace decides: gradient sample groups cut down so
that the run fits the library's own scratch, and the laws' workspaces over the
step's buffers."""
import ctypes as C

import numpy as np
import pytest
import torch

import tr_inputs as ti
from gpu_util import DEV, flat_paper, rel, rounded, say, to_dev, unfold
from oracle import brsgd, tr

pytestmark = pytest.mark.gpu

from paper_2303_16492_amd import _lib as L  # noqa: E402
from paper_2303_16492_amd import api  # noqa: E402
from paper_2303_16492_amd.driver import TRSolver  # noqa: E402


def _problem(I, R, dtype, seed=5):
    X = tr.full_tensor(ti.gaussian_cores(seed, len(I), I, R))
    X = rounded(X / np.sqrt(np.mean(X * X)), dtype)
    init = [rounded(c, dtype) for c in ti.gaussian_cores(seed + 1, len(I), I, R, scale=(1.0 / np.prod(R)) ** (1 / (2 * len(I))))]
    return X, init, to_dev(flat_paper(X), dtype)


# sizes whose preferred sample groups take the workspace past the scratch: FP32
# rows of 16 and of 4 bytes, and FP64
@pytest.mark.parametrize("I,R,prec,m", [([60, 22, 30], [12, 12, 12], "f32", 13000), ([819, 5, 4], [12, 12, 12], "f32", 3128),
                                        ([600, 23, 5], [5, 9, 5], "f32", 54000), ([3, 244, 607], [6, 16, 4], "f64", 5809)])
def test_run_with_fewer_sample_groups(I, R, prec, m):
    dtype = torch.float64 if prec == "f64" else torch.float32
    X, init, dX = _problem(I, R, dtype)
    outs = []
    for noalloc in (False, True):
        sol = TRSolver([to_dev(unfold(c), dtype) for c in init], dX, I, R, m, prec=prec, seed=3,
                       rule=api.step_rule("fixed", alpha=0.2))
        assert sol.ws.numel() <= L.TR_NOALLOC_SCRATCH_BYTES
        losses = torch.zeros(3, dtype=torch.float64, device=DEV)
        say("fewer groups", I, R, prec, m, "noalloc", noalloc)
        if noalloc:
            api.tr_run_noalloc(sol.problem, sol.config, sol.t_dev, 3, losses, sol.status)
        else:
            sol.run(3, losses)
        outs.append(([c.cpu().numpy() for c in sol.cores], losses.cpu().numpy()))
    for a, b in zip(outs[0][0], outs[1][0]):
        assert np.array_equal(a, b)
    assert np.array_equal(outs[0][1], outs[1][1])
    st = brsgd.State(init)
    cfg = brsgd.Config(m=m, alpha=0.2, seed=3)
    for _ in range(3):
        brsgd.step(st, X, cfg)
    for k in range(len(I)):
        assert rel(outs[0][0][k], unfold(st.cores[k])) < (1e-11 if prec == "f64" else 1e-4), k


@pytest.mark.parametrize("law", ["E", "L", "O"])
@pytest.mark.parametrize("m_H", [0, 150])
@pytest.mark.parametrize("shape", [([30, 25, 28], [3, 4, 3]), ([28, 28, 28], [3, 3, 3]), ([14, 70, 13], [12, 12, 12])])
def test_law_workspace_over_the_step_with_two_streams(shape, m_H, law):
    """Scaled steps under a law: the second stream's branch and the law's
    workspace change nothing, bit for bit."""
    I, R = shape
    X, init, dX = _problem(I, R, torch.float32)
    m = 6 * max(R[k] * R[(k + 1) % 3] for k in range(3))
    outs = []
    for overlap in (False, True):
        s = TRSolver([to_dev(unfold(c), torch.float32) for c in init], dX, I, R, m, law=law, scaled=True, prec="f32",
                     rule=api.step_rule("fixed", alpha=0.3), damping=1e-4, m_H=m_H and m, overlap=overlap, seed=2)
        losses = torch.zeros(8, dtype=torch.float64, device=DEV)
        say("law over the step", shape, m_H, law, "overlap", overlap)
        s.run(8, losses)
        torch.cuda.synchronize()
        outs.append(([c.clone() for c in s.cores], losses.clone(), int(s.status.item())))
    (ca, la, sa), (cb, lb, sb) = outs
    assert sa == sb and torch.equal(la, lb)
    for a, b in zip(ca, cb):
        assert torch.equal(a, b)
