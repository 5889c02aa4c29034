"""Scaled steps on one stream, where the gradient's 16-byte forms and the inverse are
one launch, against the same steps on two streams, where they are two: the same
bits, since every block does the same work in the same order."""
import pytest
import torch

import tr_inputs as ti
from gpu_util import DEV, flat_paper, rounded, say, to_dev, unfold
from oracle import tr

pytestmark = pytest.mark.gpu

from paper_2303_16492_amd import api  # noqa: E402
from paper_2303_16492_amd.driver import TRSolver  # noqa: E402


def _runs(I, R, m, prec, xdt, steps=7, law="U", m_H=0, alpha=0.5):
    dtype = torch.float64 if prec == "f64" else torch.float32
    X = rounded(tr.full_tensor(ti.gaussian_cores(1, len(I), I, R)), dtype)
    got = []
    for overlap in (True, False):
        cores = [to_dev(unfold(rounded(c, dtype)), dtype) for c in ti.gaussian_cores(2, len(I), I, R, scale=0.5)]
        s = TRSolver(cores, to_dev(flat_paper(X), dtype).to(xdt), I, R, m, law=law, scaled=True, prec=prec, m_H=m_H,
                     seed=3, rule=api.step_rule("fixed", alpha=alpha), overlap=overlap)
        losses = torch.zeros(steps, dtype=torch.float64, device=DEV)
        say("one stream", I, R, m, prec, xdt, law, m_H, "overlap", overlap)
        s.run(steps, losses)
        torch.cuda.synchronize()
        got.append((s.cores, losses, int(s.status)))
    return got


def _same(two, one):
    assert two[2] == one[2]
    assert torch.equal(two[1].view(torch.int64), one[1].view(torch.int64))
    for a, b in zip(two[0], one[0]):
        assert torch.equal(a.contiguous().view(torch.uint8), b.contiguous().view(torch.uint8))


# 3 to 8 column tiles; the largest R_n R_{n+1} 36 to 128, not every mode's the same in
# three of them; rows at the edges of a 64-row tile
SHAPES = [([30, 64, 65], [6, 6, 6]), ([63, 33, 20], [8, 8, 8]), ([40, 20, 30], [8, 10, 8]), ([40, 20, 31], [8, 12, 8]),
          ([70, 40, 33], [10, 10, 10]), ([66, 40, 35], [16, 8, 4])]


@pytest.mark.parametrize("I,R", SHAPES)
@pytest.mark.parametrize("prec,xdt", [("f32", torch.float32), ("f32", torch.float16), ("bf16", torch.float32),
                                      ("bf16", torch.float16), ("f16", torch.float32), ("f16", torch.float16)])
def test_one_stream_equals_two(I, R, prec, xdt):
    two, one = _runs(I, R, 1601, prec, xdt)
    assert two[2] == 0
    _same(two, one)


# one sample and fewer samples than R_n R_{n+1} (the damping ladder, or no update); one
# chunk of 128; a group past the last sample; 8 row tiles of 64 and 32 groups, with the
# inverse more blocks than CUs (two launches), and 7 tiles (one); an own H draw; the laws
# of the cores
@pytest.mark.parametrize("I,R,m,kw", [([30, 25, 28], [6, 6, 6], 1, {}), ([30, 25, 28], [8, 8, 8], 50, {}),
                                      ([30, 25, 28], [6, 6, 6], 128, {}), ([70, 25, 28], [6, 6, 6], 1100, {}),
                                      ([500, 12, 14], [6, 6, 6], 4096, {}), ([420, 12, 14], [6, 6, 6], 4096, {}),
                                      ([40, 35, 38], [6, 6, 6], 700, dict(m_H=333)),
                                      ([60, 70, 80], [6, 6, 6], 700, dict(law="L")),
                                      ([9, 8, 7, 10], [6, 6, 6, 6], 900, dict(law="E"))])
@pytest.mark.parametrize("prec", ["f32", "bf16"])
def test_one_stream_equals_two_at_the_edges(I, R, m, kw, prec):
    _same(*_runs(I, R, m, prec, torch.float32, **kw))
