"""The streaming FP32 gradient at the column-tile counts between 1, 2, 4, 6 and
their multiples: the largest R_n R_{n+1} in 33-48, 65-80, 129-160 and 193-224
selects kernels with 3, 5, 10 and 14 column tiles, whose LDS pitch, staging length
and column map are their own.  The gradient itself is compared with the oracle's
from the same subchain rows and samples."""
import pytest
import torch

from gpu_util import TOL, problem, rel, say, unfold
from oracle import brsgd
from paper_2303_16492_amd import _lib as L
from paper_2303_16492_amd import api

pytestmark = pytest.mark.gpu


# Every R_n R_{n+1} a multiple of 4 (rows of whole 16-byte pieces), then ranks of
# which one product is not; samples: one ragged chunk of 64, and 33001, which is 516
# chunks of 64 (the last one ragged), more than the groups that two tiles of 64 rows
# leave, so a group has several.  Both tolerances are the FP32 bar (1e-5).
@pytest.mark.parametrize("R", [[6, 6, 8], [5, 7, 6], [8, 10, 8], [8, 9, 7], [12, 12, 12], [13, 11, 12], [14, 11, 7],
                               [14, 14, 14], [15, 13, 14]])
@pytest.mark.parametrize("m", [97, 33001])
@pytest.mark.parametrize("xdt", [torch.float32, torch.float16])
def test_grad_fp32_column_tiles(R, m, xdt):
    dtype = torch.float32
    I = [70, 65, 33]
    I, R, cores, X, dcores, dX = problem(37, 3, I, R, dtype)
    dX = dX.to(xdt)
    X = dX.double().cpu().numpy().reshape(I, order="F")
    desc = api.make_desc(I, R, dtype, xdt)
    for n in range(3):
        say("grad f32", R, m, xdt, "mode", n)
        idx, pF = api.tr_sample(desc, 6, 1, n, m)
        S = api.tr_subchain(desc, n, dcores, idx, m)
        g, loss, _ = api.tr_grad(desc, n, dcores[n], dX, idx, S, pF, m, L.TR_PREC_F32)
        gref, lref = brsgd.stoch_grad(unfold(cores[n]), S.double().cpu().numpy(),
                                      brsgd.gather_fibers(X, n, idx.cpu().numpy()), pF.cpu().numpy(), brsgd.J_of(I, n))
        assert rel(g.cpu().numpy(), gref) < TOL[dtype]
        assert abs(float(loss) - lref) <= TOL[dtype] * abs(lref)
