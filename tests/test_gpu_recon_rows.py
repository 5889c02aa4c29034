"""The subchain rows of the relative error and of the reconstruction at the edges
of their two forms, against the oracle."""
import numpy as np
import pytest
import torch

from gpu_util import DEV, problem, rel, rounded, say, to_dev
from oracle import tr
from paper_2303_16492_amd import api

pytestmark = pytest.mark.gpu


# order 3, staged slices: the smallest I_2 whose columns touch eight slices of the
# last core and the first below it, columns below, at and past a block of 128, one
# row of the product per thread and several, ranks 1 and 16; then orders 6 to 8
# with ranks within 4 and 8, entries in paper order and reversed
@pytest.mark.parametrize("I,R,order", [([33, 22, 17], [2, 2, 2], "paper"), ([33, 21, 17], [2, 2, 2], "paper"),
                                       ([5, 127, 3], [5, 5, 5], "reversed"), ([40, 128, 2], [16, 4, 8], "paper"),
                                       ([70, 23, 29], [16, 2, 16], "reversed"), ([9, 1000, 2], [4, 3, 4], "paper"),
                                       ([3, 64, 5], [1, 1, 1], "paper"), ([31, 40, 3], [3, 4, 2], "reversed"),
                                       ([32, 30, 1], [8, 5, 3], "paper"), ([2, 50, 30], [1, 16, 1], "paper"),
                                       ([6, 5, 4, 3, 2, 3], [4, 3, 2, 1, 4, 2], "paper"),
                                       ([5, 4, 3, 2, 4, 3], [8, 7, 5, 8, 6, 4], "reversed"),
                                       ([3, 2, 3, 4, 2, 3, 2], [2, 2, 2, 2, 2, 2, 2], "reversed"),
                                       ([2, 3, 2, 3, 2, 3, 2, 3], [8, 2, 5, 8, 1, 6, 8, 7], "paper")])
@pytest.mark.parametrize("xdt", [torch.float32, torch.float16])
def test_error_and_reconstruction_rows(I, R, order, xdt):
    I, R, cores, X, dcores, dX = problem(57, len(I), I, R, torch.float32)
    X = rounded(X, xdt)
    strides = api.paper_strides(I)
    if order == "reversed":
        strides = [int(np.prod(I[k + 1:])) for k in range(len(I))]
    flat = torch.empty(int(np.prod(I)), dtype=xdt, device=DEV)
    flat.as_strided(I, strides).copy_(to_dev(X, xdt))
    desc = api.make_desc(I, R, torch.float32, xdt, strides)
    say("error and reconstruction rows", I, R, order, xdt)
    assert abs(float(api.tr_relerr(desc, dcores, flat)) / tr.rse(cores, X) - 1) < 1e-5
    got = api.tr_reconstruct(desc, dcores).as_strided(I, strides).double().cpu().numpy()
    want = tr.full_tensor(cores)
    assert rel(got, want) < (1e-5 if xdt == torch.float32 else 1e-3)
