"""The sampled-entry backward over uneven batches: entries concentrated on few
slices, and every split of the batch over wavefronts and workgroups."""
import numpy as np
import pytest
import torch

import tr_inputs as ti
from gpu_util import DEV, rel, rounded, say, to_dev, unfold
from oracle import brsgd, completion, entry

pytestmark = pytest.mark.gpu

from paper_2303_16492_amd import api  # noqa: E402

# Norm-wise bound of a gradient in FP32: at most 64 products summed in one FP32
# accumulator (64 roundings of 2^-24, 4e-6), the chain of the other slices
# (N R of them, 2e-6) and one rounding a partial sum, whatever the batch size.
TOL = 1e-5


def _check(N, I, R, B, idx):
    cores = [rounded(c, torch.float32) for c in ti.gaussian_cores(5, N, I, R, scale=0.6)]
    x = rounded(ti.standard_normal(7, B), torch.float32)
    desc = api.make_desc(I, R)
    dc = [to_dev(unfold(c), torch.float32) for c in cores]
    didx = to_dev(idx, torch.int32)
    resid, _ = api.tr_entry_fwd(desc, dc, didx, to_dev(x, torch.float32), B)
    grads = api.tr_entry_bwd(desc, dc, didx, resid, B)
    again = api.tr_entry_bwd(desc, dc, didx, resid, B)
    gref = entry.entry_grads(cores, idx, x)
    for k in range(N):
        assert rel(grads[k].cpu().numpy(), unfold(gref[k])) < TOL, k
        assert torch.equal(grads[k], again[k])


# 2060 slices: one wavefront a slice by their number alone.  Every entry on the
# same slices with the same value (the sum of equal terms is where a long FP32
# chain drifts most), then half of them, then none.
@pytest.mark.parametrize("share", [1.0, 0.5, 0.0])
def test_entries_concentrated_on_a_slice(share):
    N, I, R, B = 3, [2049, 5, 6], [4, 8, 4], 65537
    idx = ti.entry_indices(6, I, B)
    idx[:int(share * B)] = [2000, 3, 5]
    say("concentrated entries", share)
    cores = [rounded(c, torch.float32) for c in ti.gaussian_cores(5, N, I, R, scale=0.6)]
    x = np.zeros(B)
    desc = api.make_desc(I, R)
    dc = [to_dev(unfold(c), torch.float32) for c in cores]
    didx = to_dev(idx, torch.int32)
    resid, _ = api.tr_entry_fwd(desc, dc, didx, to_dev(x, torch.float32), B)
    grads = api.tr_entry_bwd(desc, dc, didx, resid, B)
    gref = entry.entry_grads(cores, idx, x)
    for k in range(N):
        e = rel(grads[k].cpu().numpy(), unfold(gref[k]))
        say("  core", k, e)
        assert e < TOL, k


# wavefronts of a workgroup 1, 2, 4, 8 and 16; one part of the batch and
# several, the last share ragged or empty; the smallest cores, which every entry
# falls on; more slices than one grid takes (2^22)
@pytest.mark.parametrize("N,I,R,B", [(2, [3000, 20], [3, 2], 900), (2, [1500, 20], [4, 8], 1000),
                                     (3, [500, 100, 30], [5, 3, 4], 700), (3, [300, 20, 9], [8, 8, 8], 600),
                                     (3, [20, 10, 9], [4, 4, 4], 1500), (2, [1, 1], [16, 12], 40000),
                                     (3, [40, 30, 5], [7, 9, 3], 16385), (4, [12, 9, 2, 7], [3, 4, 2, 4], 33000),
                                     (5, [14456, 826, 580, 9, 2], [3, 2, 2, 7, 8], 7975),
                                     (2, [(1 << 22) + 3, 2], [1, 1], 70)])
def test_entry_split_over_wavefronts_and_parts(N, I, R, B):
    say("entry split", N, I, R, B)
    idx = ti.entry_indices(6, I, B)
    if I[0] > 1 << 22:   # both passes over the slices
        idx[::2, 0] = I[0] - 1 - (np.arange(len(idx[::2])) % 3)
    _check(N, I, R, B, idx)


@pytest.mark.parametrize("block", [False, True])
def test_completion_step_over_parts_of_the_batch(block):
    """Two parts of the batch (more than 16 x 1024 entries): the update adds them."""
    I, R, B, steps = [40, 30, 5], [3, 4, 2], 20000, 3
    cores = [rounded(c, torch.float32) for c in ti.gaussian_cores(8, 3, I, R, scale=0.6)]
    rng = np.random.default_rng(3)
    obs_idx = np.stack([rng.integers(0, i, 6000) for i in I], axis=1).astype(np.int32)
    obs_x = rounded(rng.standard_normal(6000), torch.float32)
    cfg = completion.CompletionConfig(B=B, lam=0.05, block=block, alpha=0.02, seed=4)
    st = brsgd.State([c.copy() for c in cores])
    losses = [completion.completion_step(st, obs_idx, obs_x, cfg) for _ in range(steps)]
    dc = [to_dev(unfold(c), torch.float32) for c in cores]
    t = torch.zeros(1, dtype=torch.int64, device=DEV)
    lo = torch.zeros(steps, dtype=torch.float64, device=DEV)
    c = api.completion_config(B, block=block, lam=0.05, rule=api.step_rule("fixed", alpha=0.02), seed=4)
    say("completion over parts", block)
    api.tr_completion_run(api.make_desc(I, R), dc, None, to_dev(obs_idx, torch.int32), to_dev(obs_x, torch.float32), c,
                          t, steps, loss_out=lo)
    assert rel(lo.cpu().numpy(), np.array(losses)) < 1e-5
    for k in range(3):
        assert rel(dc[k].cpu().numpy(), unfold(st.cores[k])) < 1e-5, k
