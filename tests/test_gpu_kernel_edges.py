"""Kernel variants at the edges of their ranges (tiles, remainders, smallest
and largest sizes), against the oracle."""
import numpy as np
import pytest
import torch

import tr_inputs as ti
from gpu_util import DEV, TOL, fold, problem, rel, rounded, say, to_dev, unfold
from oracle import brsgd, entry, sampling, tr
from paper_2303_16492_amd import _lib as L
from paper_2303_16492_amd import api
from paper_2303_16492_amd.driver import TRSolver

pytestmark = pytest.mark.gpu


# R_n R_{n+1}: 144 x3; 130, 208, 160; 256, 176, 176; 240, 208, 195; 256, 16, 16;
# 154, 77, 98 - every slot count of the wide sweep, one partial last pivot
# block, tile columns far below the widest mode's.
@pytest.mark.parametrize("R", [[12, 12, 12], [10, 13, 16], [16, 16, 11], [15, 16, 13], [16, 16, 1], [14, 11, 7]])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_scaled_update_wide_sweep(R, dtype):
    I = [2 * max(R) + 5, 2 * max(R) + 4, 2 * max(R) + 3]
    I, R, cores, X, dcores, dX = problem(23, 3, I, R, dtype)
    desc = api.make_desc(I, R, dtype)
    prec = L.TR_PREC_F64 if dtype == torch.float64 else L.TR_PREC_F32
    for n in range(3):
        RRn = R[n] * R[(n + 1) % 3]
        m = 6 * RRn + 17
        say("wide sweep", R, "mode", n, "RR", RRn, dtype)
        idx, pF = api.tr_sample(desc, 8, n, n, m)
        S = api.tr_subchain(desc, n, dcores, idx, m)
        g, loss, gram = api.tr_grad(desc, n, dcores[n], dX, idx, S, pF, m, prec, want_gram=True)
        core = dcores[n].clone()
        st = api.tr_update(desc, n, core, g, gram=gram, rule=api.step_rule("fixed", alpha=0.7), t=0)
        p, sref = brsgd.scaled_direction(g.double().cpu().numpy(), gram.cpu().numpy())
        assert int(st) == sref == 0
        cond = np.linalg.cond(gram.cpu().numpy())
        assert rel(core.cpu().numpy(), unfold(cores[n]) + 0.7 * p) < max(TOL[dtype], 1e-15 * cond), cond


@pytest.mark.parametrize("R", [[12, 12, 12], [16, 16, 16]])
def test_wide_sweep_damping_ladder(R):
    """A Gram with an exactly zero row and column: the ladder takes its first
    rung, as the oracle's does, and a zero Gram leaves the core unchanged."""
    dtype = torch.float64
    rr = R[0] * R[1]
    desc = api.make_desc([40, 30, 30], R, dtype)
    rng = np.random.default_rng(4)
    A = rng.standard_normal((3 * rr, rr))
    A[:, rr // 2] = 0.0
    h = A.T @ A / (3 * rr)
    g = rng.standard_normal((40, rr))
    core0 = rng.standard_normal((40, rr))
    to = lambda a: torch.from_numpy(a).to(DEV)
    say("wide ladder", R)
    core = to(core0).clone()
    st = int(api.tr_update(desc, 0, core, to(g), gram=to(h), rule=api.step_rule("fixed", alpha=1.0)))
    p, sref = brsgd.scaled_direction(g, h)
    assert st == sref == brsgd.DEV_DAMPED
    hd = h + 1e-10 * np.trace(h) / rr * np.eye(rr)
    assert rel(core.cpu().numpy(), core0 + p) < 1e-15 * np.linalg.cond(hd)
    core = to(core0).clone()
    st = int(api.tr_update(desc, 0, core, to(g), gram=to(0.0 * h), rule=api.step_rule("fixed", alpha=1.0)))
    assert st == L.TR_DEV_NOT_SPD and np.array_equal(core.cpu().numpy(), core0)


# rows at the edges of 16-row tiles and 64-row blocks, samples at the edges of
# 16-sample tiles and 32-sample chunks (and several chunks per group), ranks at
# the edges of 16-column tiles and of every register width
@pytest.mark.parametrize("I,R,m", [([1, 16, 17], [4, 4, 4], 31), ([15, 63, 64], [1, 1, 1], 32),
                                   ([65, 16, 33], [5, 16, 5], 33), ([129, 17, 15], [9, 9, 9], 1),
                                   ([64, 48, 20], [8, 16, 8], 64), ([20, 70, 18], [13, 10, 16], 97),
                                   ([400, 12, 9], [3, 5, 2], 3001)])
def test_grad_fp64_tiles(I, R, m):
    dtype = torch.float64
    I, R, cores, X, dcores, dX = problem(33, 3, I, R, dtype)
    desc = api.make_desc(I, R, dtype)
    for n in range(3):
        say("grad f64", I, R, m, "mode", n)
        idx, pF = api.tr_sample(desc, 4, 1, n, m)
        S = api.tr_subchain(desc, n, dcores, idx, m)
        g, loss, _ = api.tr_grad(desc, n, dcores[n], dX, idx, S, pF, m, L.TR_PREC_F64)
        idn, pFn = idx.cpu().numpy(), pF.cpu().numpy()
        gref, lref = brsgd.stoch_grad(unfold(cores[n]), S.cpu().numpy(), brsgd.gather_fibers(X, n, idn), pFn,
                                      brsgd.J_of(I, n))
        assert rel(g.cpu().numpy(), gref) < TOL[dtype]
        assert abs(float(loss) - lref) <= TOL[dtype] * abs(lref)


# every column-tile count of the streaming FP32 form (R_n R_{n+1} = 16 to 256,
# with and without whole 16-byte rows), one sample to several chunks of 64 per
# group (the last one ragged), FP32 and FP16 tensors
@pytest.mark.parametrize("I,R,m", [([70, 16, 15], [4, 4, 4], 64), ([65, 17, 16], [5, 5, 5], 63),
                                   ([130, 12, 9], [10, 10, 10], 32001), ([66, 12, 9], [9, 9, 9], 40001),
                                   ([64, 12, 9], [7, 7, 7], 65), ([63, 20, 9], [11, 11, 11], 1),
                                   ([450, 20, 9], [8, 6, 7], 9001), ([70, 12, 30], [13, 11, 13], 700),
                                   ([400, 12, 9], [15, 15, 15], 10007), ([80, 33, 17], [16, 14, 16], 130)])
@pytest.mark.parametrize("xdt", [torch.float32, torch.float16])
def test_grad_fp32_streaming(I, R, m, xdt):
    dtype = torch.float32
    I, R, cores, X, dcores, dX = problem(34, 3, I, R, dtype)
    dX = dX.to(xdt)
    X = dX.double().cpu().numpy().reshape(I, order="F")
    desc = api.make_desc(I, R, dtype, xdt)
    for n in range(3):
        say("grad f32", I, R, m, xdt, "mode", n)
        idx, pF = api.tr_sample(desc, 4, 1, n, m)
        S = api.tr_subchain(desc, n, dcores, idx, m)
        g, loss, _ = api.tr_grad(desc, n, dcores[n], dX, idx, S, pF, m, L.TR_PREC_F32)
        idn, pFn = idx.cpu().numpy(), pF.cpu().numpy()
        gref, lref = brsgd.stoch_grad(unfold(cores[n]), S.double().cpu().numpy(), brsgd.gather_fibers(X, n, idn), pFn,
                                      brsgd.J_of(I, n))
        assert rel(g.cpu().numpy(), gref) < TOL[dtype]
        assert abs(float(loss) - lref) <= TOL[dtype] * abs(lref)


# sampled entries: every packing of slices (rank bounds 4, 8, 16; whole 16-byte
# slices or not), orders 2 and 8, every number of slices per workgroup (1 to
# 16), one index holding every entry, lists around 64 entries and past one
# window of the scan, large modes
@pytest.mark.parametrize("N,I,R,B", [(8, [3, 2, 4, 2, 3, 2, 2, 5], [4, 3, 2, 1, 4, 2, 3, 4], 1000),
                                     (8, [2, 3, 2, 3, 2, 3, 2, 3], [8, 5, 7, 8, 6, 8, 8, 4], 130),
                                     (2, [1, 1], [16, 12], 1025), (2, [17, 1], [4, 4], 64), (3, [1, 30, 2], [8, 8, 8], 5000),
                                     (3, [2048, 5, 6], [4, 4, 4], 3000), (3, [2049, 5, 6], [4, 8, 4], 17),
                                     (2, [32768, 6], [2, 3], 2000), (2, [32769, 6], [2, 3], 2000),
                                     (4, [9, 8, 7, 6], [12, 16, 9, 13], 40001)])
def test_entry_packs_and_lists(N, I, R, B):
    dtype = torch.float32
    cores = [rounded(c, dtype) for c in ti.gaussian_cores(5, N, I, R, scale=0.6)]
    idx = ti.entry_indices(6, I, B)
    x = rounded(ti.standard_normal(7, B), dtype)
    bad = np.zeros(B, dtype=bool)
    if B > 64:   # invalid indices: NaN residual, no gradient contribution
        bad[[3, B // 2]] = True
        idx[3, 0], idx[B // 2, N - 1] = I[0], -1
    ok = ~bad
    desc = api.make_desc(I, R, dtype)
    dc = [to_dev(unfold(c), dtype) for c in cores]
    didx = to_dev(idx, torch.int32)
    say("entries", N, I, R, B)
    resid, _ = api.tr_entry_fwd(desc, dc, didx, to_dev(x, dtype), B)
    r = resid.cpu().numpy()
    _, rref = entry.entry_loss(cores, idx[ok], x[ok])
    assert np.array_equal(np.isnan(r), bad) and rel(r[ok], rref) < 1e-5
    grads = api.tr_entry_bwd(desc, dc, didx, resid, B, scale=ok.sum() and B / ok.sum())
    again = api.tr_entry_bwd(desc, dc, didx, resid, B, scale=ok.sum() and B / ok.sum())
    gref = entry.entry_grads(cores, idx[ok], x[ok])
    for k in range(N):
        assert rel(grads[k].cpu().numpy(), unfold(gref[k])) < 1e-5, k
        assert torch.equal(grads[k], again[k])


def test_entry_infinity_stays_with_its_entries():
    """One slice of one core holds an infinity: the gradients of the rows that
    no entry through it touches stay finite and exact, packed or not."""
    N, I, R, B = 3, [8, 9, 10], [4, 4, 4], 60
    cores = [rounded(c, torch.float32) for c in ti.gaussian_cores(8, N, I, R, scale=0.6)]
    idx = ti.entry_indices(9, I, B)
    x = rounded(ti.standard_normal(10, B), torch.float32)
    keep = idx[:, 0] != 2
    dc = [to_dev(unfold(c), torch.float32) for c in cores]
    dc[0][2, 5] = float("inf")
    desc = api.make_desc(I, R, torch.float32)
    say("entries with an infinity")
    resid, _ = api.tr_entry_fwd(desc, dc, to_dev(idx, torch.int32), to_dev(x, torch.float32), B)
    grads = api.tr_entry_bwd(desc, dc, to_dev(idx, torch.int32), resid, B)
    gref = entry.entry_grads(cores, idx[keep], x[keep])
    assert np.all(np.isfinite(resid.cpu().numpy()[keep]))
    for k in range(N):
        clean = np.setdiff1d(np.arange(I[k]), idx[~keep][:, k])
        got = grads[k].cpu().numpy()[clean] * B / keep.sum()
        assert rel(got, unfold(gref[k])[clean]) < 1e-5


# ranks <= 4, 8, 16 (samples packed 4, 2 and 1 to an operand), whole 16-byte
# slices or not, orders 2 to 8, rank 1, sample counts around one block of 16
@pytest.mark.parametrize("I,R", [([5, 6], [4, 4]), ([5, 6], [3, 16]), ([5, 6, 7], [1, 4, 2]), ([5, 6, 7], [8, 4, 8]),
                                 ([5, 6, 7], [12, 16, 4]), ([5, 6, 7], [7, 1, 8]), ([3, 4, 5, 6], [5, 5, 5, 5]),
                                 ([3, 4, 5, 6, 2], [13, 2, 16, 9, 1]), ([2, 3, 2, 3, 2, 3], [4, 3, 2, 1, 4, 3]),
                                 ([2, 3, 2, 3, 2, 3, 2, 3], [8, 4, 8, 8, 4, 8, 8, 8]),
                                 ([2, 3, 2, 3, 2, 3, 2, 3], [6, 9, 16, 3, 11, 2, 7, 5])])
def test_subchain_chains_fp32(I, R):
    N = len(I)
    cores = [rounded(c, torch.float32) for c in ti.gaussian_cores(12, N, I, R, scale=0.7)]
    desc = api.make_desc(I, R, torch.float32)
    dc = [to_dev(unfold(c), torch.float32) for c in cores]
    rng = np.random.default_rng(2)
    for n in range(N):
        for m in (1, 15, 17, 70):
            idx = np.stack([rng.integers(0, i, m) for i in I], axis=1).astype(np.int32)
            say("subchain chains", I, R, "mode", n, "m", m)
            ref = brsgd.subchain_rows(cores, n, idx)
            mag = brsgd.subchain_rows([np.abs(c) for c in cores], n, idx)
            bad = np.zeros(m, dtype=bool)
            inf = np.zeros(m, dtype=bool)
            k = (n + 1) % N
            core = dc[k].clone()
            if m > 2:   # a rejected index: a row of NaN; an infinity: nobody else's
                bad[m // 2] = True
                idx[m // 2, (n + N - 1) % N] = I[(n + N - 1) % N]
                core[0, 0] = float("inf")
                inf = idx[:, k] == 0
            S = api.tr_subchain(desc, n, [core if j == k else c for j, c in enumerate(dc)], to_dev(idx, torch.int32),
                                m).cpu().numpy()
            ok = ~bad & ~inf
            assert np.all(np.isnan(S[bad])) and np.all(np.isfinite(S[ok]))
            # N - 2 products of R_k terms, each term and sum rounded once
            assert np.all(np.abs(S - ref)[ok] <= (2.0 ** -24 * sum(R) * 2 * mag)[ok])


# range ends, one to several rounds of the eight-way and of the 64-way search,
# laws with nearly all their mass in one entry (first, last or neither)
@pytest.mark.parametrize("I", [[1, 2, 7], [8, 9, 63], [64, 65, 3], [4097, 5, 512], [70001, 1, 1]])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_cdf_draws(I, dtype):
    N, m = 3, 333
    desc = api.make_desc(I, [3, 2, 4], dtype)
    rng = np.random.default_rng(6)
    for heavy in (None, 0, -1):
        w = [rng.integers(1, 1 << 20, i).astype(np.uint64) for i in I]
        if heavy is not None:
            for v in w:
                v[heavy] = 1 << 36
        up = lambda a: torch.from_numpy(np.cumsum(a, dtype=np.uint64).astype(np.int64)).to(DEV)
        for n in range(N):
            say("cdf draws", I, "mode", n, "heavy", heavy, dtype)
            idx, pF = api.tr_sample(desc, 4, 9, n, m, cdf=[up(a) for a in w])
            iref, pref = sampling.draw(4, 9, n, m, I, w_modes=w)
            assert np.array_equal(idx.cpu().numpy(), iref) and np.array_equal(pF.cpu().numpy(), pref)
            J = int(np.prod([s for k, s in enumerate(I) if k != n]))
            wJ = rng.integers(1, 1 << 12, J).astype(np.uint64)
            if heavy is not None:
                wJ[heavy] = 1 << 30
            idx, pF = api.tr_sample(desc, 4, 9, n, m, cdf_J=up(wJ))
            iref, pref = sampling.draw(4, 9, n, m, I, w_J=wJ)
            assert np.array_equal(idx.cpu().numpy(), iref) and np.array_equal(pF.cpu().numpy(), pref)


def _weights(cdf):
    return np.diff(np.concatenate([[0], cdf.cpu().numpy()])).astype(np.int64)


# the one-launch law with 1 to 4 tile columns (full and partial), tall, square
# and wide cores, row counts around batches of K steps and tiles, its largest
# I_k and the first past it; wide cores above 64 rows and above 128
@pytest.mark.parametrize("I,R", [([1, 2, 16], [4, 4, 1]), ([4096, 17, 15], [4, 4, 4]), ([4097, 17, 33], [4, 4, 4]),
                                 ([33, 32, 1000], [5, 5, 6]), ([1024, 9, 31], [8, 4, 1]), ([1025, 9, 31], [8, 4, 1]),
                                 ([455, 47, 49], [6, 8, 5]), ([256, 64, 63], [8, 8, 8]), ([257, 64, 63], [8, 8, 8]),
                                 ([60, 30, 64], [16, 16, 16]), ([66, 65, 100], [10, 10, 10]),
                                 ([150, 129, 40], [12, 13, 12]), ([256, 255, 257], [16, 16, 16])])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_leverage_forms(I, R, dtype):
    cores = [rounded(c, dtype) for c in ti.gaussian_cores(41, 3, I, R, scale=0.7)]
    desc = api.make_desc(I, R, dtype)
    for k in range(3):
        G = unfold(cores[k])
        s = np.linalg.svd(G, compute_uv=False)
        if s[-1] < 1e-5 * s[0]:   # near the rank test: covered by exact deficiency below
            continue
        say("leverage forms", I, R, dtype, "core", k)
        cdf, st = api.tr_dist(desc, k, L.TR_LAW_LEVERAGE, to_dev(G, dtype))
        wref = sampling.quantize(sampling.dist_leverage(cores[k])).astype(np.int64)
        # 64 units, and the squared condition of the Gram's rounding
        assert int(st) == 0 and np.max(np.abs(_weights(cdf) - wref)) <= 64 + 2.0 ** -10 * (s[0] / s[-1]) ** 2
        if G.shape[0] > 2:   # rows of lower rank, exactly
            H = G.copy()
            H[-1] = H[0]
            if G.shape[1] > 1:
                H[:, -1] = H[:, 0]
            say("leverage forms", I, R, dtype, "core", k, "deficient")
            cdf, st = api.tr_dist(desc, k, L.TR_LAW_LEVERAGE, to_dev(H, dtype))
            wref = sampling.quantize(sampling.dist_leverage(fold_core(H, R, k))).astype(np.int64)
            sd = np.linalg.svd(H, compute_uv=False)
            sd = sd[sd > 1e-10 * sd[0]]
            assert int(st) == 0 and np.max(np.abs(_weights(cdf) - wref)) <= 64 + 2.0 ** -10 * (sd[0] / sd[-1]) ** 2


def fold_core(G, R, k):
    return fold(G, R[k], R[(k + 1) % len(R)])


# every core's law in the first launch and the step's core after each step:
# one-launch forms and the forms of several launches
@pytest.mark.parametrize("law,I,R", [("L", [20, 30, 25], [3, 4, 5]), ("L", [90, 30, 80], [10, 9, 8]),
                                     ("E", [20, 30, 25], [3, 4, 5]), ("E", [300, 260, 40], [16, 16, 14])])
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_laws_follow_the_cores(law, I, R, prec):
    dtype = torch.float64 if prec == "f64" else torch.float32
    I, R, cores, X, dcores, dX = problem(43, 3, I, R, dtype)
    desc = api.make_desc(I, R, dtype)
    solver = TRSolver(dcores, dX, I, R, 64, law=law, prec=prec, rule=api.step_rule("fixed", alpha=1e-3), seed=5)
    code = L.TR_LAW_LEVERAGE if law == "L" else L.TR_LAW_EUCLID
    for steps in (1, 3):
        say("laws follow", law, I, R, prec, steps)
        solver.run(steps)
        for k in range(3):
            assert torch.equal(solver.cdf[k], api.tr_dist(desc, k, code, dcores[k])[0])
            pref = (sampling.dist_leverage if law == "L" else lambda c: sampling.dist_euclid(c)[0])(
                fold_core(dcores[k].double().cpu().numpy(), R, k))
            assert np.max(np.abs(_weights(solver.cdf[k]) - sampling.quantize(pref).astype(np.int64))) <= 1024
    assert int(solver.status.item()) == 0


# the optimal law's terms from the replicas: runs of columns up to and past
# kOptOuter a block (I_{n+1} from 1), orders 2 to 5, R_n R_{n+1} up to 32, past it
# and 64, I_n up to 64 and past it; J below one block of columns, and past the
# sums that every block adds itself
@pytest.mark.parametrize("I,R", [([5, 3], [4, 8]), ([70, 66], [8, 8]), ([1, 2, 40], [3, 5, 8]), ([9, 8, 7], [6, 6, 6]),
                                 ([64, 65, 11], [4, 8, 4]), ([6, 5, 4, 9], [5, 6, 7, 8]), ([30, 7, 9, 8], [5, 5, 5, 5]),
                                 ([3, 8, 2, 9, 4], [8, 1, 8, 4, 8]), ([100, 90, 80, 41], [3, 2, 3, 2])])
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_optimal_law_from_replicas(I, R, prec):
    dtype = torch.float64 if prec == "f64" else torch.float32
    I, R, cores, X, dcores, dX = problem(47, len(I), I, R, dtype)
    start = [c.clone() for c in dcores]
    for seed in (1, 2, 3, 4):
        solver = TRSolver([c.clone() for c in start], dX, I, R, 32, law="O", prec=prec,
                          rule=api.step_rule("fixed", alpha=1e-4), seed=seed)
        n = api.tr_mode(seed, 0, len(I))
        say("optimal law from replicas", I, R, prec, "mode", n)
        solver.run(1)
        J = int(np.prod([s for k, s in enumerate(I) if k != n]))
        q, _ = sampling.dist_optimal(cores, X, n)
        w = _weights(solver.cdf_J[:J])
        assert int(solver.status.item()) == 0
        assert np.max(np.abs(w - sampling.quantize(q).astype(np.int64))) <= 64 + 16 * np.max(q)


# the chains of the error kernel: ranks within 4, 8 and 16 (R_1 R_2 <= 128),
# orders 2 to 8, columns below, at and past one block of 128 and of 32, rows
# around one tile of 32; entries in paper order, reversed order and (``far``)
# more than 4 GiB apart
@pytest.mark.parametrize("I,R,order", [([33, 5], [4, 3], "paper"), ([40, 130], [8, 16], "paper"), ([31, 16, 8], [3, 4, 2], "reversed"),
                                       ([32, 43, 3], [8, 5, 7], "paper"), ([70, 9, 31], [10, 11, 16], "reversed"),
                                       ([5, 4, 3, 9], [9, 13, 2, 16], "paper"), ([9, 4, 3, 5, 6], [7, 8, 6, 7, 5], "reversed"),
                                       ([3, 2, 3, 2, 3, 2, 4], [4, 3, 9, 2, 5, 3, 4], "paper"),
                                       ([2, 3, 2, 3, 2, 3, 2, 3], [3, 2, 3, 4, 2, 3, 2, 3], "reversed"),
                                       ([6, 5, 7], [5, 4, 3], "far"), ([6, 5, 7, 3], [9, 12, 3, 4], "far")])
@pytest.mark.parametrize("xdt", [torch.float32, torch.float16])
def test_relative_error_chains(I, R, order, xdt):
    I, R, cores, X, dcores, dX = problem(53, len(I), I, R, torch.float32)
    X = rounded(X, xdt)
    strides = api.paper_strides(I)
    if order == "reversed":
        strides = [int(np.prod(I[k + 1:])) for k in range(len(I))]
    if order == "far":
        strides[-1] = 1 << 29
    flat = torch.empty(1 + sum((i - 1) * s for i, s in zip(I, strides)), dtype=xdt, device=DEV)
    flat.as_strided(I, strides).copy_(to_dev(X, xdt))
    desc = api.make_desc(I, R, torch.float32, xdt, strides)
    say("relative error chains", I, R, order, xdt)
    got = float(api.tr_relerr(desc, dcores, flat))
    assert abs(got / tr.rse(cores, X) - 1) < 1e-5
