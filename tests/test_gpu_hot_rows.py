"""Rows with very many nonzeros, and all rows of dense matrices, have several entries of the scatter
product's LDS panel: no larger error than summing every row in 256 equal runs of its nonzeros (a range
per CU over all of them; a tenth for the spread of one sample), however many panels the matrix is in,
and the same bits alone and in blocks.  Also where the extra entries just
fit, do not fit, and where every row has some.  Error bounds of a single entry: 1e-13 * sum|a||x|
(binary32 vectors 1e-5)."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spw():
    from paper_1812_00904_amd import spw as mod
    mod.load()
    assert torch.cuda.is_available()
    return mod


def by_row(A, x):
    """(first product of every row, products by row in column order)."""
    order = np.argsort(A.idx, kind="stable")
    col = np.repeat(np.arange(A.n), np.diff(A.ptr))
    return np.searchsorted(A.idx[order], np.arange(A.m + 1)), A.val[order], x[col[order]]


def in_runs(p, runs):
    """The binary64 sum of p in `runs` equal runs, each in order, then eight chains of runs and their tree."""
    cut = [len(p) * i // runs for i in range(runs + 1)]
    part = [np.add.accumulate(p[a:b])[-1] if b > a else 0.0 for a, b in zip(cut, cut[1:])]
    c = [np.add.accumulate(np.array(part[t::8]))[-1] for t in range(8)]
    return ((c[0] + c[1]) + (c[2] + c[3])) + ((c[4] + c[5]) + (c[6] + c[7]))


@pytest.mark.parametrize("rows,cols,per,alpha,positive", [
    (5_000, 300_000, 10, 1.2, True), (5_000, 300_000, 10, 1.2, False), (5_000, 300_000, 10, 0.8, True),
    (4_000, 1_500, 2_000, None, False), (20_000, 1_000, 5_000, None, True)])
def test_error_of_long_rows(spw, rows, cols, per, alpha, positive):
    A = synth.from_lengths(rows, np.full(cols, per), 4, row_alpha=alpha, values="lognormal")
    x = synth.vector(A.n, 5, 1)
    if positive:
        A.val[:] = np.abs(A.val)
        x = np.abs(x)
    at, val, xs = by_row(A, x)
    wide = val.astype(np.longdouble) * xs
    exact = np.array([wide[a:b].sum() for a, b in zip(at, at[1:])])
    runs = np.array([in_runs(val[a:b] * xs[a:b], 256) for a, b in zip(at, at[1:])])
    M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val)
    assert M.info()["n_panels"] > 1
    y = M.mv(torch.from_numpy(x).cuda()).cpu().numpy()
    M.close()
    err, ref = np.linalg.norm((y - exact).astype(np.float64)), np.linalg.norm((runs - exact).astype(np.float64))
    print("long rows %d x %d alpha=%s positive=%d: error %.2e, in 256 runs %.2e of %.2e" %
          (rows, cols, alpha, positive, err, ref, np.linalg.norm(exact.astype(np.float64))), flush=True)
    assert err <= 1.1 * ref


# panels whose columns just fit the LDS beside one another with and without room for extra entries,
# panels of one and two rows, an unnumbered matrix, and rows that all have very many nonzeros
@pytest.mark.parametrize("rows,cols,mean,alpha,opts", [
    (20_000, 60_000, 40, 1.5, {"panel_rows": p}) for p in (20_448, 20_447, 10_224, 5_112, 5_080, 1_000, 2, 1)] + [
    (3_000, 60_000, 40, 1.5, {"relabel": 0}), (20_000, 60_000, 40, 1.5, {"relabel": 0}), (40, 200_000, 20, None, {}),
    (1, 100_000, 1, None, {}), (60, 300_000, 20, 2.0, {"partition": 1}), (60, 300_000, 20, 2.0, {"partition": 2})])
def test_alone_and_in_blocks(spw, rows, cols, mean, alpha, opts):
    rng = np.random.Generator(np.random.PCG64(cols))
    A = synth.from_lengths(rows, np.minimum(rng.integers(0, 2 * mean + 1, cols), rows), 8, row_alpha=alpha)
    M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val, transpose=0, **opts)
    for dtype, tol in ((torch.float64, 1e-13), (torch.float32, 1e-5)):
        print("hot rows %d x %d %s %s" % (rows, cols, opts, dtype), flush=True)
        X = torch.from_numpy(synth.vector(A.n * 5, 3, 1).reshape(A.n, 5)).to(dtype).cuda()
        ref, d = oracle.mv_csc_batch(A.m, A.n, A.ptr, A.idx, A.val, X.double().cpu().numpy(), with_d=True)
        Y = M.mv_batch(X)
        assert np.all(np.abs(Y.double().cpu().numpy() - ref) <= tol * d)
        for c in range(5):
            assert torch.equal(Y[:, c], M.mv(X[:, c].contiguous())), c
    M.close()
