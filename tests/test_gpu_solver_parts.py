"""The solver's inner products where their number of partial sums changes (one per 2,048
elements, at most 1,024), with renumbered rows, and across an iteration that forms q = A p
directly, against the CPU oracle.  The bar is the one of two correct runs: rounding grows by
about 4 * cond(A)^2 an iteration, so 1e-12 * (4 cond^2)^iters of the largest entry, 1e-6 at most."""
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


def solve(spw, B, fmt, iters, relabel):
    code, m, n = (spw.SPW_CSC, B.m, B.n) if fmt == "csc" else (spw.SPW_CSR, B.n, B.m)
    rng = np.random.default_rng(B.n)
    b, x0 = rng.uniform(-1, 1, m), rng.uniform(-1, 1, n)
    M = spw.SpwMatrix(code, m, n, B.ptr, B.idx, B.val, relabel=relabel)
    x = torch.from_numpy(x0.copy()).cuda()
    gamma, rho = M.cgls(torch.from_numpy(b).cuda(), x, iters)
    again = torch.from_numpy(x0.copy()).cuda()
    M.cgls(torch.from_numpy(b).cuda(), again, iters, hist=False)
    assert torch.equal(x, again)                 # without a history the same solve, bit for bit
    M.close()
    return (x.cpu().numpy(), gamma, rho), oracle.cgls(fmt, m, n, B.ptr, B.idx, B.val, b, x0, iters)


@pytest.mark.parametrize("fmt", ["csc", "csr"])
@pytest.mark.parametrize("cols", [1, 100, 2047, 2048, 2049, 4097, 10_241])
@pytest.mark.parametrize("relabel", [0, 1])
def test_partial_sum_counts(spw, fmt, cols, relabel):
    B = synth.random_csc(40, cols, 5, seed=cols)
    D = synth.to_dense(B)
    sv = np.linalg.svd(D, compute_uv=False)
    sv = sv[sv > 1e-10 * sv[0]]
    tol = min(1e-12 * (4 * (sv[0] / sv[-1]) ** 2) ** 3, 1e-6)
    print("solver parts %s cols=%d relabel=%d" % (fmt, cols, relabel), flush=True)
    (x, gamma, rho), (xo, go, ro) = solve(spw, B, fmt, 3, relabel)
    assert np.max(np.abs(x - xo)) <= tol * np.max(np.abs(xo))
    assert np.all(np.abs(gamma - go) <= tol * go[0]) and np.all(np.abs(rho - ro) <= tol * ro[0])


@pytest.mark.parametrize("fmt", ["csc", "csr"])
def test_most_partial_sums(spw, fmt):
    # 2,048 * 1,024 elements and more: the number of partial sums stays at 1,024
    B = synth.random_csc(40, 2_100_000, 2, seed=9)
    (x, gamma, rho), (xo, go, ro) = solve(spw, B, fmt, 2, 1)
    assert np.max(np.abs(x - xo)) <= 1e-6 * np.max(np.abs(xo))
    assert np.all(np.abs(gamma - go) <= 1e-6 * go[0]) and np.all(np.abs(rho - ro) <= 1e-6 * ro[0])


@pytest.mark.parametrize("fmt", ["csc", "csr"])
def test_across_a_direct_product(spw, fmt):
    # iterations 49 .. 52 of a well-conditioned problem: 40 rows, 8,000 columns
    B = synth.random_csc(40, 8_000, 8, seed=4)
    for iters in (49, 50, 51, 52):
        (x, gamma, rho), (xo, go, ro) = solve(spw, B, fmt, iters, 1)
        assert gamma.size == iters + 1 and np.all(np.isfinite(gamma)) and np.all(np.isfinite(rho))
        assert np.max(np.abs(x - xo)) <= 1e-6 * np.max(np.abs(xo))
        assert np.all(np.abs(gamma - go) <= 1e-6 * go[0]) and np.all(np.abs(rho - ro) <= 1e-6 * ro[0])
