"""Blocks of 9 to 64 right-hand sides through the run kernel of the column dots: last
chunks that end at every kind of remainder (of a step, a batch, a stage, a chunk), every
column-lane shape, both chunk sizes, empty columns, columns longer than a chunk, and entries
that are not finite.  Bounds: binary64 1e-13 * sum|a||x|, binary32 vectors 1e-5."""
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


def matrix(nnz, m, seed, empty):
    """m x n with exactly nnz entries: short columns, some empty ones when asked, one of 2,500 rows."""
    rng = np.random.Generator(np.random.PCG64(seed))
    lengths = []
    left = nnz
    while left > 0:
        ln = 0 if empty and rng.random() < 0.4 else int(min(rng.geometric(0.15), m))
        if len(lengths) == 20 and left > 2500:
            ln = 2500
        ln = min(ln, left)
        lengths.append(ln)
        left -= ln
    return synth.from_lengths(m, np.array(lengths + [0, 0] if empty else lengths), seed)


def compare(spw, M, A, k, dtype, tol, what):
    X, V = synth.vector(A.n * k, 5, 1).reshape(A.n, k), synth.vector(A.m * k, 5, 2).reshape(A.m, k)
    if dtype == torch.float32:
        X, V = (a.astype(np.float32).astype(np.float64) for a in (X, V))
    Yr, dY = oracle.mv_csc_batch(A.m, A.n, A.ptr, A.idx, A.val, X, with_d=True)
    Ur, dU = oracle.vtm_csc_batch(A.m, A.n, A.ptr, A.idx, A.val, V, with_d=True)
    vdt = spw.SPW_F64 if dtype == torch.float64 else spw.SPW_F32
    for op in (spw.SPW_OP_MV, spw.SPW_OP_VTM):
        M.set_batch_plan(op, vdt, k, spw.SPW_PLAN_TILE)
    for op, inp, ref, d in ((M.mv_batch, X, Yr, dY), (M.vtm_batch, V, Ur, dU)):
        t = torch.from_numpy(inp).to(dtype).cuda()
        out = torch.full((ref.shape[0], k + 1), float("nan"), dtype=dtype, device="cuda")
        got = op(t, out[:, :k]).double().cpu().numpy()
        assert np.all(np.abs(got - ref) <= tol * d), what
        assert torch.isnan(out[:, k]).all(), what


@pytest.mark.parametrize("rest", [0, 1, 7, 8, 15, 16, 17, 255, 256, 257, 1023])
@pytest.mark.parametrize("empty", [False, True])
def test_last_chunk_remainders(spw, rest, empty):
    A = matrix(4 * 1024 + rest, 2_600, rest + 1, empty)
    for chunk in (1024, 512):
        M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val, transpose=1, chunk_nnz=chunk, relabel=chunk == 512)
        for k in (9, 20, 64):
            for dtype, tol in ((torch.float64, 1e-13), (torch.float32, 1e-5)):
                print("run blocks rest=%d empty=%d chunk=%d k=%d %s" % (rest, empty, chunk, k, dtype), flush=True)
                compare(spw, M, A, k, dtype, tol, (rest, empty, chunk, k, dtype))
        M.close()


@pytest.mark.parametrize("storage", [0, 1, 2])
@pytest.mark.parametrize("k", [10, 16, 17, 18, 31, 32, 33, 36, 47, 62, 63])
def test_every_shape(spw, storage, k):
    # 5,000 renumbered rows and 300,000 columns: two blocks of the transpose, 4-byte indices there
    A = synth.random_csc(5_000, 300_000, 3, seed=k, empty_frac=0.2, row_alpha=0.8)
    M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val, transpose=1, value_storage=storage)
    B = synth.Sparse(A.m, A.n, A.ptr, A.idx, spw.spw_round_values(storage, A.val))
    for dtype, tol in ((torch.float64, 1e-13), (torch.float32, 1e-5)):
        print("run shapes storage=%d k=%d %s" % (storage, k, dtype), flush=True)
        compare(spw, M, B, k, dtype, tol, (storage, k, dtype))
    M.close()


def test_entries_that_are_not_finite(spw):
    # one infinite and one NaN row of V reach exactly the columns that hold those rows
    A = synth.random_csc(3_000, 2_000, 6, seed=3)
    M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val)
    V = torch.ones((A.m, 12), dtype=torch.float64, device="cuda")
    rows = (0, int(A.idx[7]))
    V[rows[0], 3], V[rows[1], 5] = float("inf"), float("nan")
    U = M.vtm_batch(V).cpu().numpy()
    col = np.repeat(np.arange(A.n), np.diff(A.ptr))
    for c in range(12):
        holds = np.isin(np.arange(A.n), col[A.idx == {3: rows[0], 5: rows[1]}.get(c, -1)])
        assert np.array_equal(~np.isfinite(U[:, c]), holds), c
    M.close()


@pytest.mark.parametrize("k", [9, 10, 15, 16, 17, 31, 32, 33, 64])
@pytest.mark.parametrize("rest", [0, 7, 16, 255, 1023])
def test_long_columns(spw, k, rest):
    # 40 nonzeros a column: every width takes the run kernel over the matrix's own storage
    rng = np.random.Generator(np.random.PCG64(k))
    lengths = rng.integers(30, 51, 400)
    lengths[rng.random(400) < 0.1] = 0
    lengths[-1] += (rest - int(lengths.sum())) % 1024
    A = synth.from_lengths(6_000, lengths, rest + 1)
    assert A.ptr[-1] % 1024 == rest
    for chunk in (512, 1024):
        M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val, transpose=1, chunk_nnz=chunk)
        print("run long k=%d rest=%d chunk=%d" % (k, rest, chunk), flush=True)
        compare(spw, M, A, k, torch.float64, 1e-13, (k, rest, chunk))
        M.close()


@pytest.mark.parametrize("n", [100_000, 300_000])
def test_transpose_narrow_blocks(spw, n):
    # enough nonzeros for the narrow blocks of the kept transpose, with and without several row blocks
    A = synth.random_csc(700, n, 1_400_000 // n, seed=n, row_alpha=0.5)
    M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val, transpose=1)
    for k in (12, 16):
        for dtype, tol in ((torch.float64, 1e-13), (torch.float32, 1e-5)):
            print("run narrow n=%d k=%d %s" % (n, k, dtype), flush=True)
            compare(spw, M, A, k, dtype, tol, (n, k, dtype))
    M.close()


@pytest.mark.parametrize("mean", [3, 5, 6, 7, 8, 9, 29, 31])
def test_either_side_of_the_rule(spw, mean):
    # both kernels give the same result within the bound wherever the line between them lies
    A = synth.from_lengths(1_000, np.full(900, mean), mean)
    M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val, transpose=1)
    for k in (16, 32, 64):
        print("run rule mean=%d k=%d" % (mean, k), flush=True)
        compare(spw, M, A, k, torch.float64, 1e-13, (mean, k))
    M.close()
