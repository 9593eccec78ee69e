"""Scatter product of several columns at once (A x of a wide matrix with k right-hand
sides): every number of columns that can share an LDS panel, streams of less than
one, of one or two and of many blocks, and row strides past 32-bit byte offsets.
Each column equals the single-vector product bit for bit, and the oracle within
the library's bound for binary64, 1e-13 * sum|a||x| (binary32 vectors: 1e-5)."""
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


# rows per panel -> columns that fit beside one another: 20,448 entries of LDS
PANELS = {20448: 1, 20447: 1, 10224: 2, 6816: 3, 5112: 4, 1000: 4, 0: 4}
# mean column length of a 20,000 x 6,000 matrix: streams of 30 nonzeros, of one or two
# blocks (1,024 each) with a remainder, and of three and more
LENGTHS = {"part": 5, "two": 300, "many": 700}


@pytest.mark.parametrize("panel", sorted(PANELS))
@pytest.mark.parametrize("length", sorted(LENGTHS))
def test_columns_share_a_panel(spw, panel, length):
    A = synth.random_csc(20_000, 6_000, LENGTHS[length], seed=panel + len(length), row_alpha=0.8)
    M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val, panel_rows=panel)
    for k, pad in ((2, 0), (3, 1), (5, 0), (7, 2), (8, 0)):
        X = synth.vector(A.n * k, 3, k).reshape(A.n, k)
        ref, d = oracle.mv_csc_batch(A.m, A.n, A.ptr, A.idx, A.val, X, with_d=True)
        for dtype, tol in ((torch.float64, 1e-13), (torch.float32, 1e-5)):
            print("scatter columns panel=%d %s k=%d %s" % (panel, length, k, dtype), flush=True)
            full = torch.full((A.n, k + pad), float("nan"), dtype=dtype, device="cuda")
            full[:, :k] = torch.from_numpy(X).to(dtype)
            Y = M.mv_batch(full[:, :k])
            if dtype == torch.float32:
                X32 = X.astype(np.float32).astype(np.float64)
                ref, d = oracle.mv_csc_batch(A.m, A.n, A.ptr, A.idx, A.val, X32, with_d=True)
            assert np.all(np.abs(Y.double().cpu().numpy() - ref) <= tol * d)
            for c in range(k):
                assert torch.equal(Y[:, c], M.mv(full[:, c].contiguous())), (panel, length, k, c)
    M.close()


@pytest.mark.parametrize("ld", [8191, 8192, 16384])
def test_wide_row_stride(spw, ld):
    # 8,192 binary64 (16,384 binary32) entries a row: byte offsets inside a block leave 32 bits
    A = synth.random_csc(5_000, 2_500, 40, seed=ld)
    M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val)
    for dtype in (torch.float64, torch.float32):
        print("scatter columns row stride %d %s" % (ld, dtype), flush=True)
        full = torch.full((A.n, ld), float("nan"), dtype=dtype, device="cuda")
        full[:, :5] = torch.from_numpy(synth.vector(A.n * 5, 4, 1).reshape(A.n, 5)).to(dtype)
        Y = M.mv_batch(full[:, :5])
        for c in range(5):
            assert torch.equal(Y[:, c], M.mv(full[:, c].contiguous())), (ld, dtype, c)
    M.close()


def test_empty_rows_and_infinite_entries(spw):
    # an infinite x entry reaches exactly the rows its column holds; padding slots of a block
    # read the block's first column and must not spread it
    ptr = np.array([0, 2, 2, 3, 5], dtype=np.int64)
    idx = np.array([0, 3, 1, 0, 4], dtype=np.int32)
    M = spw.SpwMatrix(spw.SPW_CSC, 6, 4, ptr, idx, np.ones(5))
    X = torch.ones((4, 3), dtype=torch.float64, device="cuda")
    X[0, 1] = float("inf")
    want = torch.tensor([[2, float("inf"), 2], [1, 1, 1], [0, 0, 0], [1, float("inf"), 1], [1, 1, 1], [0, 0, 0]],
                        dtype=torch.float64)
    assert torch.equal(M.mv_batch(X).cpu(), want)
    M.close()
