"""The reduction of the scatter product's partial sums by one thread a row (panels of at most eight
workgroup ranges): from one to nine ranges a panel, panels smaller and larger than a workgroup and of
uneven numbers of rows, several columns.  Same order of additions as by eight threads a row, so a
column alone, in a block and through the oracle's bound agree: bits between the first two, 1e-13 *
sum|a||x| (binary32 vectors 1e-5) for the last."""
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


# 256 ranges over the panels: 300 panels of one, 125 of two or three, 37 of six or seven, 32 of eight, 29 of eight or nine
@pytest.mark.parametrize("rows,panels", [(300, 300), (5_000, 125), (4_001, 37), (9_000, 32), (9_001, 29), (600_000, 30)])
@pytest.mark.parametrize("relabel", [0, 1])
def test_ranges_of_a_panel(spw, rows, panels, relabel):
    A = synth.random_csc(rows, 3_000, 60, seed=rows + panels, empty_frac=0.1)
    M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val, panel_rows=-(-rows // panels), relabel=relabel)
    assert M.info()["n_panels"] == panels
    for dtype, tol in ((torch.float64, 1e-13), (torch.float32, 1e-5)):
        print("ranges of a panel rows=%d panels=%d relabel=%d %s" % (rows, panels, relabel, dtype), flush=True)
        X = torch.from_numpy(synth.vector(A.n * 9, 3, 1).reshape(A.n, 9)).to(dtype).cuda()
        ref, d = oracle.mv_csc_batch(A.m, A.n, A.ptr, A.idx, A.val, X.double().cpu().numpy(), with_d=True)
        Y = M.mv_batch(X)
        assert np.all(np.abs(Y.double().cpu().numpy() - ref) <= tol * d)
        for c in (0, 3, 8):
            assert torch.equal(Y[:, c], M.mv(X[:, c].contiguous())), c
    M.close()
