"""Column dots of chunks of 512 by what their waves stage: binary64 vectors 256 segments a chunk or 512
(more than one chunk in eight with over 256), binary32 ones none or 512 (short columns, or empty ones
all over and all rows beside the stages), on either side of each rule, with chunks that the
smaller stage does not take among the others and empty columns inside.  Bounds: binary64 1e-13 *
sum|a||x|, binary32 vectors 1e-5; empty columns exactly zero, nothing else written.  And explicit
chunks of 512 with binary32 vectors over many rows keep their hot rows: no slower than a third over
chunks of 1,024 (two thirds over with every wave staging)."""
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


def mixed(chunks, short, gaps):
    """Column lengths of `chunks` chunks of 512: one in every `short` of single nonzeros, the others of eight
    (or all of eight); `gaps`: an empty column after every tenth."""
    out = []
    for c in range(chunks):
        out += [1] * 512 if short and c % short == 0 else [8] * 64
    lengths = []
    for i, ln in enumerate(out):
        lengths += [ln, 0] if gaps and i % 10 == 9 else [ln]
    return np.array(lengths)


@pytest.mark.parametrize("rows", [400, 15_000, 30_000])
@pytest.mark.parametrize("short", [0, 4, 8, 9, 20])
@pytest.mark.parametrize("gaps", [False, True])
def test_stage_rules(spw, rows, short, gaps):
    A = synth.from_lengths(rows, mixed(120, short, gaps), rows + short)
    for storage in (0, 1, 2):
        M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val, chunk_nnz=512, value_storage=storage)
        val = spw.spw_round_values(storage, A.val)
        for dtype, tol in ((torch.float64, 1e-13), (torch.float32, 1e-5)):
            for k in (1, 3):
                print("stage rows=%d short=%d gaps=%d storage=%d k=%d %s" % (rows, short, gaps, storage, k, dtype), flush=True)
                V = torch.from_numpy(synth.vector(A.m * k, 7, 2).reshape(A.m, k)).to(dtype).cuda()
                ref, d = oracle.vtm_csc_batch(A.m, A.n, A.ptr, A.idx, val, V.double().cpu().numpy(), with_d=True)
                full = torch.full((A.n + 2, k), float("nan"), dtype=dtype, device="cuda")
                if k == 1:
                    M.vtm(V[:, 0].contiguous(), full[1:-1, 0])
                else:
                    M.vtm_batch(V, full[1:-1])
                got = full[1:-1].double().cpu().numpy()
                assert np.all(np.abs(got - ref) <= tol * d) and not got[np.diff(A.ptr) == 0].any()
                assert torch.isnan(full[0]).all() and torch.isnan(full[-1]).all()
        M.close()


def test_hot_rows_beside_the_stages(spw):
    A = synth.from_lengths(50_000, np.full(1_000_000, 20), 7)
    v, u = torch.rand(A.m, dtype=torch.float32, device="cuda"), torch.empty(A.n, dtype=torch.float32, device="cuda")
    best = {}
    for chunk in (512, 1024):
        M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val, chunk_nnz=chunk, value_storage=1, transpose=0)
        times = []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                M.vtm(v, u)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) * 100)
        best[chunk] = min(times)
        M.close()
    print("explicit chunks, us: %s" % best, flush=True)
    assert best[512] < 4 / 3 * best[1024]
