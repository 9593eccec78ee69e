"""Column dots of matrices with empty columns: chunks whose segments are staged fill short
gaps with zeros themselves, a list takes the rest.  Gaps around the longest one filled,
empty first and last columns, segment counts around what a chunk stages, shares of empty
columns on both sides of where chunks fill gaps, and output strides on both sides of what
the staged copy takes.  Bounds: binary64 1e-13 * sum|a||x|, binary32 vectors 1e-5; an
empty column is exactly zero and nothing else is written."""
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


def lengths_of(filled, gaps, lead):
    """Column lengths: `filled` in turn, after each the next count of empty columns of `gaps`."""
    out = [0] * lead
    for i, ln in enumerate(filled):
        out += [int(ln)] + [0] * gaps[i % len(gaps)]
    return np.array(out)


def check(spw, A, chunk, k, dtype, ld, what):
    # ld: entries from one output row to the next (None: k and one of padding, k = 1 contiguous)
    tol = 1e-13 if dtype == torch.float64 else 1e-5
    V = synth.vector(A.m * k, 7, 2).reshape(A.m, k)
    if dtype == torch.float32:
        V = V.astype(np.float32).astype(np.float64)
    ref, d = oracle.vtm_csc_batch(A.m, A.n, A.ptr, A.idx, A.val, V, with_d=True)
    M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val, chunk_nnz=chunk)
    Vd = torch.from_numpy(V).to(dtype).cuda()
    if k == 1:
        full = torch.full((A.n + 2,), float("nan"), dtype=dtype, device="cuda")
        M.vtm(Vd[:, 0].contiguous(), full[1:-1])
        assert torch.isnan(full[0]) and torch.isnan(full[-1]), what
        got = full[1:-1, None].double().cpu().numpy()
    else:
        M.set_batch_plan(spw.SPW_OP_VTM, spw.SPW_F64 if dtype == torch.float64 else spw.SPW_F32, k, spw.SPW_PLAN_PASSES)
        full = torch.full((A.n, ld or k + 1), float("nan"), dtype=dtype, device="cuda")
        M.vtm_batch(Vd, full[:, :k])
        assert torch.isnan(full[:, k:]).all(), what
        got = full[:, :k].double().cpu().numpy()
    assert np.all(np.abs(got - ref) <= tol * d), what
    assert not got[np.diff(A.ptr) == 0].any(), what
    M.close()


@pytest.mark.parametrize("chunk", [512, 1024])
@pytest.mark.parametrize("gaps", [[0, 1, 2], [1, 0, 0, 0, 0, 31], [0, 32, 0, 0, 0, 0, 0, 0, 0, 0, 0, 33],
                                  [2, 3, 4], [3], [4], [31, 32, 33, 0]])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_gaps(spw, chunk, gaps, dtype):
    rng = np.random.Generator(np.random.PCG64(sum(gaps)))
    for lead, filled in ((3, rng.integers(1, 4, 2_500)), (0, np.r_[rng.integers(1, 6, 900), 1_500, rng.integers(1, 6, 900)])):
        A = synth.from_lengths(2_000, lengths_of(filled, gaps, lead), 11)
        for k in (1, 3):
            print("gaps chunk=%d gaps=%s lead=%d k=%d %s" % (chunk, gaps, lead, k, dtype), flush=True)
            check(spw, A, chunk, k, dtype, None, (chunk, gaps, lead, k, dtype))


@pytest.mark.parametrize("chunk", [512, 1024])
@pytest.mark.parametrize("per", [254, 255, 256, 257, 511, 512])
def test_segments_of_a_chunk(spw, chunk, per):
    # every chunk holds exactly `per` columns, cut at its ends or not
    if per > chunk:
        per = chunk
    one = np.full(per, chunk // per)
    one[: chunk - int(one.sum())] += 1
    for cut in (0, 1):
        filled = np.tile(one, 5)
        filled[0] += cut                              # shifts every later chunk by one position
        for gaps in ([0], [0, 0, 0, 1], [1, 1]):
            A = synth.from_lengths(300, lengths_of(filled, gaps, 1), 5)
            for dtype in (torch.float64, torch.float32):
                print("segments chunk=%d per=%d cut=%d gaps=%s %s" % (chunk, per, cut, gaps, dtype), flush=True)
                for k in (1, 2):
                    check(spw, A, chunk, k, dtype, None, (chunk, per, cut, gaps, dtype, k))


@pytest.mark.parametrize("chunk,dtype,limit", [(512, torch.float64, 1 << 16), (1024, torch.float64, 1 << 15),
                                               (512, torch.float32, 1 << 17), (1024, torch.float32, 1 << 16)])
def test_wide_output_rows(spw, chunk, dtype, limit):
    rng = np.random.Generator(np.random.PCG64(3))
    A = synth.from_lengths(500, lengths_of(rng.integers(1, 4, 1_200), [0, 1, 0, 2], 1), 3)
    for ld in (limit, limit + 1):
        print("wide chunk=%d ld=%d %s" % (chunk, ld, dtype), flush=True)
        check(spw, A, chunk, 2, dtype, ld, (chunk, dtype, ld))


@pytest.mark.parametrize("n,mean,storage,chunk", [(190_000, 8.1, 0, 512), (200_000, 8.1, 0, 1024), (700_000, 7.5, 0, 512),
                                                  (500_000, 3.4, 1, 1024), (700_000, 2.9, 1, 512), (30_000, 40, 2, 512)])
def test_automatic_chunk(spw, n, mean, storage, chunk):
    # few nonzeros, short columns (below eight with binary64 values, three otherwise), or the full chunk
    lengths = np.full(n, int(mean))
    lengths[: int(round(n * (mean - int(mean))))] += 1
    A = synth.from_lengths(400, lengths, 9)
    M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val, value_storage=storage)
    assert M.info()["chunk_nnz"] == chunk
    M.close()
