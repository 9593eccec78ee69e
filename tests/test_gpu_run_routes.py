"""Which kernel a block of 9 to 64 right-hand sides takes (by the library's own profile), and the run
kernel where that is it: every storage and index type and chunk size, every width's lanes, last chunks
that end at every kind of remainder, entries that are not finite, narrow blocks of a transpose with
2-byte rows on both sides of its row stride limit; and the tile kernel where single chunks have so many
column starts that the run kernel's waves would end late.  Bounds: binary64 1e-13 * sum|a||x|, binary32
vectors 1e-5."""
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


def kernel_of(spw, call):
    """The block kernel that `call` runs and its result."""
    spw.spw_profile_enable(True)
    spw.spw_profile_reset()
    out = call()
    torch.cuda.synchronize()
    names = set(spw.spw_profile_read()) & {"cdot_run", "cdot_tile"}
    spw.spw_profile_enable(False)
    assert len(names) == 1, names
    return names.pop(), out


def check(spw, M, A, op, k, dtype, kernel, what, ld=None, val=None):
    tol = 1e-13 if dtype == torch.float64 else 1e-5
    rows = A.m if op == "vtm" else A.n
    V = torch.from_numpy(synth.vector(rows * k, 7, k).reshape(rows, k)).to(dtype).cuda()
    if ld:
        wide = torch.full((rows, ld), float("nan"), dtype=dtype, device="cuda")
        wide[:, :k] = V
        V = wide[:, :k]
    code = spw.SPW_OP_VTM if op == "vtm" else spw.SPW_OP_MV
    M.set_batch_plan(code, spw.SPW_F64 if dtype == torch.float64 else spw.SPW_F32, k, spw.SPW_PLAN_TILE)
    print("run routes %s %s k=%d %s ld=%s" % (what, op, k, dtype, ld), flush=True)
    out = torch.full((A.n if op == "vtm" else A.m, k + 1), float("nan"), dtype=dtype, device="cuda")
    name, _ = kernel_of(spw, lambda: (M.vtm_batch if op == "vtm" else M.mv_batch)(V, out[:, :k]))
    assert name == kernel, (what, op, k, dtype, ld)
    ref, d = (oracle.vtm_csc_batch if op == "vtm" else oracle.mv_csc_batch)(
        A.m, A.n, A.ptr, A.idx, A.val if val is None else val, V.double().cpu().numpy(), with_d=True)
    assert np.all(np.abs(out[:, :k].double().cpu().numpy() - ref) <= tol * d), (what, op, k, dtype, ld)
    assert torch.isnan(out[:, k]).all()


def lengths_for(rest, mean=40, cols=450, empty=True):
    rng = np.random.Generator(np.random.PCG64(rest + mean))
    lengths = rng.integers(mean - mean // 4, mean + mean // 4 + 1, cols)
    if empty:
        lengths[rng.random(cols) < 0.1] = 0
    lengths[-1] += (rest - int(lengths.sum())) % 1024
    return lengths


# 2-byte and 4-byte rows, every storage type, both chunk sizes, the widths of every shape and either side
@pytest.mark.parametrize("rows", [3_000, 70_000])
@pytest.mark.parametrize("storage", [0, 1, 2])
@pytest.mark.parametrize("chunk", [512, 1024])
def test_own_storage(spw, rows, storage, chunk):
    A = synth.from_lengths(rows, lengths_for(rows + storage), 5)
    M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val, chunk_nnz=chunk, value_storage=storage, transpose=0)
    val = spw.spw_round_values(storage, A.val)
    for k in (9, 15, 16, 17, 31, 32, 33, 47, 64):
        check(spw, M, A, "vtm", k, torch.float64, "cdot_run", (rows, storage, chunk), val=val)
    M.close()


@pytest.mark.parametrize("rest", [0, 1, 7, 8, 15, 16, 17, 255, 256, 257, 511, 512, 513, 1023])
def test_remainders(spw, rest):
    A = synth.from_lengths(3_000, lengths_for(rest), rest + 1)
    assert A.ptr[-1] % 1024 == rest
    for chunk in (512, 1024):
        M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val, chunk_nnz=chunk, transpose=0)
        for k in (9, 20, 64):
            check(spw, M, A, "vtm", k, torch.float64, "cdot_run", ("rest", rest, chunk))
        M.close()


@pytest.mark.parametrize("k", [12, 24, 48])
@pytest.mark.parametrize("rest", [0, 5, 300])
def test_entries_that_are_not_finite(spw, k, rest):
    # padding positions of the last chunk gather row 0: an infinite and a NaN entry there and in another
    # row reach exactly the columns that hold those rows
    A = synth.from_lengths(2_500, lengths_for(rest, empty=False), rest + 2)
    M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val, relabel=0, transpose=0)
    V = torch.ones((A.m, k), dtype=torch.float64, device="cuda")
    at = {3: 0, 5: int(A.idx[7]), 8: 0}
    for (c, row), x in zip(at.items(), (float("inf"), float("nan"), float("-inf"))):
        V[row, c] = x
    name, U = kernel_of(spw, lambda: M.vtm_batch(V))
    assert name == "cdot_run"
    col = np.repeat(np.arange(A.n), np.diff(A.ptr))
    for c in range(k):
        holds = np.isin(np.arange(A.n), col[A.idx == at.get(c, -1)])
        assert np.array_equal(~np.isfinite(U[:, c].cpu().numpy()), holds), c
    M.close()


# enough nonzeros for narrow blocks over the transpose: 2-byte rows up to 65,536 columns, 4-byte past them
@pytest.mark.parametrize("n", [50_000, 65_536, 65_537])
def test_narrow_blocks_of_a_transpose(spw, n):
    A = synth.from_lengths(700, np.full(n, 28), n)
    M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val, transpose=1)
    for dtype, es in ((torch.float64, 8), (torch.float32, 4)):
        for k in (12, 16):
            check(spw, M, A, "mv", k, dtype, "cdot_run", ("narrow", n))
        # rows of 65,536 bytes and more have no 32-bit byte offsets
        for k, ld in ((16, 65536 // es - 4), (16, 65536 // es), (32, 65536 // es)):
            if n == 50_000:
                check(spw, M, A, "mv", k, dtype, "cdot_run" if ld * es < 65536 else "cdot_tile", ("stride", n), ld=ld)
    M.close()


@pytest.mark.parametrize("storage", [0, 1, 2])
@pytest.mark.parametrize("k", [16, 20, 32, 36, 64])
def test_transpose_shapes(spw, storage, k):
    # two blocks of the transpose, binary64 partial sums of binary32 columns
    A = synth.from_lengths(700, np.full(300_000, 5), k)
    M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val, transpose=1, value_storage=storage)
    val = spw.spw_round_values(storage, A.val)
    for dtype in (torch.float64, torch.float32):
        check(spw, M, A, "mv", k, dtype, "cdot_run", ("transpose", storage), val=val)
    M.close()


@pytest.mark.parametrize("order,kernel", [("random", "cdot_run"), ("descending", "cdot_tile"), ("ascending", "cdot_tile")])
def test_columns_by_length(spw, order, kernel):
    # a third of the columns hold one nonzero each: chunks of up to a thousand column starts where they
    # are together, of about forty where not
    rng = np.random.Generator(np.random.PCG64(1))
    lengths = rng.permutation(np.r_[np.full(8_000, 1), rng.integers(20, 100, 16_000)])
    if order != "random":
        lengths = np.sort(lengths)[::-1 if order == "descending" else 1]
    A = synth.from_lengths(4_000, lengths, 3)
    M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val, transpose=0)
    for k in (16, 32, 64):
        check(spw, M, A, "vtm", k, torch.float64, kernel, order)
    M.close()
