"""What a kept transpose costs in device memory: its values, indices, column-start bits, chunk and segment
tables, one list of its empty columns and its zones; the lists that only single-vector products read are
for the matrix's own storage."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spw():
    from paper_1812_00904_amd import spw as mod
    mod.load()
    assert torch.cuda.is_available()
    return mod


def test_one_list_of_empty_columns(spw):
    # 40,000 rows in two blocks of the transpose, half of the (block, row) columns empty, mostly fifty in a
    # row: a second list, of those in long gaps, would hold nearly all of them
    rng = np.random.Generator(np.random.PCG64(2))
    n, m = 300_000, 40_000
    rows = np.flatnonzero((np.arange(m) // 50 % 2 == 0) & (np.arange(m) % 25 > 0))
    idx = np.sort(rng.choice(rows, (n, 2)), axis=1)
    idx[idx[:, 0] == idx[:, 1], 1] = rows[-1]
    idx = np.sort(idx, axis=1).astype(np.int32).reshape(-1)
    ptr = np.arange(0, 2 * n + 1, 2, dtype=np.int64)
    keep = np.r_[True, (idx[1:] != idx[:-1]) | (np.arange(1, 2 * n) % 2 == 0)]
    ptr = np.r_[0, np.cumsum(keep)][ptr]
    idx = idx[keep]
    nnz = len(idx)
    total = {}
    for t in (0, 1):
        M = spw.SpwMatrix(spw.SPW_CSC, m, n, ptr, idx, np.ones(nnz), transpose=t, relabel=0)
        total[t] = M.info()["device_bytes"]
        M.close()
    # the transpose's own arrays, 1,024 nonzeros a chunk
    block = np.searchsorted(np.arange(0, n, 1 << 18)[1:], np.repeat(np.arange(n), np.diff(ptr)), side="right")
    counts = np.bincount(block * m + idx, minlength=2 * m)
    ends = np.cumsum(counts)
    starts = ends - counts
    chunks = -(-nnz // 1024)
    pad = -(-nnz // 4096) * 4096
    filled = counts > 0
    segs = int(((ends[filled] - 1) // 1024 - starts[filled] // 1024 + 1).sum())
    zones = int(((ends[filled] - 1) // 1024 > starts[filled] // 1024).sum())
    arrays = [pad * 4, pad * 8, chunks * 64 * 2, chunks * 16, (segs + 1) * 4, int((~filled).sum()) * 4] + [zones * 4] * 3
    want = sum(arrays)
    # its carries may replace the matrix's own (two a chunk); scratch is otherwise the same
    assert total[1] - total[0] <= want + 16 * chunks, (total, want)
