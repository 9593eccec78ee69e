"""Creating a matrix costs about the same whatever its partition and its number of row panels: the
panels' nonzeros are sorted out once, not searched panel by panel.  The bound is a multiple of the
cheapest creation of the same matrix that a panel-by-panel search misses by more than ten times, and
products are checked against the CPU oracle (1e-13 * sum|a||x|)."""
import time

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


# long columns in many panels under each partition; very many panels; one panel
@pytest.mark.parametrize("rows,cols,mean,opts", [
    (20_000, 1_000, 5_000, {"partition": 2}), (20_000, 1_000, 5_000, {"partition": 1}),
    (20_000, 200_000, 20, {"panel_rows": 4}), (20_000, 200_000, 20, {"panel_rows": 4, "partition": 2}),
    (20_000, 200_000, 20, {"panel_rows": 20_000}), (3, 50_000, 2, {"panel_rows": 1})])
def test_cost_and_result(spw, rows, cols, mean, opts):
    rng = np.random.Generator(np.random.PCG64(7))
    lengths = np.minimum(rng.integers(0, 2 * mean + 1, cols), rows)
    A = synth.from_lengths(rows, lengths, 5)
    x = synth.vector(A.n, 3, 1)
    ref, d = oracle.mv_csc(A.m, A.n, A.ptr, A.idx, A.val, x, with_d=True)

    def create(**o):
        t = time.perf_counter()
        M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val, transpose=0, **o)
        return M, time.perf_counter() - t

    create(panel_rows=20_000)[0].close()              # the process's first
    plain = []
    for _ in range(3):
        M, t = create(panel_rows=20_000)
        plain.append(t)
        M.close()
    M, t = create(**opts)
    print("create %d x %d %s: %.3f s, one panel %.3f s" % (rows, cols, opts, t, min(plain)), flush=True)
    assert t < 5 * min(plain) + 0.2
    y = M.mv(torch.from_numpy(x).cuda()).cpu().numpy()
    assert np.all(np.abs(y - ref) <= 1e-13 * d)
    M.close()
