"""A matrix serves one stream at a time: while its last call is pending on one stream a call on
another is refused, whatever kernel the pending call ends in, on its first call and on
later ones; once that work is done the other stream is served."""
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


def refused(spw, busy, call, other):
    """Whether `other` is refused after `call` behind a bounded spin on `busy`; the spin can
    end early on an idle device, so a try counts only if it is still running afterwards."""
    for _ in range(8):
        torch.cuda.synchronize()
        with torch.cuda.stream(busy):
            torch.cuda._sleep(50_000_000)
        call()
        try:
            other()
            was_refused = False
        except spw.SpwError as e:
            assert e.status_name == "SPW_ERR_BUSY"
            was_refused = True
        if not busy.query():
            return was_refused
    pytest.skip("the spin never outlasted two calls")


# products that end in the column dots, in their zone sums, in the reduction of the scatter
# product, in a tile kernel, and blocks of several passes (11 columns: 8 and 3)
@pytest.mark.parametrize("op,k", [("vtm", 1), ("mv", 1), ("vtm", 3), ("mv", 3), ("vtm", 11), ("mv", 11), ("vtm", 7)])
@pytest.mark.parametrize("long_columns", [False, True])
def test_pending_call_refuses_another_stream(spw, op, k, long_columns):
    A = synth.random_csc(2_000, 1_000 if long_columns else 60_000, 900 if long_columns else 4, seed=k, empty_frac=0.1)
    M = spw.SpwMatrix(spw.SPW_CSC, A.m, A.n, A.ptr, A.idx, A.val)
    if k in (3, 11):
        M.set_batch_plan(spw.SPW_OP_VTM if op == "vtm" else spw.SPW_OP_MV, spw.SPW_F64, k, spw.SPW_PLAN_PASSES)
    n_in, n_out = (A.m, A.n) if op == "vtm" else (A.n, A.m)
    x = torch.rand((n_in, k) if k > 1 else (n_in,), dtype=torch.float64, device="cuda")
    y, z = (torch.empty((n_out, k) if k > 1 else (n_out,), dtype=torch.float64, device="cuda") for _ in range(2))
    run = getattr(M, op if k == 1 else op + "_batch")
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    for call in range(3):
        print("busy %s k=%d long=%d call %d" % (op, k, long_columns, call), flush=True)
        assert refused(spw, sa, lambda: run(x, y, stream=sa), lambda: run(x, z, stream=sb)), call
    torch.cuda.synchronize()
    run(x, z, stream=sb)
    torch.cuda.synchronize()
    assert torch.equal(y, z)
    M.close()
