"""A matrix serves one stream at a time: while its last call is pending on one stream a call on
another is refused, whatever kernel the pending call ends in, on its first call and on
later ones; once that work is done the other stream is served."""
import threading

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


@pytest.mark.parametrize("fmt", ["csc", "csr"])
def test_solve_being_issued_refuses_another_stream(spw, fmt):
    # x moves once the first iteration has run; thousands of launches are then still to be issued, and the
    # call's event comes after the last.  A new matrix: no earlier call's event stands in for it.
    A = synth.random_csc(50, 2_000, 6, seed=3)
    code, m, n = (spw.SPW_CSC, A.m, A.n) if fmt == "csc" else (spw.SPW_CSR, A.n, A.m)
    b, v, u = (torch.rand(s, dtype=torch.float64, device="cuda") for s in (m, m, n))
    alone = torch.zeros(n, dtype=torch.float64, device="cuda")
    iters = 5_000
    for used_before in (False, True):
        M = spw.SpwMatrix(code, m, n, A.ptr, A.idx, A.val)
        sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
        x = torch.zeros(n, dtype=torch.float64, device="cuda")
        if used_before:
            M.vtm(v, u, stream=sb)
        torch.cuda.synchronize()
        print("solve being issued %s used=%d" % (fmt, used_before), flush=True)
        errs = []

        def solve():
            try:
                M.cgls(b, x, iters, hist=False, stream=sa)
            except spw.SpwError as e:
                errs.append(e)

        t = threading.Thread(target=solve)
        t.start()
        with torch.cuda.stream(sb):
            while t.is_alive() and not x.any().item():
                pass
        refusals = 0
        for call in (lambda: M.vtm(v, u, stream=sb), lambda: M.mv(u, v, stream=sb),
                     lambda: M.cgls(b, torch.zeros_like(x), 1, hist=False, stream=sb)):
            with pytest.raises(spw.SpwError) as e:
                call()
            assert e.value.status_name == "SPW_ERR_BUSY"
            refusals += t.is_alive()
        t.join()
        assert refusals and not errs                      # refused while the solve was being issued
        torch.cuda.synchronize()
        M.cgls(b, alone.zero_(), iters, hist=False, stream=sb)
        torch.cuda.synchronize()
        assert torch.equal(x.view(torch.int64), alone.view(torch.int64))   # and the solve was not disturbed
        M.close()
