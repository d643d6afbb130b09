"""GPU test of the served form with more apply work items queued than one round's
table holds (2^20): the rest of the burst waits for the next round.

3700 requests of one A (253953 x 128 FP32, d = 129: 9 strips of 32 row slices each,
1065600 items), one step each, submitted while the first request's inputs are
still being written on another stream, so that the scheduler finds them all."""
import pytest

pytestmark = pytest.mark.gpu


def test_burst_past_the_apply_table():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_03070_amd as sap
    if torch.cuda.mem_get_info()[0] < 64 << 30:
        pytest.skip("needs 64 GB of free device memory")
    m, n, d, count = 253953, 128, 129, 3700
    print(f"serve-burst m={m} n={n} d={d} count={count}", flush=True)
    ctx = sap.Context(0)
    sap.sap_serve_start(48 << 30, 4096, ctx=ctx)
    A = torch.randn(m, n, device="cuda")
    b = torch.randn(m, device="cuda", dtype=torch.float64)
    x = torch.zeros(count, n, dtype=torch.float64, device="cuda")
    W = torch.randn(16384, 16384, device="cuda", dtype=torch.bfloat16)
    busy = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(busy):
        for _ in range(80):  # about half a second
            W = W @ W
        tickets = [sap.sap_submit(A, b, d, 8, 7, tol=1e-12, maxiter=1, ctx=ctx, x=x[0])]
    tickets += [sap.sap_submit(A, b, d, 8, 7, tol=1e-12, maxiter=1, ctx=ctx, x=x[k]) for k in range(1, count)]
    states = {sap.sap_poll(t, wait=True, ctx=ctx)[0] for t in tickets}
    torch.cuda.synchronize()
    assert states == {sap.SAP_NOT_CONVERGED}  # one step of a rate near 1
    # the same problem and seed throughout: one step's iterate, to the rounding of the sketch's sums
    ref = x[0]
    assert torch.isfinite(ref).all() and ref.norm() > 0
    assert ((A.double() @ (x - ref).T).norm(dim=0) <= 1e-9 * b.norm()).all()
    ctx.close()
