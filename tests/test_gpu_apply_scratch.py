"""GPU tests of the sketch apply's optional scratch: a call that has to do without
it gives the same result and says nothing of it."""
import pytest

from test_gpu_apply_forms import _run, sap  # noqa: F401

pytestmark = pytest.mark.gpu


def test_no_error_text_without_scratch(sap):  # noqa: F811
    """The budget holds the scatter form's two row slices (24.1 MB) and no lists."""
    import torch
    ctx = sap.Context(0, 26 << 20)
    m, n, d = 130001, 301, 5003
    A = torch.randint(-8, 9, (m, n), device="cuda").double()
    idx, sign = sap.sps_generate(m, d, 8, 3)
    Y = sap.sps_apply(idx, sign, d, 8, A, None, ctx=ctx)
    assert ctx.last_error() == ""
    ref = sap.sps_apply(idx, sign, d, 8, A, None)
    torch.cuda.synchronize()
    assert torch.equal(Y, ref)
    ctx.close()


def test_workspace_keeps_its_claim(sap):  # noqa: F811
    """A workspace that fits the budget only without the optional scratch gets it:
    the apply's slices (18.1 MB, beside the 8.9 MB that it needs) first, then a QR
    whose panels take 12 MB, of 28 MB."""
    import torch
    ctx = sap.Context(0, 28 << 20)
    m, n, d = 120001, 64, 600
    print(f"scratch-claim m={m} n={n} d={d}", flush=True)
    A = torch.randint(-8, 9, (m, n), device="cuda").double()
    idx, sign = sap.sps_generate(m, d, 8, 3)
    ref = sap.sps_apply(idx, sign, d, 8, A, None)
    F = torch.randn(1300, 4200, device="cuda", dtype=torch.float64)
    for _ in range(2):
        assert torch.equal(sap.sps_apply(idx, sign, d, 8, A, None, ctx=ctx), ref)
        G, H = F.clone(), F.clone()
        sap.sap_qr(G, ctx=ctx)
        sap.sap_qr(H)
        torch.cuda.synchronize()
        assert torch.equal(G, H)
    ctx.close()
