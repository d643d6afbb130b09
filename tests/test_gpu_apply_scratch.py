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


def _exact_case(sap, m, n, d, adt, seed):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    A = torch.randint(-8, 9, (m, n), generator=g, device="cuda").to(adt)
    idx, sign = sap.sps_generate(m, d, 8, seed)
    ref = sap.sps_apply(idx, sign, d, 8, A, None, y_dtype=torch.float64)
    torch.cuda.synchronize()
    return A, idx, sign, d, ref


def test_streams_share_scratch(sap):  # noqa: F811
    """Asynchronous applies on three streams of one context, the null stream among them, with lists, slices and
    packed rows of their own sizes."""
    import torch
    ctx = sap.Context(0)
    cases = [_exact_case(sap, 131072, 1024, 4000, torch.float32, 1), _exact_case(sap, 131072, 1024, 4001, torch.float32, 2),
             _exact_case(sap, 90001, 1030, 2400, torch.float32, 3)]
    print("scratch-streams", flush=True)
    streams = [torch.cuda.Stream(), torch.cuda.default_stream(), torch.cuda.Stream()]
    outs = []
    for rep in range(6):
        for k, (A, idx, sign, d, ref) in enumerate(cases):
            Y = torch.full_like(ref, float("nan"))
            st = streams[(rep * 2 + k + k // 2) % 3]
            st.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(st):
                sap.sps_apply(idx, sign, d, 8, A, None, ctx=ctx, Y=Y, y_dtype=torch.float64)
            outs.append((Y, ref))
    torch.cuda.synchronize()
    for Y, ref in outs:
        assert torch.equal(Y, ref)
    ctx.close()


def test_captured_apply(sap):  # noqa: F811
    """A captured apply that needs no workspace, replayed between eager ones that
    use the context's scratch."""
    import torch
    ctx = sap.Context(0)
    A, idx, sign, d, ref = _exact_case(sap, 131072, 1024, 4000, torch.float32, 1)
    B, idx2, sign2, d2, ref2 = _exact_case(sap, 90001, 1030, 2400, torch.float32, 3)
    print("scratch-capture", flush=True)
    Y, Y2 = torch.empty_like(ref), torch.empty_like(ref2)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        sap.sps_apply(idx, sign, d, 8, A, None, ctx=ctx, Y=Y, y_dtype=torch.float64)
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        sap.sps_apply(idx, sign, d, 8, A, None, ctx=ctx, Y=Y, y_dtype=torch.float64)
    for rep in range(4):
        Y.fill_(float("nan"))
        graph.replay()
        sap.sps_apply(idx2, sign2, d2, 8, B, None, ctx=ctx, Y=Y2, y_dtype=torch.float64)
        torch.cuda.synchronize()
        assert torch.equal(Y, ref), rep
        assert torch.equal(Y2, ref2), rep
    ctx.close()
