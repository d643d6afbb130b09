"""GPU test of sap_choose_d's price of the sketch apply: it is timed on a slab of
65536 rows, and the whole problem may take another form than the slab.

The slab's timing is scaled by the ratio of two of the apply's own estimates,
each fitted to measurements within about 10%; the bar is a quarter."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,ks,dtype", [(1 << 20, 500, (4, 8, 10), "float64"), (1 << 19, 1000, (3, 4, 5), "float64"),
                                          (1 << 19, 700, (2, 4, 6), "float32")])
def test_apply_price(m, n, ks, dtype):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_03070_amd as sap
    print(f"choose-price m={m} n={n} {dtype}", flush=True)
    ctx = sap.Context(0)
    A = torch.randn(m, n, device="cuda", dtype=torch.float32).to(getattr(torch, dtype))
    b = torch.randn(m, device="cuda", dtype=torch.float64)
    sap.sap_choose_d(A, b, 8, 1e-12, ctx=ctx)
    prob = sap._problem(A, b)
    for k in ks:
        d = k * n
        price = ctypes.c_double(0.0)
        assert sap.lib().sap_internal_price_apply(ctx.handle, ctypes.byref(prob), 8, d, ctypes.byref(price)) == 0
        idx, sign = sap.sps_generate(m, d, 8, 3, ctx=ctx)
        Y = torch.empty(n + 1, d, dtype=torch.float64, device="cuda")
        times = []
        for _ in range(6):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            sap.sps_apply(idx, sign, d, 8, A, b, y_dtype=torch.float64, ctx=ctx, Y=Y)
            e1.record()
            e1.synchronize()
            times.append(e0.elapsed_time(e1))
        ms = sorted(times[1:])[2]
        print(f"  d={d}: priced {price.value:.3f} ms, takes {ms:.3f} ms", flush=True)
        assert abs(price.value / ms - 1.0) <= 0.25
    torch.cuda.synchronize()
    ctx.close()
