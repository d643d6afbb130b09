"""GPU parity of the sketch apply's packed rows (16-byte sketch rows, zeta = 8),
single and batched, at every strip width, with ragged last batches of rows,
last strips without and with b's column, padded rows and foreign sketches.

Integer A and b keep every partial sum exact, so a single apply's Y must equal
the exact sums times 1/sqrt(zeta) bit for bit.  The batched form is held to the
oracle after a fixed count of 8 steps, where the iterate still depends on every
row of the sketch, at the FP64 bars of the batched form's other tests."""
import numpy as np
import pytest

import inputs
from test_gpu_apply_forms import _out_of_range, _run, sap  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,d,adt,ydt,with_b,pad", [
    (200003, 64, 600, "f64", "f64", True, 0),     # 32 columns; b alone in the last strip
    (200003, 95, 600, "f32", "f64", True, 1),     # b in a full last strip
    (120001, 150, 1024, "bf16", "f64", True, 3),  # 16
    (100001, 160, 1100, "f64", "f64", False, 2),  # 16, no b, whole strips
    (90007, 163, 2052, "f32", "f32", False, 0),   # 8, no b, 3 columns in the last
    (60011, 302, 2499, "f64", "f64", True, 5),    # 4, below the gather's d
    (20011, 401, 8191, "f32", "f64", True, 0),    # 2
    (20011, 301, 16385, "f64", "f32", True, 0),   # 1, above the gather's d
])
@pytest.mark.parametrize("spoil", [None, _out_of_range])
def test_packed_single_exact(sap, m, n, d, adt, ydt, with_b, pad, spoil):  # noqa: F811
    import torch
    print(f"packed m={m} n={n} d={d} A={adt} Y={ydt} b={with_b} pad={pad} spoil={spoil is not None}", flush=True)
    Y, ref = _run(sap, m, n, d, 8, adt, ydt, with_b, pad, spoil=spoil)
    assert torch.equal(Y, ref)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("zeta", [8, 5])
def test_batch_strip_widths(sap, orc, dtype, zeta):  # noqa: F811
    """Problems whose strips are 32, 16, 8 and 4 columns wide in one batch."""
    import torch
    shapes = [(5003, 16, 200), (9001, 150, 600), (20001, 31, 400), (6001, 40, 1100), (5001, 20, 2400),
              (7001, 60, 4096), (4097, 64, 256)]
    print(f"batch widths dtype={np.dtype(dtype).name} zeta={zeta} shapes={shapes}", flush=True)
    probs = [inputs.make_problem(m, n, kind="colscale", cond=1e4, noise=1e-8, seed=7300 + k, dtype=dtype)
             for k, (m, n, d) in enumerate(shapes)]
    As = [torch.from_numpy(np.ascontiguousarray(p.A)).cuda() for p in probs]
    bs = [torch.from_numpy(p.b).cuda() for p in probs]
    T = 8
    xs, st, infos = sap.sap_solve_batch(As, bs, [d for _, _, d in shapes], zeta, 31, tol=0.0, maxiter=T, fixed_iters=T)
    torch.cuda.synchronize()
    for k, p in enumerate(probs):
        A64 = p.A.astype(np.float64)
        x_or, _ = orc.solve(A64, p.b, shapes[k][2], zeta, 31, tol=0.0, maxiter=T, stream=k)
        x = xs[k].cpu().numpy()
        assert infos[k]["iters"] == T, infos[k]
        assert np.linalg.norm(A64 @ (x - x_or)) <= 1e-11 * np.linalg.norm(p.b), k
        assert np.linalg.norm(x - x_or) <= 1e-8 * np.linalg.norm(x_or), k
