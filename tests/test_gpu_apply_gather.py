"""GPU parity of every gather kernel of the sketch apply: 3, 4 and 8 slots of 4
columns and 16 slots of 2, each A and Y type, and its fall-back to the scatter.
Each row asserts that the gather is the form that runs.

Integer A and b keep every partial sum exact, so Y must equal the exact sums
times 1/sqrt(zeta) bit for bit.  A non-finite entry of A must reach its zeta rows
of its own column of Y and nothing else, in either form."""
import ctypes

import numpy as np
import pytest

from test_gpu_apply_forms import _few_rows, _out_of_range, sap  # noqa: F401

pytestmark = pytest.mark.gpu
DT = {"f64": "float64", "f32": "float32", "bf16": "bfloat16"}
CODE = {"f64": 0, "f32": 1, "bf16": 2}
GATHER, SCATTER = 2, 1


def _form(sap, m, zeta, d, n, lda, with_b, adt, ydt):
    f = sap.lib().sap_internal_apply_form
    f.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int64] + [ctypes.c_int] * 3
    return f(sap.default_context().handle, m, zeta, d, n, lda, int(with_b), CODE[adt], CODE[ydt])


def _case(sap, m, n, d, zeta, adt, ydt, with_b, first=0, pad=0, spoil=None, hurt=None, form=GATHER, noalloc=False):
    """Y and the exact result; A starts `first` columns into a row of its storage."""
    import torch
    print(f"apply-gather m={m} n={n} d={d} zeta={zeta} A={adt} Y={ydt} b={with_b} first={first} pad={pad} "
          f"spoil={spoil.__name__ if spoil else None}", flush=True)
    lda = first + n + pad
    assert _form(sap, m, zeta, d, n, lda, with_b, adt, ydt) == form
    g = torch.Generator(device="cuda")
    g.manual_seed(m + d)
    A = torch.randint(-8, 9, (m, lda), generator=g, device="cuda").to(getattr(torch, DT[adt]))[:, first:first + n]
    b = torch.randint(-8, 9, (m,), generator=g, device="cuda").to(torch.float64) if with_b else None
    idx, sign = sap.sps_generate(m, d, zeta, 5)
    if spoil:
        spoil(idx)
    if hurt:
        for i, j, v in hurt:
            A[i, j] = v
    apply = sap.sps_apply_noalloc if noalloc else sap.sps_apply
    Y = apply(idx, sign, d, zeta, A, b, y_dtype=getattr(torch, DT[ydt]))
    Ab = torch.cat([A.double(), b[:, None]], 1) if with_b else A.double()
    exact = torch.zeros(d, Ab.shape[1], dtype=torch.float64, device="cuda")
    for k in range(zeta):
        r = idx[:, k].long()
        keep = (r >= 0) & (r < d)
        sg = ((sign >> k) & 1).double() * 2 - 1
        exact.index_add_(0, r[keep], (Ab * sg[:, None])[keep])
    torch.cuda.synchronize()
    h = 1.0 / np.sqrt(float(zeta))
    if ydt == "f64":
        ref = (exact * h).T
    else:
        assert exact.nan_to_num(0, 0, 0).abs().max() < 2 ** 24
        ref = (exact.to(torch.float32) * torch.tensor(np.float32(h), device="cuda")).T
    return Y, ref.contiguous()


def _equal(Y, ref):
    """Bit for bit, any NaN for any NaN."""
    import torch
    nan = torch.isnan(ref)
    return torch.equal(torch.isnan(Y), nan) and torch.equal(Y[~nan], ref[~nan])


SHAPES = {  # m, n, d; ragged last tiles and strips
    "3x4": (131071, 1022, 3001),
    "4x4": (131071, 1023, 4001),
    "8x4": (151665, 261, 5003),
    "16x2": (131071, 1001, 16000),
}


@pytest.mark.parametrize("adt", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("ydt", ["f64", "f32"])
@pytest.mark.parametrize("slots", list(SHAPES))
def test_gather_exact(sap, slots, adt, ydt):  # noqa: F811
    m, n, d = SHAPES[slots]
    Y, ref = _case(sap, m, n, d, 8, adt, ydt, True, pad=1)
    assert _equal(Y, ref)


@pytest.mark.parametrize("m,n,d,zeta,adt,with_b", [
    (201868, 163, 10000, 8, "f64", False),  # 2-column strips, the last of one column, no b
    (137877, 260, 16384, 8, "f64", True),   # 16 slots full
    (65536, 1000, 8192, 16, "f32", True),   # 8 slots full, whole tiles, zeta that is not 8
    (114001, 601, 12001, 5, "f32", True),
])
def test_gather_edges(sap, m, n, d, zeta, adt, with_b):  # noqa: F811
    Y, ref = _case(sap, m, n, d, zeta, adt, "f64", with_b)
    assert _equal(Y, ref)


@pytest.mark.parametrize("spoil", [_few_rows, _out_of_range])
@pytest.mark.parametrize("slots,adt,ydt", [("8x4", "f32", "f64"), ("8x4", "f32", "f32"), ("16x2", "f32", "f64"),
                                           ("16x2", "f64", "f64"), ("3x4", "bf16", "f64")])
def test_gather_foreign_sketch(sap, spoil, slots, adt, ydt):  # noqa: F811
    m, n, d = SHAPES[slots]
    Y, ref = _case(sap, m, n, d, 8, adt, ydt, True, spoil=spoil)
    assert _equal(Y, ref)


@pytest.mark.parametrize("slots,adt", [("8x4", "f64"), ("16x2", "f32"), ("4x4", "bf16")])
def test_gather_noalloc(sap, slots, adt):  # noqa: F811
    m, n, d = SHAPES[slots]
    Y, ref = _case(sap, m, n, d, 8, adt, "f64", True, noalloc=True)
    assert _equal(Y, ref)


INF, NAN = float("inf"), float("nan")


@pytest.mark.parametrize("m,n,d,zeta,adt,ydt,form", [
    (131071, 1022, 3001, 8, "f64", "f64", GATHER), (151665, 261, 5003, 8, "f32", "f32", GATHER),
    (131071, 1001, 16000, 8, "f32", "f64", GATHER), (151665, 261, 5003, 8, "bf16", "f64", GATHER),
    (200003, 64, 600, 8, "f64", "f64", SCATTER),    # packed rows, 32 columns
    (120001, 150, 1024, 8, "bf16", "f64", SCATTER),  # 16
    (90007, 163, 2052, 8, "f32", "f32", SCATTER),    # 8
    (20011, 401, 8191, 8, "f32", "f64", SCATTER),    # 2
    (20000, 100, 400, 8, "f64", "f64", SCATTER),     # no packed copy
])
def test_nonfinite_entries(sap, m, n, d, zeta, adt, ydt, form):  # noqa: F811
    """The last row, the last column, a whole tile's first row; two infinities of one column."""
    hurt = [(m - 1, n - 1, INF), (0, 0, NAN), (8192, 3, -INF), (4096, 2, INF), (4097, 2, -INF), (m // 2, n - 2, NAN)]
    Y, ref = _case(sap, m, n, d, zeta, adt, ydt, True, hurt=hurt, form=form)
    assert _equal(Y, ref)


@pytest.mark.parametrize("m,n,d,form", [(151665, 261, 5003, GATHER), (131071, 1001, 16000, GATHER),
                                        (120001, 150, 1024, SCATTER), (60011, 302, 2499, SCATTER)])
@pytest.mark.parametrize("pad", [0, 1])
def test_bf16_odd_base(sap, m, n, d, form, pad):  # noqa: F811
    """A BF16 A whose rows start 2 bytes past a 4-byte boundary."""
    Y, ref = _case(sap, m, n, d, 8, "bf16", "f64", True, first=1, pad=pad, form=form)
    assert _equal(Y, ref)
