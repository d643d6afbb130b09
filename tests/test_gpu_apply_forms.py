"""GPU parity of the sketch apply's two forms (lists and gather above d = 2500
where it pays, LDS scatter otherwise) and of the fall-back between them.

Integer A and b keep every partial sum exact, so Y must equal the exact sums
times 1/sqrt(zeta) bit for bit, whatever form ran and in any order."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
DT = {"f64": "float64", "f32": "float32", "bf16": "bfloat16"}


def _run(sap, m, n, d, zeta, adt, ydt, with_b, pad, spoil=None, seed=5, noalloc=False):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    A = torch.randint(-8, 9, (m, n + pad), generator=g, device="cuda").to(getattr(torch, DT[adt]))[:, :n]
    b = torch.randint(-8, 9, (m,), generator=g, device="cuda").to(torch.float64) if with_b else None
    idx, sign = sap.sps_generate(m, d, zeta, seed)
    if spoil:
        spoil(idx)
    f = sap.sps_apply_noalloc if noalloc else sap.sps_apply
    Y = f(idx, sign, d, zeta, A, b, y_dtype=getattr(torch, DT[ydt]))
    Ab = torch.cat([A.double(), b[:, None]], 1) if with_b else A.double()
    exact = torch.zeros(d, Ab.shape[1], dtype=torch.float64, device="cuda")
    for k in range(zeta):
        r = idx[:, k].long()
        keep = (r >= 0) & (r < d)
        sg = (((sign >> k) & 1).double() * 2 - 1) * keep
        exact.index_add_(0, torch.where(keep, r, 0), Ab * sg[:, None])
    torch.cuda.synchronize()
    h = 1.0 / np.sqrt(float(zeta))
    if ydt == "f64":
        ref = (exact * h).T
    else:
        assert exact.abs().max() < 2 ** 24
        ref = (exact.to(torch.float32) * torch.tensor(np.float32(h), device="cuda")).T
    return Y, ref.contiguous()


@pytest.fixture(scope="module")
def sap():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_03070_amd as sap
    sap.lib()
    return sap


@pytest.mark.parametrize("m,n,d,zeta,adt,ydt,with_b,pad", [
    (130001, 301, 5003, 8, "f64", "f64", True, 3),    # gather, 8 slots, last strip of one column
    (130001, 303, 5003, 8, "f32", "f32", True, 1),    # FP32 tiles, FP32 Y
    (150000, 257, 3001, 12, "f64", "f64", False, 0),  # 3 slots, zeta that is not 8, no b
    (98304, 300, 9001, 8, "f32", "f64", True, 0),     # 2-column strips; whole tiles only
    (90001, 302, 9001, 8, "f64", "f64", True, 0),
    (120000, 511, 4096, 5, "bf16", "f64", True, 1),   # 4 slots full
    (70000, 602, 16384, 8, "f64", "f64", True, 0),    # 16 slots full
    (40961, 2050, 8192, 16, "f32", "f64", True, 2),   # 8 slots full, slices of tiles
    (33000, 129, 2499, 8, "f32", "f32", True, 0),     # scatter: FP32 Y from FP64 sums
    (300007, 65, 2052, 8, "f32", "f32", True, 0),     # scatter, re-chosen slices
    (600, 7, 40, 8, "f64", "f64", True, 0),           # fewer rows than two slices
    (20000, 33, 21000, 8, "f32", "f32", True, 0),     # row ranges (d past one FP64 strip)
])
def test_apply_forms_exact(sap, m, n, d, zeta, adt, ydt, with_b, pad):
    import torch
    print(f"apply-forms m={m} n={n} d={d} zeta={zeta} A={adt} Y={ydt} b={with_b} pad={pad}", flush=True)
    Y, ref = _run(sap, m, n, d, zeta, adt, ydt, with_b, pad)
    assert torch.equal(Y, ref)


def _few_rows(idx):  # every nonzero in 16 rows: the lists of one group pass their share
    idx.remainder_(16)


def _out_of_range(idx):
    idx[::7, 1] = 1 << 30
    idx[::11, 2] = -3
    idx[::5, 0] = idx[::5, 3]  # the same row twice


@pytest.mark.parametrize("spoil", [_few_rows, _out_of_range])
@pytest.mark.parametrize("adt", ["f64", "f32"])
def test_apply_gather_foreign_sketch(sap, spoil, adt):
    """Caller-supplied sketches: too uneven for the lists (the scatter form takes
    over), out-of-range and repeated rows."""
    import torch
    print(f"apply-foreign {spoil.__name__} A={adt}", flush=True)
    Y, ref = _run(sap, 130001, 301, 5003, 8, adt, "f64", True, 0, spoil=spoil)
    assert torch.equal(Y, ref)


def test_apply_forms_noalloc(sap):
    """The allocation-free entry point takes the gather where its buffer has room."""
    import torch
    Y, ref = _run(sap, 130001, 301, 5003, 8, "f64", "f64", True, 0, noalloc=True)
    assert torch.equal(Y, ref)


def test_apply_tight_budget(sap):
    """A context whose budget holds what the scatter form needs (two row slices
    of the 5003 x 301 sketch: 24.1 MB) and not the lists beside them."""
    import torch
    ctx = sap.Context(0, 26 << 20)
    m, n, d = 130001, 301, 5003
    A = torch.randint(-8, 9, (m, n), device="cuda").double()
    idx, sign = sap.sps_generate(m, d, 8, 3)
    Y = sap.sps_apply(idx, sign, d, 8, A, None, ctx=ctx)
    assert torch.equal(Y, sap.sps_apply(idx, sign, d, 8, A, None))
    torch.cuda.synchronize()
    ctx.close()
