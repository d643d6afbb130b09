"""GPU tests of the chained QR's hand-over from block to block (places marked
with a signalling NaN and read until overwritten), at every register block
height: the factor against the input's Gram matrix, the same bits on every run,
and inputs that are NaN, the marking pattern among them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
SHAPES = [(300, 40), (700, 61), (1500, 130), (2049, 301), (4096, 77), (6000, 40), (12000, 12)]


def _sap():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_03070_amd as sap
    return sap


@pytest.mark.parametrize("rows,cols", SHAPES)
def test_handover_same_bits(rows, cols):
    import torch
    sap = _sap()
    print(f"qr-handover rows={rows} cols={cols}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(rows)
    Y = torch.randn(cols, rows, generator=g, device="cuda", dtype=torch.float64)
    runs = []
    for _ in range(4):
        F = Y.clone()
        tau = sap.sap_qr(F)
        torch.cuda.synchronize()
        runs.append((F, tau))
    for F, tau in runs[1:]:
        assert torch.equal(F, runs[0][0]) and torch.equal(tau, runs[0][1])
    R = torch.triu(runs[0][0].T[:cols])
    assert torch.linalg.norm(R.T @ R - Y @ Y.T) <= 1e-12 * torch.linalg.norm(R) ** 2


@pytest.mark.parametrize("bits", [0x7FF4D15C00000000, 0x7FF4D15C00000001, 0x7FF8000000000000])
@pytest.mark.parametrize("rows,cols", [(300, 40), (1500, 130), (4096, 77)])
def test_handover_nan_input(rows, cols, bits):
    """A NaN in column c makes R's columns from c on non-finite and leaves those
    before it as they are."""
    import torch
    sap = _sap()
    print(f"qr-handover nan rows={rows} cols={cols} bits={bits:x}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(rows + 1)
    Y = torch.randn(cols, rows, generator=g, device="cuda", dtype=torch.float64)
    ref = Y.clone()
    sap.sap_qr(ref)
    c = cols // 2
    bad = Y.clone()
    bad.view(torch.int64)[c, rows - 3] = bits
    sap.sap_qr(bad)
    torch.cuda.synchronize()
    nb = c // 4 * 4  # whole blocks before the column
    assert torch.equal(bad[:nb], ref[:nb])
    assert not torch.isfinite(torch.diagonal(bad)[c:]).any()
