"""GPU test of the QR with a non-finite entry: R above a column's own block does
not depend on the block's other columns, so it stays what it is without the entry."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf"), 1e200])
@pytest.mark.parametrize("rows,cols", [(300, 40), (1500, 66), (4096, 40), (6000, 40)])
def test_qr_nonfinite_neighbour(rows, cols, value):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_03070_amd as sap
    print(f"qr-nonfinite rows={rows} cols={cols} value={value}", flush=True)
    nb = 4 if rows <= 4096 else 2
    g = torch.Generator(device="cuda")
    g.manual_seed(rows + 2)
    Y = torch.randn(cols, rows, generator=g, device="cuda", dtype=torch.float64)
    ref = Y.clone()
    sap.sap_qr(ref)
    c0 = cols // 2 // nb * nb  # the first column of a block, which has columns to its right
    bad = Y.clone()
    bad[c0, rows - 3] = value
    sap.sap_qr(bad)
    torch.cuda.synchronize()
    assert torch.equal(bad[:c0], ref[:c0])
    assert torch.equal(bad[c0 + 1:c0 + nb, :c0], ref[c0 + 1:c0 + nb, :c0])
    if not np.isfinite(value):
        assert not torch.isfinite(torch.diagonal(bad)[c0:]).any()
