"""GPU parity of the QR panels' Gram form and of its refusal.

A panel whose columns keep a quarter of their squared norm below the diagonal
is factored from its Gram matrix; any other (nearly dependent, triangular,
tiny or nearly square panels) column by column.  Both must meet the bars of the
other QR tests: ||R^T R - R_or^T R_or|| <= 1e-12 ||R_or||^2, ||Q R - Y|| <=
1e-12 ||Y|| sqrt(rows) / 10, and Q orthogonal to 1e-12 sqrt(cols).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _matrix(kind, rows, cols):
    rng = np.random.default_rng(rows * 13 + cols)
    Y = rng.standard_normal((rows, cols))
    if kind == "pairs":        # dependent to 1e-9 inside every 4-column panel
        Y[:, 1::2] = Y[:, 0:2 * (cols // 2):2] + 1e-9 * Y[:, 1::2]
    elif kind == "edge":       # column shares kept around the limit of the Gram form
        t = np.linspace(0.05, 0.95, cols // 2)
        Y[:, 1::2] = np.sqrt(1 - t) * Y[:, 0:2 * (cols // 2):2] + np.sqrt(t) * Y[:, 1::2]
    elif kind == "vandermonde":
        Y = np.linspace(0.1, 1.0, rows)[:, None] ** np.arange(cols)[None, :]
    elif kind == "identity":
        Y = np.eye(rows, cols)
    elif kind == "upper":      # nothing below the diagonal
        Y = np.triu(Y)
    elif kind == "tiny":       # squared norms below the normal range in every third column
        Y[:, ::3] *= 1e-150
    elif kind == "scaled":
        Y *= np.logspace(0, -12, cols)[None, :]
    return Y


@pytest.mark.parametrize("kind,rows,cols", [
    ("pairs", 900, 66), ("edge", 1100, 64), ("vandermonde", 600, 40), ("identity", 300, 33), ("upper", 520, 50),
    ("tiny", 700, 31), ("scaled", 2100, 65), ("gauss", 16, 4), ("gauss", 15, 4), ("gauss", 17, 6),
    ("gauss", 512, 127), ("gauss", 513, 513), ("gauss", 4096, 70), ("gauss", 4097, 70), ("pairs", 4500, 40),
    ("gauss", 9000, 20), ("pairs", 9000, 20)])
def test_qr_gram_form(orc, kind, rows, cols):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_03070_amd as sap
    print(f"qr-gram {kind} rows={rows} cols={cols}", flush=True)
    Y = _matrix(kind, rows, cols)
    Yt = torch.from_numpy(np.ascontiguousarray(Y.T)).cuda()
    tau = sap.sap_qr(Yt)
    torch.cuda.synchronize()
    F = Yt.cpu().numpy().T
    tau = tau.cpu().numpy()
    Fo, _ = orc.householder_qr(Y)
    R, Ro = np.triu(F[:cols]), np.triu(Fo[:cols])
    assert np.linalg.norm(R.T @ R - Ro.T @ Ro) <= 1e-12 * np.linalg.norm(Ro) ** 2
    Q = orc.q_factor(F, tau)
    assert np.linalg.norm(Q @ R - Y) <= 1e-12 * np.linalg.norm(Y) * max(1, np.sqrt(rows) / 10)
    assert np.linalg.norm(Q.T @ Q - np.eye(Q.shape[1])) <= 1e-12 * np.sqrt(cols)
    if kind in ("identity", "upper"):  # every reflector is trivial: the factor is Y itself
        assert np.all(tau == 0.0) and np.array_equal(R, np.triu(Y[:cols]))
