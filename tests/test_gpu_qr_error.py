"""GPU test of the QR's error against 80-bit arithmetic: a panel factored from its
Gram matrix must be as exact as one factored column by column.

Q is formed from the reflectors in 80 bits, so that what is measured is the
reflectors' own error.  On these matrices the column-by-column form, run on the
CPU with the same order of sums, has ||Q^T Q - I|| = 1.9 to 2.2 u sqrt(cols)
(u = 2^-53), whatever the columns' correlation, and max ||(Q R - Y)_j|| / ||Y_j||
= 2.6 to 4.6 u; the bars leave a tenth on the first and a third on the second.
Norms that come out of G with a rounding at every step, or that lost three
quarters of what G was summed for, miss them (2.4 to 7.3, and up to 13)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


def _matrix(kind, rows, cols, seed):
    Y = np.random.default_rng(seed).standard_normal((rows, cols))
    if kind == "scaled":  # columns of norms 1 to 1e-4, as a sketch of column-scaled data
        return Y * np.logspace(0, -4, cols)[None, :]
    share = float(kind)   # every column keeps this share of its squared norm beside the one before
    for j in range(1, cols):
        Y[:, j] = np.sqrt(1 - share) * Y[:, j - 1] / np.linalg.norm(Y[:, j - 1]) + np.sqrt(share) * Y[:, j] / np.linalg.norm(Y[:, j])
    return Y


def _errors(Y, F, tau):
    rows, cols = Y.shape
    B = np.zeros((rows, 2 * cols), dtype=np.longdouble)  # [I R], then Q times it
    B[:cols, :cols] = np.eye(cols)
    B[:cols, cols:] = np.triu(F[:cols])
    for k in range(cols - 1, -1, -1):
        v = F[k:, k].astype(np.longdouble)
        v[0] = 1.0
        B[k:] -= np.outer(v, np.longdouble(tau[k]) * (v @ B[k:]))
    Q = B[:, :cols]
    orth = np.linalg.norm((Q.T @ Q - np.eye(cols)).astype(np.float64))
    back = np.sqrt(((B[:, cols:] - Y) ** 2).sum(0) / (Y.astype(np.longdouble) ** 2).sum(0)).max()
    return orth / (U * np.sqrt(cols)), float(back) / U


@pytest.mark.parametrize("kind,rows,cols", [("scaled", 400, 101), ("scaled", 1026, 129), ("scaled", 4500, 64),
                                            ("0.3", 600, 64), ("0.5", 2100, 65), ("0.8", 900, 65)])
def test_qr_error(kind, rows, cols):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_03070_amd as sap
    got = []
    for seed in (1, 2, 3):
        Y = _matrix(kind, rows, cols, seed)
        Yt = torch.from_numpy(np.ascontiguousarray(Y.T)).cuda()
        tau = sap.sap_qr(Yt)
        torch.cuda.synchronize()
        got.append(_errors(Y, Yt.cpu().numpy().T, tau.cpu().numpy()))
    orth, back = np.mean(got, axis=0)
    print(f"qr-error {kind} rows={rows} cols={cols}: orthogonality {orth:.2f}, backward {back:.2f}", flush=True)
    assert orth <= 2.4 and back <= 6.0
