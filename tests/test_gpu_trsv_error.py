"""GPU test of the triangular solves' error against 80-bit arithmetic.

sap_trsv multiplies by the inverse of each 64 x 64 diagonal block, whose columns
are back substitutions.  The reference inverts the one block of an n = 64 R the
same way on the CPU, in FP64, column by column; over 24 sketches with singular
values 1 to 1e-k the solves' mean error may be a quarter larger than the
reference's (their sums are ordered differently; blocks joined by products with
inverses come out 1.4 to 1.6 times as far off at k = 10)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _sketch_r(n, k, seed):
    g = np.random.default_rng(seed)
    V, _ = np.linalg.qr(g.standard_normal((n, n)))
    return np.triu(np.linalg.qr((g.standard_normal((4 * n, n)) * np.logspace(0, -k, n)) @ V.T, mode="r")), g.standard_normal(n)


def _solve80(R, b, trans):
    A = (R.T if trans else R).astype(np.longdouble)
    x = np.zeros(len(b), dtype=np.longdouble)
    for i in (range(len(b)) if trans else range(len(b) - 1, -1, -1)):
        x[i] = (b[i] - (A[i] * x).sum()) / A[i, i]
    return x


def _column_inverse(R):
    n = len(R)
    X = np.zeros((n, n))
    for r in range(n - 1, -1, -1):
        X[r, r] = 1.0 / R[r, r]
        for k in range(r + 1, n):  # ascending, one product after the other
            X[r, r + 1:] -= R[r, k] * X[k, r + 1:]
        X[r, r + 1:] /= R[r, r]
    return X


def _errors(solve, trans, k, seeds=24):
    mine, ref = [], []
    for seed in range(seeds):
        R, b = _sketch_r(64, k, 1000 * k + seed)
        x = _solve80(R, b, trans)
        X = _column_inverse(R)
        norm = float(np.linalg.norm(x.astype(np.float64)))
        mine.append(float(np.linalg.norm((solve(R, b, trans) - x).astype(np.float64))) / norm)
        ref.append(float(np.linalg.norm(((X.T if trans else X) @ b - x).astype(np.float64))) / norm)
    return np.mean(mine), np.mean(ref)


@pytest.mark.parametrize("trans", [0, 1])
@pytest.mark.parametrize("k", [3, 6, 10])
def test_trsv_error(trans, k):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_03070_amd as sap

    def solve(R, b, trans):
        Rt = torch.from_numpy(np.ascontiguousarray(R.T)).cuda()
        x = sap.sap_trsv(Rt, torch.from_numpy(b).cuda(), trans=trans)
        torch.cuda.synchronize()
        return x.cpu().numpy()

    mine, ref = _errors(solve, trans, k)
    print(f"trsv-error trans={trans} k={k}: {mine:.2e}, column by column on the CPU {ref:.2e}", flush=True)
    assert mine <= 1.25 * ref
