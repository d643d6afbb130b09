"""GPU parity of a batch whose sketches are generated by both launches (packed at
zeta = 8, words otherwise), held to the oracle after a fixed count of 8 steps at
the FP64 bars of the batched form's other tests."""
import numpy as np
import pytest

import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("zetas", [(8, 4, 8, 16, 1), (4, 8, 33), (64, 8), (5, 12)])
def test_batch_mixed_zetas(orc, zetas):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_03070_amd as sap
    print(f"batch-zetas {zetas}", flush=True)
    shapes = [(4000 + 257 * k, 20 + 7 * k, 96 + 31 * k) for k in range(len(zetas))]
    probs = [inputs.make_problem(m, n, kind="colscale", cond=1e4, noise=1e-8, seed=900 + k) for k, (m, n, _) in enumerate(shapes)]
    As = [torch.from_numpy(np.ascontiguousarray(p.A)).cuda() for p in probs]
    bs = [torch.from_numpy(p.b).cuda() for p in probs]
    T = 8
    xs, _, infos = sap.sap_solve_batch(As, bs, [d for _, _, d in shapes], list(zetas), 31, tol=0.0, maxiter=T, fixed_iters=T)
    torch.cuda.synchronize()
    for k, p in enumerate(probs):
        x_or, _ = orc.solve(p.A, p.b, shapes[k][2], zetas[k], 31, tol=0.0, maxiter=T, stream=k)
        x = xs[k].cpu().numpy()
        assert infos[k]["iters"] == T, infos[k]
        assert np.linalg.norm(p.A @ (x - x_or)) <= 1e-11 * np.linalg.norm(p.b), k
        assert np.linalg.norm(x - x_or) <= 1e-8 * np.linalg.norm(x_or), k
