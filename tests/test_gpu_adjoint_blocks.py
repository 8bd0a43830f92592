"""The adjoint where its triangular products run on 128 x 128 blocks (at least
512 of them), in place on the lower triangle, with a last block that is not
full.  Formulas and bound as for the smaller sizes: 5 (m' + n) u cond(R)^2 <
1e-10.
"""
import numpy as np
import pytest

import synth
from oracle import coded_qr as oc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("m,n", [(3072, 3008), (4096, 3040)])
def test_backward_blocks(m, n):
    from paper_2311_11943_amd import cqr
    print(f"[case] backward m={m} n={n}", flush=True)
    v = synth.q_generator_draws(1, 4, 0)
    q = cqr.CodedQR(cqr.Config(m, n, 4, 1, 1, 0, 4), v, None)
    gv = torch.from_numpy(oc.q_generator(v)).cuda()
    mp = q.cfg.mp
    g = torch.Generator(device="cuda:0").manual_seed(m + n)
    rand = lambda r, c: torch.rand(c, r, dtype=torch.float64, device="cuda:0", generator=g).t()
    R = (torch.triu(2 * rand(n, n) - 1, 1) / (2 * n)).t().contiguous().t()
    R.diagonal().copy_(1 + rand(n, 1)[:, 0])
    Q, dQ, dR = (rand(mp, n) - 0.5) / np.sqrt(mp), rand(mp, n) - 0.5, rand(n, n) - 0.5
    dA = q.backward(Q, R, dQ, dR)
    torch.cuda.synchronize()
    q.close()
    M = R @ torch.triu(dR).T.contiguous() - dQ.T.contiguous() @ Q
    S = torch.tril(M) + torch.tril(M, -1).T
    X = torch.linalg.solve_triangular(R, (dQ + Q @ S).T.contiguous(), upper=True).T
    ref = X[:m] + (gv.T.contiguous() @ X[m:].reshape(1, -1)).reshape(m, n)
    err = (torch.linalg.norm(dA - ref) / torch.linalg.norm(ref)).item()
    print(f"    error {err:.2e}", flush=True)
    assert err <= 1e-10
