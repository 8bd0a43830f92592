"""Panels wider than a leaf, split in two until they are leaves.  With
lookahead the plan chooses 64 columns for these matrices, without it takes b, so
both are run: b of two, three, four and five leaves, and b that leaves do not
divide.  A has singular values in [1, 2]; bounds as for the small
factorizations (a few m u, 1e-11).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("m,n,b", [(700, 512, 128), (801, 576, 192), (700, 512, 256), (960, 640, 320), (900, 720, 240),
                                   (500, 288, 96), (641, 320, 160)])
@pytest.mark.parametrize("lookahead", [0, 1])
def test_wide_panels(m, n, b, lookahead):
    from paper_2311_11943_amd import cqr
    print(f"[case] wide panels {m}x{n} b={b} lookahead={lookahead}", flush=True)
    rng = np.random.default_rng(m + n)
    U, _ = np.linalg.qr(rng.standard_normal((m, n)))
    V, _ = np.linalg.qr(rng.standard_normal((n, n)))
    A = U @ (np.linspace(1, 2, n)[:, None] * V)
    q = cqr.CodedQR(cqr.Config(m, n, 1, 1, 0, 0, b, lookahead=lookahead))
    Q, R, _, _ = q.run(torch.from_numpy(A).cuda())
    torch.cuda.synchronize()
    assert q.info() == 0
    q.close()
    Q, R = Q.cpu().numpy(), R.cpu().numpy()
    Rn = np.linalg.qr(A)[1]
    Rn *= np.sign(np.diag(Rn))[:, None]
    worst = max(np.linalg.norm(Q.T @ Q - np.eye(n)), np.linalg.norm(A - Q @ R) / np.linalg.norm(A),
                np.linalg.norm(R - Rn) / np.linalg.norm(Rn))
    print(f"    worst {worst:.2e}", flush=True)
    assert worst <= 1e-11
