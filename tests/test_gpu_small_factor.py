"""Factorizations of small matrices at the edges of the small products' tiles:
16 x 16 outputs, 16 rows of depth at a time, depths around the largest that
takes them (2048 rows), odd leading dimensions, panels narrower and wider than
a tile, one to several panels.

A has singular values in [1, 2].  |Q^T Q - I| and |A - Q R| / |A| stay within a
few m u (re-projection, two Cholesky-QR passes), and R, unique with a positive
diagonal, within that times cond(A) of NumPy's: below 50 m u < 3e-11 for
these sizes (3e-10 at 26000 rows); 1e-11 is asserted up to 1000 rows, 5e-11 above.  A second run
gives the same bits.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("m,n,b", [
    (1, 1, 1), (7, 5, 5), (16, 16, 16), (17, 16, 8), (33, 33, 11), (64, 48, 16), (65, 51, 17), (100, 96, 48),
    (255, 63, 21), (257, 130, 65), (320, 320, 16), (321, 128, 128), (333, 192, 64), (512, 260, 20),
    (1007, 105, 35), (1386, 165, 33), (2047, 64, 16), (2048, 96, 32), (2049, 96, 32), (2064, 35, 7),
    (1025, 1024, 16), (1300, 1280, 40), (5121, 130, 65), (20500, 64, 16), (2304, 256, 128), (9216, 128, 64), (26000, 208, 16),
])
@pytest.mark.parametrize("lookahead", [0, 1])
def test_small_factor(m, n, b, lookahead):
    from paper_2311_11943_amd import cqr
    print(f"[case] factor {m}x{n} b={b} lookahead={lookahead}", flush=True)
    rng = np.random.default_rng(m + n)
    U, _ = np.linalg.qr(rng.standard_normal((m, n)))
    V, _ = np.linalg.qr(rng.standard_normal((n, n)))
    A = U @ (np.linspace(1, 2, n)[:, None] * V)
    q = cqr.CodedQR(cqr.Config(m, n, 1, 1, 0, 0, b, lookahead=lookahead))
    Q, R, _, _ = q.run(torch.from_numpy(A).cuda())
    again = q.run(torch.from_numpy(A).cuda())
    torch.cuda.synchronize()
    assert q.info() == 0
    q.close()
    assert torch.equal(Q, again[0]) and torch.equal(R, again[1])
    Q, R = Q.cpu().numpy(), R.cpu().numpy()
    Rn = np.linalg.qr(A)[1]
    Rn *= np.sign(np.diag(Rn))[:, None]
    tol = 1e-11 if m <= 1000 else 5e-11
    worst = max(np.linalg.norm(Q.T @ Q - np.eye(n)), np.linalg.norm(A - Q @ R) / np.linalg.norm(A),
                np.linalg.norm(R - Rn) / np.linalg.norm(Rn))
    print(f"    worst {worst:.2e}", flush=True)
    assert worst <= tol
