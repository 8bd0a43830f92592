"""The adjoint's kernels at the edges of their tiles and through each of its
routes: the triangular inverse's 64-row blocks and doubling levels (batched up
to 512, one by one above), the 64 x 64 and 128 x 128 products with triangular
operands, and the general kernels that odd heights fall back to.

R is upper triangular with a diagonal that dominates its rows (condition number
below 4).  The reference evaluates the formulas in NumPy / SciPy, FP64.  Every
product has at most m' + n terms and there are five in a row, so the relative
error in the 2-norm stays below 5 (m' + n) u cond(R)^2 < 1e-10 for the largest
size here; 1e-10 is asserted.
"""
import numpy as np
import pytest

import synth
from oracle import coded_qr as oc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
linalg = pytest.importorskip("scipy.linalg")


def _upper(n, rng):
    return np.triu(rng.uniform(-1, 1, (n, n)), 1) / (2 * n) + np.diag(rng.uniform(1, 2, n))


def _engine(m, n):
    from paper_2311_11943_amd import cqr
    v = synth.q_generator_draws(1, 4, 0)
    return cqr, cqr.CodedQR(cqr.Config(m, n, 4, 1, 1, 0, 4), v, None), oc.q_generator(v)


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("m,n", [(64, 16), (72, 60), (128, 64), (132, 68), (160, 96), (256, 128), (260, 192),
                                 (404, 196), (700, 320), (1300, 576), (2304, 1152), (6400, 1088)])
def test_backward_sizes(m, n):
    cqr, q, gv = _engine(m, n)
    print(f"[case] backward m={m} n={n}", flush=True)
    rng = np.random.default_rng(m + n)
    mp, bs = q.cfg.mp, q.cfg.bs
    R, dR = _upper(n, rng), rng.standard_normal((n, n))
    Q, dQ = rng.standard_normal((mp, n)) / np.sqrt(mp), rng.standard_normal((mp, n))
    dev = lambda x: cqr.to_device_colmajor(x, "cuda:0")
    dA = q.backward(dev(Q), dev(R), dev(dQ), dev(dR))
    torch.cuda.synchronize()
    q.close()
    M = R @ np.triu(dR).T - dQ.T @ Q
    S = np.tril(M) + np.tril(M, -1).T
    X = linalg.solve_triangular(R, (dQ + Q @ S).T).T
    ref = X[:m] + np.kron(gv, np.eye(bs)).T @ X[m:] if m < 1000 else \
        X[:m] + (gv.T @ X[m:].reshape(1, -1)).reshape(m, n)
    err = _rel(dA.cpu().numpy(), ref)
    print(f"    error {err:.2e}", flush=True)
    assert err <= 1e-10


@pytest.mark.parametrize("n", [16, 60, 64, 68, 128, 132, 260, 388])
@pytest.mark.parametrize("nrhs", [1, 4, 5])
@pytest.mark.parametrize("odd", [False, True])
def test_solve_backward_sizes(n, nrhs, odd):
    m = n + 8
    cqr, q, gv = _engine(m, n)
    print(f"[case] solve_backward n={n} nrhs={nrhs} odd={odd}", flush=True)
    rng = np.random.default_rng(n + nrhs)
    R = _upper(n, rng)
    Qp, Bp = rng.standard_normal((m, n)), rng.standard_normal((m, nrhs))
    X, dX = rng.standard_normal((n, nrhs)), rng.standard_normal((n, nrhs))
    dev = lambda x: cqr.to_device_colmajor(x, "cuda:0")
    Rn = R + np.tril(np.full((n, n), np.nan), -1)      # nothing below the diagonal is used
    Rd = dev(np.vstack([Rn, np.zeros((1, n))]))[:n] if odd else dev(Rn)   # an odd leading dimension
    dQ, dR, dB = q.solve_backward(dev(Qp), Rd, dev(Bp), dev(X), dev(dX))
    torch.cuda.synchronize()
    q.close()
    G0 = np.kron(oc.g0_tilde(gv), np.eye(q.cfg.bs))
    dy = linalg.solve_triangular(R, dX, trans="T")
    assert _rel(dQ[:m].cpu().numpy(), G0 @ (Bp @ dy.T)) <= 1e-10
    assert not dQ[m:].any()
    assert _rel(dR.cpu().numpy(), -np.triu(dy @ X.T)) <= 1e-10
    assert _rel(dB.cpu().numpy(), G0 @ (Qp @ dy)) <= 1e-10
