"""The coded solve's kernels at the edges of their blocks: 64-row inverted
diagonal blocks, 128-row blocks of the back substitution, groups of four
right-hand sides.

R is upper triangular with a diagonal that dominates its rows (condition number
below 4), with NaN below the diagonal, which the solve must not read.  The
reference is NumPy / SciPy in FP64.  With |Y - Y^| <= m u |Qpost|^T |Bpost| and
the substitution's |R X^ - Y^| <= n u |R| |X^|, the relative error in the
2-norm stays below (m + n) u cond(R) sqrt(n) < 3e-12 for these sizes; 1e-11 is
asserted.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
linalg = pytest.importorskip("scipy.linalg")


@pytest.mark.parametrize("n", [16, 60, 64, 68, 124, 128, 132, 192, 196, 256, 388])
@pytest.mark.parametrize("nrhs", [1, 3, 4, 5])
def test_solve_blocks(n, nrhs):
    from paper_2311_11943_amd import cqr
    m = n + 4
    print(f"[case] solve n={n} nrhs={nrhs}", flush=True)
    rng = np.random.default_rng(100 * n + nrhs)
    R = np.triu(rng.uniform(-1, 1, (n, n)), 1) / (2 * n) + np.diag(rng.uniform(1, 2, n))
    Q = rng.standard_normal((m, n))
    B = rng.standard_normal((m, nrhs))
    q = cqr.CodedQR(cqr.Config(m, n, 4, 4, 1, 1, 4), synth.q_generator_draws(1, 4, 0), synth.r_generator_draws(4, 1, 0))
    dev = lambda x: cqr.to_device_colmajor(x, "cuda:0")
    Rd = dev(R + np.tril(np.full((n, n), np.nan), -1))
    Qd, Bd = dev(Q), dev(B)
    X = q.solve(Qd, Rd, Bd)
    again = q.solve(Qd, Rd, Bd)
    torch.cuda.synchronize()
    q.close()
    ref = linalg.solve_triangular(R, Q.T @ B)
    err = np.linalg.norm(X.cpu().numpy() - ref) / np.linalg.norm(ref)
    print(f"    error {err:.2e}", flush=True)
    assert torch.equal(X, again)
    assert err <= 1e-11
