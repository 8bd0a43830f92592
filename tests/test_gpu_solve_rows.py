"""The solve's product Qpost^T Bpost at the edges of its batches of rows: 512
rows a batch with one wave a column (more than 1024 columns), 2048 with four.

With R_1 the identity the solution is that product: sums of m terms below 64.
Each rounding is at most u of a partial sum, which stays below 64 m, and m of
them meet; for random terms partial sums and their errors grow with sqrt(m), so
the difference to NumPy's stays below 64 m u by far; 64 m 1e-15 is asserted.
"""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def solver(m, n, nrhs, seed=0):
    from paper_2311_11943_amd import cqr
    q = cqr.CodedQR(cqr.Config(m, n, 1, 1, 0, 0, 1))
    rng = np.random.default_rng(seed)
    Q, B = np.clip(rng.standard_normal((m, n)), -8, 8), np.clip(rng.standard_normal((m, nrhs)), -8, 8)
    Qd, Bd, Rd = (cqr.to_device_colmajor(x, "cuda:0") for x in (Q, B, np.eye(n)))
    X, ws = cqr.col_major(n, nrhs, "cuda:0"), q.solve_workspace(nrhs)
    return Q, B, X, lambda: q.solve(Qd, Rd, Bd, X, ws)


@pytest.mark.parametrize("m,n,nrhs", [
    (1, 1, 1), (63, 5, 3), (64, 64, 4), (65, 64, 5), (255, 7, 1), (257, 64, 9), (1023, 33, 2), (1793, 64, 4),
    (2047, 64, 5), (2048, 64, 1), (2049, 16, 6), (2305, 64, 4), (4095, 3, 4), (6145, 8, 3),
    (1025, 1025, 1), (1088, 1025, 5), (1535, 1030, 4), (1536, 1030, 2), (1537, 1030, 3),
])
def test_rows(m, n, nrhs):
    print(f"[case] product {m}x{n} nrhs={nrhs}", flush=True)
    Q, B, X, run = solver(m, n, nrhs)
    run()
    torch.cuda.synchronize()
    assert np.abs(X.cpu().numpy() - Q.T @ B).max() <= 1e-15 * m * 64


def test_fewer_rows_take_no_longer():
    """1024 rows (no whole batch) against 4096 (two), 1024 right-hand sides."""
    t = {}
    for m in (1024, 4096):
        print(f"[case] time of {m} rows", flush=True)
        run = solver(m, 64, 1024)[3]
        run()
        best = np.inf
        for _ in range(5):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(5):
                run()
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
        t[m] = best / 5
    print(f"    {1e6 * t[1024]:.0f} us, {1e6 * t[4096]:.0f} us", flush=True)
    assert t[1024] <= 1.1 * t[4096]
