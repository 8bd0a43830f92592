"""Erasure and recovery at the edges of their launches' argument sizes (1 and 4
lines, 32 and 256 coefficients; 16, 64 and 256 erased blocks) and of the way
threads run down a block's columns (blocks of one row, of odd height, of fewer
and of more elements than a workgroup).

A recovered block is G_hat^{-1} applied to sums of at most 32 terms; with
condition at most 1e5 of the erased submatrices (checked) its error stays below
32 u 1e5 max|.| < 1e-9.
"""
import numpy as np
import pytest

from tests.gpu_helpers import host, make_inputs, gpu_config
from oracle import coded_qr as oc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def column(rows, j):
    return [(i, j) for i in rows]


# n, m, grid, K, lost nodes (out-of-node storage)
RECOVER = [
    (4, 4, 4, 1, [(2, 1)]),                                        # one element a block
    (24, 40, 8, 2, [(5, 5)]),                                      # one line of 8 coefficients
    (120, 200, 8, 2, column((0, 3), 2)),                           # one of 16 in Q, two of 8 in R
    (16 * 9, 16 * 33, 16, 2, column((4, 9), 1)),                   # 32 coefficients
    (17 * 5, 17 * 31, 17, 2, column((4, 9), 1)),                   # 34
    (8 * 21, 8 * 21, 8, 2, [(0, 0), (1, 1), (2, 2), (3, 3)]),      # four lines
    (8 * 21, 8 * 21, 8, 2, [(0, 0), (1, 1), (2, 2), (3, 3), (4, 4)]),
    (24 * 3, 24 * 5, 24, 8, column(range(0, 24, 3), 7) + column((1, 5), 9)),       # 240 coefficients
    (24 * 3, 24 * 5, 24, 8, column(range(0, 24, 3), 7) + column((1, 5, 8), 9)),    # 264
]


@pytest.mark.parametrize("n,m,p,K,nodes", RECOVER, ids=[f"{c[1]}x{c[0]}_{c[2]}_{len(c[4])}" for c in RECOVER])
def test_recover(n, m, p, K, nodes):
    from paper_2311_11943_amd import cqr
    print(f"[case] recover n={n} m={m} {p}x{p} K={K} {nodes}", flush=True)
    A, v, gh, lay = make_inputs(n, p, K, p, "out", seed=11, m=m)
    gv, ghm = oc.q_generator(v), oc.r_generator(gh, lay.storage)
    lost = {j: sorted(i for i, jj in nodes if jj == j) for _, j in nodes}
    cond = max([np.linalg.cond(gv[:len(r)][:, r]) for r in lost.values()])
    assert cond <= 1e5
    q = cqr.CodedQR(gpu_config(cqr, lay, 1), v, gh)
    At, R = q.alloc()
    At.copy_(cqr.to_device_colmajor(oc.encode(A, gv, ghm, lay), "cuda:0"))
    Rh = np.random.default_rng(1).standard_normal((n, n))
    R.copy_(cqr.to_device_colmajor(np.hstack([Rh, Rh @ np.kron(ghm, np.eye(n // p))]), "cuda:0"))
    Q0, R0 = host(At), host(R)
    q.erase(At, R, nodes)
    Qe, Re = Q0.copy(), R0.copy()
    oc.erase(Qe, Re, nodes, lay)
    assert np.array_equal(host(At), Qe, equal_nan=True) and np.array_equal(host(R), Re, equal_nan=True)
    q.recover(At, R, nodes)
    torch.cuda.synchronize()
    q.close()
    keep = ~np.isnan(Qe)
    assert np.array_equal(host(At)[keep], Q0[keep])
    dq, dr = np.abs(host(At) - Q0).max() / np.abs(Q0).max(), np.abs(host(R) - R0).max() / np.abs(R0).max()
    print(f"    restored Q {dq:.2e} R {dr:.2e}", flush=True)
    assert dq <= 1e-9 and dr <= 1e-9


@pytest.mark.parametrize("blocks", [1, 16, 17, 64, 65, 256, 257])
@pytest.mark.parametrize("h,w", [(1, 3), (33, 7), (64, 2), (258, 3)])
def test_erase(blocks, h, w):
    from paper_2311_11943_amd import cqr
    print(f"[case] erase {blocks} blocks of {h}x{w}", flush=True)
    p = 17
    n, m = p * w, p * max(h, w)
    A, v, gh, lay = make_inputs(n, p, 1, p, "out", seed=3, m=m)
    q = cqr.CodedQR(gpu_config(cqr, lay, 1), v, gh)
    At, R = q.alloc()
    At.fill_(1.0)
    R.fill_(2.0)
    every = [(i, j) for j in range(p) for i in range(p)]
    nodes = [every[k] for k in np.random.default_rng(blocks).permutation(len(every))[:blocks]]
    q.erase(At, R, nodes)
    torch.cuda.synchronize()
    q.close()
    Qe, Re = np.full(At.shape, 1.0), np.full(R.shape, 2.0)
    oc.erase(Qe, Re, nodes, lay)
    assert np.array_equal(host(At), Qe, equal_nan=True) and np.array_equal(host(R), Re, equal_nan=True)
