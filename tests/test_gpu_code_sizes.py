"""Encoding, erasure and recovery at the edges of their kernels' shapes: blocks
shorter than a wavefront, odd heights (one row a thread) and even ones (two),
grids on either side of the encoding's 8, 16 and 32 block columns, and failure
patterns whose lines take one launch or several.

The encoded matrix is compared with the oracle's: sums of at most p terms, and
sums of those, so |difference| <= 2 p^2 u max|g|^2 max|A| < 1e-12 here.  A
recovered block is G_hat^{-1} applied to sums of p terms; with the condition of
these generators' erased submatrices (checked below 1e4) its error stays below
p u 1e4 max|.| < 1e-9.
"""
import numpy as np
import pytest

import synth
from oracle import coded_qr as oc
from tests.gpu_helpers import gpu_config, host, make_inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# m, n, pr, pc, K, storage, failed nodes
CASES = [
    (20, 20, 4, 4, 1, "out", [(1, 2)]),
    (60, 60, 4, 4, 2, "out", [(0, 1), (2, 1), (0, 3)]),
    (135, 105, 5, 7, 2, "out", [(4, 6), (1, 0)]),
    (128, 64, 8, 8, 2, "in", [(3, 3), (6, 1)]),
    (272, 272, 16, 16, 4, "out", synth.reverse_diagonal(16, 4)),
    (544, 544, 17, 17, 2, "out", synth.reverse_diagonal(17, 2)),
    (690, 690, 23, 23, 3, "out", synth.reverse_diagonal(23, 3)),
    (1152, 576, 9, 9, 4, "in", synth.reverse_diagonal(9, 1)),
    (2080, 1040, 16, 16, 8, "in", synth.reverse_diagonal(16, 4)),
]


@pytest.mark.parametrize("m,n,pr,pc,K,storage,nodes", CASES, ids=[f"{c[0]}x{c[1]}_{c[2]}x{c[3]}_{c[5]}" for c in CASES])
def test_encode_erase_recover(m, n, pr, pc, K, storage, nodes):
    from paper_2311_11943_amd import cqr
    print(f"[case] code m={m} n={n} grid {pr}x{pc} K={K} {storage}", flush=True)
    A, v, gh, lay = make_inputs(n, pr, K, pr, storage, seed=5, m=m, pc=pc)
    b = next(w for w in (8, 7, 6, 5, 4, 3, 2, 1) if n % w == 0)
    gv, ghm = oc.q_generator(v), oc.r_generator(gh, lay.storage)
    q = cqr.CodedQR(gpu_config(cqr, lay, b), v, gh)
    At, R = q.alloc()
    At[:m, :n].copy_(cqr.to_device_colmajor(A, "cuda:0"))
    q.encode(At)
    ref = oc.encode(A, gv, ghm, lay)
    scale = max(np.abs(gv).max(), 1) * max(np.abs(ghm).max(), 1) * np.abs(A).max() * pr * pc
    assert np.abs(host(At) - ref).max() <= 1e-14 * scale
    Rh = np.random.default_rng(1).standard_normal((n, n))
    Rh = np.hstack([Rh, np.kron(np.ones((1, 1)), Rh) @ np.kron(ghm, np.eye(n // pc))])
    R.copy_(cqr.to_device_colmajor(Rh, "cuda:0"))
    Q0, R0 = host(At), host(R)
    q.erase(At, R, nodes)
    Qe, Re = Q0.copy(), R0.copy()
    oc.erase(Qe, Re, nodes, lay)
    assert np.array_equal(np.isnan(host(At)), np.isnan(Qe)) and np.array_equal(np.isnan(host(R)), np.isnan(Re))
    q.recover(At, R, nodes)
    torch.cuda.synchronize()
    q.close()
    dq, dr = np.abs(host(At) - Q0).max() / np.abs(Q0).max(), np.abs(host(R) - R0).max() / np.abs(R0).max()
    print(f"    restored Q {dq:.2e} R {dr:.2e}", flush=True)
    assert dq <= 1e-9 and dr <= 1e-9
