"""The column-wise panel kernels (CGS2, ICGS, MGS) at the edges of their shapes:
leaf widths around the 16 columns a wave holds, row counts around the 64-row
blocks and the steps in the number of workgroups.

Against the oracle's column-by-column panel on the same matrix.  For these
Gaussian inputs (m >= 2 n) the condition number stays below 10, so Q and R agree
to about 10 n u times the columns' norm ratio; 1e-11 relative is asserted, and
1e-12 for ||I - Q~^T Q~||_F with CGS2 and ICGS.
"""
import numpy as np
import pytest

from oracle import coded_qr as oc
from tests.gpu_helpers import gpu_config, host, make_inputs, oracle_state, rel

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MODES = [(1, "cgs2"), (2, "icgs"), (3, "mgs")]


@pytest.mark.parametrize("mode,name", MODES, ids=[m[1] for m in MODES])
@pytest.mark.parametrize("m,n,b", [(32, 4, 1), (40, 8, 2), (64, 16, 16), (132, 60, 15), (256, 68, 17), (260, 128, 64),
                                   (1024, 96, 48), (1700, 64, 32), (3300, 132, 33), (14000, 32, 16)])
def test_column_panels(m, n, b, mode, name):
    from paper_2311_11943_amd import cqr
    print(f"[case] {name} m={m} n={n} b={b}", flush=True)
    A, v, gh, lay = make_inputs(n, 4, 1, b, "out", seed=9, m=m)
    q = cqr.CodedQR(gpu_config(cqr, lay, b, panel=mode), v, gh)
    At, R = q.alloc()
    At[:m, :n].copy_(cqr.to_device_colmajor(A, "cuda:0"))
    q.encode(At)
    q.factor(At, R)
    info = q.info()
    q.close()
    _, Qo, Ro, _, _ = oracle_state(A, v, gh, lay, b, n // b, panel=name)
    Q, Rg = host(At)[:, :n], host(R)[:n]
    eq, er = rel(Q, Qo[:, :n]), rel(Rg, Ro)
    orth = np.linalg.norm(np.eye(n) - Q.T @ Q)
    print(f"    Q {eq:.2e} R {er:.2e} orth {orth:.2e}", flush=True)
    assert info == 0
    assert eq <= 1e-11 and er <= 1e-11
    assert not np.tril(Rg[:, :n], -1).any()
    assert orth <= 1e-12 or name == "mgs"
