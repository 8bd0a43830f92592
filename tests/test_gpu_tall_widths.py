"""Many rows and few columns: a plan's own widths and streams (lookahead) take no
longer than panels of b on one stream.
"""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("m,n", [(1600000, 192), (1600000, 128), (400000, 448)])
def test_own_widths_take_no_longer(m, n):
    from paper_2311_11943_amd import cqr
    print(f"[case] time {m}x{n}", flush=True)
    A = torch.randn(n, m, dtype=torch.float64, device="cuda:0").t()
    best = {}
    for lookahead in (0, 1):
        q = cqr.CodedQR(cqr.Config(m, n, 1, 1, 0, 0, 64, lookahead=lookahead))
        best[lookahead] = np.inf
        for _ in range(6):
            torch.cuda.synchronize()
            t = time.perf_counter()
            q.run(A)
            torch.cuda.synchronize()
            best[lookahead] = min(best[lookahead], time.perf_counter() - t)
        q.close()
    print(f"    one stream {1e3 * best[0]:.2f} ms, two {1e3 * best[1]:.2f} ms", flush=True)
    assert best[1] <= 1.1 * best[0]
