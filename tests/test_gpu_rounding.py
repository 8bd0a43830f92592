"""How far the widths that a plan chooses let rounding grow.  A plan with
lookahead factors columns in widths of its own (leaves in pairs, or 512 at
once); one without factors b columns at a time.  On the same input and failures
the first may leave no more in A~ - Q~ R and in the post-orthogonalized basis
than the second: both measures sum the rounding of over 10^6 independent
updates, which vary by a few per cent between two orders, whereas sums twice as
deep raise their squares by a third or more.  The bound, 10%, lies between.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# m, n, grid, K, storage (1: in-node), b, failures a grid row and event, events
@pytest.mark.parametrize("m,n,p,K,storage,b,lost,events", [
    (4096, 4096, 16, 8, 1, 64, 4, 2),       # pairs of leaves
    (8192, 8192, 16, 8, 1, 256, 4, 3),      # 512 columns at once
    (8192, 8192, 16, 8, 1, 128, 4, 3),
    (49152, 4096, 8, 2, 0, 128, 2, 3),      # the coefficients' sums over many rows
    (20480, 5120, 8, 2, 0, 64, 2, 3),
], ids=["pairs_4096", "wide_8192_b256", "wide_8192_b128", "wide_49152x4096", "wide_20480x5120_b64"])
def test_rounding_of_the_chosen_width(m, n, p, K, storage, b, lost, events):
    from paper_2311_11943_amd import cqr
    print(f"[case] rounding {m}x{n} b={b}", flush=True)
    r = np.random.default_rng(7919)
    v, gh = r.uniform(0, 1, (K, p - K)), r.uniform(0, 1, (p, K))
    g = torch.Generator(device="cuda:0").manual_seed(1)
    A = torch.randn(n, m, dtype=torch.float64, device="cuda:0", generator=g).t()
    nodes = [(i, (p - 1 - i - k) % p) for i in range(p) for k in range(lost)]
    sched = [(n // b * (e + 1) // (events + 1), nodes) for e in range(events)]
    eye = torch.eye(n, dtype=torch.float64, device="cuda:0")
    out = {}
    for la in (0, 1):
        q = cqr.CodedQR(cqr.Config(m, n, p, p, K, K, b, storage, lookahead=la), v, gh)
        Qpost = q.run(A)[2]
        post = torch.linalg.norm(eye - Qpost.T @ Qpost).item()
        del Qpost
        Q, R, _, _ = q.run(A, sched)
        D = A.clone()
        for c in range(0, n, 256):
            D -= Q[:m, c:c + 256] @ R[c:c + 256, :n]
        out[la] = ((torch.linalg.norm(D) / torch.linalg.norm(A)).item(), post)
        assert q.info() == 0
        q.close()
        del Q, R, D
    print(f"    residual {out[0][0]:.3e} {out[1][0]:.3e}  post-orthogonalized {out[0][1]:.3e} {out[1][1]:.3e}", flush=True)
    assert out[1][0] <= 1.1 * out[0][0] and out[1][1] <= 1.1 * out[0][1]
