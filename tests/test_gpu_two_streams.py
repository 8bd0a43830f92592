"""The two-stream schedule where it is taken (an encoded matrix of at least 80 M
elements x panel width; panels updated in pairs from 160 MB on, 240 MB with odd
leading dimensions): against the one-stream plan on the same input and
failures, and with panels that break down beside it.

Matrices are Gaussian with at least 1.25 rows per column (condition number below
20).  Both plans' R are the unique factor of nearly the same matrix: with
residuals e and orthogonalities o their difference stays below cond (e0 + e1 +
o0 + o1), here at most 20 times that sum, which is asserted.  Decoding amplifies
the checksum drift of both alike, so residuals with failures, and all measures
with nearly dependent columns, are bounded by four times the one-stream plan's.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def factors(lookahead, A, m, n, pr, pc, K, kh, b, storage, sched):
    """(residual, |I - Q~^T Q~|, |I - Q_post^T Q_post|), R, fallbacks"""
    from paper_2311_11943_amd import cqr
    r = np.random.default_rng(7919)
    v = r.uniform(0, 1, (K, pr - K)) if K else None
    gh = r.uniform(0, 1, (pc, kh)) if kh else None
    q = cqr.CodedQR(cqr.Config(m, n, pr, pc, K, kh, b, storage, lookahead=lookahead), v, gh)
    Q, R, Qpost, _ = q.run(A, sched)
    torch.cuda.synchronize()
    assert q.info() == 0
    eye = torch.eye(n, dtype=torch.float64, device="cuda:0")
    out = [torch.linalg.norm(A - Q[:m, :n] @ R[:n, :n]) / torch.linalg.norm(A),
           torch.linalg.norm(eye - Q[:, :n].T.contiguous() @ Q[:, :n])]
    if K:
        out.append(torch.linalg.norm(eye - Qpost.T.contiguous() @ Qpost))
    fallbacks = q.panel_fallbacks()
    q.close()
    return [x.item() for x in out], R[:n, :n].clone(), fallbacks


def gaussian(m, n, seed=1):
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    return torch.randn(n, m, dtype=torch.float64, device="cuda:0", generator=g).t()


# m, n, pr, pc, K, K_h, b, storage, panels at which a node fails
SHAPES = [
    (1280, 1024, 8, 8, 2, 2, 64, 1, []),             # 64-column panels, even
    (1280, 1024, 8, 8, 2, 2, 64, 1, [3, 8]),
    (1525, 1200, 5, 5, 1, 1, 48, 0, [7]),            # early updates end in half tiles, near launches below one
    (1525, 1200, 5, 5, 1, 1, 40, 0, []),
    (4095, 1575, 7, 7, 3, 3, 35, 0, [11, 30]),       # odd leading dimension
    (2401, 1920, 1, 1, 0, 0, 60, 0, []),
    (26624, 416, 4, 1, 1, 0, 32, 0, [5]),            # tall: splits of the early update summed first
    (5120, 4096, 8, 8, 2, 2, 64, 1, [17, 40]),       # pairs; a call that ends inside one
    (6000, 4800, 5, 5, 1, 1, 48, 0, [33]),           # pairs of 48: N = 120 panels
    (6000, 4800, 5, 5, 1, 1, 60, 0, [14, 31]),       # 120 products in two sums, no LDS-staged kernel
    (5765, 4590, 5, 5, 2, 2, 51, 0, [7, 20, 43]),    # odd leading dimension, N = 126 panels
    (6307, 5040, 7, 7, 1, 1, 63, 0, [9]),
    (6307, 5040, 7, 7, 1, 1, 30, 0, [21]),           # pairs no deeper than a slab
]


@pytest.mark.parametrize("m,n,pr,pc,K,kh,b,storage,fails", SHAPES,
                         ids=[f"{c[0]}x{c[1]}_b{c[6]}_{len(c[8])}" for c in SHAPES])
def test_matches_one_stream(m, n, pr, pc, K, kh, b, storage, fails):
    print(f"[case] two streams {m}x{n} grid {pr}x{pc} b={b} failures at {fails}", flush=True)
    A = gaussian(m, n)
    sched = [(t, [(t % pr, t % pc)]) for t in fails]
    one, R1, _ = factors(0, A, m, n, pr, pc, K, kh, b, storage, sched)
    two, R2, _ = factors(1, A, m, n, pr, pc, K, kh, b, storage, sched)
    diff = (torch.linalg.norm(R1 - R2) / torch.linalg.norm(R1)).item()
    print(f"    one stream {one}\n    two        {two}\n    R {diff:.2e}", flush=True)
    assert one[0] <= 1e-11 and one[1] <= 1e-11
    assert two[0] <= max(1e-14, 4 * one[0]) and two[1] <= max(1e-12, 4 * one[1])
    assert diff <= 20 * (one[0] + two[0] + one[1] + two[1])


# m, n, pr, pc, K, K_h, b, storage, nearly dependent columns, panels at which a node fails
BREAKDOWNS = [
    (1024, 1024, 8, 8, 2, 2, 64, 1, (12, 37), []),           # first panel
    (1024, 1024, 8, 8, 2, 2, 64, 1, (140, 170), []),         # a panel with an early update
    (1024, 1024, 8, 8, 2, 2, 64, 1, (140, 170), [6]),
    (1024, 1024, 8, 8, 2, 2, 64, 1, (963, 990), []),         # last panel
    (1200, 1200, 5, 5, 1, 1, 48, 0, (97, 130), []),          # panels of three 16-column blocks
    (4096, 4096, 8, 8, 2, 2, 64, 1, (260, 300), []),         # first and second panel of a pair
    (4096, 4096, 8, 8, 2, 2, 64, 1, (325, 380), []),
    (28672, 448, 4, 1, 1, 0, 64, 0, (130, 190), []),         # splits of the early update summed first
]


@pytest.mark.parametrize("m,n,pr,pc,K,kh,b,storage,cols,fails", BREAKDOWNS,
                         ids=[f"{c[0]}x{c[1]}_{c[8][0]}_{len(c[9])}" for c in BREAKDOWNS])
def test_breakdown(m, n, pr, pc, K, kh, b, storage, cols, fails):
    print(f"[case] breakdown beside the update {m}x{n} b={b} columns {cols} failures at {fails}", flush=True)
    A = gaussian(m, n, 5)
    A[:, cols[1]] = A[:, cols[0]] + 1e-9 * gaussian(m, 1, 6)[:, 0]
    sched = [(t, [(t % pr, t % pc)]) for t in fails]
    one, _, f1 = factors(0, A, m, n, pr, pc, K, kh, b, storage, sched)
    two, _, f2 = factors(1, A, m, n, pr, pc, K, kh, b, storage, sched)
    print(f"    one stream {one} fallbacks {f1}\n    two        {two} fallbacks {f2}", flush=True)
    assert f1 >= 1 and f2 >= 1
    assert two[0] <= max(1e-12, 4 * one[0])
    for x, y in zip(one[1:], two[1:]):
        assert y <= max(1e-12, 4 * x)
