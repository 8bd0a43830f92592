"""Buffers that the library writes whole come unfilled: with torch filling every
unfilled tensor with NaN, run() and the autograd functions give the bits they
give without, over grids with and without each checksum."""
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = [
    # m, n, b, pr, pc, kv, kh, nodes lost after one panel
    (96, 64, 16, 4, 4, 1, 1, [(1, 1)]),
    (105, 45, 3, 5, 3, 2, 0, [(4, 2)]),
    (64, 64, 16, 2, 4, 0, 2, []),
    (80, 40, 10, 1, 1, 0, 0, []),
]


@pytest.fixture
def nan_filled():
    kept = torch.are_deterministic_algorithms_enabled(), torch.utils.deterministic.fill_uninitialized_memory
    yield
    torch.use_deterministic_algorithms(kept[0])
    torch.utils.deterministic.fill_uninitialized_memory = kept[1]


@pytest.mark.parametrize("m,n,b,pr,pc,kv,kh,nodes", CASES)
def test_bits_with_nan_in_unfilled(nan_filled, m, n, b, pr, pc, kv, kh, nodes):
    from paper_2311_11943_amd import autograd, cqr
    print(f"[case] unfilled {m}x{n} grid {pr}x{pc} checksums {kv},{kh}", flush=True)
    q = cqr.CodedQR(cqr.Config(m, n, pr, pc, kv, kh, b),
                    synth.q_generator_draws(kv, pr, 0), synth.r_generator_draws(pc, kh, 0))
    torch.manual_seed(m)
    A = torch.randn(m, n, dtype=torch.float64, device="cuda")
    B = torch.randn(2, m, dtype=torch.float64, device="cuda").t()
    W = torch.randn(n, 2, dtype=torch.float64, device="cuda")
    schedule = [(1, nodes)] if nodes else []

    def once(fill):
        torch.use_deterministic_algorithms(fill, warn_only=True)
        torch.utils.deterministic.fill_uninitialized_memory = fill
        out = [t for t in q.run(A, schedule, B) if t is not None]
        if kv > 0:
            a, x = A.clone().requires_grad_(), B.clone().requires_grad_()
            Q, R1 = autograd.coded_qr(a, q, schedule)
            (autograd.coded_solve(Q, R1, x, q) * W).sum().backward()
            out += [a.grad, x.grad]
        torch.cuda.synchronize()
        return out

    want, got = once(False), once(True)
    q.close()
    assert len(want) == len(got)
    for u, v in zip(want, got):
        assert torch.equal(u, v) and torch.isfinite(v).all()
