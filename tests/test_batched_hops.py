"""The exchange of the batched register tile at the edges of its rule (16 slices, 256 rows), and its step over many
slices, which must not be read by one thread a row."""
import pytest

import oracle
from paper_2203_10838_amd import inputs
from parity import alpha_star, check_iterate, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,eta,G", [(256, 40, 16), (272, 40, 17), (1024, 256, 16), (1024, 257, 16), (1088, 256, 17),
                                     (64, 5, 4), (15, 3, 1)])
def test_hops_match_the_oracle(cuda, rsk_lib, n, eta, G):
    from paper_2203_10838_amd import rsk
    m, K, lam = 2 * n + eta, 12, 0.2
    s = inputs.dense_system(m, n, max(1, n // 20), dtype="f32", seed=n + eta)
    idx = inputs.index_stream(inputs.row_sampling_weights(s["A"]), K, eta, 5)
    alpha = alpha_star(s["A"], eta)
    ld = n + (-n) % 4
    import torch
    A = torch.full((m, ld), float("nan"), device=cuda)
    A[:, :n] = to_dev(s["A"], cuda)
    sys_ = [rsk.BatchSystem(A=A[:, :n], b=to_dev(s["b"], cuda), index_stream=to_dev(idx, cuda), eta=eta, K=K,
                            alpha=alpha, lam=lam) for _ in range(3)]
    wg = eta * n * 4 // G
    assert rsk.plan_batched(sys_, wg_bytes=wg, kernel=2)["groups"] == [G] * 3
    res = rsk.solve_batched(sys_, wg_bytes=wg, kernel=2)
    ref = oracle.rska_dense(s["A"], s["b"], lam, eta, alpha, K, idx)
    for i in range(3):
        assert torch.equal(res.x_star[i], res.x_star[0])
        check_iterate(res.x_star[i], res.x[i], ref, lam, 1e-4, min_support=0)


def test_a_step_over_many_slices_costs_no_more_than_over_few(cuda, rsk_lib):
    """64 columns a slice, 32 rows a step: 256 slices took 27 us a step against 6 for 16 where each thread read
    all the slices' partials of its row; with two hops about as long."""
    import torch
    from paper_2203_10838_amd import rsk
    eta, K, per_step = 32, 60, {}
    for G in (16, 256):
        m, n = 600, 64 * G
        A = torch.randn(m, n, device=cuda)
        sys_ = [rsk.BatchSystem(A=A, b=torch.randn(m, device=cuda), eta=eta, K=K, alpha=1.0, lam=0.1,
                                index_stream=torch.randint(0, m, (K * eta,), dtype=torch.int32, device=cuda))]
        wg = eta * n * 4 // G
        assert rsk.plan_batched(sys_, wg_bytes=wg, kernel=2)["groups"] == [G]
        best = float("inf")
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(4):
                rsk.solve_batched(sys_, wg_bytes=wg, kernel=2, check=False)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) / (4 * K))
        per_step[G] = best
    assert per_step[256] <= 2.0 * per_step[16], per_step
