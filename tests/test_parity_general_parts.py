"""The column sums of the general kernel at the edge of their two forms: up to eight parts of a slice added one after
another, more of them by several lanes; float64 against the oracle, one workgroup and a batch."""
import pytest

import oracle
from paper_2203_10838_amd import inputs
from parity import alpha_star, check_iterate, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,parts", [(512, 1), (258, 1), (256, 2), (64, 8), (56, 9), (30, 17), (32, 16), (2, 256)])
def test_parts_of_a_slice(cuda, rsk_lib, n, parts):
    from paper_2203_10838_amd import rsk
    assert 256 // (n // 2) == parts  # threads of a workgroup over chunks of two columns
    K, lam, eta, m = 8, 0.05, 40, 700
    s = inputs.dense_system(m, n, max(1, n // 20), dtype="f64", seed=n)
    idx = inputs.index_stream(inputs.row_sampling_weights(s["A"]), K, eta, n)
    alpha = alpha_star(s["A"], eta)
    A, b, ix = to_dev(s["A"], cuda), to_dev(s["b"], cuda), to_dev(idx, cuda)
    ref = oracle.rska_dense(s["A"], s["b"], lam, eta, alpha, K, idx)
    r = rsk.solve_dense(A, b, lam=lam, eta=eta, alpha=alpha, K=K, index_stream=ix, kernel=1, grid=1)
    check_iterate(r.x_star, r.x, ref, lam, 1e-10, min_support=0)
    rb = rsk.solve_batched([rsk.BatchSystem(A=A, b=b, index_stream=ix, eta=eta, K=K, alpha=alpha, lam=lam)],
                           wg_bytes=1 << 20)
    check_iterate(rb.x_star[0], rb.x[0], ref, lam, 1e-10, min_support=0)
