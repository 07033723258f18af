"""The built-in column splits of the multi-RHS products: at least 128 columns a split while the tiles of all
splits fit one round on the CUs, never fewer splits than at 256 columns; and the results at such splits."""
import pytest

import oracle
from paper_2203_10838_amd import inputs
from parity import alpha_star, check_columns, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,R,eta", [(300, 128, 8, 13), (300, 132, 64, 14), (500, 260, 4, 70), (900, 1000, 60, 101)])
def test_short_splits_match_the_oracle(cuda, rsk_lib, m, n, R, eta):
    from paper_2203_10838_amd import rsk
    K, lam = 6, 0.05
    s = inputs.multirhs_system(m, n, R, max(1, n // 20), seed=n)
    A = to_dev(s["A"], cuda)
    plan = rsk.plan_multirhs(A, R, eta=eta)
    assert plan["kernel"] == 1 and -(-n // 256) <= plan["S"] <= -(-n // 112) and plan["kspan"] % 16 == 0
    idx = inputs.index_stream(inputs.row_sampling_weights(s["A"]), K, eta, 3)
    alpha = alpha_star(s["A"], eta)
    res = rsk.solve_multirhs(A, to_dev(s["B"], cuda), lam=lam, eta=eta, alpha=alpha, K=K,
                             index_stream=to_dev(idx, cuda))
    assert res.status == 0 and res.k_done == K
    ref = oracle.rska_multirhs(s["A"], s["B"], lam, eta, alpha, K, idx)
    check_columns(res.x_star, res.x, ref, lam, 1e-4)
