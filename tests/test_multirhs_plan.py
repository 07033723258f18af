"""The built-in kernel and column splits of the multi-RHS products: for R <= 64 the wide tiles only where the 64 x 64 ones,
in splits of 128 columns, are more than two rounds on the CUs; wide tiles in whole XCD rounds where that is free; and the
results at a shape on each side."""
import pytest

import oracle
from paper_2203_10838_amd import inputs
from parity import alpha_star, check_columns, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,eta,R,kernel,S", [
    (4096, 820, 64, 1, None), (6000, 601, 64, 1, None), (32768, 128, 64, 1, None), (32768, 128, 16, 1, None),
    (8192, 820, 64, 3, 32), (20000, 200, 64, 3, None), (32768, 129, 64, 3, None),
    (8192, 820, 256, 3, 16), (4096, 410, 192, 3, 16), (6000, 601, 192, 3, 16), (16384, 820, 128, 3, 32),
    (12000, 820, 256, 3, 18), (32768, 820, 256, 3, 18),  # 16 splits would be longer than 18 by a pair of stages or more
    (8192, 127, 256, 1, None), (1000, 128, 68, 3, 8),
])
def test_built_in_plan(cuda, rsk_lib, n, eta, R, kernel, S):
    import torch
    from paper_2203_10838_amd import rsk
    plan = rsk.plan_multirhs(torch.empty(2 * eta, n, device=cuda), R, eta=eta)
    assert plan["kernel"] == kernel and (S is None or plan["S"] == S), plan


@pytest.mark.parametrize("m,n,R,eta,kernel", [(400, 2048, 64, 130, 1), (1700, 2052, 192, 700, 3), (900, 4100, 64, 1100, 3)])
def test_both_sides_match_the_oracle(cuda, rsk_lib, m, n, R, eta, kernel):
    from paper_2203_10838_amd import rsk
    K, lam = 4, 0.05
    s = inputs.multirhs_system(m, n, R, max(1, n // 20), seed=n)
    A = to_dev(s["A"], cuda)
    assert rsk.plan_multirhs(A, R, eta=eta)["kernel"] == kernel
    idx = inputs.index_stream(inputs.row_sampling_weights(s["A"]), K, eta, 3)
    alpha = alpha_star(s["A"], eta)
    res = rsk.solve_multirhs(A, to_dev(s["B"], cuda), lam=lam, eta=eta, alpha=alpha, K=K, index_stream=to_dev(idx, cuda))
    ref = oracle.rska_multirhs(s["A"], s["B"], lam, eta, alpha, K, idx)
    check_columns(res.x_star, res.x, ref, lam, 1e-4)
