"""The one-workgroup kernel's row sums: every tile shape (1, 2, 4 and 8 columns a thread) with rows that do and
do not fill its folds of four, against the oracle."""
import pytest

import oracle
from paper_2203_10838_amd import inputs
from parity import alpha_star, check_iterate, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,tol", [("f64", 1e-10), ("f32", 1e-4)])
@pytest.mark.parametrize("n", [3, 256, 257, 513, 1500])
def test_row_sums_of_the_one_workgroup_kernel(cuda, rsk_lib, dtype, tol, n):
    from paper_2203_10838_amd import rsk
    K, lam, m = 9, 0.05, 400
    most = 32 if n <= 256 else 16 if n <= 512 else 8 if n <= 1024 else 4
    s = inputs.dense_system(m, n, max(1, n // 20), dtype=dtype, seed=n)
    for eta in sorted({1, 2, 3, most // 2 + 1, most - 1, most}):
        idx = inputs.index_stream(inputs.row_sampling_weights(s["A"]), K, eta, eta)
        alpha = alpha_star(s["A"], eta)
        r = rsk.solve_dense(to_dev(s["A"], cuda), to_dev(s["b"], cuda), lam=lam, eta=eta, alpha=alpha, K=K,
                            index_stream=to_dev(idx, cuda), kernel=4)
        assert r.status == 0 and r.k_done == K
        ref = oracle.rska_dense(s["A"], s["b"], lam, eta, alpha, K, idx)
        check_iterate(r.x_star, r.x, ref, lam, tol, min_support=0, what=f"eta {eta}")
