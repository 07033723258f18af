"""The general kernel's exchange and column sums over its grids: one row a wave or several, slices of one
chunk to more than a wave's, 1 to 256 workgroups; float64 against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2203_10838_amd import inputs
from parity import alpha_star, check_iterate, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,eta,grid", [
    (600, 40, 256), (600, 40, 65), (600, 300, 64), (600, 300, 2),   # one row a wave; several; G around 64
    (520, 257, 129), (515, 9, 200), (8, 70, 4),                     # odd rows (single elements), one chunk a slice
    (1000, 33, 31), (2048, 20, 5), (2050, 12, 2),                   # slices around 64 chunks and above 256
])
def test_general_kernel_over_its_grids(cuda, rsk_lib, n, eta, grid):
    from paper_2203_10838_amd import rsk
    K, lam = 8, 0.05
    m = max(2 * eta, 700)
    s = inputs.dense_system(m, n, max(1, n // 20), dtype="f64", seed=n + eta)
    idx = inputs.index_stream(inputs.row_sampling_weights(s["A"]), K, eta, grid)
    alpha = alpha_star(s["A"], eta)
    r = rsk.solve_dense(to_dev(s["A"], cuda), to_dev(s["b"], cuda), lam=lam, eta=eta, alpha=alpha, K=K,
                        index_stream=to_dev(idx, cuda), kernel=1, grid=grid)
    assert r.status == 0 and r.k_done == K
    ref = oracle.rska_dense(s["A"], s["b"], lam, eta, alpha, K, idx)
    check_iterate(r.x_star, r.x, ref, lam, 1e-10, min_support=0)


def test_default_grid_of_large_float64_steps(cuda, rsk_lib):
    import torch
    from paper_2203_10838_amd import rsk
    A = torch.zeros((300, 6000), device=cuda, dtype=torch.float64)
    got = [rsk.plan_dense(A, eta=eta)["G"] for eta in (64, 65, 66, 170, 180)]
    assert got == [128, 128, 192, 192, 256], got
