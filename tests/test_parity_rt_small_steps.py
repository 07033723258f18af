"""Register tile on small steps, against the oracle: rows per wave on both sides of one, one and two
exchange hops, and grids rounded down to a power of two."""
import numpy as np
import pytest

import oracle
from paper_2203_10838_amd import inputs
from parity import alpha_star, check_iterate

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,eta,G,hops", [
    (200, 64, 16, 4, 1), (200, 64, 17, 4, 2), (200, 64, 64, 4, 2), (300, 64, 256, 4, 2),
    (200, 508, 16, 32, 1), (200, 512, 33, 32, 2), (300, 1000, 16, 32, 1), (400, 1020, 200, 64, 2),
    (300, 1500, 16, 64, 1), (300, 3332, 4, 209, 1), (300, 3332, 8, 209, 2), (300, 3332, 16, 128, 2), (500, 4092, 300, 256, 2),
])
@pytest.mark.parametrize("weights", [False, True])
def test_small_steps_match_the_oracle(cuda, rsk_lib, m, n, eta, G, hops, weights):
    import torch
    from paper_2203_10838_amd import rsk
    K, lam = 30, 0.02
    s = inputs.dense_system(m, n, max(1, n // 20), dtype="f32", seed=n + eta, noise_rel=0.01)
    idx = inputs.index_stream(inputs.row_sampling_weights(s["A"]), K, eta, eta)
    A, b, it = (torch.from_numpy(v).to(cuda) for v in (s["A"], s["b"], idx))
    plan = rsk.plan_dense(A, eta=eta)
    assert (plan["kernel"], plan["G"], plan["hops"]) == (2, G, hops), plan
    w = inputs.row_weights(m, 3) if weights else None
    alpha = alpha_star(s["A"], eta)
    res = rsk.solve_dense(A, b, lam=lam, eta=eta, alpha=alpha, K=K, index_stream=it,
                          row_w=None if w is None else torch.from_numpy(w).to(cuda))
    assert res.status == 0 and res.k_done == K
    ref = oracle.rska_dense(s["A"], s["b"], lam, eta, alpha, K, idx, row_w=w)
    check_iterate(res.x_star, res.x, ref, lam, 1e-4)  # the float32 bar of the other parity tests


def test_small_step_faults(cuda, rsk_lib):
    """A zero row and an index out of range among the rows a wave fetches together."""
    import torch
    from paper_2203_10838_amd import rsk
    m, n, eta, K = 200, 64, 64, 20
    s = inputs.dense_system(m, n, 5, dtype="f32", seed=1)
    A = torch.from_numpy(s["A"]).to(cuda)
    b = torch.from_numpy(s["b"]).to(cuda)
    idx = torch.randint(0, m - 1, (K * eta,), dtype=torch.int32, device=cuda)
    bad = idx.clone()
    bad[7 * eta + 50] = m
    zero = idx.clone()
    zero[3 * eta + 49] = m - 1
    Az = A.clone()
    Az[m - 1] = 0
    for M, ix, name, step in ((A, bad, "RSK_ERR_INDEX_RANGE", 7), (Az, zero, "RSK_ERR_ZERO_ROW", 3)):
        r = rsk.solve_dense(M, b, lam=0.1, eta=eta, alpha=1.0, K=K, index_stream=ix, check=False)
        code, done = r.status_dev.tolist()
        assert rsk._abi.STATUS_NAMES[code] == name and done == step
