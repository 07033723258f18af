"""The wide-tile products (float32 by three bfloat16 pieces): edges of their tiles and stages, and their
accuracy against float64 beside the float32 matrix cores'."""
import numpy as np
import pytest

import oracle
from paper_2203_10838_amd import inputs
from parity import alpha_star, check_columns, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,R,eta", [
    (40, 4, 4, 1), (60, 28, 8, 31), (60, 32, 64, 32), (80, 36, 68, 33),   # stages of 32 columns and rows
    (300, 132, 132, 127), (300, 260, 60, 129), (700, 516, 124, 257),      # tiles of 128, both R edges
    (900, 1160, 256, 300),                                                # several column splits
])
def test_wide_products_match_the_oracle(cuda, rsk_lib, m, n, R, eta):
    import torch
    from paper_2203_10838_amd import rsk
    K, lam = 6, 0.05
    s = inputs.multirhs_system(m, n, R, max(1, n // 8), seed=m + n)
    idx = inputs.index_stream(inputs.row_sampling_weights(s["A"]), K, eta, 3)
    alpha = alpha_star(s["A"], eta)
    full = torch.full((m + 1, n + 4), float("nan"), device=cuda)  # the padding of the rows is never used
    full[:m, :n] = to_dev(s["A"], cuda)
    res = rsk.solve_multirhs(full[:m, :n], to_dev(s["B"], cuda), lam=lam, eta=eta, alpha=alpha, K=K,
                             index_stream=to_dev(idx, cuda), kernel=3)
    assert res.status == 0 and res.k_done == K
    ref = oracle.rska_multirhs(s["A"], s["B"], lam, eta, alpha, K, idx)
    check_columns(res.x_star, res.x, ref, lam, 1e-4)  # the float32 bar of the other multi-RHS tests


@pytest.mark.parametrize("scale", [1e-12, 1.0, 1e12])
@pytest.mark.parametrize("kind", ["normal", "positive", "wide"])
def test_split_products_are_as_accurate_as_float32(cuda, rsk_lib, kind, scale):
    """One step from zero and one more: the error of x* against float64 is no larger than that of the
    float32 products (kernel 1), over entries of one sign, of both, and of very different sizes."""
    import torch
    from paper_2203_10838_amd import rsk
    m, n, R, eta, K = 600, 1024, 128, 256, 2
    g = np.random.default_rng(5)
    A = g.standard_normal((m, n))
    if kind == "positive":
        A = np.abs(A)
    if kind == "wide":
        A *= 2.0 ** g.integers(-12, 13, size=(m, n))
    A = (A * scale).astype(np.float32)
    B = (A.astype(np.float64) @ g.standard_normal((n, R))).astype(np.float32)
    idx = g.integers(0, m, K * eta).astype(np.int32)
    ref = oracle.rska_multirhs(A, B, 0.0, eta, 1.0, K, idx)["z"]
    err = {}
    for kernel in (1, 3):
        r = rsk.solve_multirhs(to_dev(A, cuda), to_dev(B, cuda), lam=0.0, eta=eta, alpha=1.0, K=K,
                               index_stream=to_dev(idx, cuda), kernel=kernel)
        err[kernel] = np.linalg.norm(r.x_star.double().cpu().numpy() - ref) / np.linalg.norm(ref)
    # "no larger" up to the spread of two roundings of the same sums
    assert err[3] <= 1.25 * err[1] + 2.0 ** -24, err


def test_a_nonfinite_row_is_reported(cuda, rsk_lib):
    import torch
    from paper_2203_10838_amd import rsk
    m, n, R, eta, K = 300, 256, 128, 130, 4
    s = inputs.multirhs_system(m, n, R, 20, seed=2)
    idx = inputs.index_stream(np.ones(m - 1), K, eta, 3)
    idx[2 * eta + 129] = m - 1
    for bad in (np.inf, np.nan):
        A = to_dev(s["A"], cuda)
        r2 = rsk.rownorm2(A)
        A[m - 1, 100] = bad
        r = rsk.solve_multirhs(A, to_dev(s["B"], cuda), lam=0.1, eta=eta, alpha=1.0, K=K, rownorm2_t=r2,
                               index_stream=to_dev(idx, cuda), kernel=3, check=False)
        code, done = r.status_dev.tolist()
        assert rsk._abi.STATUS_NAMES[code] == "RSK_ERR_NONFINITE" and done == 2
        assert torch.isfinite(r.x_star).all()
