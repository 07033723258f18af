"""The two products of a wide multi-RHS step, seen alone and element by element, over short sums.

With row norms of one, alpha = eta and lambda = 0 a step is C = A_tau X - B_tau, X* -= A_tau^T C. Columns of A that
hold a unit matrix over the sampled rows, where X is zero, show C itself in X*; B alone (X = 0) shows A^T B.
"""
import numpy as np
import pytest

from parity import to_dev

pytestmark = pytest.mark.gpu

# a = b = this leaves most outside the first two bfloat16 pieces of a truncating split
WORST = np.float32(1 + 2.0 ** -7 - 2.0 ** -15 + 2.0 ** -16 - 2.0 ** -23)


def _entries(g, shape, kind):
    if kind == "worst":
        return (WORST * g.choice([-1.0, 1.0], size=shape)).astype(np.float32)
    v = g.standard_normal(shape)
    if kind == "small":  # products of 2^-60 and, of small mantissas, less: all their terms are normal numbers
        v *= 2.0 ** -30
    return v.astype(np.float32)


def _sparse(g, rows, R, nnz, kind):
    x = np.zeros((rows, R), dtype=np.float32)
    for r in range(R):
        x[g.choice(rows, nnz, replace=False), r] = _entries(g, nnz, kind)
    return x


def _error(cuda, kernel, which, A, S, eta):
    """max and rms over the elements of |product - float64| / (sum of the terms' sizes)"""
    import torch
    from paper_2203_10838_amd import rsk
    A64, S64 = A.astype(np.float64), S.astype(np.float64)
    R = S.shape[1]
    kw = dict(lam=0.0, eta=eta, alpha=float(eta), K=1, kernel=kernel,
              index_stream=torch.arange(eta, dtype=torch.int32, device=cuda),
              rownorm2_t=torch.ones(eta, device=cuda))
    if which == "A X":
        full = np.concatenate([A, np.eye(eta, dtype=np.float32)], axis=1)
        X0 = np.concatenate([S, np.zeros((eta, R), np.float32)])
        r = rsk.solve_multirhs(to_dev(full, cuda), torch.zeros(eta, R, device=cuda), X_star=to_dev(X0, cuda),
                               warm_start=True, **kw)
        got, want, size = -r.x_star[A.shape[1]:].double().cpu().numpy(), A64 @ S64, np.abs(A64) @ np.abs(S64)
    else:
        r = rsk.solve_multirhs(to_dev(A, cuda), to_dev(S, cuda), **kw)
        got, want, size = r.x_star.double().cpu().numpy(), A64.T @ S64, np.abs(A64).T @ np.abs(S64)
    e = np.abs(got - want) / size
    return e.max(), np.sqrt((e * e).mean())


@pytest.mark.parametrize("which", ["A X", "At C"])
@pytest.mark.parametrize("kind", ["normal", "worst", "small"])
@pytest.mark.parametrize("nnz", [1, 2, 4])
@pytest.mark.parametrize("R", [64, 128])
def test_short_sums_round_as_float32(cuda, rsk_lib, R, nnz, kind, which):
    g = np.random.default_rng(7 * nnz + R)
    eta, n = 128, 384
    A = _entries(g, (eta, n), kind)
    S = _sparse(g, n if which == "A X" else eta, R, nnz, kind)
    top3, rms3 = _error(cuda, 3, which, A, S, eta)
    top1, rms1 = _error(cuda, 1, which, A, S, eta)
    # one rounding of half a unit (2^-24) for the sum and a unit (the matrix cores may truncate) for each
    # addition of a term to another, and the small terms' 2^-28
    bound = (2 * nnz - 1) * 2.0 ** -24 + 2.0 ** -27
    assert top3 <= bound and top1 <= bound, (top3 * 2 ** 24, top1 * 2 ** 24)
    # the same roundings in another order: their mean square is that of the float32 matrix cores', up to the
    # spread of 16 thousand of them
    assert rms3 <= 1.0625 * rms1 + 2.0 ** -28, (rms3 * 2 ** 24, rms1 * 2 ** 24)
