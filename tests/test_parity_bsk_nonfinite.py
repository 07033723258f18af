"""A NaN in a sampled row of the block sparse Kaczmarz method is reported at its step, wherever the row stands in
its block, and the steps before it are those of the shorter run."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("eta", [3, 17, 64])
@pytest.mark.parametrize("at", ["first", "middle", "last"])
def test_a_nan_row_is_nonfinite_at_its_step(cuda, rsk_lib, dtype, eta, at):
    import torch
    from paper_2203_10838_amd import rsk
    dt = {"f32": torch.float32, "f64": torch.float64}[dtype]
    g = np.random.default_rng(eta)
    m, n, K, bad = 200, 70, 5, 2
    A = torch.from_numpy(g.standard_normal((m, n))).to(cuda, dt)
    A[m - 1, 33] = float("nan")
    b = torch.from_numpy(g.standard_normal(m)).to(cuda, dt)
    idx = g.integers(0, m - 1, K * eta).astype(np.int32)
    idx[bad * eta + {"first": 0, "middle": eta // 2, "last": eta - 1}[at]] = m - 1
    it = torch.from_numpy(idx).to(cuda)
    kw = dict(lam=0.1, eta=eta, w=1.0, index_stream=it)
    x_star = torch.full((n,), float("nan"), dtype=dt, device=cuda)
    with pytest.raises(rsk.RskError) as e:
        rsk.bsk_solve(A, b, K=K, x_star=x_star, **kw)
    assert e.value.name == "RSK_ERR_NONFINITE"
    want = rsk.bsk_solve(A, b, K=bad, **kw)
    assert want.k_done == bad and torch.equal(x_star, want.x_star)
