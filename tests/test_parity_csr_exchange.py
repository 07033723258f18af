"""The CSR kernel with two exchanges a step against the one with three barriers, bit for bit: the
latter runs where a workgroup holds more rows than one pass (a smaller grid), with the same sums."""
import numpy as np
import pytest

import oracle
from paper_2203_10838_amd import inputs
from parity import check_vec

pytestmark = pytest.mark.gpu


def _t(a, dev):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to(dev)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("m,n,lo,hi,eta,K", [
    (40, 30, 0, 8, 4, 50),          # empty rows are never drawn (weight 0)
    (200, 150, 1, 100, 9, 60),      # rows longer than 32 entries, a last workgroup of one row
    (300, 60, 3, 9, 200, 40),       # every column hit many times, rows drawn repeatedly
    (3000, 5000, 30, 70, 512, 30),
    (6000, 2000, 5, 40, 2048, 8),   # 256 workgroups
])
@pytest.mark.parametrize("dual", [False, True])
def test_two_exchanges_equal_three_barriers(cuda, rsk_lib, dtype, m, n, lo, hi, eta, K, dual):
    import torch
    from paper_2203_10838_amd import rsk
    c = inputs.csr_system_ragged(m, n, lo, hi, max(1, n // 20), seed=m + eta, dtype=dtype)
    w = inputs.csr_sampling_weights(c["row_ptr"], c["val"])
    idx = inputs.index_stream(w, K, eta, 7)
    args = (_t(c["row_ptr"], cuda), _t(c["col"], cuda), _t(c["val"], cuda), n, _t(c["b"], cuda))
    rw = _t(inputs.row_weights(m, 5, dtype, lo=0.5), cuda)
    xr = _t(c["xhat"], cuda)

    def run(grid, **kw):
        y = torch.zeros(m, dtype=args[2].dtype, device=cuda) if dual else None
        r = rsk.solve_csr(*args, lam=0.05, eta=eta, alpha=0.5 * eta ** 0.5, index_stream=_t(idx, cuda), row_w=rw,
                          x_ref=xr, check_every=5, y_out=y, grid=grid, kernel=2, **kw)
        return r.x_star, r.x, r.err_hist, y

    G = -(-eta // 8)
    small = max(1, (G + 1) // 2) if G > 1 else 0
    one = run(0, K=K)
    if small:  # two passes
        three = run(small, K=K)
        for u, v in zip(one[:2] + one[3:], three[:2] + three[3:]):
            assert u is None or torch.equal(u, v)
        # the monitor sums by workgroup blocks: equal to rounding
        assert torch.allclose(one[2], three[2], rtol=1e-12, atol=0)
    # resumed: the pending step is folded at the end of each call
    h = rsk.solve_csr(*args, lam=0.05, eta=eta, alpha=0.5 * eta ** 0.5, K=K // 2, index_stream=_t(idx, cuda),
                      row_w=rw, kernel=2)
    r = rsk.solve_csr(*args, lam=0.05, eta=eta, alpha=0.5 * eta ** 0.5, K=K - K // 2, index_stream=_t(idx, cuda),
                      stream_offset=K // 2 * eta, row_w=rw, kernel=2, x_star=h.x_star.clone(), warm_start=True)
    assert torch.equal(r.x_star, one[0]) and torch.equal(r.x, one[1])
    ref = oracle.rska_csr(c["row_ptr"], c["col"], c["val"], n, c["b"], 0.05, eta, 0.5 * eta ** 0.5, K, idx,
                          row_w=rw.cpu().numpy())
    check_vec(one[0], ref["z"], {"f32": 1e-4, "f64": 1e-10}[dtype], what="x*")


@pytest.mark.parametrize("what,name", [("index", "RSK_ERR_INDEX_RANGE"), ("column", "RSK_ERR_INDEX_RANGE"),
                                       ("zero", "RSK_ERR_ZERO_ROW")])
def test_fault_ends_the_run_at_its_step(cuda, rsk_lib, what, name):
    import torch
    from paper_2203_10838_amd import rsk
    m, n, eta, K, at = 400, 300, 40, 12, 5
    c = inputs.csr_system(m, n, 40, 10, seed=3)
    idx = inputs.index_stream(np.ones(m - 1), K, eta, 4)  # row m - 1 is never drawn
    val, col = c["val"].copy(), c["col"].copy()
    idx[at * eta + 17] = m if what == "index" else m - 1
    if what == "zero":
        val[-40:] = 0
    if what == "column":
        col[-3] = n
    args = (_t(c["row_ptr"], cuda), _t(col, cuda), _t(val, cuda), n, _t(c["b"], cuda))
    kw = dict(lam=0.05, eta=eta, alpha=5.0, index_stream=_t(idx, cuda), kernel=2, check=False)
    r = rsk.solve_csr(*args, K=K, **kw)
    code, done = r.status_dev.tolist()
    assert rsk._abi.STATUS_NAMES[code] == name and done == at
    good = rsk.solve_csr(*args, K=at, **kw)
    assert torch.equal(r.x_star, good.x_star) and torch.equal(r.x, good.x)
