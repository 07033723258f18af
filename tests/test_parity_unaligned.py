"""Float32 register tile on rows that are not whole 16-byte chunks: odd row lengths, odd pitches and
bases off a 16-byte boundary, against the FP64 oracle and against the kernel for aligned rows."""
import numpy as np
import pytest

import oracle
from paper_2203_10838_amd import inputs
from parity import check_iterate

pytestmark = pytest.mark.gpu

TOL = 1e-4  # the float32 bar of the other parity tests, relative to the largest element of x*


def _alpha(m, n, eta):
    smax2 = (np.sqrt(m) + np.sqrt(n)) ** 2
    return eta / (1.0 + (eta - 1.0) * smax2 / (m * n))


def _system(m, n, ld, off, eta, K, cuda, seed):
    import torch
    s = inputs.dense_system(m, n, max(1, n // 20), dtype="f32", seed=seed, noise_rel=0.01)
    idx = inputs.index_stream(inputs.row_sampling_weights(s["A"]), K, eta, seed + 1)
    full = torch.full((m, ld), float("nan"), dtype=torch.float32, device=cuda)  # the padding is never used
    full[:, off:off + n] = torch.from_numpy(s["A"]).to(cuda)
    return s, idx, full[:, off:off + n]


@pytest.mark.parametrize("m,n,ld,off,eta,K", [
    (60, 17, 17, 0, 40, 60),         # a slice that holds one column
    (300, 65, 67, 1, 33, 50),        # likewise, with a pitch and an offset
    (300, 18, 19, 0, 34, 30),        # the last chunk shares two columns with the one before
    (300, 130, 130, 0, 70, 40),
    (1500, 1283, 1283, 0, 1024, 12),  # 512 threads, 8 row passes, the last one full
    (1500, 1286, 1286, 0, 897, 12),   # the last pass holds one row
    (900, 20479, 20479, 0, 300, 10),  # two row groups, slices of 160 columns, slots left to HBM
    (900, 20477, 20477, 0, 250, 10),  # one group, the whole next tile in LDS
    (700, 9999, 9999, 0, 334, 20),
])
def test_unaligned_rows_match_the_oracle(cuda, rsk_lib, m, n, ld, off, eta, K):
    import torch
    from paper_2203_10838_amd import rsk
    lam = 0.02
    s, idx, A = _system(m, n, ld, off, eta, K, cuda, 4000 + n + eta)
    assert rsk.plan_dense(A, eta=eta)["kernel"] in (2, 3)
    b, it = torch.from_numpy(s["b"]).to(cuda), torch.from_numpy(idx).to(cuda)
    xr = torch.from_numpy(s["xhat"]).to(cuda)
    kw = dict(lam=lam, eta=eta, alpha=_alpha(m, n, eta), index_stream=it, rownorm2_t=rsk.rownorm2(A))
    res = rsk.solve_dense(A, b, K=K, x_ref=xr, check_every=K // 2, **kw)
    assert res.status == 0 and res.k_done == K
    ref = oracle.rska_dense(s["A"], s["b"], lam, eta, _alpha(m, n, eta), K, idx, check_every=K // 2, xref=s["xhat"])
    check_iterate(res.x_star, res.x, ref, lam, TOL)
    assert np.allclose(res.err_hist.cpu().numpy(), ref["hist"], rtol=1e-3)
    # the same bits again, and over a resumed run
    again = rsk.solve_dense(A, b, K=K, **kw)
    half = rsk.solve_dense(A, b, K=K // 2, **kw)
    rest = rsk.solve_dense(A, b, K=K - K // 2, x_star=half.x_star.clone(), warm_start=True,
                           stream_offset=(K // 2) * eta, **kw)
    for r in (again, rest):
        assert torch.equal(r.x_star, res.x_star) and torch.equal(r.x, res.x)


@pytest.mark.parametrize("m,n,eta,K,groups", [(300, 128, 33, 40, 1), (900, 20480, 300, 10, 2),
                                              (1500, 1280, 1000, 10, 1), (900, 5120, 700, 10, 1)])
def test_unaligned_pitch_gives_the_aligned_bits(cuda, rsk_lib, m, n, eta, K, groups):
    """Whole chunks at an odd pitch: the same plan and the same sums as with aligned rows."""
    import torch
    from paper_2203_10838_amd import rsk
    s, idx, A = _system(m, n, n + 3, 1, eta, K, cuda, 77 + n)
    assert A.data_ptr() % 16 and rsk.plan_dense(A, eta=eta)["row_groups"] == groups
    b, it = torch.from_numpy(s["b"]).to(cuda), torch.from_numpy(idx).to(cuda)
    kw = dict(lam=0.02, eta=eta, alpha=_alpha(m, n, eta), K=K, index_stream=it, rownorm2_t=rsk.rownorm2(A))
    got = rsk.solve_dense(A, b, **kw)
    want = rsk.solve_dense(A.contiguous(), b, kernel=groups + 1, **kw)
    assert torch.equal(got.x_star, want.x_star) and torch.equal(got.x, want.x)
    assert (want.x != 0).any()


@pytest.mark.parametrize("n,eta,kernel", [(3, 3, 4), (16, 32, 4), (16, 33, 1), (17, 33, 2), (503, 16, 4), (503, 17, 2),
                                          (2047, 4, 4), (2047, 5, 2), (2049, 1, 2)])
def test_kernel_of_ragged_rows(cuda, rsk_lib, n, eta, kernel):
    """Both sides of the rule's edges, each against the oracle."""
    import torch
    from paper_2203_10838_amd import rsk
    lam, m, K = 0.02, 120, 30
    s, idx, A = _system(m, n, n | 1, 0, eta, K, cuda, 50 + n + eta)
    assert rsk.plan_dense(A, eta=eta)["kernel"] == kernel
    alpha = _alpha(m, n, eta)
    res = rsk.solve_dense(A, torch.from_numpy(s["b"]).to(cuda), lam=lam, eta=eta, alpha=alpha, K=K,
                          index_stream=torch.from_numpy(idx).to(cuda))
    ref = oracle.rska_dense(s["A"], s["b"], lam, eta, alpha, K, idx)
    check_iterate(res.x_star, res.x, ref, lam, TOL)


def test_explicit_register_tile_still_asks_for_aligned_rows(cuda, rsk_lib):
    from paper_2203_10838_amd import rsk
    _, _, A = _system(100, 65, 65, 0, 8, 1, cuda, 9)
    for kernel in (2, 3):
        with pytest.raises(rsk.RskError) as e:
            rsk.plan_dense(A, eta=8, kernel=kernel)
        assert e.value.name == "RSK_ERR_UNSUPPORTED"
