"""Edges of the set-up kernels: row norms over chunk remainders and pitches, and the sampler's
two-level search around its pivot count."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("m,n,ld", [(3, 1, 1), (5, 3, 3), (7, 255, 257), (6, 2048, 2048), (9, 2049, 2051),
                                    (4, 4103, 4103), (70000, 9, 9)])
def test_row_norms_over_chunk_edges(cuda, rsk_lib, dtype, m, n, ld):
    import torch
    from paper_2203_10838_amd import rsk
    dt = {"f32": torch.float32, "f64": torch.float64}[dtype]
    g = torch.Generator().manual_seed(m + n)
    full = torch.full((m, ld), float("nan"), dtype=dt)
    full[:, :n] = torch.randn((m, n), generator=g, dtype=dt)
    A = full.to(cuda)[:, :n]
    ref = full[:, :n].double().square().sum(1).numpy()
    got = rsk.rownorm2(A).double().cpu().numpy()
    # double sums in two orders, then one rounding to the type
    eps = {"f32": 2.0 ** -24, "f64": 2.0 ** -53}[dtype]
    assert np.all(np.abs(got - ref) <= (eps + 2 * n * 2.0 ** -53) * ref)
    cdf = rsk.sampling_cdf(A).cpu().numpy()
    assert np.all(np.abs(cdf - np.cumsum(ref)) <= 2 * (n + m) * 2.0 ** -53 * np.cumsum(ref))


@pytest.mark.parametrize("m", [1, 2, 4095, 4096, 4097, 8191, 8193, 60001])
@pytest.mark.parametrize("K,eta", [(1, 1), (3, 1365), (5, 4099)])
def test_two_level_search_equals_the_oracle(cuda, rsk_lib, m, K, eta):
    import torch
    from paper_2203_10838_amd import rsk
    w = np.random.default_rng(m + eta).random(m) ** 8 + 1e-12  # very uneven weights
    w[m // 3: m // 2] = 0.0 if m > 6 else w[m // 3: m // 2]
    cdf = oracle.sampling_cdf(w)
    got = rsk.sample_stream(torch.from_numpy(cdf).to(cuda), seed=5, K=K, eta=eta, k0=7).cpu().numpy()
    assert np.array_equal(got, oracle.sample_stream(cdf, 5, K, eta, k0=7))
