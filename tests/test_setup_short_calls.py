"""Set-up calls away from the long rows and streams their kernels are made for: both sides of the rules that choose
between the two forms, and the time of short ones beside long ones."""
import numpy as np
import pytest

import oracle
from parity import to_dev

pytestmark = pytest.mark.gpu


def _us(fn, reps=8, inner=10):
    import torch
    fn()
    best = float("inf")
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(inner):
            fn()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / inner)
    return best


@pytest.mark.parametrize("m,K,eta", [
    (1, 1024, 1024), (999, 1024, 1024), (1000, 1024, 1024),     # fewest rows of the two-level search
    (4097, 1023, 1025), (4097, 1024, 1025),                     # fewest draws
    (4095, 1024, 1025), (4096, 1025, 1024), (8191, 1049, 1001), (8193, 1024, 1024), (60001, 257, 4099),  # its pivots
    (1 << 20, 1024, 1024), ((1 << 20) + 1, 1024, 1024),         # most rows
])
def test_draws_on_both_sides_of_the_rule(cuda, rsk_lib, m, K, eta):
    from paper_2203_10838_amd import rsk
    w = np.random.default_rng(m + eta).random(m) ** 8 + 1e-12  # very uneven weights, some rows never drawn
    w[m // 3: m // 2] = 0.0
    cdf = oracle.sampling_cdf(w)
    got = rsk.sample_stream(to_dev(cdf, cuda), seed=11, K=K, eta=eta, k0=5).cpu().numpy()
    assert np.array_equal(got, oracle.sample_stream(cdf, 11, K, eta, k0=5))


def test_few_draws_from_many_rows_cost_what_few_rows_do(cuda, rsk_lib):
    """64 draws: from 10^7 rows 67 us against 16 from 1000 where every workgroup read 4096 pivots first; 13
    and 13 without."""
    import torch
    from paper_2203_10838_amd import rsk
    us = {}
    for m in (1000, 10_000_000):
        cdf = torch.rand(m, dtype=torch.float64, device=cuda).cumsum(0)
        out = torch.empty(64, dtype=torch.int32, device=cuda)
        us[m] = _us(lambda: rsk.sample_stream(cdf, seed=5, K=1, eta=64, out=out))
    assert us[10_000_000] <= 2.5 * us[1000], us
