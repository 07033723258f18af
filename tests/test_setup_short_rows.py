"""Row norms of short rows: the lengths around the line between one element and one chunk a load, and their time."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("n", [1, 63, 65, 255, 256, 257, 319, 320, 321, 512])
def test_norms_around_the_line(cuda, rsk_lib, dtype, n):
    import torch
    from paper_2203_10838_amd import rsk
    dt = {"f32": torch.float32, "f64": torch.float64}[dtype]
    m = 37
    full = torch.full((m, n + 3), float("nan"), dtype=dt, device=cuda)
    full[:, 1:n + 1] = torch.from_numpy(np.random.default_rng(n).standard_normal((m, n))).to(cuda, dt)
    A = full[:, 1:n + 1]
    ref = (A.double() ** 2).sum(1)
    # n additions in double, then one rounding to the type
    eps = n * 2.0 ** -53 + (2.0 ** -24 if dtype == "f32" else 0.0)
    assert ((rsk.rownorm2(A).double() - ref).abs() <= eps * ref).all()
    cdf = rsk.sampling_cdf(A)
    assert ((cdf - ref.cumsum(0)).abs() <= (n + m) * 2.0 ** -53 * cdf).all()


def test_short_rows_take_less_time_than_long_ones(cuda, rsk_lib):
    """300000 float32 rows of 16 and of 400: 124 and 131 us where the short ones issued the long ones' loads, 46 and
    131 without."""
    import torch
    from paper_2203_10838_amd import rsk
    us = {}
    for n in (16, 400):
        A = torch.randn(300_000, n, device=cuda)
        best = float("inf")
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                rsk.rownorm2(A)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 200)
        us[n] = best
    assert us[16] <= 0.65 * us[400], us
