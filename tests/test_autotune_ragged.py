"""Tuned dense entries of float32 rows that are not whole 16-byte chunks and of aligned rows of the same shape do not
replace or serve one another."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def clean_table(cuda, rsk_lib):
    from paper_2203_10838_amd import autotune
    autotune.clear()
    yield
    autotune.clear()


@pytest.fixture
def views(cuda):
    """One shape (n a multiple of 4) at an aligned and at an odd pitch; the odd one's built-in launch is the register
    tile, several times faster than the general kernel it can ask for by name."""
    import torch
    m, n, eta, steps = 2000, 2048, 400, 10
    full = torch.randn(m, n + 1, device=cuda)
    kw = dict(eta=eta, lam=0.1, alpha=1.0, steps=steps, reps=2,
              index_stream=torch.randint(0, m, (steps * eta,), dtype=torch.int32, device=cuda))
    return full[:, :n].contiguous(), full[:, :n], torch.randn(m, device=cuda), kw


def test_tuning_ragged_rows_leaves_the_aligned_entry(views):
    from paper_2203_10838_amd import _abi, autotune, rsk
    aligned, ragged, b, kw = views
    eta = kw["eta"]
    out = autotune.tune_dense(aligned, b, candidates=[(2, 64), (2, 32)], **kw)
    tuned = rsk.plan_dense(aligned, eta=eta)
    default = rsk.plan_dense(ragged, eta=eta)
    assert (tuned["kernel"], tuned["G"]) == out["choice"]
    got = autotune.tune_dense(ragged, b, candidates=[(1, 16), (1, 32)], **kw)
    assert got["choice"] == (0, 0), got          # the built-in launch beats the candidates
    assert rsk.plan_dense(ragged, eta=eta) == default
    assert rsk.plan_dense(aligned, eta=eta) == tuned


def test_an_entry_of_ragged_rows_is_theirs_alone(views, tmp_path):
    from paper_2203_10838_amd import _abi, autotune, rsk
    aligned, ragged, b, kw = views
    eta, (m, n) = kw["eta"], aligned.shape
    before = rsk.plan_dense(aligned, eta=eta)
    autotune.set_entry(_abi.RSK_TUNE_DENSE, _abi.RSK_F32, m=m, n=n, eta=eta, R=1, v0=1, v1=24)
    assert rsk.plan_dense(aligned, eta=eta) == before
    assert rsk.plan_dense(ragged, eta=eta)["G"] == 24
    f = str(tmp_path / "tune.txt")
    autotune.save(f)
    autotune.clear()
    autotune.load(f)
    assert rsk.plan_dense(aligned, eta=eta) == before
    assert rsk.plan_dense(ragged, eta=eta)["G"] == 24
    # a timing that installs nothing leaves what was there
    autotune.tune_dense(ragged, b, candidates=[(1, 16)], install=False, **kw)
    assert rsk.plan_dense(ragged, eta=eta)["G"] == 24
    autotune.clear()
    autotune.tune_dense(ragged, b, candidates=[(1, 16)], install=False, **kw)
    assert autotune.get_entry(_abi.RSK_TUNE_DENSE, _abi.RSK_F32, m=m, n=n, eta=eta, R=1) is None


def test_an_entry_of_the_shape_serves_ragged_rows_without_their_own(views):
    """A cache file written before ragged rows had entries of their own."""
    from paper_2203_10838_amd import _abi, autotune, rsk
    aligned, ragged, b, kw = views
    eta, (m, n) = kw["eta"], aligned.shape
    default = rsk.plan_dense(ragged, eta=eta)
    autotune.set_entry(_abi.RSK_TUNE_DENSE, _abi.RSK_F32, m=m, n=n, eta=eta, v0=1, v1=24)
    assert rsk.plan_dense(ragged, eta=eta)["G"] == 24
    autotune.set_entry(_abi.RSK_TUNE_DENSE, _abi.RSK_F32, m=m, n=n, eta=eta, v0=2, v1=24)  # does not apply to them
    assert rsk.plan_dense(ragged, eta=eta) == default
