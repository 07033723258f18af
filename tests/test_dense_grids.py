"""The built-in workgroup counts of dense solves where a larger or smaller grid costs more than it gives."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,eta,G", [(1008, 1024, 63), (1008, 769, 63), (1008, 768, 32), (2000, 1024, 125),
                                     (2000, 512, 64), (3344, 1000, 209), (3344, 334, 128)])
def test_slices_of_the_512_thread_form_stay_narrow(cuda, rsk_lib, n, eta, G):
    """63 slices of 16 columns against 32 of 32, 1024 rows: 8.8 and 12.2 us a step."""
    import torch
    from paper_2203_10838_amd import rsk
    plan = rsk.plan_dense(torch.empty(4 * eta, n, device=cuda), eta=eta)
    assert plan["row_groups"] == 2 or plan["G"] == G, plan
    assert plan["threads"] == (512 if eta > 768 else 1024)


@pytest.mark.parametrize("dtype,n,eta,G", [
    ("f64", 500, 800, 128), ("f64", 1000, 400, 128), ("f64", 1000, 786, 128), ("f64", 2000, 256, 128),  # as many lanes a row
    ("f64", 8000, 50, 128), ("f64", 350, 1142, 128), ("f32", 1000, 1100, 128),
    ("f64", 700, 571, 192), ("f64", 1500, 349, 192), ("f64", 5000, 100, 192), ("f32", 1500, 1100, 192),  # half as many
])
def test_192_workgroups_where_they_halve_the_lanes_of_a_row(cuda, rsk_lib, dtype, n, eta, G):
    """n = 1000, 400 rows: 12.4 us a step with 128, 14.3 with 192; n = 5000, 80 rows: 12.5 and 10.5."""
    import torch
    from paper_2203_10838_amd import rsk
    A = torch.empty((2 * eta, n), device=cuda, dtype={"f32": torch.float32, "f64": torch.float64}[dtype])
    plan = rsk.plan_dense(A, eta=eta)
    assert (plan["kernel"], plan["G"]) == (1, G), plan
