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
