"""The batched register tile at the edges of its exchange (one hop, a row a thread, against two) and of its
index prefetch two steps ahead."""
import numpy as np
import pytest

import oracle
from paper_2203_10838_amd import inputs
from parity import check_iterate, to_dev

pytestmark = pytest.mark.gpu

# (m, n, eta, K, wg_bytes)
EDGES = [
    (40, 8, 1, 1, 0), (40, 8, 1, 2, 0), (60, 20, 3, 3, 0),             # one workgroup, the first steps
    (600, 164, 33, 7, 0), (700, 640, 64, 7, 0), (900, 516, 128, 7, 0),  # whole passes and one row more
    (900, 516, 129, 7, 0), (1200, 640, 256, 7, 0), (1200, 640, 257, 7, 0), (1400, 640, 512, 7, 0),
    (1200, 512, 256, 7, 16384), (1200, 528, 256, 7, 16384),            # 32 and 33 slices: 8192 words and more
    (1100, 1040, 20, 7, 1024), (900, 1028, 3, 7, 256),                 # more slices than lanes of a poll
]


def test_batched_exchange_edges(cuda, rsk_lib):
    """All edges in batches of one, and all together in one launch: the oracle's iterates at the float32 bar,
    and the same bits whether a system runs alone or beside the others."""
    from paper_2203_10838_amd import rsk
    by_wg = {}
    for i, (m, n, eta, K, wg) in enumerate(EDGES):
        s = inputs.dense_system(m, n, max(1, n // 20), dtype="f32", seed=60 + i)
        idx = inputs.index_stream(inputs.row_sampling_weights(s["A"]), K, eta, 600 + i)
        alpha = oracle.optimal_alpha(eta, float((s["A"].astype(np.float64) ** 2).sum()),
                                     float(np.linalg.norm(s["A"].astype(np.float64), 2) ** 2))
        sy = dict(A=to_dev(s["A"], cuda), b=to_dev(s["b"], cuda), index_stream=to_dev(idx, cuda), eta=eta, K=K,
                  alpha=alpha, lam=0.1)
        one = rsk.solve_batched([rsk.BatchSystem(**sy)], wg_bytes=wg, kernel=2)
        assert one.status == [0] and one.k_done == [K]
        ref = oracle.rska_dense(s["A"], s["b"], 0.1, eta, alpha, K, idx)
        check_iterate(one.x_star[0], one.x[0], ref, 0.1, 1e-4, min_support=0, what=f"{(m, n, eta, K)}")
        by_wg.setdefault(wg, []).append((sy, one.x_star[0].clone()))
    for wg, group in by_wg.items():
        r = rsk.solve_batched([rsk.BatchSystem(**sy) for sy, _ in group] * 3, wg_bytes=wg, kernel=2)
        for i, (_, x1) in enumerate(group * 3):
            assert (r.x_star[i] == x1).all()


def test_batched_bad_index_in_each_of_the_first_steps(cuda, rsk_lib):
    """An index out of range is reported at its own step, whichever buffer it was fetched into."""
    import torch
    from paper_2203_10838_amd import rsk
    m, n, eta, K = 300, 100, 40, 5
    s = inputs.dense_system(m, n, 5, dtype="f32", seed=9)
    idx = inputs.index_stream(inputs.row_sampling_weights(s["A"]), K, eta, 3)
    A, b = to_dev(s["A"], cuda), to_dev(s["b"], cuda)
    for k in range(K):
        for bad in (-1, m):
            ix = idx.copy()
            ix[k * eta + eta - 1] = bad
            r = rsk.solve_batched([rsk.BatchSystem(A=A, b=b, index_stream=to_dev(ix, cuda), eta=eta, K=K, alpha=1.0,
                                                   lam=0.1)], kernel=2, check=False)
            code, done = r.status_dev[0].tolist()
            assert rsk._abi.STATUS_NAMES[code] == "RSK_ERR_INDEX_RANGE" and done == k, (k, bad, code, done)
            assert torch.isfinite(r.x_star[0]).all()
