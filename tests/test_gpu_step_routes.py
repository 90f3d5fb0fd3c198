"""The routes of w2v_step_batch (atomic, staged, pulled): each against the
oracle and against the sorted batch, with the route that ran asserted."""
import numpy as np
import pytest

import oracle
from paper_1611_06172_amd import inputs, w2v
from gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,N,K,V,D,route", [
    (12_000, 10, 5, 15_000, 300, "pulled"),
    (1_500, 10, 5, 100_000, 300, "staged"),
    (300, 10, 5, 3_000, 64, "atomic"),
])
@pytest.mark.parametrize("views", ["same", "next row", "shared columns"])
def test_matrices_that_share_rows(B, N, K, V, D, route, views):
    """One matrix passed as M_in and M_out (tied embeddings) and views that
    share rows or columns: both updates reach every shared element, whatever
    the route of separate matrices of this size. Each element is M0 plus up to
    two sums with a rounding each: 1e-5 of both sums' magnitudes."""
    import torch
    t, c, n = inputs.kernel_batch(B, N, K, V, 1.0, 7)
    ld = D + 8
    assert w2v.debug_step_route(B, N, K, V, D, ld) == route
    base = inputs.init_matrix(V + 1, ld, "normal", 4)
    cut = {"same": (0, 0), "next row": (1, 0), "shared columns": (0, 5)}[views]
    buf = to_dev(base)
    M_in = buf[:V, :D]
    M_out = buf[cut[0]:cut[0] + V, cut[1]:cut[1] + D]
    h_in = np.ascontiguousarray(base[:V, :D])
    h_out = np.ascontiguousarray(base[cut[0]:cut[0] + V, cut[1]:cut[1] + D])
    oi, oo, S_in, S_out = oracle.step_batch(t, c, n, h_in, h_out, 0.025)
    want = base.astype(np.float64)
    scale = np.abs(want)
    want[:V, :D] += oi.astype(np.float64) - h_in
    scale[:V, :D] += S_in
    want[cut[0]:cut[0] + V, cut[1]:cut[1] + D] += oo.astype(np.float64) - h_out
    scale[cut[0]:cut[0] + V, cut[1]:cut[1] + D] += S_out
    w2v.step_batch(to_dev(t), to_dev(c), to_dev(n), M_in, M_out, 0.025)
    torch.cuda.synchronize()
    assert float(np.max(np.abs(buf.cpu().numpy() - want) / scale)) <= 1e-5
