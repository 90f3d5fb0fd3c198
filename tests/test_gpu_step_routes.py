"""The routes of w2v_step_batch (atomic, staged, pulled): each against the
oracle and against the sorted batch, with the route that ran asserted."""
import numpy as np
import pytest

import oracle
from paper_1611_06172_amd import inputs, w2v
from gpu_util import expect_device_flag, scaled_error, to_dev

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


# |gpu - oracle| <= 1e-5 S, S the magnitude of the summands of an element.
BAR = 1e-5


@pytest.mark.parametrize("B,N,K,V,D,pad,absent,route", [
    (10_000, 10, 5, 15_000, 300, 0, 0.0, "pulled"),     # one output block
    (25_000, 10, 5, 100_000, 100, 3, 0.3, "pulled"),    # unaligned rows, gaps
    (60_000, 3, 7, 100_000, 63, 0, 0.0, "pulled"),      # several blocks, spans of chunks
    (10_000, 32, 3, 100_000, 128, 0, 0.2, "pulled"),    # 17 to 32 inputs
    (15_000, 16, 9, 100_000, 200, 0, 0.1, "pulled"),    # 11 to 16 inputs, two blocks
    (6_000, 10, 7, 15_000, 512, 0, 0.0, "pulled"),      # C = 8, blocks of 4
    (10_000, 10, 5, 8_000, 400, 0, 0.0, "pulled"),      # C = 8, one block
    (6_000, 10, 12, 30_000, 600, 40, 0.0, "pulled"),    # C = 10, blocks of 4
    (25_000, 1, 1, 3_000, 640, 0, 0.0, "pulled"),       # fewest partners
    (12_000, 1, 63, 50_000, 100, 0, 0.0, "pulled"),     # a partner in every lane
    (1_500, 10, 5, 100_000, 300, 20, 0.2, "staged"),
    (2_500, 20, 5, 60_000, 100, 0, 0.0, "staged"),
    (1_000, 10, 12, 15_000, 600, 0, 0.0, "staged"),
    (1_000, 31, 20, 60_000, 128, 0, 0.3, "staged"),
    (12_000, 1, 64, 50_000, 100, 0, 0.0, "atomic"),     # 65 columns: no lane each
    (2_000, 10, 5, 300, 64, 0, 0.0, "atomic"),
    (3_000, 16, 25, 2_000, 200, 0, 0.2, "atomic"),
    (70, 2, 0, 3_000, 385, 15, 0.0, "atomic"),
])
def test_every_route_of_the_snapshot_batch(B, N, K, V, D, pad, absent, route):
    """w2v_step_batch by the route its sizes take: the oracle's result,
    skipped minibatches counted, untouched elements and row padding bit for
    bit; staged and pulled batches the sorted batch's bits (the same sums in
    the same order), the atomic ones one fp32 step from them at most (fp64
    sums in another order, rounded once)."""
    import torch
    assert w2v.debug_step_route(B, N, K, V, D, D + pad) == route
    t, c, n = inputs.kernel_batch(B, N, K, V, 1.0, 7)
    rng = np.random.Generator(np.random.PCG64(8))
    c[rng.random(c.shape) < absent] = -1
    t[1], c[3, 0] = V, -2                      # two minibatches are skipped
    bad = [1, 3]
    M_in = inputs.init_matrix(V, D, "normal", 4)
    M_out = inputs.init_matrix(V, D, "normal", 5)
    ok = np.setdiff1d(np.arange(B), bad)
    oi, oo, S_in, S_out = oracle.step_batch(t[ok], c[ok], n[ok], M_in, M_out, 0.025)
    got = []
    for srt in (False, True):
        full = [torch.full((V, D + pad), 9.0, device="cuda") for _ in range(2)]
        m = [f[:, :D] for f in full]
        for x, y in zip(m, (M_in, M_out)):
            x.copy_(to_dev(y))
        stats = torch.zeros(5, dtype=torch.int64, device="cuda")
        w2v.step_batch(to_dev(t), to_dev(c), to_dev(n), m[0], m[1], 0.025, stats=stats,
                       sorted=srt)
        expect_device_flag()
        got.append([x.cpu().numpy() for x in m] + [stats.cpu().numpy()])
        assert all(bool((f[:, D:] == 9.0).all()) for f in full)
    for g, o, S, M0 in zip(got[0], (oi, oo), (S_in, S_out), (M_in, M_out)):
        assert scaled_error(g, o, S) <= BAR
        rest = S == np.abs(M0.astype(np.float64))   # no summands
        assert np.array_equal(g[rest].view(np.uint32), M0[rest].view(np.uint32))
    assert np.array_equal(got[0][2], got[1][2]) and got[0][2][3] == len(bad)
    for g, h in zip(got[0][:2], got[1][:2]):
        if route == "atomic":
            assert np.all(np.abs(g - h) <= np.spacing(np.maximum(np.abs(g), np.abs(h))))
        else:
            assert np.array_equal(g.view(np.uint32), h.view(np.uint32))


@pytest.mark.parametrize("B,N,K,V,D,route", [
    (12_000, 10, 5, 15_000, 300, "pulled"),
    (15_000, 16, 9, 100_000, 200, "pulled"),
    (6_000, 10, 7, 15_000, 512, "pulled"),
    (1_500, 10, 5, 100_000, 300, "staged"),
    (1_000, 10, 12, 15_000, 600, "staged"),
    (2_000, 10, 5, 300, 64, "atomic"),
    (3_000, 16, 25, 2_000, 200, "atomic"),
])
@pytest.mark.parametrize("srt", [False, True])
def test_infinities_and_nans_stay_where_they_belong(B, N, K, V, D, route, srt):
    """Infinities and NaNs in a few rows of both matrices reach the elements
    that the oracle's products carry them to and no others: missing rows and
    columns of a tile are left out, not multiplied by zero errors."""
    assert w2v.debug_step_route(B, N, K, V, D, D) == route
    t, c, n = inputs.kernel_batch(B, N, K, V, 1.0, 9)
    rng = np.random.Generator(np.random.PCG64(10))
    c[rng.random(c.shape) < 0.3] = -1
    M_in = inputs.init_matrix(V, D, "normal", 4)
    M_out = inputs.init_matrix(V, D, "normal", 5)
    # rare rows (few minibatches hold them), one of each matrix for each value
    for k, v in enumerate((np.inf, -np.inf, np.nan)):
        M_in[V // 2 + 7 * k, (5 * k) % D] = v
        M_out[V // 3 + 7 * k, (3 * k + D - 1) % D] = v
        t[10 + k], c[20 + k, 0], n[30 + k, 0] = V // 3 + 7 * k, V // 2 + 7 * k, V // 3 + 7 * k
    with np.errstate(all="ignore"):
        oi, oo, S_in, S_out = oracle.step_batch(t, c, n, M_in, M_out, 0.025)
    gi, go = to_dev(M_in), to_dev(M_out)
    w2v.step_batch(to_dev(t), to_dev(c), to_dev(n), gi, go, 0.025, sorted=srt)
    touched = 0
    for g, o, S, M0 in ((gi.cpu().numpy(), oi, S_in, M_in), (go.cpu().numpy(), oo, S_out, M_out)):
        fin = np.isfinite(o)
        touched += int((~fin).sum()) - int((~np.isfinite(M0)).sum())
        assert np.array_equal(np.isfinite(g), fin)
        assert scaled_error(g[fin], o[fin], S[fin]) <= BAR
    assert touched > 0


@pytest.mark.parametrize("B,N,K,V,D,route", [
    (10_000, 10, 5, 15_000, 300, "pulled"),
    (1_500, 10, 5, 100_000, 300, "staged"),
    (2_000, 10, 5, 300, 64, "atomic"),
])
def test_every_route_replays_from_a_graph(B, N, K, V, D, route):
    """A captured call replayed with eager work in between: each replay leaves
    what the eager call leaves (the atomic route's fp64 sums come in another
    order: one fp32 step)."""
    import torch
    assert w2v.debug_step_route(B, N, K, V, D, D) == route
    t, c, n = (to_dev(x) for x in inputs.kernel_batch(B, N, K, V, 1.0, 11))
    start = [to_dev(inputs.init_matrix(V, D, "normal", s)) for s in (4, 5)]
    want = [x.clone() for x in start]
    ws = w2v.step_batch(t, c, n, want[0], want[1], 0.025)
    m = [x.clone() for x in start]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        w2v.step_batch(t, c, n, m[0], m[1], 0.025, workspace=ws)
    for _ in range(3):
        for x, y in zip(m, start):
            x.copy_(y)
        other = [x.clone() for x in start]
        w2v.step_batch(t, c, n, other[0], other[1], 0.025)   # eager, its own workspace
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for g, h in zip(m, want):
            if route == "atomic":
                g, h = g.cpu().numpy(), h.cpu().numpy()
                assert np.all(np.abs(g - h) <= np.spacing(np.maximum(np.abs(g), np.abs(h))))
            else:
                assert torch.equal(g, h)
