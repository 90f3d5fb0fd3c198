"""The vocabulary's rewrite of long streams (2^24 tokens on), which keeps the
most frequent words' ranks in a table per workgroup: bit for bit against the
reference."""
import numpy as np
import pytest

import oracle
from paper_1611_06172_amd import inputs, w2v

pytestmark = pytest.mark.gpu

T = (1 << 24) + 7


@pytest.mark.parametrize("V_raw,kind,min_count,skip", [
    (300_000, "zipf", 5, 0),
    (300_000, "zipf", 1, 1),          # input and output not aligned alike
    (8_193, "uniform", 0, 0),         # one id more than the table has slots
    (2_000_000, "uniform", 7, 2),     # no head: nearly every token is gathered
    (50_000, "zipf", T + 1, 0),       # every word dropped: an empty table
    (1 << 20, "strided", 2, 0),       # ids that share few table slots
])
def test_long_streams_match_the_reference(V_raw, kind, min_count, skip):
    import torch
    n = T + skip
    if kind == "zipf":
        perm = np.random.default_rng(V_raw).permutation(V_raw)
        raw = perm[inputs.zipf_ids(n, V_raw, 1.0, 3)].astype(np.int32)
    elif kind == "uniform":
        raw = np.random.default_rng(5).integers(0, V_raw, n, dtype=np.int32)
    else:
        raw = (np.random.default_rng(6).integers(0, 64, n) * 16_384).astype(np.int32)
    raw[::997] = V_raw + 5                # ids outside [0, V_raw)
    raw[5::1009] = -3
    raw[11::5003] = np.iinfo(np.int32).min
    raw[13::7001] = np.iinfo(np.int32).max
    ranked, rank_of, V, corpus = oracle.build_vocab(raw[skip:], V_raw, min_count)
    out = w2v.build_vocab(torch.from_numpy(raw).cuda()[skip:], V_raw, min_count)
    assert out["V"] == V
    assert np.array_equal(out["ranked_counts"].cpu().numpy(), ranked)
    assert np.array_equal(out["rank_of"].cpu().numpy(), rank_of)
    assert np.array_equal(out["corpus"].cpu().numpy(), corpus)


@pytest.mark.parametrize("in_skip,out_skip", [(1, 1), (3, 3), (2, 6), (1, 2), (0, 3)])
def test_streams_that_start_inside_a_quad(in_skip, out_skip):
    """raw and corpus_out alike in their 16-byte alignment (head tokens, quads
    and a tail, with the tables) and not (every token on its own): the
    reference's corpus, and nothing written around it."""
    import torch
    V_raw = 9_000
    raw = torch.from_numpy(np.random.default_rng(V_raw).permutation(V_raw)[
        inputs.zipf_ids(T + 8, V_raw, 1.0, 4)].astype(np.int32)).cuda()
    x = raw[in_skip:in_skip + T]
    buf = torch.full((T + 16,), -9, dtype=torch.int32, device="cuda")
    ranked = torch.empty(V_raw, dtype=torch.int64, device="cuda")
    rank_of = torch.empty(V_raw, dtype=torch.int32, device="cuda")
    kept = torch.empty(1, dtype=torch.int32, device="cuda")
    L = w2v.lib()
    ws = torch.empty(int(L.w2v_build_vocab_workspace_bytes(V_raw, T)), dtype=torch.uint8,
                     device="cuda")
    rc = L.w2v_build_vocab(x.data_ptr(), T, V_raw, 3, ranked.data_ptr(), rank_of.data_ptr(),
                           kept.data_ptr(), buf[out_skip:].data_ptr(), ws.data_ptr(),
                           ws.numel(), torch.cuda.current_stream().cuda_stream)
    assert rc == w2v.OK
    want = oracle.build_vocab(x.cpu().numpy(), V_raw, 3)
    got = buf.cpu().numpy()
    assert np.array_equal(got[out_skip:out_skip + T], want[3])
    assert np.all(got[:out_skip] == -9) and np.all(got[out_skip + T:] == -9)
