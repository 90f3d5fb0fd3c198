"""The workloads whose speed is tracked, each run through the public entry
points of paper_1611_06172_amd.w2v as a training program calls them.

Five kinds of call:

  epoch   w2v.train_epoch over a corpus that is resident on the GPU: HogBatch
          (update rows pending in LDS, or every update written at once), the
          paper's per-pair Algorithm 1, or negatives shared by a group of
          targets; Hogwild at the library's default concurrency, or one
          sentence at a time (`inflight` 1), which is reproducible
  batch   w2v.step_batch: one deterministic batch of independent minibatches,
          with fp64 atomic sums or with the fixed-order sorted reduction
  vocab   w2v.build_vocab: count, rank, cut and rewrite a raw id stream

Sizes are those of paper_1611_06172_amd.configs (tiny, kernel test, planted,
large vocabulary, sweep) with the corpora cut to what a second or less
trains. Corpora are i.i.d. Zipf streams. A reproducible epoch starts as
training starts (M_in uniform in +-0.5/D, M_out zero, the full learning
rate); a Hogwild epoch is the last of five over matrices that hold values of
a trained model's size (normal, 0.1), where the order in which concurrent
sentences meet matters least; the snapshot batches have the kernel test's
matrices (normal, 0.1).
"""
import math

import numpy as np
import torch

from paper_1611_06172_amd import configs, inputs, w2v

_TINY = configs.Tiny()
_KT = configs.KernelTest()
_PL = configs.Planted()
_LV = configs.LargeVocab()
_SW = configs.Sweep()


def _epoch(name, T, V, D, window, K, zipf, sample, **over):
    c = {"name": name, "kind": "epoch", "T": T, "V": V, "D": D, "window": window,
         "K": K, "zipf": zipf, "sample": sample, "algorithm": "hogbatch", "group": 1,
         "inflight": 0, "sentence": 1000, "table": 10_000_000, "tiers": "model",
         "tol": 0.05, "padded": True, "loss": True}
    c.update(over)
    return c


def listed():
    return [
        # A reproducible run, one sentence at a time: what a test, a debugging
        # session or a bit-exact resume of a small model does. Two sentences,
        # so launches and one wavefront's latency are all there is.
        _epoch("serial_d64", 2_000, _TINY.V, _TINY.D, _TINY.window, _TINY.K,
               _TINY.zipf_s, 0.0, inflight=1, table=1_000_000, tiers="plain"),
        # The tiny configuration whole, with the binding's defaults (every
        # update atomic): a small vocabulary allows only 15 sentences at once.
        _epoch("tiny_d64", _TINY.T, _TINY.V, _TINY.D, _TINY.window, _TINY.K,
               _TINY.zipf_s, _TINY.sample, table=1_000_000, tiers="atomic"),
        # A mid-sized corpus with the planted configuration's shape: wide
        # window, many negatives, rows of 200 floats, 71,290 words.
        _epoch("planted_d200_w8_k25", 2_000_000, _PL.V, _PL.D, _PL.window, _PL.K,
               _PL.topic_zipf_s, _PL.sample),
        # The throughput workload (a tenth of its tokens): the paper's
        # hyper-parameters over 10^6 words, launched as bench.py launches it.
        _epoch("large_d300_k5", 100_000_000, _LV.V, _LV.D, _LV.window, _LV.K,
               _LV.zipf_s, _LV.sample, table=_LV.table_size, tol=0.5),
        # Three cells of the shape sweep: short rows, long rows with several
        # output blocks, and the largest number of negatives.
        _epoch("sweep_d100_k5", 40_000_000, _SW.V, 100, _SW.window, 5, _SW.zipf_s,
               _SW.sample),
        _epoch("sweep_d600_k15", 6_000_000, _SW.V, 600, _SW.window, 15, _SW.zipf_s,
               _SW.sample),
        _epoch("sweep_d100_k64", 4_000_000, _SW.V, 100, _SW.window, 64, _SW.zipf_s,
               _SW.sample),
        # Negatives shared by four targets, the faster variant of the method.
        _epoch("grouped_d300_g4", 40_000_000, _LV.V, _LV.D, _LV.window, _LV.K,
               _LV.zipf_s, _LV.sample, group=4),
        # The paper's baseline algorithm, which HogBatch is compared with.
        _epoch("pairwise_d300", 6_000_000, _LV.V, _LV.D, _LV.window, _LV.K,
               _LV.zipf_s, _LV.sample, algorithm="pairwise"),
        # The kernel-test snapshot batch: bit-reproducible, and with atomics.
        {"name": "batch_sorted_b65536", "kind": "batch", "B": _KT.B, "N": _KT.N,
         "K": _KT.K, "V": _KT.V, "D": _KT.D, "zipf": _KT.zipf_s, "absent": 0.0,
         "sorted": True, "padded": True, "alphas": False, "stats": False},
        {"name": "batch_atomic_b65536", "kind": "batch", "B": _KT.B, "N": _KT.N,
         "K": _KT.K, "V": _KT.V, "D": _KT.D, "zipf": _KT.zipf_s, "absent": 0.0,
         "sorted": False, "padded": True, "alphas": False, "stats": False},
        # The vocabulary of a billion-token corpus over 2 million raw words.
        {"name": "vocab_1e9", "kind": "vocab", "T": 1_000_000_000, "V": 2_000_000,
         "zipf": _LV.zipf_s, "min_count": 5, "remap": True},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["epoch", "epoch", "epoch", "batch", "vocab"])
    if kind == "vocab":
        T = _log(rng, 5_000, 400_000_000) + rng.randrange(3)
        return {"kind": "vocab", "T": T, "V": _log(rng, 500, min(3_000_000, 4 * T)),
                "zipf": rng.choice([1.0, 1.07]), "min_count": rng.choice([0, 1, 5]),
                "remap": rng.random() < 0.8}
    if kind == "batch":
        N = rng.randrange(1, 11) if rng.random() < 0.7 else rng.randrange(11, 33)
        D = _log(rng, 20, {True: 640, False: 320 if N <= 16 else 128}[N <= 10])
        K = rng.choice([0, 1, 5, 5, 10, 15, 25])
        B = _log(rng, 64, min(65_536, int(2e8 / (D * (N + K + 1)))))
        return {"kind": "batch", "B": B, "N": N, "K": K,
                "V": _log(rng, 2_000, 400_000), "D": D, "zipf": 1.0,
                "absent": rng.choice([0.0, 0.3]), "sorted": rng.random() < 0.5,
                "padded": rng.random() < 0.7, "alphas": rng.random() < 0.5,
                "stats": rng.random() < 0.3}
    algorithm = rng.choice(["hogbatch"] * 5 + ["hogbatch_immediate", "pairwise", "group"])
    window = rng.choice([2, 3, 5, 5, 5, 5, 8, 12])
    K = rng.choice([0, 3, 5, 5, 5, 10, 15, 25, 64])
    group = 1
    if algorithm == "group":
        algorithm, group, window, K = "hogbatch", rng.choice([2, 4]), 5, rng.choice([3, 5])
    D = _log(rng, 24, 640 if window <= 5 else 320 if window <= 8 else 128)
    V = _log(rng, 3_000, 1_000_000)
    # Tokens: what about a quarter of a second trains, at some microseconds a
    # minibatch and wavefront with the library's caps on concurrency.
    waves = max(1.0, min(2048.0, V / (4.0 * group * (2 * window + K + 1)), 131072.0 / (K + 1)))
    step = 8e-6 * (1 + 0.01 * D) * (1 + K / 12.0) * (window if algorithm == "pairwise" else 1)
    T = _log(rng, 10_000, max(20_000, min(30_000_000, 0.25 * waves / step)))
    c = _epoch("", T + rng.randrange(2), V, D, window, K, rng.choice([1.0, 1.07]),
               rng.choice([0.0, 1e-4, 1e-4]), algorithm=algorithm, group=group,
               sentence=rng.choice([1000, 1000, 40, 257]),
               tiers="atomic" if rng.random() < 0.25 else "model",
               padded=rng.random() < 0.7, loss=rng.random() < 0.7)
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs --

def _corpus(T, V, zipf, seed):
    return inputs.zipf_corpus_hashed(T, V, zipf, seed % (1 << 22), "cuda")


def _matrix(V, D, padded, init, generator):
    if padded:
        M = w2v.alloc_matrix(V, D, "cuda")
    else:
        M = torch.zeros((V, D), dtype=torch.float32, device="cuda")
    if init == "uniform":
        M.copy_((torch.rand((V, D), generator=generator, device="cuda") - 0.5) / D)
    elif init == "normal":
        M.copy_(torch.randn((V, D), generator=generator, device="cuda") * 0.1)
    return M


def _prepare_epoch(c, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    corpus = _corpus(c["T"], c["V"], c["zipf"], seed)
    counts = torch.bincount(corpus, minlength=c["V"]).cpu().numpy().astype(np.int64)
    table, thr = w2v.build_tables(counts, 0.75, c["sample"], c["table"],
                                  want_thresh=c["sample"] > 0)
    first = c["inflight"] == 1
    M_in = _matrix(c["V"], c["D"], c["padded"], "uniform" if first else "normal", g)
    M_out = _matrix(c["V"], c["D"], c["padded"], "zeros" if first else "normal", g)
    hot, split = c["V"], 0
    if c["tiers"] == "plain":
        hot = 0
    elif c["tiers"] == "model":
        kw = dict(sample_t=c["sample"], window=c["window"], K=c["K"],
                  inflight=w2v.default_inflight(c["D"], c["window"], c["K"], V=c["V"],
                                                group=c["group"]))
        hot = w2v.hot_rows(counts, tol=c["tol"], **kw)
        if c["algorithm"] != "pairwise":
            split = min(2, w2v.hot_rows(counts, tol=128.0, **kw))
    dev = corpus.device
    ws = w2v.train_epoch_workspace_bytes(split, M_in.stride(0))
    return {"kind": "epoch", "corpus": corpus, "M_in": M_in, "M_out": M_out,
            "table": torch.from_numpy(table).to(dev),
            "thr": None if thr is None else torch.from_numpy(thr.view(np.int32)).to(dev),
            "loss": torch.zeros((10, 2), dtype=torch.float64, device=dev)
            if c["loss"] else None,
            "stats": torch.zeros(5, dtype=torch.int64, device=dev),
            "kw": dict(window=c["window"], K=c["K"], seed=seed,
                       epoch=0 if first else 4, n_epochs=1 if first else 5,
                       sentence_len=c["sentence"], max_inflight=c["inflight"],
                       hot_rows=hot, split_rows=split, algorithm=c["algorithm"],
                       group=c["group"],
                       workspace=torch.empty(ws, dtype=torch.uint8, device=dev)
                       if ws else None)}


def _prepare_batch(c, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    B, N, K, V = c["B"], c["N"], c["K"], c["V"]
    ids = _corpus(B * (1 + N + K), V, c["zipf"], seed).reshape(B, 1 + N + K)
    contexts = ids[:, 1:1 + N].contiguous()
    if c["absent"]:
        gone = torch.rand((B, N), generator=g, device="cuda") < c["absent"]
        contexts = torch.where(gone, torch.full_like(contexts, -1), contexts)
    # The batch's updates are summed, so the step is one of learning rate 1
    # (half to one and a half, where minibatches have their own) over the
    # mean gradient.
    alpha = 1.0 / B
    if c["alphas"]:
        alpha = (torch.rand(B, generator=g, device="cuda") + 0.5) / B
    M_in = _matrix(V, c["D"], c["padded"], "normal", g)
    M_out = _matrix(V, c["D"], c["padded"], "normal", g)
    ld = M_in.stride(0)
    ws = (w2v.step_batch_sorted_workspace_bytes(B, N, K, V, ld) if c["sorted"]
          else w2v.step_batch_workspace_bytes(V, ld))
    return {"kind": "batch", "targets": ids[:, 0].contiguous(), "contexts": contexts,
            "negatives": ids[:, 1 + N:].contiguous(), "M_in": M_in, "M_out": M_out,
            "alpha": alpha, "sorted": c["sorted"],
            "ws": torch.empty(ws, dtype=torch.uint8, device="cuda"),
            "stats": torch.zeros(5, dtype=torch.int64, device="cuda")
            if c["stats"] else None}


def _prepare_vocab(c, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    # Raw ids come in no order of frequency.
    perm = torch.randperm(c["V"], generator=g, device="cuda").to(torch.int32)
    raw = _corpus(c["T"], c["V"], c["zipf"], seed)
    step = 1 << 26
    for b in range(0, raw.numel(), step):
        raw[b:b + step] = perm[raw[b:b + step].long()]
    return {"kind": "vocab", "raw": raw, "V": c["V"], "min_count": c["min_count"],
            "remap": c["remap"]}


def prepare(case, seed):
    return {"epoch": _prepare_epoch, "batch": _prepare_batch,
            "vocab": _prepare_vocab}[case["kind"]](case, int(seed))


# -------------------------------------------------------------------- run --

def run(state):
    if state["kind"] == "epoch":
        w2v.train_epoch(state["corpus"], state["M_in"], state["M_out"], state["table"],
                        state["thr"], loss_buckets=state["loss"], stats=state["stats"],
                        **state["kw"])
        out = {"M_in": state["M_in"], "M_out": state["M_out"], "stats": state["stats"]}
        if state["loss"] is not None:
            out["loss"] = state["loss"]
        return out
    if state["kind"] == "batch":
        w2v.step_batch(state["targets"], state["contexts"], state["negatives"],
                       state["M_in"], state["M_out"], state["alpha"],
                       workspace=state["ws"], stats=state["stats"],
                       sorted=state["sorted"])
        out = {"M_in": state["M_in"], "M_out": state["M_out"]}
        if state["stats"] is not None:
            out["stats"] = state["stats"]
        return out
    voc = w2v.build_vocab(state["raw"], state["V"], state["min_count"],
                          remap=state["remap"])
    if voc["corpus"] is None:
        del voc["corpus"]
    return voc


# ------------------------------------------------- work, tolerance, exact --

def _kept(c):
    """Expected share of kept tokens, and of words seen at least once."""
    p = inputs.zipf_pmf(c["V"], c["zipf"])
    seen = float(np.sum(1.0 - np.exp(-p * c["T"])))
    if c["sample"] <= 0:
        return 1.0, seen
    r = c["sample"] / p
    return float(np.sum(p * np.minimum(1.0, np.sqrt(r) + r))), seen


def work(case):
    c = case
    if c["kind"] == "vocab":
        # ids in, ids out, and per raw word its count and rank
        return {"bytes": 4.0 * c["T"] * (2 if c["remap"] else 1) + 12.0 * c["V"],
                "flops": float(c["T"])}
    if c["kind"] == "batch":
        n = c["N"] * (1 - c["absent"])
        p = inputs.zipf_pmf(c["V"], c["zipf"])
        rows = sum(float(np.sum(1.0 - np.exp(-p * c["B"] * k))) for k in (n, c["K"] + 1))
        return {"bytes": 8.0 * c["D"] * rows + 4.0 * c["B"] * (c["N"] + c["K"] + 1),
                "flops": 6.0 * c["B"] * n * (c["K"] + 1) * c["D"]}
    kept, seen = _kept(c)
    targets = c["T"] * kept
    pairs = targets * (c["window"] + 1) * (c["K"] + 1)
    return {"bytes": 4.0 * c["T"] + 16.0 * c["D"] * seen
            + 4.0 * min(targets * c["K"], c["table"]),
            "flops": 6.0 * pairs * c["D"]}


def tolerance(case):
    if case["kind"] == "vocab":
        return "exact"
    if case["kind"] == "batch":
        return {"rel": 1e-7, "max": 1e-6}
    if case["inflight"] == 1:
        return {"rel": 1e-6, "max": 1e-4}
    # Concurrent sentences update the matrices without locks, in an order
    # that differs from run to run: two runs over the same inputs are up to
    # 0.009 (largest element 0.4) apart from 4e7 tokens on, 0.004 (0.2) below.
    return {"rel": 0.03, "max": 0.99} if case["T"] > 2e7 else {"rel": 0.016, "max": 0.7}


def _mulhi(a, b):
    m = np.uint64(0xFFFFFFFF)
    s = np.uint64(32)
    al, ah, bl, bh = a & m, a >> s, b & m, b >> s
    t = al * bl
    u = ah * bl + (t >> s)
    v = al * bh + (u & m)
    return ah * bh + (u >> s) + (v >> s)


def _philox(seed, pos, block):
    """Words 8 block .. 8 block + 7 of every position's stream, uint32 [n, 8]
    (Philox4x64-10: Salmon, Moraes, Dror and Shaw, SC'11)."""
    c0 = pos.astype(np.uint64)
    c1 = np.zeros_like(c0)
    c2 = np.full_like(c0, block)
    c3 = np.zeros_like(c0)
    k0, k1 = int(seed), 0
    ma, mb = np.uint64(0xD2E7470EE14C6C93), np.uint64(0xCA5A826395121157)
    for _ in range(10):
        ka, kb = np.uint64(k0), np.uint64(k1)
        c0, c1, c2, c3 = (_mulhi(mb, c2) ^ c1 ^ ka, mb * c2,
                          _mulhi(ma, c0) ^ c3 ^ kb, ma * c0)
        k0 = (k0 + 0x9E3779B97F4A7C15) % (1 << 64)
        k1 = (k1 + 0xBB67AE8584CAA73B) % (1 << 64)
    out = np.stack([c0, c1, c2, c3], axis=1)
    low = (out & np.uint64(0xFFFFFFFF)).astype(np.uint32)
    high = (out >> np.uint64(32)).astype(np.uint32)
    return np.stack([low, high], axis=2).reshape(len(pos), 8)


def _exact_epoch(c, seed):
    """The epoch one minibatch after the other in 64 bits."""
    s = _prepare_epoch(c, seed)
    corpus = s["corpus"].cpu().numpy()
    table = s["table"].cpu().numpy()
    A, O = s["M_in"].double().cpu().numpy(), s["M_out"].double().cpu().numpy()
    T, w, K, L = c["T"], c["window"], c["K"], c["sentence"]
    pos = np.arange(T)
    blocks = np.concatenate([_philox(seed, pos, b) for b in range((K + 9) // 8)], axis=1)
    keep = np.ones(T, dtype=bool)
    if s["thr"] is not None:
        keep = blocks[:, 0] <= s["thr"].cpu().numpy().view(np.uint32)[corpus]
    half = w - ((blocks[:, 1].astype(np.int64) * w) >> 32)
    negs = table[(blocks[:, 2:2 + K].astype(np.uint64) * np.uint64(len(table)))
                 >> np.uint64(32)]
    alphas = np.float32(np.float64(np.float32(0.025)) * np.maximum(
        np.float64(np.float32(1e-4)), 1.0 - pos.astype(np.float64) / float(T)))
    loss = np.zeros((10, 2))
    for b in range(0, T, L):
        kept = b + np.nonzero(keep[b:b + L])[0]
        words = corpus[kept]
        for q, p in enumerate(kept):
            lo, hi = max(q - half[p], 0), min(q + half[p], len(kept) - 1)
            if lo == hi:
                continue
            ins = np.concatenate([words[lo:q], words[q + 1:hi + 1]])
            outs = np.concatenate([words[q:q + 1], negs[p][negs[p] != words[q]]])
            a, o = A[ins], O[outs]
            z = a @ o.T
            z[:, 0] *= -1.0
            e = -1.0 / (1.0 + np.exp(-z))
            e[:, 0] *= -1.0
            e *= float(alphas[p])
            np.add.at(A, ins, e @ o)
            np.add.at(O, outs, e.T @ a)
            k = p * 10 // T
            loss[k] += np.logaddexp(0.0, z).sum(), len(ins)
    return {"M_in": A, "M_out": O, "stats": None, "loss": loss}


def _exact_batch(c, seed):
    s = _prepare_batch(c, seed)
    A, O = s["M_in"].double(), s["M_out"].double()
    dA, dO = torch.zeros_like(A), torch.zeros_like(O)
    B = c["B"]
    alpha = s["alpha"] if isinstance(s["alpha"], torch.Tensor) else \
        torch.full((B,), s["alpha"], device="cuda")
    step = max(1, (1 << 26) // (c["D"] * (c["N"] + c["K"] + 1)))
    for b in range(0, B, step):
        t, n = s["targets"][b:b + step].long(), s["negatives"][b:b + step].long()
        i = s["contexts"][b:b + step].long()
        there, i = i >= 0, i.clamp(min=0)
        outs = torch.cat([t[:, None], n], dim=1)
        a, o = A[i], O[outs]
        z = torch.bmm(a, o.transpose(1, 2).contiguous())
        label = torch.zeros_like(z)
        label[:, :, 0] = 1.0
        e = (label - torch.sigmoid(z)) * alpha[b:b + step].double()[:, None, None]
        used = torch.ones_like(outs, dtype=torch.bool)
        used[:, 1:] = n != t[:, None]
        e = e * there[:, :, None] * used[:, None, :]
        dA.index_add_(0, i.reshape(-1), torch.bmm(e, o).reshape(-1, c["D"]))
        dO.index_add_(0, outs.reshape(-1), torch.bmm(
            e.transpose(1, 2).contiguous(), a).reshape(-1, c["D"]))
    return {"M_in": A + dA, "M_out": O + dO}


def _exact_vocab(c, seed):
    s = _prepare_vocab(c, seed)
    counts = torch.zeros(c["V"], dtype=torch.int64, device="cuda")
    step = 1 << 27
    for b in range(0, c["T"], step):
        counts += torch.bincount(s["raw"][b:b + step], minlength=c["V"])
    ranked, order = torch.sort(counts, descending=True, stable=True)
    keep = ranked >= max(c["min_count"], 1)
    rank_of = torch.full((c["V"],), -1, dtype=torch.int32, device="cuda")
    v = int(keep.sum())
    rank_of[order[:v]] = torch.arange(v, dtype=torch.int32, device="cuda")
    out = {"ranked_counts": torch.where(keep, ranked, torch.zeros_like(ranked)),
           "rank_of": rank_of, "V": v}
    if c["remap"]:
        corpus = torch.empty_like(s["raw"])
        for b in range(0, c["T"], step):
            corpus[b:b + step] = rank_of[s["raw"][b:b + step].long()]
        out["corpus"] = corpus
    return out


def exact(case, seed):
    """What run() returns for these inputs, in 64 bits; None where the result
    depends on how concurrent sentences interleave."""
    if case["kind"] == "batch":
        return _exact_batch(case, int(seed))
    if case["kind"] == "vocab":
        return _exact_vocab(case, int(seed))
    if case["inflight"] == 1 and case["algorithm"] == "hogbatch" and case["group"] == 1 \
            and case["T"] <= 20_000:
        return _exact_epoch(case, int(seed))
    return None
