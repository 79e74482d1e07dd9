"""What this library's speed is measured on: calls of its public entry points
over the sizes, workload laws, storage types and stages that a program
training or serving a self-organizing map uses.

A training pass refreshes the codebook norms, then per CSR batch orders the
documents, plans and searches them and accumulates the update, and at the end
of an epoch blurs the accumulators into new weights; batches that come back
every epoch are planned once and searched with their plan.  Serving calls the
search on a few documents at a time.  The documents are binary term vectors
with frequency-ordered feature ids (truncated Zipf law, exponent 1.1), either
over one vocabulary or as mixtures of one to three of 256 topics of 2,000
features each; a codebook is either the random initial one or one whose
weights follow the features' document frequencies, as training makes them.
"""

import math

import torch

from paper_2609_05138_amd import som

ZIPF = 1.1
TOPICS, TOPIC_SIZE = 256, 2000

# The cost of the largest listed search, in weights added (documents x mean
# features x neurons): no drawn case goes beyond half of it (the topic law and
# small tiles cost more per added weight).
LARGEST = 262144 * 80 * 262144


def listed():
    return [
        # Serving: a handful of documents against a medium map, allocation-free
        # entry point (a tight serving loop or a captured graph).
        dict(name="serve-16docs-128sq", kind="noalloc", rows=128, cols=128, F=20000, B=16, nnz=80, law="poisson",
             book="trained", f16=False, top2=False),
        # The smallest training pass: norms, order, search with its plan.
        dict(name="pass-32sq-10k", kind="pass", rows=32, cols=32, F=2048, B=10000, nnz=20, law="poisson",
             book="initial", f16=False, top2=False),
        # Ragged everything: odd map sides, vocabulary and batch; best and
        # second-best unit (what the topographic error needs), input order.
        dict(name="top2-63x65-odd", kind="search", rows=63, cols=65, F=4999, B=9973, nnz=70, law="lognormal",
             book="trained", f16=False, top2=True),
        # One batch of the 128 x 128 map's pass, ordered and searched.
        dict(name="pass-128sq-64k", kind="pass", rows=128, cols=128, F=20000, B=65536, nnz=80, law="poisson",
             book="initial", f16=False, top2=False),
        # A large corpus on a small map: ordering and planning count as much
        # as the search does.
        dict(name="pass-32sq-1M", kind="pass", rows=32, cols=32, F=20000, B=1048576, nnz=80, law="poisson",
             book="initial", f16=False, top2=False),
        # A batch of the 256 x 256 map that returns every epoch: its plan is kept.
        dict(name="planned-256sq-256k", kind="planned", rows=256, cols=256, F=20000, B=262144, nnz=70,
             law="lognormal", book="trained", f16=False, top2=False),
        # The 512 x 512 map, a quarter of one batch of its pass.
        dict(name="planned-512sq-256k", kind="planned", rows=512, cols=512, F=20000, B=262144, nnz=80, law="poisson",
             book="initial", f16=False, top2=False),
        # The same map on the topic corpus (no globally frequent features).
        dict(name="planned-512sq-topics", kind="planned", rows=512, cols=512, F=20000, B=131072, nnz=80,
             law="topics", book="initial", f16=False, top2=False),
        # Half-precision codebook storage, whole call with ordering and plan.
        dict(name="pass-512sq-f16", kind="pass", rows=512, cols=512, F=20000, B=262144, nnz=80, law="poisson",
             book="initial", f16=True, top2=False),
        # The update's scatter: one searched batch of a million documents.
        dict(name="accumulate-256sq-1M", kind="accumulate", rows=256, cols=256, F=20000, B=1048576, nnz=80,
             law="poisson"),
        # End of a late epoch: narrow neighbourhood, new weights, their norms.
        dict(name="finish-256sq-s2", kind="finish", rows=256, cols=256, F=20000, B=1048576, nnz=80, law="poisson",
             sigma=2.0, f16=False),
        # End of an early epoch: wide neighbourhood, half-precision weights.
        dict(name="finish-128sq-s16-f16", kind="finish", rows=128, cols=128, F=20000, B=262144, nnz=80,
             law="poisson", sigma=16.0, f16=True),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["noalloc", "search", "search", "pass", "pass", "pass", "planned", "planned", "planned",
                       "accumulate", "finish"])
    law = rng.choice(["poisson", "lognormal", "topics"])
    F = _log_uniform(rng, 2000, 20000)
    nnz = max(4, min(rng.randint(15, 90), F // 40))
    if kind in ("accumulate", "finish"):
        rows, cols = _log_uniform(rng, 30, 256), _log_uniform(rng, 30, 256)
        case = dict(kind=kind, rows=rows, cols=cols, F=F, B=_log_uniform(rng, 5000, 1048576), nnz=nnz, law=law)
        if kind == "finish":
            case.update(sigma=round(math.exp(rng.uniform(math.log(0.5), math.log(16.0))), 2),
                        f16=rng.random() < 0.5)
            if rng.random() < 0.1:
                case["sigma"] = 0.0
        return case
    rows, cols = _log_uniform(rng, 30, 512), _log_uniform(rng, 30, 512)
    f16 = rng.random() < 0.3 and kind != "noalloc"
    if kind == "noalloc":
        B = _log_uniform(rng, 1, 40000)
    else:
        B = _log_uniform(rng, 500, 1048576)
    B = max(1, min(B, int(LARGEST / 2 / (rows * cols * nnz))))
    return dict(kind=kind, rows=rows, cols=cols, F=F, B=B, nnz=nnz, law=law,
                book=rng.choice(["initial", "trained"]), f16=f16,
                top2=kind in ("search", "planned") and rng.random() < 0.25)


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _documents(case, g, dev):
    """CSR batch (indptr, indices) as int32 tensors: i.i.d. draws per document
    from its law with repeats dropped, ids ascending within a document."""
    B, F, law = case["B"], case["F"], case["law"]
    size = min(TOPIC_SIZE, F) if law == "topics" else F
    w = torch.arange(1, size + 1, dtype=torch.float64, device=dev) ** -ZIPF
    cdf = torch.cumsum(w, 0)
    cdf /= cdf[-1].clone()
    # draws per document: the mean number of distinct features they give is
    # solved for the wanted one from the law itself
    p = (w / w.sum()).cpu()
    lo, hi = 1.0, 1.0e5
    for _ in range(50):
        mid = 0.5 * (lo + hi)
        if float((1.0 - torch.exp(-mid * p)).sum()) < case["nnz"]:
            lo = mid
        else:
            hi = mid
    mean = hi
    if law == "poisson":
        draws = torch.poisson(torch.full((B,), mean, device=dev), generator=g)
    else:
        z = torch.randn(B, device=dev, generator=g)
        draws = torch.round(mean * torch.exp((0.7 if law == "topics" else 0.6) * z))
    draws = draws.clamp_(1, 4000).to(torch.int64)
    if law == "topics":
        table = torch.stack([torch.randperm(F, device=dev, generator=g)[:size] for _ in range(TOPICS)])
        mix = torch.randint(1, 4, (B,), device=dev, generator=g)
        topic = torch.randint(0, TOPICS, (B, 3), device=dev, generator=g)
    keys = []
    bound = torch.cumsum(draws, 0)
    step = max(1, (1 << 25) * B // max(1, int(bound[-1])))   # documents per block of about 2^25 draws
    for b0 in range(0, B, step):
        n = draws[b0:b0 + step]
        doc = torch.repeat_interleave(torch.arange(b0, b0 + n.numel(), device=dev), n)
        u = torch.rand(doc.numel(), device=dev, dtype=torch.float64, generator=g)
        rank = torch.searchsorted(cdf, u).clamp_(max=size - 1)
        if law == "topics":
            pick = (torch.rand(doc.numel(), device=dev, generator=g) * mix[doc]).to(torch.int64).clamp_(max=2)
            rank = table[topic[doc, pick], rank]
        keys.append(torch.unique(doc * F + rank))
    key = torch.cat(keys)
    indices = (key % F).to(torch.int32)
    count = torch.bincount(torch.div(key, F, rounding_mode="floor"), minlength=B)
    indptr = torch.zeros(B + 1, dtype=torch.int32, device=dev)
    indptr[1:] = torch.cumsum(count, 0).to(torch.int32)
    return indptr, indices


def _codebook(case, g, dev):
    """Feature-major [F, ldw] codebook at the recommended row stride."""
    F, N = case["F"], case["rows"] * case["cols"]
    W = torch.zeros((F, som.som_codebook_ldw(N)), dtype=torch.float16 if case["f16"] else torch.float32, device=dev)
    df = (18.5 * torch.arange(1, F + 1, device=dev, dtype=torch.float32) ** -ZIPF).clamp_(max=1.0)
    for a in range(0, F, 512):
        rows = min(512, F - a)
        block = torch.rand((rows, N), device=dev, generator=g)
        if case["book"] == "trained":      # near a feature's frequency, a few units far above it
            block = (df[a:a + rows, None] * (0.25 + block * block * block * block * 4.0)).clamp_(max=1.0)
        W[a:a + rows, :N] = block.to(W.dtype)
    return W


def prepare(case, seed):
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(1000003 * int(seed) + 17)
    N, F, B = case["rows"] * case["cols"], case["F"], case["B"]
    indptr, indices = _documents(case, g, dev)
    s = dict(case=case, N=N, F=F, indptr=indptr, indices=indices)
    kind = case["kind"]
    if kind in ("accumulate", "finish"):
        # best-matching units: some units catch far more documents than others
        u = torch.rand(B, device=dev, generator=g)
        unit = torch.randperm(N, device=dev, generator=g)[(u * u * N).to(torch.int64).clamp_(max=N - 1)]
        s["bmu"] = unit.to(torch.int32)
        s["acc"] = torch.zeros((F, som.som_codebook_ldw(N)), dtype=torch.int32, device=dev)
        s["count"] = torch.zeros(N, dtype=torch.int32, device=dev)
        if kind == "finish":
            som.som_update_accumulate(indptr, indices, s["bmu"], F, N, s["acc"], s["count"])
            W = torch.empty((F, som.som_codebook_ldw(N)), dtype=torch.float16 if case["f16"] else torch.float32,
                            device=dev)
            for a in range(0, F, 512):
                W[a:a + 512] = torch.rand((min(512, F - a), W.shape[1]), device=dev, generator=g).to(W.dtype)
            s["W"] = W
            s["norms"] = torch.empty(N, dtype=torch.float32, device=dev)
            s["ws"] = torch.empty(som.som_update_workspace_bytes(F, N), dtype=torch.uint8, device=dev)
        return s
    s["W"] = _codebook(case, g, dev)
    s["norms"] = som.som_codebook_norms(s["W"], N=N)
    s["outs"] = dict(bmu=torch.empty(B, dtype=torch.int32, device=dev),
                     dist=torch.empty(B, dtype=torch.float32, device=dev))
    if case["top2"]:
        s["outs"].update(bmu2=torch.empty(B, dtype=torch.int32, device=dev),
                         dist2=torch.empty(B, dtype=torch.float32, device=dev))
    nnz = indices.numel()
    if kind == "planned":
        knobs = dict(storage=1 if case["f16"] else 0)
        perm = som.som_cluster_order(indptr, indices, F)
        s["plan"] = som.som_plan(indptr, indices, F, perm=perm, **knobs)
        s["ws"] = torch.empty(som.som_bmu_search_planned_workspace_bytes(N, B, **knobs), dtype=torch.uint8,
                              device=dev)
    elif kind in ("pass", "search"):
        s["ws"] = torch.empty(som.som_bmu_workspace_bytes(F, N, B, nnz), dtype=torch.uint8, device=dev)
    if kind == "pass":
        s["perm"] = torch.empty(B, dtype=torch.int32, device=dev)
        s["cluster_ws"] = torch.empty(som.som_cluster_workspace_bytes(B, F, nnz), dtype=torch.uint8, device=dev)
    return s


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "accumulate":
        som.som_update_accumulate(s["indptr"], s["indices"], s["bmu"], s["F"], s["N"], s["acc"], s["count"])
        return {"acc": s["acc"], "count": s["count"]}
    if kind == "finish":
        som.som_update_finish(s["W"], case["rows"], case["cols"], case["sigma"], s["acc"], s["count"], ws=s["ws"])
        som.som_codebook_norms(s["W"], N=s["N"], norms=s["norms"])
        return {"W": s["W"], "norms": s["norms"]}
    search = som.som_bmu_search_top2 if case["top2"] else som.som_bmu_search
    if kind == "noalloc":
        som.som_bmu_search_noalloc(s["W"], s["norms"], s["indptr"], s["indices"], N=s["N"], **s["outs"])
    elif kind == "search":
        search(s["W"], s["norms"], s["indptr"], s["indices"], N=s["N"], ws=s["ws"], **s["outs"])
    elif kind == "pass":
        som.som_codebook_norms(s["W"], N=s["N"], norms=s["norms"])
        som.som_cluster_order(s["indptr"], s["indices"], s["F"], perm=s["perm"], ws=s["cluster_ws"])
        search(s["W"], s["norms"], s["indptr"], s["indices"], N=s["N"], perm=s["perm"], ws=s["ws"], **s["outs"])
        return {**s["outs"], "perm": s["perm"], "norms": s["norms"]}
    else:
        planned = som.som_bmu_search_top2_planned if case["top2"] else som.som_bmu_search_planned
        planned(s["W"], s["norms"], s["indptr"], s["plan"], N=s["N"], ws=s["ws"], **s["outs"])
    return s["outs"]


# ---------------------------------------------------------------------------
# What a pass cannot do without, and how exactly it is computed
# ---------------------------------------------------------------------------

def work(case):
    N, F, B, nnz = case["rows"] * case["cols"], case["F"], case["B"], case["B"] * case["nnz"]
    csr = 4 * (nnz + B + 1)
    if case["kind"] == "accumulate":
        # a counter read and written per distinct (feature, unit): at most the
        # nonzeros, at most the whole accumulator
        return {"bytes": csr + 4 * B + 8 * min(nnz, F * N) + 8 * N, "flops": nnz + B}
    size = 2 if case["f16"] else 4
    if case["kind"] == "finish":
        taps = 2 * min(math.ceil(3 * case["sigma"]), max(case["rows"], case["cols"])) + 1
        return {"bytes": F * N * (4 + size) + 8 * N, "flops": 2 * F * N * (2 * taps + 1)}
    # the rows of the features that some document holds, once each: all of
    # them for a large batch
    rows = min(F, nnz)
    bytes_ = csr + size * rows * N + 4 * N + (16 if case["top2"] else 8) * B
    flops = nnz * N + 3 * B * N
    if case["kind"] == "pass":
        bytes_ += 4 * N + 4 * B
        flops += 2 * F * N
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    if case["kind"] == "accumulate":
        return "exact"
    if case["kind"] == "finish":
        # two 32-bit tap sums and a division (7e-8 from 64 bits, the norms of
        # drawn sizes 2.4e-7); half-precision weights are rounded to 11 bits
        # once more (1.2e-4, half a unit in the last place is 4.9e-4)
        if case["f16"]:
            return {"rel": 4e-4, "max": 2e-3}
        return {"rel": 1e-6, "max": 3e-6}
    # distances from 32-bit sums: measured 1.5e-7 from 64 bits and 1.4e-7 (at
    # most 7e-7) between two orders of summation; units at almost equal
    # distances swapped in 1.2e-5 of the documents
    return {"rel": 5e-7, "max": 3e-6, "differ": 1e-4}


def exact(case, seed):
    N, F, B = case["rows"] * case["cols"], case["F"], case["B"]
    if case["kind"] == "accumulate":
        return None
    if case["kind"] == "finish":
        taps = math.ceil(3 * case["sigma"])
        if float(F) * N * (min(taps, case["rows"]) + min(taps, case["cols"])) > 1e12:
            return None
        s = prepare(case, seed)
        return _exact_finish(s, case)
    if float(B) * N * F > 1.2e14:
        return None
    s = prepare(case, seed)
    dev = s["W"].device
    W = s["W"][:, :N].double()
    norms = (W * W).sum(0)
    best = torch.empty(B, dtype=torch.float64, device=dev)
    second = torch.empty(B, dtype=torch.float64, device=dev)
    ip = s["indptr"].to(torch.int64)
    step = max(1, min(8192, (1 << 30) // max(N, F)))
    for b0 in range(0, B, step):
        n = min(step, B - b0)
        X = torch.zeros((n, F), dtype=torch.float64, device=dev)
        a, b = int(ip[b0]), int(ip[b0 + n])
        doc = torch.repeat_interleave(torch.arange(n, device=dev), ip[b0 + 1:b0 + n + 1] - ip[b0:b0 + n])
        X[doc, s["indices"][a:b].to(torch.int64)] = 1.0
        d = X.sum(1, keepdim=True) + norms[None, :] - 2.0 * (X @ W)
        v = torch.topk(d, min(2, N), dim=1, largest=False, sorted=True).values
        best[b0:b0 + n] = v[:, 0]
        second[b0:b0 + n] = v[:, -1]
        del X, d
    out = dict(bmu=None, dist=best)
    if case["top2"]:
        out.update(bmu2=None, dist2=second if N > 1 else torch.full_like(best, math.inf))
    if case["kind"] == "pass":
        out.update(perm=None, norms=norms)
    return out


def _exact_finish(s, case):
    """Neighbourhood-weighted means of the accumulated documents in 64 bits."""
    rows, cols, N, F, sigma = case["rows"], case["cols"], s["N"], s["F"], case["sigma"]
    dev = s["W"].device

    def band(n):
        k = torch.arange(n, device=dev, dtype=torch.float64)
        d = (k[:, None] - k[None, :]).abs()
        if sigma == 0:
            return (d == 0).double()
        return torch.where(d <= math.ceil(3 * sigma), torch.exp(-d * d / (2.0 * sigma * sigma)), torch.zeros_like(d))

    R, C = band(rows), band(cols)
    den = R @ s["count"].double().reshape(rows, cols) @ C
    W = s["W"].double()
    norms = torch.zeros(N, dtype=torch.float64, device=dev)
    for a in range(0, F, 256):
        n = min(256, F - a)
        plane = s["acc"][a:a + n, :N].double().reshape(n * rows, cols) @ C
        plane = plane.reshape(n, rows, cols).transpose(1, 2).reshape(n * cols, rows) @ R
        num = plane.reshape(n, cols, rows).transpose(1, 2)
        new = torch.where(den > 0, num / den, W[a:a + n, :N].reshape(n, rows, cols)).reshape(n, N)
        W[a:a + n, :N] = new
        norms += (new * new).sum(0)
    if case["f16"]:
        norms = None      # of the rounded weights, not of these
    return dict(W=W, norms=norms)
