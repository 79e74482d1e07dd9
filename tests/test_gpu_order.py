"""The order in which the automatic launch sums below 65,536 documents: that of
kernel 3 with 64-document super-tiles for fp32 and of kernel 1 with 8-document
tiles for fp16, whichever kernel it takes, so that a batch's units do not depend
on it.  Two nearly equal distances change places with the order of a sum, and one
changed unit is much of a small batch; so the bits must agree, on random
codebooks, where almost every document's sum shows its order.

Sizes: where the launch changes form, super-tiles and tiles that are ragged,
empty or cut by an XCD's share of the launch, and long documents, whose
super-tiles start far into their unions."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2609_05138_amd as som
else:  # collected on CPU-only machines, never run there
    som = None

DEV = "cuda:0"


def _docs(rng, B, F, mean, hole=False):
    n = np.minimum(rng.poisson(mean, B), F)
    n[rng.random(B) < 0.02] = 0
    n[rng.random(B) < 0.005] = min(F, 5 * mean + 70)
    if hole:
        n[64:192] = 0               # a super-tile and more with no feature
    doc = np.repeat(np.arange(B, dtype=np.int64), n)
    ids = np.minimum((F * rng.random(doc.size) ** 3).astype(np.int64), F - 1)
    key = np.unique(doc * F + ids)
    count = np.bincount(key // F, minlength=B)
    indptr = np.concatenate([[0], np.cumsum(count)])
    return (torch.from_numpy(indptr.astype(np.int32)).to(DEV), torch.from_numpy((key % F).astype(np.int32)).to(DEV))


def _book(rng, F, N, dtype):
    W = torch.zeros((F, som.som_codebook_ldw(N)), dtype=dtype, device=DEV)
    W[:, :N] = torch.from_numpy(rng.random((F, N), dtype=np.float32)).to(DEV).to(dtype)
    return W, som.som_codebook_norms(W, N=N)


def _same(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


FORMER = {torch.float32: dict(kernel=3), torch.float16: dict(kernel=1, tile_docs=8)}


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("B,F,N,mean", [
    (1, 50, 70, 10), (32, 900, 65537, 30), (33, 900, 65537, 30), (64, 3000, 300, 60), (64, 900, 65536, 30),
    (65, 3000, 300, 60), (256, 700, 16385, 30), (257, 700, 16385, 30), (512, 5000, 200, 80), (512, 700, 12288, 30), (400, 5000, 12289, 60),
    (513, 5000, 200, 80), (1023, 4000, 300, 60), (1024, 4000, 300, 60), (1100, 20000, 130, 80),
    (1600, 65536, 130, 90), (1600, 65537, 130, 90), (2049, 65, 129, 20), (2500, 63, 129, 4), (5000, 2000, 257, 15),
    (5120, 900, 16385, 40), (5121, 900, 16385, 40), (9973, 4999, 130, 70), (10000, 2048, 1024, 20),
    (12288, 20000, 64, 80), (12289, 20000, 64, 80), (40000, 20000, 64, 80), (65535, 3000, 64, 40)])
def test_automatic_launch_sums_in_the_former_order(dtype, B, F, N, mean):
    rng = np.random.default_rng(B + F)
    ip, ix = _docs(rng, B, F, mean, hole=B % 3 == 0)
    W, norms = _book(rng, F, N, dtype)
    perm = som.som_cluster_order(ip, ix, F)
    for p in (None, perm):
        want = som.som_bmu_search_top2(W, norms, ip, ix, N=N, perm=p, **FORMER[dtype])
        for sweep in (0, 2):
            assert _same(som.som_bmu_search_top2(W, norms, ip, ix, N=N, perm=p, sweep=sweep), want), (sweep, p is None)
            assert _same(som.som_bmu_search(W, norms, ip, ix, N=N, perm=p, sweep=sweep), want[:2]), (sweep, p is None)
    if dtype == torch.float32 and B <= 9973:
        assert _same(som.som.som_bmu_search_noalloc(W, norms, ip, ix, N=N, perm=perm), want[:2])
    # a plan for either storage type, searched with this one
    for storage in (0, 1):
        former = dict(kernel=3) if storage == 0 else dict(kernel=1, tile_docs=8)
        plan = som.som_plan(ip, ix, F, perm=perm, storage=storage)
        ref = som.som_plan(ip, ix, F, perm=perm, storage=storage, **former)
        assert _same(som.som_bmu_search_top2_planned(W, norms, ip, plan, N=N),
                     som.som_bmu_search_top2_planned(W, norms, ip, ref, N=N)), storage


def test_orders_differ_in_bits():
    # what the comparison above rests on: another order shows in the distances
    rng = np.random.default_rng(3)
    B, F, N = 9973, 4999, 130
    ip, ix = _docs(rng, B, F, 70)
    W, norms = _book(rng, F, N, torch.float32)
    a = som.som_bmu_search(W, norms, ip, ix, N=N)
    b = som.som_bmu_search(W, norms, ip, ix, N=N, sweep=1)
    assert float((a[1] != b[1]).float().mean()) > 0.01
