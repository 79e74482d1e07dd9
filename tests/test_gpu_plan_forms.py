"""A plan searched with a codebook of more rows than it was made for.  som_plan
takes the vocabulary of the batch; the search only asks for a codebook of at least
as many rows.  Up to 65,536 features the automatic plan may be of the list form and
beyond it is a tile plan, so the search must go by the plan and not by its own
codebook's rows: a list plan read as a tile plan gives row numbers out of range."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2609_05138_amd as som
else:  # collected on CPU-only machines, never run there
    som = None

DEV = "cuda:0"


def _docs(rng, B, F, mean):
    doc = np.repeat(np.arange(B, dtype=np.int64), rng.poisson(mean, B))
    key = np.unique(doc * F + np.minimum((F * rng.random(doc.size) ** 3).astype(np.int64), F - 1))
    indptr = np.concatenate([[0], np.cumsum(np.bincount(key // F, minlength=B))])
    return (torch.from_numpy(indptr.astype(np.int32)).to(DEV), torch.from_numpy((key % F).astype(np.int32)).to(DEV))


# features of the plan, rows of the codebook
@pytest.mark.parametrize("F,rows", [(300, 65537), (65536, 65537), (65537, 65537), (65537, 70000), (400, 65536)])
@pytest.mark.parametrize("B,storage", [(500, 0), (1700, 0), (66000, 0), (60, 1), (1700, 1), (66000, 1)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
def test_plans_serve_codebooks_with_more_rows(F, rows, B, storage, dtype):
    rng = np.random.default_rng(F + B)
    N = 70
    ip, ix = _docs(rng, B, F, 12)
    W = torch.zeros((rows, som.som_codebook_ldw(N)), dtype=dtype, device=DEV)
    W[:, :N] = torch.from_numpy(rng.integers(0, 4, (rows, N)) / 4).to(DEV).to(dtype)   # dyadic: exact sums
    norms = som.som_codebook_norms(W, N=N)
    perm = som.som_cluster_order(ip, ix, F)
    want = som.som_bmu_search_top2(W, norms, ip, ix, N=N, perm=perm, kernel=1, sweep=1)
    for sweep in (0, 1):
        plan = som.som_plan(ip, ix, F, perm=perm, storage=storage, sweep=sweep)
        listed = int(plan.buf[:4].view(torch.int32)) < 0          # the mark of a list plan
        assert listed == (F <= 65536 and (B >= 65536 or (storage == 0 and sweep == 0 and 256 < B <= 5120)))
        got = som.som_bmu_search_top2_planned(W, norms, ip, plan, N=N)
        assert all(torch.equal(x, y) for x, y in zip(got, want)), sweep
        best = som.som_bmu_search_planned(W, norms, ip, plan, N=N)
        assert all(torch.equal(x, y) for x, y in zip(best, want)), sweep
