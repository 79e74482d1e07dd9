"""Clustering parity where the document-frequency histogram's cuts fall: batches
of one run of indices, one more and many, and vocabularies of one LDS window
and of three (integer work: bit-exact)."""

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2609_05138_amd as som
else:  # collected on CPU-only machines, never run there
    som = None


@pytest.mark.parametrize("nnz", [1, 4095, 4096, 4097, 8191, 70001])
@pytest.mark.parametrize("F", [3, 32768, 32769, 70000])
def test_cluster_order_at_the_histogram_cuts(nnz, F):
    rng = np.random.default_rng(nnz + F)
    rows = []
    left = nnz
    while left:
        k = min(left, F, int(rng.integers(0, 9)))
        rows.append(np.sort(rng.choice(F, k, replace=False)) if F < 100 else
                    np.sort(rng.choice(np.concatenate([np.arange(50), rng.integers(50, F, 50)]), k, replace=False)))
        rows[-1] = np.unique(rows[-1])
        left -= len(rows[-1])
    indptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    indices = np.concatenate(rows).astype(np.int32)
    assert len(indices) == nnz
    got = som.som_cluster_order(torch.from_numpy(indptr).to("cuda:0"), torch.from_numpy(indices).to("cuda:0"), F)
    assert got.cpu().numpy().tolist() == oracle.cluster_order(indptr, indices, F).tolist()
