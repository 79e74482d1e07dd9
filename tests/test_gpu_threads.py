"""Calls from several threads, each on its own stream: a kernel's limit of dynamic
LDS belongs to the process, so calls of different sizes side by side must not set
it under each other."""

import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2609_05138_amd as som
else:  # collected on CPU-only machines, never run there
    som = None

DEV = "cuda:0"
# features, documents, map and neighbourhood: small and large LDS needs of the
# histogram, both plan kernels and the wide blur
SIZES = [(40, 1600, 8, 9, 6.0), (60000, 1600, 300, 9, 6.0), (32768, 300, 16, 200, 30.0), (300, 300, 500, 3, 40.0)]


def _work(F, B, rows, cols, sigma, seed):
    """Inputs of one thread and a function that runs every step on them."""
    rng = np.random.default_rng(seed)
    N = rows * cols
    doc = np.repeat(np.arange(B, dtype=np.int64), rng.poisson(8, B))
    key = np.unique(doc * F + rng.integers(0, F, doc.size))
    ip = torch.from_numpy(np.concatenate([[0], np.cumsum(np.bincount(key // F, minlength=B))]).astype(np.int32)).to(DEV)
    ix = torch.from_numpy((key % F).astype(np.int32)).to(DEV)
    W = torch.rand((F, som.som_codebook_ldw(N)), device=DEV)
    norms = som.som_codebook_norms(W, N=N)
    acc = torch.randint(0, 5, (20, N), device=DEV, dtype=torch.int32)
    count = torch.randint(0, 5, (N,), device=DEV, dtype=torch.int32)
    blurred = torch.zeros((20, som.som_codebook_ldw(N)), device=DEV)

    def run():
        perm = som.som_cluster_order(ip, ix, F)
        out = som.som_bmu_search(W, norms, ip, ix, N=N, perm=perm)
        tiles = som.som_bmu_search(W, norms, ip, ix, N=N, perm=perm, kernel=3, sweep=1)
        V = blurred.clone()
        som.som_update_finish(V, rows, cols, sigma, acc, count)
        return (perm, *out, *tiles, V)

    return run


def test_calls_of_different_sizes_side_by_side():
    runs = [_work(*size, seed) for seed, size in enumerate(SIZES)]
    want = [run() for run in runs]
    torch.cuda.synchronize()
    failed = []

    def body(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream(device=DEV)):
                for _ in range(20):
                    got = runs[i]()
                    torch.cuda.current_stream().synchronize()
                    if not all(torch.equal(x, y) for x, y in zip(got, want[i])):
                        failed.append((i, "another result"))
        except Exception as e:   # noqa: BLE001 (reported by the main thread)
            failed.append((i, repr(e)))

    threads = [threading.Thread(target=body, args=(i,)) for i in range(len(runs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed
