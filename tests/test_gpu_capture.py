"""The allocation-free search and the steps around it under HIP graph capture, on
each side of the automatic launch's lines: every replay must give the eager
result, on inputs changed between the replays, with eager work in between."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2609_05138_amd as som
else:  # collected on CPU-only machines, never run there
    som = None

DEV = "cuda:0"


@pytest.mark.parametrize("B,N", [(16, 300), (400, 300), (400, 12352), (700, 300), (3000, 300), (6000, 16448), (70000, 64)])
def test_replays_give_the_eager_result(B, N):
    rng = np.random.default_rng(B)
    F, per = 500, 9
    ix = torch.from_numpy(np.sort(np.stack([rng.choice(F, per, replace=False) for _ in range(B)]), 1)
                          .astype(np.int32).reshape(-1)).to(DEV)
    ip = torch.arange(0, B * per + 1, per, dtype=torch.int32, device=DEV)
    W = torch.rand((F, som.som_codebook_ldw(N)), device=DEV)
    norms = torch.empty(N, device=DEV)
    perm = torch.empty(B, dtype=torch.int32, device=DEV)
    bmu = torch.empty(B, dtype=torch.int32, device=DEV)
    dist = torch.empty(B, device=DEV)
    ws = torch.empty(som.som_cluster_workspace_bytes(B, F, ix.numel()), dtype=torch.uint8, device=DEV)

    def step():
        som.som_codebook_norms(W, N=N, norms=norms)
        som.som_cluster_order(ip, ix, F, perm=perm, ws=ws)
        som.som.som_bmu_search_noalloc(W, norms, ip, ix, N=N, perm=perm, bmu=bmu, dist=dist)

    side = torch.cuda.Stream(device=DEV)
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()                                  # (the scratch array's first lookup, outside the capture)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for k in range(4):
        W.uniform_()
        ix.copy_(ix.view(B, per).roll(1, 0).reshape(-1))
        bmu.fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        got = [t.clone() for t in (norms, perm, bmu, dist)]
        step()
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(got, (norms, perm, bmu, dist))), k
