"""Codebook norms at the edges of the launch's three shapes (64, 16 or 4 lanes
per row): the last narrow map and the first wide one of each, and row counts
around a whole pass of a workgroup's waves and chains."""

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2609_05138_amd as som
else:  # collected on CPU-only machines, never run there
    som = None

E = {torch.float32: 4, torch.float16: 8}     # weights per 128-bit load


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("lanes,groups", [(4, 1), (16, 128), (64, 256)])
@pytest.mark.parametrize("F", [1, 31, 33, 1023, 1025])
def test_norms_at_the_shape_edges(dtype, lanes, groups, F):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(F * 7 + lanes)
    first = E[dtype] * lanes * (groups - 1) + 1          # neurons of the narrowest map of this shape
    for N in (first, first + 2, max(1, first - 1)):
        W = torch.rand((F, som.som_codebook_ldw(N)), device="cuda:0", generator=g).to(dtype)
        got = som.som_codebook_norms(W, N=N)
        want = (W[:, :N].double() ** 2).sum(0)
        # 64-bit sums in another order, rounded once: the same fp32 value or,
        # next to a half-way point, its neighbour
        w32 = want.float()
        ulps = (got.view(torch.int32) - w32.view(torch.int32)).abs()
        assert int(ulps.max()) <= 1 and int((ulps > 0).sum()) <= max(1, N // 1000), N
