"""GPU checks of the automatic launch's list form (tiles of 256 documents for
fp32, 128 for fp16; per-wave entry lists) at the sizes where it can go wrong:
the batch sizes its forms start at (fp32: 513 documents, in kernel 3's order, and
65,536, in its own; fp16: 65,536) and ragged last tiles, unions of one stage and of
one row more, documents with no feature and with more than two 64-lane reads of
them, maps around the slice width, the largest vocabulary it takes, rows of 4 GB
and more, and plans searched with the other storage type.

The codebooks are dyadic (W in {0, 1/4, 1/2, 3/4}), so every fp32 sum is exact
and every order of summation must give kernel 1's bits; kernel 1 faces the
oracle in the parity tests.  On a random codebook the ascending sweep must give
kernel 1's bits as well."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2609_05138_amd as som
else:  # collected on CPU-only machines, never run there
    som = None

DEV = "cuda:0"
# batches from which a form of the list kernel is taken
FORMS = [(np.float32, 513), (np.float32, 65536), (np.float16, 65536)]


def _csr(key, B, F):
    """CSR tensors of the distinct (document, feature) pairs in key = document * F + feature."""
    key = np.unique(key)
    indptr = np.concatenate([[0], np.cumsum(np.bincount(key // F, minlength=B))])
    return (torch.from_numpy(indptr.astype(np.int32)).to(DEV), torch.from_numpy((key % F).astype(np.int32)).to(DEV))


def _docs(rng, B, F):
    """CSR batch: mostly short documents over frequent ids, every 37th empty,
    every 101st with as many features as F allows up to 300."""
    n = np.minimum(rng.poisson(min(12, F / 2), B), F)
    n[::37] = 0
    n[1::101] = min(F, 300)
    short = n <= F // 4
    doc = np.repeat(np.arange(B, dtype=np.int64)[short], n[short])
    keys = [doc * F + np.minimum((F * rng.random(doc.size) ** 3).astype(np.int64), F - 1)]
    for d in np.flatnonzero(~short):                      # exactly n[d] distinct features
        keys.append(d * F + rng.choice(F, n[d], replace=False))
    return _csr(np.concatenate(keys), B, F)


def _book(rng, F, N, dtype, ldw=None, dyadic=True):
    W = torch.zeros((F, ldw or som.som_codebook_ldw(N)), dtype=torch.float16 if dtype == np.float16 else torch.float32,
                    device=DEV)
    v = rng.integers(0, 4, (F, N)) / 4 if dyadic else rng.random((F, N), dtype=np.float32)
    W[:, :N] = torch.from_numpy(v.astype(dtype)).to(DEV)
    return W, som.som_codebook_norms(W, N=N)


def _auto(top2, W, norms, ip, ix, N, perm=None, sweep=0):
    """The automatic search, and that it took the list form where it should: its
    plan, at the start of the workspace, then bears the list plan's mark."""
    B, F = ip.numel() - 1, W.shape[0]
    ws = torch.empty(som.som_bmu_workspace_bytes(F, N, B, ix.numel(), sweep=sweep), dtype=torch.uint8, device=DEV)
    got = (som.som_bmu_search_top2 if top2 else som.som_bmu_search)(W, norms, ip, ix, N=N, perm=perm, ws=ws, sweep=sweep)
    listed = F <= 65536 and (B >= 65536 or (W.dtype == torch.float32 and sweep != 1 and 512 < B <= 12288))
    if F > 1:      # (one feature: the list plan does not fit the fp16 tile plan's bytes)
        assert (int(ws[:4].view(torch.int32)) < 0) == listed
    return got


def _equal(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("dtype,least", FORMS)
@pytest.mark.parametrize("extra,F,N", [(-1, 300, 200), (0, 64, 128), (1, 65, 127), (255, 2000, 129), (256, 64, 1),
                                       (300, 65536, 300), (130, 5000, 513), (1000, 1, 2)])
def test_list_form_matches_kernel_1(dtype, least, extra, F, N):
    rng = np.random.default_rng(F * 1000 + N)
    B = least + extra
    ip, ix = _docs(rng, B, F)
    perm = som.som_cluster_order(ip, ix, F)
    W, norms = _book(rng, F, N, dtype)
    for p in (None, perm):
        want = som.som_bmu_search_top2(W, norms, ip, ix, N=N, perm=p, kernel=1, sweep=1)
        for sweep in (0, 1):
            assert _equal(_auto(True, W, norms, ip, ix, N, p, sweep), want), (sweep, p is None)
            assert _equal(_auto(False, W, norms, ip, ix, N, p, sweep), want[:2]), sweep


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("B", [6000, 66000])
def test_list_form_ascending_bits_and_reuse_of_a_plan(dtype, B):
    rng = np.random.default_rng(7)
    F, N = 3000, 1000
    ip, ix = _docs(rng, B, F)
    perm = som.som_cluster_order(ip, ix, F)
    W, norms = _book(rng, F, N, dtype, dyadic=False)
    want = som.som_bmu_search_top2(W, norms, ip, ix, N=N, perm=perm, kernel=1, sweep=1)
    assert _equal(som.som_bmu_search_top2(W, norms, ip, ix, N=N, perm=perm, sweep=1), want)
    # a plan made for either storage type serves both, with the same bits
    other = W.to(torch.float16 if dtype == np.float32 else torch.float32)
    other_norms = som.som_codebook_norms(other, N=N)
    for storage in (0, 1):
        for sweep in (0, 1):
            plan = som.som_plan(ip, ix, F, perm=perm, storage=storage, sweep=sweep)
            mine = som.som_bmu_search_top2_planned(W, norms, ip, plan, N=N)
            assert _equal(som.som_bmu_search_planned(W, norms, ip, plan, N=N), mine[:2])
            if sweep == 1:
                assert _equal(mine, want), storage
            half = som.som_bmu_search_top2_planned(other, other_norms, ip, plan, N=N)
            if dtype == np.float16:      # the widened codebook holds the same values
                assert _equal(half, mine), (storage, sweep)


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("B", [1, 2, 3, 64, 65, 512, 513, 700, 767, 768, 1023])
def test_small_batches_match_kernel_1(dtype, B):
    # two-document tiles of kernel 1 (up to 512 documents, fp16 64), and the
    # kernels between them and the list form
    rng = np.random.default_rng(B)
    F, N = 900, 700
    ip, ix = _docs(rng, B, F)
    W, norms = _book(rng, F, N, dtype)
    want = som.som_bmu_search_top2(W, norms, ip, ix, N=N, kernel=1, tile_docs=8, sweep=1)
    assert _equal(som.som_bmu_search_top2(W, norms, ip, ix, N=N), want)
    plan = som.som_plan(ip, ix, F, storage=1 if dtype == np.float16 else 0)
    assert _equal(som.som_bmu_search_planned(W, norms, ip, plan, N=N), want[:2])
    if dtype == np.float32:
        assert _equal(som.som.som_bmu_search_noalloc(W, norms, ip, ix, N=N), want[:2])


def test_list_form_rows_of_4_gib():
    rng = np.random.default_rng(11)
    F, N, B = 2, 300, 1700
    ip, ix = _docs(rng, B, F)
    W, norms = _book(rng, F, N, np.float32, ldw=(1 << 30) + 64)
    want = som.som_bmu_search_top2(W, norms, ip, ix, N=N, kernel=1, sweep=1)
    assert _equal(_auto(True, W, norms, ip, ix, N), want)
    assert _equal(_auto(False, W, norms, ip, ix, N), want[:2])


def test_list_form_on_more_slices_than_one_launch_takes():
    # 128-neuron slices: a grid holds 65,535 of them, a wider map takes two
    rng = np.random.default_rng(13)
    F, N, B = 2, 65535 * 128 + 300, 520
    ip, ix = _docs(rng, B, F)
    W = torch.zeros((F, som.som_codebook_ldw(N)), device=DEV)
    W[0, :N] = (torch.arange(N, device=DEV) % 4096) / 4096      # dyadic, the minima in the last slices
    W[1, :N] = 1.0
    W[:, N - 200:N - 1] = torch.tensor([[0.75], [0.5]], device=DEV)
    norms = som.som_codebook_norms(W, N=N)
    norms[N - 200:] -= 2.0                                       # (norms are an input: these units win)
    want = som.som_bmu_search_top2(W, norms, ip, ix, N=N, kernel=1, sweep=1)
    assert int(want[0].min()) > 65535 * 128
    got = som.som_bmu_search_top2(W, norms, ip, ix, N=N)
    assert _equal(got, want)
    assert _equal(som.som_bmu_search(W, norms, ip, ix, N=N), want[:2])


@pytest.mark.parametrize("dtype,least", FORMS)
@pytest.mark.parametrize("dense,share,F", [(15, 0.5, 400), (16, 0.4, 400), (17, 1.0, 32768), (64, 0.3, 65), (63, 0.3, 300),
                                           (100, 0.5, 3000), (40, 0.25, 500), (64, 1.0, 64), (40, 0.5, 32769)])
def test_rows_that_many_documents_hold(dtype, least, dense, share, F):
    # such rows of a tile (from 16 of them on, at most 64) are summed on the matrix
    # cores (fp32, from 65,536 documents on)
    rng = np.random.default_rng(dense * 7 + F)
    B, N = least + 300, 300
    hot = np.sort(rng.choice(F, dense, replace=False))
    at = np.flatnonzero(rng.random(B * dense) < share)
    doc = np.repeat(np.arange(B, dtype=np.int64), rng.integers(0, 9, B))
    key = np.concatenate([at // dense * F + hot[at % dense], doc * F + rng.integers(0, F, doc.size)])
    key = key[(key // F != 5) & (key // F != B - 1)]
    ip, ix = _csr(key, B, F)
    W, norms = _book(rng, F, N, dtype)
    for special in (False, True):
        if special:   # 0 times an infinity or a NaN is no 0; finite norms, so that they show
            # (the NaN in the last neuron of every kernel's lane: a lane takes its
            # first neuron before it compares, whatever its distance)
            W[hot[0], 3], W[hot[1], 7], W[hot[-1], 70], W[hot[2], 299] = np.inf, np.nan, -np.inf, np.inf
            norms[:N:3] *= 0.5
        want = som.som_bmu_search_top2(W, norms, ip, ix, N=N, kernel=1, sweep=1)
        for sweep in (0, 1):
            assert _equal(_auto(True, W, norms, ip, ix, N, sweep=sweep), want), (special, sweep)
            assert _equal(_auto(False, W, norms, ip, ix, N, sweep=sweep), want[:2]), (special, sweep)


@pytest.mark.parametrize("dtype,least", FORMS)
@pytest.mark.parametrize("N", [1, 2, 3, 5, 127, 129, 130, 131, 257, 260, 261, 510])
def test_what_lies_between_the_rows_is_never_a_unit(dtype, least, N):
    # the columns from N to the row stride hold no neuron: a NaN there whose sign
    # bit is set would come before every distance
    rng = np.random.default_rng(N)
    B, F = least + 77, 200
    ip, ix = _docs(rng, B, F)
    W, norms = _book(rng, F, N, dtype)
    W[:, N:].view(torch.int16 if dtype == np.float16 else torch.int32).fill_(-1)
    want = som.som_bmu_search_top2(W, norms, ip, ix, N=N, kernel=1, sweep=1)
    for sweep in (0, 1):
        assert _equal(_auto(True, W, norms, ip, ix, N, sweep=sweep), want), sweep
        assert _equal(_auto(False, W, norms, ip, ix, N, sweep=sweep), want[:2]), sweep
    # where no distance is a number, there is no best unit, but the answer is one of the map
    for bits in (0x7fc00000, -1):
        norms.view(torch.int32).fill_(bits)
        bmu, _, bmu2, _ = som.som_bmu_search_top2(W, norms, ip, ix, N=N)
        assert 0 <= int(bmu.min()) and int(bmu.max()) < N
        assert -1 <= int(bmu2.min()) and int(bmu2.max()) < N
