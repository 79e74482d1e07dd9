"""The wide-neighbourhood blur (radii above 16) where its launch changes form:
single cells, rows and columns, maps narrower than the radius, ragged groups of
eight outputs, 32- and 16-column strips, and the strip that exceeds the LDS.

Every numerator and denominator is two fp32 sums of at most 2 R + 1 positive
terms with taps rounded once, so each is within (4 R + 8) u of the exact one (u =
2^-24), their quotient within twice that and u; fp16 weights round once more."""

import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2609_05138_amd as som
else:  # collected on CPU-only machines, never run there
    som = None

DEV = "cuda:0"


def _band(n, sigma):
    k = torch.arange(n, dtype=torch.float64, device=DEV)
    d = (k[:, None] - k[None, :]).abs()
    return torch.where(d <= math.ceil(3 * sigma), torch.exp(-d * d / (2 * sigma * sigma)), torch.zeros_like(d))


@pytest.mark.parametrize("f16", [False, True])
@pytest.mark.parametrize("rows,cols,sigma", [(1, 1, 6.0), (1, 50, 6.0), (50, 1, 6.0), (7, 9, 20.0), (8, 16, 5.5),
                                             (33, 65, 5.5), (17, 2100, 6.0), (600, 40, 9.0), (700, 24, 60.0),
                                             (1024, 33, 200.0), (3, 16384, 400.0)])
def test_wide_blur_matches_the_exact_means(rows, cols, sigma, f16):
    g = torch.Generator(device=DEV)
    g.manual_seed(rows * 31 + cols)
    F, N = 3, rows * cols
    acc = torch.randint(0, 5, (F, N + 5), device=DEV, dtype=torch.int32, generator=g)
    count = torch.randint(0, 5, (N,), device=DEV, dtype=torch.int32, generator=g)
    W0 = torch.rand((F, som.som_codebook_ldw(N)), device=DEV, generator=g)
    W = W0.half() if f16 else W0.clone()
    old = W.clone()
    som.som_update_finish(W, rows, cols, sigma, acc, count)
    R, C = _band(rows, sigma), _band(cols, sigma)
    den = R @ count.double().reshape(rows, cols) @ C
    radius = math.ceil(3 * sigma)
    u = 2.0 ** -24
    tol = 2 * (4 * min(radius, max(rows, cols)) + 8) * u + u + (2.0 ** -11 if f16 else 0)
    for f in range(F):
        num = R @ acc[f, :N].double().reshape(rows, cols) @ C
        want = torch.where(den > 0, num / den, old[f, :N].double().reshape(rows, cols)).reshape(-1)
        got = W[f, :N].double()
        # the smallest fp16 steps are 2^-24 apart
        assert bool(((got - want).abs() <= tol * want.abs() + (2.0 ** -25 if f16 else 1e-30)).all()), f
    assert torch.equal(W[:, N:], old[:, N:])
