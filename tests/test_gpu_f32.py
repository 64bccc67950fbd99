"""The fp32 assignment against 64 bits: the nearest centroid up to fp32 rounding,
at every row width it is built for and at the edges of its tiles, stages and
point blocks; and no more rounding than one per product and add."""
from __future__ import annotations

import pytest
import torch

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -24  # half an ulp, relative


@pytest.fixture(scope="module")
def km():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_2608_12629_amd import kmeans
    return kmeans


def _check(X, C, idx, md):
    """Every rounding of a sum of D products is at most EPS of the partial sum, which
    stays within |x|^2 + |c|^2 and grows evenly: a standard deviation of EPS sqrt(D / 3)
    / sqrt(3) of that, and one more EPS for |x|^2, |c|^2 and the last step; six of them
    as the bound of one value, one of them for all together."""
    X, C = X.double(), C.double()
    D = X.shape[1]
    xn, cn = (X * X).sum(1), (C * C).sum(1)
    d = xn[:, None] - 2 * X @ C.T + cn[None]
    best, ib = d.min(1)
    got = d.gather(1, idx.long()[:, None])[:, 0]
    sd = EPS * (D ** 0.5 / 3 + 1) * (xn + torch.maximum(cn[ib], cn[idx.long()]))
    assert bool((got - best <= 6 * sd).all()), float(((got - best) / sd).max())
    err = ((md.double() - got.clamp(min=0)) / sd).abs()
    assert float(err.max()) <= 6, float(err.max())
    assert float(err.square().mean().sqrt()) <= 1, float(err.square().mean().sqrt())


WIDTHS = [1, 3, 16, 32, 48, 64, 80, 96, 97, 112, 128, 144, 160, 176, 192, 208, 224, 240, 256]
SIZES = [(1, 1), (127, 33), (129, 64), (700, 65), (257, 129)]
# enough points for the larger point blocks of rows up to 64 and up to 128
# elements; an even and an odd number of stages
LARGE = [(16, 262200, 70), (48, 262200, 129), (64, 262200, 70), (96, 131100, 129), (128, 131100, 70)]


@pytest.mark.parametrize("D,N,K", [(D, N, K) for D in WIDTHS for N, K in SIZES] + LARGE)
def test_f32_assignment(km, D, N, K):
    g = torch.Generator(device="cuda").manual_seed(D * K + N)
    X = torch.randn((1, N, D), generator=g, device="cuda") + 3.0
    C = torch.randn((1, K, D), generator=g, device="cuda") + 3.0
    if K > 40:
        C[0, 40] = C[0, 7]  # equal rows: the lower index
        X[0, 0] = C[0, 7]
        C[0, 5, 0] = float("nan")
    idx, md = km.kmeans_assign(X, C)
    keep = torch.isfinite(C[0]).all(1)
    Cd = C[0].clone()
    Cd[~keep] = 1e3  # never nearest
    _check(X[0], Cd, idx[0], md[0])
    if K > 40:
        assert int(idx[0, 0]) == 7
        assert int((idx == 5).sum()) == 0 and int((idx == 40).sum()) == 0


# magnitudes far from 1
@pytest.mark.parametrize("e", [-30, 0, 30])
def test_f32_scales(km, e):
    g = torch.Generator(device="cuda").manual_seed(e + 100)
    X = torch.randn((1, 500, 64), generator=g, device="cuda") * 2.0 ** e
    C = torch.randn((1, 100, 64), generator=g, device="cuda") * 2.0 ** e
    idx, md = km.kmeans_assign(X, C)
    _check(X[0] * 2.0 ** -e, C[0] * 2.0 ** -e, idx[0], md[0].double() * 4.0 ** -e)


# rows and centroids whose scales differ by 2^40: each point's error is bounded
# by its own norm and that of the centroids it decides between
def test_f32_mixed_scales(km):
    g = torch.Generator(device="cuda").manual_seed(7)
    sx = 2.0 ** torch.randint(-20, 21, (600, 1), generator=g, device="cuda")
    sc = 2.0 ** torch.randint(-20, 21, (100, 1), generator=g, device="cuda")
    X = torch.randn((600, 64), generator=g, device="cuda") * sx
    C = torch.randn((100, 64), generator=g, device="cuda") * sc
    idx, md = km.kmeans_assign(X[None], C[None])
    _check(X, C, idx[0], md[0])


# One coordinate in use, x near c / 2 and c of 12 bits (c^2 / 2 exact): the score
# x c - c^2 / 2 is nearly 0 and, as one multiply-add, exact to its own half ulp, so
# min_dist = |x|^2 - 2 s has the rounding of |x|^2 and of the last step only.
# A product rounded by itself, or without its lowest bits, is off by up to four
# times that.
@pytest.mark.parametrize("D", [16, 32, 64, 96, 128, 256])
@pytest.mark.parametrize("N", [1000, 131100])
def test_f32_rounds_once_per_product(km, D, N):
    g = torch.Generator(device="cuda").manual_seed(D + N)
    for c, j in ((1.0 + 683 / 2048, 0), (1.0 + 1365 / 2048, D - 1)):
        X = torch.zeros((1, N, D), device="cuda")
        X[0, :, j] = 0.5 * c * (1 + 2.0 ** -6 * torch.rand(N, generator=g, device="cuda"))
        C = torch.zeros((1, 1, D), device="cuda")
        C[0, 0, j] = c
        _, md = km.kmeans_assign(X, C)
        x = X[0, :, j].double()
        s, want = x * c - c * c / 2, (x - c) ** 2
        tol = EPS * (x * x + want) * (1 + 2.0 ** -20) + 2 * EPS * s.abs()
        err = ((md[0].double() - want).abs() / tol).max()
        assert float(err) <= 1, float(err)


# a run equals its steps bit for bit
@pytest.mark.parametrize("B,N,D,K", [(1, 500, 3, 1), (2, 900, 16, 5), (1, 3000, 64, 63), (1, 3000, 64, 600),
                                     (3, 2500, 128, 300), (1, 2000, 256, 500), (1, 1200, 256, 1150)])
def test_f32_lloyd_equals_steps(km, B, N, D, K):
    g = torch.Generator(device="cuda").manual_seed(N + K)
    X = torch.randn((B, N, D), generator=g, device="cuda")
    C = X[:, :K].clone()
    out = km.kmeans_lloyd(X, C.clone(), 3)
    for _ in range(3):
        idx, md = km.kmeans_assign(X, C)
        C, n = km.kmeans_update(X, idx, C)
    assert torch.equal(out[1], idx) and torch.equal(out[2], md) and torch.equal(out[3], n)
    assert torch.equal(out[0].view(torch.int32), C.view(torch.int32))
