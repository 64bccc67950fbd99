"""The fp32 assignment in three bf16 pieces, against 64 bits: the nearest centroid
up to fp32 rounding, at every row width it is built for and at the edges of its
tiles, stages and point blocks."""
from __future__ import annotations

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def km():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_2608_12629_amd import kmeans
    return kmeans


def _check(X, C, idx, md, scale):
    X, C = X.double(), C.double()
    d = (X * X).sum(1)[:, None] - 2 * X @ C.T + (C * C).sum(1)[None]
    best = d.min(1).values
    got = d.gather(1, idx.long()[:, None])[:, 0]
    # fp32 sums of D products and of |c|^2 / 2: a few ulp of |x||c| + |c|^2, twice over
    tol = 2e-6 * scale
    assert bool((got - best <= tol).all()), float((got - best).max() / scale)
    assert bool(((md.double() - got.clamp(min=0)).abs() <= tol).all())


@pytest.mark.parametrize("D", [1, 3, 16, 32, 48, 64, 80, 96, 97, 112, 128, 144, 160, 176, 192, 208, 224, 240, 256])
@pytest.mark.parametrize("N,K", [(1, 1), (127, 33), (129, 64), (700, 65), (257, 129), (131100, 70)])
def test_f32_assignment(km, D, N, K):
    if N > 10000 and D not in (16, 48, 64, 96):
        pytest.skip("two point tiles a wave: few widths")
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
    _check(X[0], Cd, idx[0], md[0], 10.0 * 4 * D)
    if K > 40:
        assert int(idx[0, 0]) == 7
        assert int((idx == 5).sum()) == 0 and int((idx == 40).sum()) == 0


# magnitudes far from 1, and rows whose scales differ by 2^40
@pytest.mark.parametrize("e", [-30, 0, 30])
def test_f32_scales(km, e):
    g = torch.Generator(device="cuda").manual_seed(e + 100)
    X = torch.randn((1, 500, 64), generator=g, device="cuda") * 2.0 ** e
    C = torch.randn((1, 100, 64), generator=g, device="cuda") * 2.0 ** e
    idx, md = km.kmeans_assign(X, C)
    _check(X[0] * 2.0 ** -e, C[0] * 2.0 ** -e, idx[0], md[0].double() * 4.0 ** -e, 4.0 * 64)


# images that the update rewrites, with padding rows shared out (K = 1 .. 63),
# and images that do not fit beside the sums (prepared by each iteration) or at
# all (the fp32 matrix instructions): a run equals its steps bit for bit
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
