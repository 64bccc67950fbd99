"""Calls with few points, whose centroids are shared out among workgroups: the
same points among so many instances that nothing is shared give the same bits."""
from __future__ import annotations

import pytest
import torch

pytestmark = pytest.mark.gpu
DT = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}


@pytest.fixture(scope="module")
def km():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_2608_12629_amd import kmeans
    return kmeans


# one point; a block and one more; 64-row stages (D = 256) with a short last
# share; four point tiles a wave (D <= 64); widths that are padded; rows past
# 256 elements, whose workgroups take fewer centroid blocks; tie-heavy
# duplicates are in every case (the second half of C
# repeats the first)
@pytest.mark.parametrize("N,D,K,dt,B", [
    (1, 128, 2050, "bf16", 513), (257, 128, 4100, "f16", 260), (130, 256, 3001, "bf16", 260),
    (513, 32, 5000, "f16", 260), (100, 100, 2500, "bf16", 520), (65, 200, 2222, "f16", 520),
    (100, 320, 2500, "bf16", 260), (300, 512, 1100, "f16", 300),
    (100, 64, 1100, "f32", 520), (257, 96, 1030, "f32", 300), (200, 128, 600, "f32", 400),
])
def test_shared_centroids_same_bits(km, N, D, K, dt, B):
    g = torch.Generator().manual_seed(N + D + K)
    X = torch.randn((1, N, D), generator=g)
    if N > 4:
        X[0, 1] = float("nan")
        X[0, 2, 0] = float("inf")
    if N > 256:
        X[0, 256:] *= 100.0  # a block whose norms spread widely, and its own point shifts
        X[0, 3] *= 100.0
    C = torch.randn((1, K, D), generator=g)
    C[0, K // 2:] = C[0, :K - K // 2].clone()
    C[0, 7] = float("nan")
    X, C = X.to(DT[dt]).cuda(), C.cuda()
    idx, md = km.kmeans_assign(X, C)
    Xb, Cb = X.expand(B, N, D).contiguous(), C.expand(B, K, D).contiguous()
    idx_b, md_b = km.kmeans_assign(Xb, Cb)
    assert torch.equal(idx_b, idx.expand(B, N))
    assert torch.equal(md_b.view(torch.int32), md.view(torch.int32).expand(B, N))
    ok = idx[0] >= 0
    assert int((~ok).sum()) == (2 if N > 4 else 0)
    d = (X[0].double()[ok][:, None] - C[0].to(DT[dt]).double()[None].nan_to_num(1e4)).square().sum(-1)
    best = d.min(1).values
    got = d.gather(1, idx[0][ok].long()[:, None])[:, 0]
    xn = X[0].double()[ok].square().sum(-1)
    assert bool((got - best <= 1e-3 * xn).all())
    # objective and state of a Lloyd step, one instance against many
    J = torch.empty((1, 1), dtype=torch.float64, device="cuda")
    Jb = torch.empty((B, 1), dtype=torch.float64, device="cuda")
    C1, Cb1 = C.clone(), Cb.clone()
    km.kmeans_lloyd(X, C1, 1, objective=J)
    km.kmeans_lloyd(Xb, Cb1, 1, objective=Jb)
    assert torch.equal(Jb, J.expand(B, 1))
    assert torch.equal(Cb1.view(torch.int32), C1.view(torch.int32).expand(B, K, D))


# rows past 256 elements: point blocks in either order (79 and 136 plain, 258 in
# super-tiles, 60 in one), few enough for fewer centroid blocks a workgroup: a
# point's bits do not depend on the others of its call
@pytest.mark.parametrize("D,K", [(288, 300), (320, 2100)])
def test_wide_block_orders_same_bits(km, D, K):
    g = torch.Generator(device="cuda").manual_seed(D)
    X = torch.randn((1, 66_000, D), generator=g, device="cuda").to(torch.bfloat16)
    C = torch.randn((1, K, D), generator=g, device="cuda")
    idx, md = km.kmeans_assign(X, C)
    for N in (1, 256, 2_049, 15_300, 20_001, 34_600, 50_100, 65_800):
        i, m = km.kmeans_assign(X[:, :N].contiguous(), C)
        assert torch.equal(i, idx[:, :N]) and torch.equal(m, md[:, :N]), N
    n = 2_000  # and the bits are those of the nearest centroids
    x, c = X[0, -n:].double(), C[0].to(torch.bfloat16).double()
    d = (x * x).sum(1)[:, None] - 2 * x @ c.T + (c * c).sum(1)[None]
    got = d.gather(1, idx[0, -n:].long()[:, None])[:, 0]
    assert bool((got - d.min(1).values <= 1e-3 * (x * x).sum(1)).all())


# the update's sort: one pass (9 and 10 bits, a chunk, a chunk and one), the
# largest one-bit-short and full digit, two passes from 1,025 clusters on and
# where a batch has too many bins; every K with ids outside [0, K) among idx
@pytest.mark.parametrize("B,N,K", [(1, 4097, 257), (1, 4096, 512), (2, 9001, 513), (1, 12289, 1000),
                                   (3, 5000, 1024), (1, 9001, 1025), (9, 4500, 1024), (1, 5000, 160)])
def test_update_sort_passes(km, B, N, K):
    D = 128
    g = torch.Generator().manual_seed(N + K)
    X = torch.randn((B, N, D), generator=g).to(torch.bfloat16)
    idx = torch.randint(-1, K + 1, (B, N), generator=g, dtype=torch.int32)
    idx[:, : N // 3] = K - 1  # one cluster longer than any slice
    C = torch.randn((B, K, D), generator=g)
    out, n = km.kmeans_update(X.cuda(), idx.cuda(), C.cuda())
    ref, cnt = torch.zeros((B, K, D), dtype=torch.float64), torch.zeros((B, K), dtype=torch.int64)
    for b in range(B):
        ok = (idx[b] >= 0) & (idx[b] < K)
        i = idx[b][ok].long()
        ref[b].index_add_(0, i, X[b][ok].double())
        cnt[b] = torch.bincount(i, minlength=K)
    assert torch.equal(n.cpu().long(), cnt)
    ref = torch.where(cnt[..., None] > 0, ref / cnt[..., None].clamp(min=1), C.double())
    # fp32 sums of up to 4,000 unit normals: errors stay near 2^-24 sqrt(n) of a mean of |x| = 0.8
    err = (out.cpu().double() - ref).abs().max()
    assert float(err) < 1e-5, float(err)
