"""Assignment of 16-bit rows of any width read in place: the same bits as on rows
the caller padded with zeros to the kernels' width."""
from __future__ import annotations

import pytest
import torch

pytestmark = pytest.mark.gpu
DT = {"bf16": torch.bfloat16, "f16": torch.float16}


@pytest.fixture(scope="module")
def km():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_2608_12629_amd import kmeans
    return kmeans


# one element into a 16-element piece, one short of it, half of it, each for
# 1, 2 and 4 point tiles a wave; instances that start off a 16-byte boundary;
# one point; K <= 256 past D = 96 and K > 256 (the kernel that reads in place)
@pytest.mark.parametrize("D", [17, 31, 40, 63, 65, 88, 95, 100, 113, 127, 129, 145, 200, 241, 255])
@pytest.mark.parametrize("B,N,K,dt", [(1, 1, 300, "f16"), (3, 517, 260, "bf16"), (1, 1000, 2100, "f16")])
def test_ragged_rows_same_bits(km, D, B, N, K, dt):
    g = torch.Generator().manual_seed(D * N + K)
    X = torch.randn((B, N, D), generator=g).to(DT[dt])
    C = torch.randn((B, K, D), generator=g)
    X[:, N // 2:] *= 30 if B == 3 else 1  # blocks whose norms spread widely
    if N > 1:
        X[0, 5, D - 1] = float("nan")
        C[0, 9, D - 1] = float("inf")
    Dk = -(-D // 16) * 16
    Xp = torch.zeros((B, N, Dk), dtype=X.dtype)
    Cp = torch.zeros((B, K, Dk))
    Xp[..., :D], Cp[..., :D] = X, C
    idx, md = km.kmeans_assign(X.cuda(), C.cuda())
    idx_p, md_p = km.kmeans_assign(Xp.cuda(), Cp.cuda())
    assert torch.equal(idx, idx_p)
    assert torch.equal(md.view(torch.int32), md_p.view(torch.int32))
    assert int((idx < 0).sum()) == (1 if N > 1 else 0)
