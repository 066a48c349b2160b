"""GPU k-means on both sides of the lines between its forms: the smallest calls run in one launch; launched step by
step, small bf16 calls assign every row exactly, larger ones filter first (and, with the list threshold at 1, small
ones too), in workgroups of two or four waves. The forms give the same labels, counts and centroids bit for bit, also for strided rows and
with text rows, and the labels are the oracle's."""
import numpy as np
import pytest
import torch

from oracle import svgear_oracle as orc
from helpers import KMEANS_FORMS, dev, kmeans_as, to_np

pytestmark = pytest.mark.gpu


def _rows(H, N, d, dtype, strided, seed):
    g = torch.Generator().manual_seed(seed)
    mu = torch.randn(24, d, generator=g)
    x = (mu[torch.randint(0, 24, (H, N), generator=g)] + 0.3 * torch.randn(H, N, d, generator=g)).to(dtype)
    if strided:  # heads interleaved along a token, as a projection leaves them
        return x.transpose(0, 1).contiguous().to(dev()).transpose(0, 1)[None]
    return x[None].to(dev())


@pytest.mark.parametrize("H,N,tail,C,d,dtype", [
    (2, 32768, 0, 128, 64, torch.bfloat16), (2, 32769, 0, 128, 64, torch.bfloat16),   # 256 and 258 blocks of 256 rows
    (2, 700, 37, 128, 128, torch.bfloat16), (2, 700, 37, 129, 128, torch.bfloat16),   # two and three chunks of centroids
    (1, 16384, 0, 40, 128, torch.bfloat16), (1, 16385, 1, 40, 128, torch.bfloat16),   # 64 and 65 blocks
    (3, 33, 0, 33, 64, torch.bfloat16), (1, 2, 1, 1, 128, torch.bfloat16),
    (1, 16384, 0, 70, 64, torch.float32), (1, 16385, 0, 70, 64, torch.float32), (4, 650, 11, 130, 128, torch.float32),
])
@pytest.mark.parametrize("strided", [False, True])
def test_forms_agree(H, N, tail, C, d, dtype, strided):
    x, x2 = _rows(H, N, d, dtype, strided, 1), _rows(H, N, d, dtype, strided, 2)
    start = torch.stack([x[0, h, : N - tail][torch.randperm(N - tail, generator=torch.Generator().manual_seed(h))[:C].to(dev())]
                         for h in range(H)])[None].float().contiguous()
    for iters in (1, 4):
        got = []
        for form in KMEANS_FORMS:
            c = start.clone()
            labels, counts, c2 = kmeans_as(form, x, c, iters, tail, x2=x2)
            torch.cuda.synchronize()
            got.append((labels, counts, c, c2))
        for a, b, e in zip(*got):
            assert torch.equal(a, b) and torch.equal(a, e)
        if iters == 1:
            for h in range(H):
                assert np.array_equal(to_np(got[0][0][0, h]), orc.kmeans_assign(to_np(x[0, h])[: N - tail], to_np(start[0, h])))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,N,C", [(1, 63, 9), (2, 65, 40), (3, 2049, 33), (2, 4096, 130), (1, 6001, 700), (2, 3000, 5)])
@pytest.mark.parametrize("spread", [0.3, 3.0])
def test_candidate_lists_over_many_iterations(H, N, C, d, spread):
    """Rows tested against candidate lists only where moved neighbours do not prove their label (a bit per row, words of
    64; clusters of more than the 256 positions a wave takes; lists of one to more than 128 centroids): after every
    number of iterations the same labels and centroids as testing every centroid."""
    g = torch.Generator().manual_seed(N + C)
    mu = torch.randn(max(2, C // 4), d, generator=g)
    x = (mu[torch.randint(0, len(mu), (H, N), generator=g)] + spread * torch.randn(H, N, d, generator=g)).bfloat16()[None].to(dev())
    start = x[:, :, torch.randperm(N, generator=g)[:C].to(dev())].float().contiguous()
    for iters in (3, 4, 5, 9, 14):
        got = []
        for form in ("lists", "steps"):
            c = start.clone()
            labels, counts, _ = kmeans_as(form, x, c, iters)
            torch.cuda.synchronize()
            got.append((labels, counts, c))
        for a, b in zip(*got):
            assert torch.equal(a, b)
