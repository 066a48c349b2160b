"""GPU k-means of small calls (all iterations in one launch) against the paths that launch every step: labels, counts,
centroids and the second tensor's means are the same bits, at the edges of blocks of centroids (32), groups of clusters
(2, 4, 8), tiles, clusters summed in parts, with text rows, strides, empty and lopsided clusters, iterations that leave
clusters as they are and rows without a finite score."""
import pytest
import torch

import paper_2603_08982_amd as sv
from helpers import dev, kmeans_as

pytestmark = pytest.mark.gpu


def _both(x, start, iters, tail, x2):
    got = []
    for form in ("one launch", "steps"):
        c = start.clone()
        labels, counts, c2 = kmeans_as(form, x, c, iters, tail, x2=x2)
        torch.cuda.synchronize()
        got.append((labels, counts, c) + ((c2,) if x2 is not None else ()))
    for a, b in zip(*got):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))


def _rows(H, N, d, dtype, seed, spread=40):
    g = torch.Generator().manual_seed(seed)
    mu = torch.randn(spread, d, generator=g)
    return (mu[torch.randint(0, spread, (H, N), generator=g)] + 0.3 * torch.randn(H, N, d, generator=g)).to(dtype)[None].to(dev())


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,N,tail,C", [
    (1, 2, 1, 1), (1, 33, 0, 33), (2, 257, 5, 2), (3, 640, 7, 31), (2, 667, 37, 32), (2, 700, 0, 33), (1, 4096, 0, 64),
    (1, 900, 3, 65), (5, 1000, 0, 129), (1, 2049, 1, 8), (2, 5000, 0, 3), (12, 1200, 0, 100), (17, 650, 9, 90),
    (1, 16384, 0, 80), (1, 16385, 0, 80), (8, 9600, 0, 24), (1, 4999, 0, 10), (2, 9600, 0, 100), (1, 9000, 0, 1000), (40, 600, 0, 10), (300, 64, 0, 5),
    (24, 3528, 0, 24), (8, 2376, 0, 226), (1, 13300, 0, 20), (5, 6000, 1, 9),
])
def test_small_calls_agree_with_the_step_by_step_paths(H, N, tail, C, d, dtype):
    x, x2 = _rows(H, N, d, dtype, 1), _rows(H, N, d, dtype, 2)
    g = torch.Generator().manual_seed(3)
    start = torch.stack([x[0, h, torch.randperm(N - tail, generator=g)[:C].to(dev())].float() for h in range(H)])[None].contiguous()
    if C > 2:
        start[0, 0, 1] = 1e6  # a cluster without rows
    for iters in (1, 2, 5, 12):
        _both(x, start, iters, tail, x2 if iters != 2 else None)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,N,C", [(2, 3000, 6), (2, 3000, 40), (16, 1200, 40), (24, 1200, 48)])  # 4, 4, 2, 1 waves a cluster
def test_lopsided_clusters_strided_and_nonfinite_rows(H, N, C, d):
    x = _rows(H, N, d, torch.bfloat16, 5, spread=1)  # one blob: nearly all rows go to the centroid in its middle
    start = x[:, :, :C].float() * 3.0
    start[:, :, C // 2] = x.float().mean(2)
    x = x[0].transpose(0, 1).contiguous().transpose(0, 1)[None]  # heads interleaved along a token
    _both(x, start.contiguous(), 4, 11, x)
    x[0, 0, 100, 3], x[0, 1, 200, 5] = float("nan"), float("inf")
    _both(x, start.contiguous(), 1, 0, None)


def test_more_iterations_than_the_one_launch_counts():
    """65,537 iterations, past the last of which the tasks of a launch are no longer sure to be counted in 32 bits."""
    x = _rows(1, 64, 64, torch.float32, 8)
    start = x[:, :, :3].contiguous()
    got = []
    for iters in (65537, 100):
        c = start.clone()
        labels, counts, _ = sv.kmeans(x, c, iters)
        got.append((labels, counts, c))
    for a, b in zip(*got):
        assert torch.equal(a, b)
