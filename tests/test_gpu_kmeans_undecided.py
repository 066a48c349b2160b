"""GPU k-means, bf16: the rows that the bf16 filter cannot decide, by number of candidates, and the same rows
where every score is exact (one launch; steps of up to 128 centroids). Repeated centroids tie exactly (the
lowest index wins); a few of them stay within the candidate list of a workgroup, many overflow it. Labels are
whole numbers and equal the oracle's."""
import numpy as np
import pytest
import torch

from oracle import svgear_oracle as orc
from helpers import KMEANS_FORMS, dev, kmeans_as, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", KMEANS_FORMS)  # ("lists": the filter at any number of centroids)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("copies", [1, 2, 10, 16, 17, 40, 130])
def test_labels_among_repeated_centroids(d, copies, form):
    rng = np.random.default_rng(copies + d)
    base, N = 7, 1000
    cent = rng.standard_normal((base, d)).astype(np.float32)
    C = base * copies
    order = rng.permutation(C)
    table = np.repeat(cent, copies, 0)[order]
    x = torch.from_numpy(cent[rng.integers(0, base, N)] + 0.2 * rng.standard_normal((N, d)).astype(np.float32)).to(torch.bfloat16)
    # rows near the middle of two centroids, and rows of zeros
    for i in range(0, 200):
        a, b = rng.choice(base, 2, replace=False)
        x[i] = torch.from_numpy(0.5 * (cent[a] + cent[b])).to(torch.bfloat16)
    x[500:520] = 0
    g = torch.from_numpy(np.stack([table, table[::-1].copy()])).unsqueeze(0).to(dev())
    X = x[None, None].expand(1, 2, N, d).contiguous().to(dev())
    labels, _, _ = kmeans_as(form, X, g, 1)
    torch.cuda.synchronize()
    for h, t in enumerate((table, table[::-1].copy())):
        assert np.array_equal(to_np(labels[0, h]), orc.kmeans_assign(x.float().numpy(), t))


@pytest.mark.parametrize("form", KMEANS_FORMS)
@pytest.mark.parametrize("C", [3, 200])
def test_rows_without_a_finite_score_go_to_centroid_0(C, form):
    rng = np.random.default_rng(C)
    d, N = 128, 700
    x = torch.from_numpy(rng.standard_normal((N, d)).astype(np.float32)).to(torch.bfloat16)
    bad = rng.choice(N, 90, replace=False)
    x[bad[:45], 3] = float("nan")
    x[bad[45:], 5] = float("inf")
    cent = np.abs(rng.standard_normal((C, d))).astype(np.float32) * -1.0  # +inf rows: every score is +inf
    g = torch.from_numpy(cent)[None, None].contiguous().to(dev())
    labels, _, _ = kmeans_as(form, x[None, None].to(dev()), g, 1)
    torch.cuda.synchronize()
    got = to_np(labels[0, 0])
    assert not got[bad].any()
    good = np.setdiff1d(np.arange(N), bad)
    assert np.array_equal(got[good], orc.kmeans_assign(x.float().numpy()[good], cent))
