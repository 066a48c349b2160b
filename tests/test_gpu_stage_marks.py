"""attention_layer(mark=...): a stage's mark comes after the work of both streams in that stage."""
import pytest
import torch

import paper_2603_08982_amd as sv
from helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("overlap", [False, True])
def test_the_kmeans_mark_waits_for_the_queries_side(overlap):
    """Thousands of query clusters and two key clusters: K's side is done long before Q's. What the caller's stream sees at the
    mark are the final centroids of both."""
    g = torch.Generator(device=dev()).manual_seed(1)
    Q, K, V = (torch.randn(1, 8, 20000, 128, generator=g, device=dev()).bfloat16() for _ in range(3))
    start_q, start_k = Q[:, :, :4000].float().contiguous(), K[:, :, :2].float().contiguous()
    for _ in range(2):  # (the first pass loads code)
        cq, ck, seen = start_q.clone(), start_k.clone(), {}
        O, r = sv.attention_layer(Q, K, V, cq, ck, 6, 20000 * 2000, overlap=overlap,
                                  mark=lambda name: seen.setdefault(name, (cq.clone(), ck.clone())))
        torch.cuda.synchronize()
    assert list(seen) == ["kmeans", "permute", "probe_route", "attention", "unpermute"]
    for a, b in seen.values():
        assert torch.equal(a, cq) and torch.equal(b, ck)
    cq, ck = start_q.clone(), start_k.clone()
    plain, _ = sv.attention_layer(Q, K, V, cq, ck, 6, 20000 * 2000, overlap=overlap)
    assert torch.equal(O, plain)
