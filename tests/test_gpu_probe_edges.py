"""GPU probe where its tiles can go wrong: key clusters of 0 to a few hundred keys around the 32-key
blocks and the four waves that take them, query centroids around the groups of 32 and 128, both types,
head sizes and estimates, against the definition in 64 bits."""
import numpy as np
import pytest
import torch

import paper_2603_08982_amd as sv
from helpers import dev, to_np

pytestmark = pytest.mark.gpu

K_SIZES = [0, 1, 31, 32, 33, 64, 127, 128, 129, 160, 257, 3, 0, 20, 96]


def _definition(q, kb, vb, K, V, sizes, scale, plain):
    S = np.where(sizes[None] > 0, (q @ kb.T) * scale, -np.inf)
    m = S.max(1, keepdims=True)
    W, w = np.exp(S - m), np.exp((q @ K.T) * scale - m)
    out = np.zeros((len(q), len(sizes)))
    at = 0
    for b, n in enumerate(sizes):
        u, x = W[:, b: b + 1], w[:, at: at + n]
        if n and plain:
            out[:, b] = ((u - x) ** 2).sum(1) / n
        elif n:
            diff = u[:, :, None] * vb[b][None, None] - x[:, :, None] * V[at: at + n][None]
            out[:, b] = (diff ** 2).sum((1, 2)) / n
        at += n
    return out


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Cq", [1, 31, 33, 128, 129, 300])
@pytest.mark.parametrize("plain", [False, True])
def test_scores_at_the_edges_of_tiles(dtype, d, Cq, plain):
    g = torch.Generator().manual_seed(Cq + d)
    sizes, tail, H = np.array(K_SIZES), 9, 2
    Ck, n = len(sizes), int(sizes.sum())
    q = torch.randn(1, H, Cq, d, generator=g)
    kb, vb = torch.randn(1, H, Ck, d, generator=g), torch.randn(1, H, Ck, d, generator=g)
    lab = torch.from_numpy(np.repeat(np.arange(Ck), sizes))
    K, V = (torch.cat([t[:, :, lab] + 0.3 * torch.randn(1, H, n, d, generator=g), torch.randn(1, H, tail, d, generator=g)], 2)
            .to(dtype) for t in (kb, vb))
    koff = torch.from_numpy(np.concatenate([[0], np.cumsum(sizes), [n + tail]]).astype(np.int32)).expand(1, H, -1).contiguous()
    qoff = torch.arange(Cq + 2, dtype=torch.int32).expand(1, H, -1).contiguous()
    # centroid values need no more than 4-byte alignment
    vb_dev = torch.empty(vb.numel() + 1, device=dev())[1:].view_as(vb).copy_(vb)
    r = sv.probe_route(q.to(dev()), kb.to(dev()), vb_dev, K.to(dev()), V.to(dev()), qoff.to(dev()), koff.to(dev()),
                       n * Cq // 4, d ** -0.5, flags=sv.PROBE_PLAIN if plain else 0)
    torch.cuda.synchronize()
    for h in range(H):
        f = lambda t: t[0, h].double().numpy()
        ref = _definition(f(q), f(kb), f(vb), f(K)[:n], f(V)[:n], sizes, d ** -0.5, plain)
        got = to_np(r["scores"][0, h]).astype(np.float64)
        assert not got[:, sizes == 0].any()
        # a logit of size s is off by s 2^-22 or so after d products, its exponential relatively by as much
        assert np.linalg.norm(got - ref) <= 1e-5 * np.linalg.norm(ref)
        assert (np.abs(got - ref) <= 2e-4 * ref + 1e-6 * ref.max(1, keepdims=True)).all()


def test_many_heads_give_the_scores_of_one_head():
    """Enough workgroups of 32 query centroids switch the centroid logits to the matrix cores: bit for bit
    the vector-ALU chain of a head by itself."""
    H, Cq, Ck, d, n = 9, 1000, 51, 128, 500
    g = torch.Generator().manual_seed(5)
    sizes = np.full(Ck, n // Ck)
    sizes[7], sizes[50] = 0, n - n // Ck * (Ck - 2)
    koff = torch.from_numpy(np.concatenate([[0], np.cumsum(sizes), [n]]).astype(np.int32)).expand(1, H, -1).contiguous().to(dev())
    qoff = torch.arange(Cq + 2, dtype=torch.int32).expand(1, H, -1).contiguous().to(dev())
    for dtype in (torch.float32, torch.bfloat16):
        q, kb, vb = (torch.randn(1, H, c, d, generator=g).to(dev()) for c in (Cq, Ck, Ck))
        K, V = (torch.randn(1, H, n, d, generator=g).to(dtype).to(dev()) for _ in range(2))
        for p in (None, 0.6):
            r = sv.probe_route(q, kb, vb, K, V, qoff, koff, n * Cq // 4, d ** -0.5, top_p=p)
            for h in (0, 4, 8):
                one = sv.probe_route(*(t[:, h: h + 1].contiguous() for t in (q, kb, vb, K, V, qoff, koff)), n * Cq // 4,
                                     d ** -0.5, top_p=p)
                torch.cuda.synchronize()
                for key in ("scores", "mask_bits", "row_ptr", "routed_cost") + (("row_budget",) if p else ()):
                    assert torch.equal(r[key][:, h: h + 1], one[key]), key


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_errors_beyond_fp32_are_infinite(dtype, d):
    """Values whose squared norm leaves fp32: the scores are +inf for every number of keys in a cluster's
    last 32-key block, never NaN."""
    sizes, Cq, H = np.array([1, 20, 32, 33, 63, 64, 95, 0, 130]), 40, 1
    Ck, n = len(sizes), int(sizes.sum())
    g = torch.Generator().manual_seed(d)
    q, kb = torch.randn(1, H, Cq, d, generator=g), torch.randn(1, H, Ck, d, generator=g)
    lab = torch.from_numpy(np.repeat(np.arange(Ck), sizes))
    vb = torch.full((1, H, Ck, d), 2.0 ** 65)
    K, V = (kb[:, :, lab] + 0.3 * torch.randn(1, H, n, d, generator=g)).to(dtype), vb[:, :, lab].to(dtype)
    off = lambda s: torch.from_numpy(np.concatenate([[0], np.cumsum(s), [np.sum(s)]]).astype(np.int32))[None, None].to(dev())
    r = sv.probe_route(*(t.to(dev()).contiguous() for t in (q, kb, vb, K, V)), off(np.full(Cq, 3)), off(sizes), n, d ** -0.5)
    torch.cuda.synchronize()
    got = to_np(r["scores"][0, 0])
    assert np.isposinf(got[:, sizes > 0]).all() and not got[:, sizes == 0].any()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,Cq", [(1, 40), (9, 1000)])  # centroid logits on the vector ALU and on the matrix cores
@pytest.mark.parametrize("plain", [False, True])
def test_fp32_clusters_of_equal_keys_have_no_error(d, H, Cq, plain):
    """The logit of a key that equals its cluster's centroid is the centroid's, bit for bit: the score is 0."""
    sizes = np.array([1, 1, 4, 1, 2, 32, 1, 64])
    Ck, n = len(sizes), int(sizes.sum())
    g = torch.Generator().manual_seed(d)
    q, kb, vb = (torch.randn(1, H, c, d, generator=g).to(dev()) for c in (Cq, Ck, Ck))
    lab = torch.from_numpy(np.repeat(np.arange(Ck), sizes)).to(dev())
    off = lambda s: torch.from_numpy(np.concatenate([[0], np.cumsum(s), [np.sum(s)]]).astype(np.int32)).expand(1, H, -1).contiguous().to(dev())
    r = sv.probe_route(q, kb, vb, kb[:, :, lab].contiguous(), vb[:, :, lab].contiguous(), off(np.ones(Cq)), off(sizes), n,
                       d ** -0.5, flags=sv.PROBE_PLAIN if plain else 0)
    torch.cuda.synchronize()
    assert not r["scores"].any()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Ck,Cq", [(255, 20), (257, 33), (259, 150)])  # a workgroup per cluster; four clusters in one
@pytest.mark.parametrize("plain", [False, True])
def test_fp32_scores_of_many_small_clusters(d, Ck, Cq, plain):
    rng = np.random.default_rng(Ck)
    H, sizes = 4, rng.integers(0, 70, Ck)
    n = int(sizes.sum())
    assert n <= 40 * Ck
    g = torch.Generator().manual_seed(d)
    q, kb, vb = (torch.randn(1, H, c, d, generator=g) for c in (Cq, Ck, Ck))
    lab = torch.from_numpy(np.repeat(np.arange(Ck), sizes))
    K, V = (t[:, :, lab] + 0.3 * torch.randn(1, H, n, d, generator=g) for t in (kb, vb))
    off = lambda s: torch.from_numpy(np.concatenate([[0], np.cumsum(s), [np.sum(s)]]).astype(np.int32)).expand(1, H, -1).contiguous().to(dev())
    r = sv.probe_route(*(t.to(dev()).contiguous() for t in (q, kb, vb, K, V)), off(np.ones(Cq)), off(sizes), n, d ** -0.5,
                       flags=sv.PROBE_PLAIN if plain else 0)
    torch.cuda.synchronize()
    for h in (0, H - 1):
        ref = _definition(*(t[0, h].double().numpy() for t in (q, kb, vb, K, V)), sizes, d ** -0.5, plain)
        got = to_np(r["scores"][0, h]).astype(np.float64)
        assert not got[:, sizes == 0].any()
        assert np.linalg.norm(got - ref) <= 1e-5 * np.linalg.norm(ref)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,Ck,Cq", [(35, 30, 40), (36, 29, 40), (70, 30, 130), (75, 28, 31), (300, 28, 40), (290, 29, 130)])
def test_scores_do_not_depend_on_the_clusters_a_workgroup_takes(H, Ck, Cq, d):
    """Few heads give a workgroup one key cluster, many two, four or eight, side by side with the other groups of 128
    query centroids: every head's scores are those of a call with that head alone, bit for bit."""
    g = torch.Generator().manual_seed(H + d)
    sizes = torch.randint(0, 70, (H, Ck), generator=g)
    sizes[:, 0] = 70 * Ck - sizes[:, 1:].sum(1)  # the same number of keys in every head
    n = 70 * Ck
    q, kb, vb = (torch.randn(1, H, c, d, generator=g) for c in (Cq, Ck, Ck))
    lab = torch.stack([torch.repeat_interleave(torch.arange(Ck), s) for s in sizes])
    rows = lambda t: (torch.gather(t[0], 1, lab[:, :, None].expand(H, n, d)) + 0.3 * torch.randn(H, n, d, generator=g)).bfloat16()[None]
    koff = torch.cat([torch.zeros(H, 1, dtype=torch.int64), sizes.cumsum(1), torch.full((H, 1), n)], 1).int()[None]
    qoff = torch.cat([torch.arange(Cq + 1) * 3, torch.tensor([3 * Cq])]).int().expand(1, H, Cq + 2)
    a = [t.contiguous().to(dev()) for t in (q, kb, vb, rows(kb), rows(vb), qoff, koff)]
    got = sv.probe_route(*a, n, d ** -0.5, Nq=3 * Cq)["scores"]
    for h in (0, 1, H // 2, H - 1):
        one = sv.probe_route(*(t[:, h:h + 1].contiguous() for t in a), n, d ** -0.5, Nq=3 * Cq)["scores"]
        torch.cuda.synchronize()
        assert torch.isfinite(one).all() and torch.equal(got[:, h:h + 1], one)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("case,value", [("cap", 0.0), ("cap", 1e-3), ("low", 1e4)])
def test_scores_at_both_ends_of_the_weights(case, value, d):
    """bf16 errors that a float holds although the weights' squares alone, summed over the cluster or not, would leave its
    range: thousands of keys at the cap of e^40 with values of (almost) nothing, and weights below e^-50 with large
    values. Keys and query have one dim that is not 0, so a logit is one product."""
    n0, n1 = 16400, 300
    g = torch.Generator().manual_seed(d)
    step = 0.25 * d ** 0.5  # a logit of 1/4
    k = torch.zeros(n0 + n1, d)
    if case == "cap":
        k[:n0, 0] = torch.where(torch.arange(n0) % 2 == 0, 200.0, -200.0) * step  # logits +-50 around a centroid at 0
    else:
        k[:n0, 0] = -206.0 * step + step * torch.randint(-4, 5, (n0,), generator=g)  # around -51.5
    k = k.bfloat16().float()
    v = torch.randn(n0 + n1, d, generator=g)
    if case == "low":
        v = 1.0 + 0.1 * v
    v = (value * v).bfloat16().float()
    if case == "cap":
        v[:n0] = v[0]
    kb, vb = (torch.stack([t[:n0].double().mean(0), t[n0:].double().mean(0)]).float() for t in (k, v))
    q = torch.zeros(1, d)
    q[0, 0] = 1.0
    scale = d ** -0.5
    logits = (k.double() @ q[0].double()) * scale
    lb = (kb.double() @ q[0].double()) * scale
    ref = []
    for b, (lo, hi) in enumerate(((0, n0), (n0, n0 + n1))):
        W, w = (torch.clamp(x - lb.max(), max=40.0).exp() for x in (lb[b], logits[lo:hi]))
        ref.append(float(((W * vb[b].double() - w[:, None] * v[lo:hi].double()) ** 2).sum() / (hi - lo)))
    at = lambda t, ty=torch.float32: t[None, None].to(ty).contiguous().to(dev())
    koff = at(torch.tensor([0, n0, n0 + n1, n0 + n1]), torch.int32)
    qoff = at(torch.tensor([0, 5, 5]), torch.int32)
    got = to_np(sv.probe_route(at(q), at(kb), at(vb), at(k, torch.bfloat16), at(v, torch.bfloat16), qoff, koff, 1, scale, Nq=5)["scores"][0, 0, 0])
    # a weight's error is its logit's (50 x a few 2^-24) and the exponential's; squares double it
    assert np.isfinite(got).all() and np.allclose(got.astype(np.float64), ref, rtol=1e-4, atol=0), (got, ref)


def test_more_key_clusters_than_one_grid_dimension_holds():
    """2,050 heads of 8,192 key clusters, 2^24 and more in one launch: heads of few keys, nearly all clusters empty; the
    last head's scores are those of a call with that head alone."""
    H, Ck, d, n = 2050, 8192, 64, 40
    g = torch.Generator(device=dev()).manual_seed(0)
    r = lambda *s: torch.randn(1, H, *s, d, generator=g, device=dev())
    q, kb, vb, k, v = r(1), r(Ck), r(Ck), r(n).bfloat16(), r(n).bfloat16()
    koff = torch.zeros(1, H, Ck + 2, dtype=torch.int32, device=dev())
    koff[..., 1:100] = 7
    koff[..., 100:] = n - 3
    koff[..., -1] = n
    qoff = torch.tensor([0, 5, 5], dtype=torch.int32, device=dev()).expand(1, H, 3).contiguous()
    got = sv.probe_route(q, kb, vb, k, v, qoff, koff, 100, 0.125, Nq=5)["scores"]
    for h in (0, H - 1):
        one = sv.probe_route(*(t[:, h:h + 1].contiguous() for t in (q, kb, vb, k, v, qoff, koff)), 100, 0.125, Nq=5)["scores"]
        assert int((one != 0).sum()) == 2 and torch.equal(got[:, h:h + 1], one)
