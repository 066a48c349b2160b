"""GPU attention kernels where their tiles and lists can go wrong: query clusters of 1 to a few
hundred rows around the tile heights (32-row blocks, tiles of 128 and 384 rows), key clusters
around the 32- and 64-key tiles, empty ones, text rows, no / some / all blocks routed, few query
tiles with many keys (the keys of a tile split over workgroups) and the reverse, against the
definition in 64 bits."""
import numpy as np
import pytest
import torch

import paper_2603_08982_amd as sv
from helpers import dev, mask_to_bits, csr_from_mask

pytestmark = pytest.mark.gpu

Q_EDGES = [1, 31, 0, 32, 33, 64, 127, 128, 129, 0, 383, 385]
K_EDGES = [0, 1, 31, 32, 33, 63, 64, 65, 0, 127, 200, 5, 17, 96, 255, 0]
# rel-L2 of the output. fp32: d products and N weights per sum, each rounded to 2^-24, errors of either
# sign: a few 1e-7 (measured 7e-7); bf16: rounded probabilities, values and outputs, 2^-9 each
TOL = {torch.float32: 3e-6, torch.bfloat16: 1e-2}


def _lse_tol(dtype, d):
    """Largest log-sum-exp error. bf16 products are exact in fp32, so a logit below 8 is off by a few 2^-21 in
    either type and the fp32 sum of the weights by less; bf16 heads of 128 sum rounded weights, 2^-9 each."""
    return 2e-2 if dtype == torch.bfloat16 and d == 128 else 2e-5


def _sizes(name, rng):
    if name == "edges":
        return Q_EDGES, K_EDGES, 13
    if name == "few_rows":  # a handful of tiles over thousands of keys
        return [40, 3], list(rng.integers(1, 90, 120)), 0
    if name == "many_rows":
        return list(rng.integers(1, 70, 150)), [7, 90], 1
    if name == "split_keys":  # a few tiles over keys enough for every number of splits
        return [200, 1, 129], list(rng.integers(1, 250, 80)), 5
    if name == "full_tiles":  # clusters of several tiles; d = 64: tiles of 384 rows
        return list(rng.integers(385, 800, 40)), [30, 64, 500], 3
    if name == "large_tiles":  # 16 heads: tiles of 384 rows at d = 128 too (more than 1,024 of 128), a few dozen a work list
        return Q_EDGES + list(rng.integers(385, 800, 20)), K_EDGES, 13
    if name == "ranked":  # 256 items over both heads
        return list(rng.integers(1, 200, 127)), [64, 0, 300], 2
    if name == "fine_splits":  # a few hundred tiles over 8,192 keys and more
        return list(rng.integers(1, 3, 400)), list(rng.integers(1, 400, 42)) + [1000], 9
    if name == "spread_splits":  # more than a thousand over 16,384 and more
        return list(rng.integers(0, 3, 1100)), list(rng.integers(1, 600, 86)) + [300], 0
    return [130, 64], list(rng.integers(0, 3, 900)), 40  # hundreds of tiny clusters


def _definition(Q, K, V, kbar, vbar, qs, ks, mask, scale):
    rows_of = np.repeat(np.arange(len(qs)), qs)
    keys_of = np.repeat(np.arange(len(ks)), ks)
    on = torch.from_numpy(mask)
    s = (Q @ K.t()) * scale
    s.masked_fill_(~on[rows_of][:, keys_of], -np.inf)
    n = torch.tensor(ks[:-1], dtype=torch.float64)
    c = (Q @ kbar.t()) * scale + torch.log(n)[None]
    c.masked_fill_(on[rows_of][:, : len(ks) - 1] | torch.from_numpy(rows_of == len(qs) - 1)[:, None], -np.inf)
    lse = torch.logsumexp(torch.cat([s, c], 1), 1, keepdim=True)
    return torch.exp(s - lse) @ V + torch.exp(c - lse) @ vbar, lse[:, 0]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("name", ["edges", "few_rows", "many_rows", "tiny_clusters", "split_keys", "full_tiles", "large_tiles",
                                  "ranked", "fine_splits", "spread_splits"])
@pytest.mark.parametrize("density", [0.0, 0.3, 1.0])
def test_attention_at_the_edges_of_tiles_and_lists(dtype, d, name, density):
    rng = np.random.default_rng(3)
    qs, ks, tail = _sizes(name, rng)
    qs, ks = np.array(list(qs) + [tail]), np.array(list(ks) + [tail])
    Cq, Ck, Nq, Nk = len(qs) - 1, len(ks) - 1, int(qs.sum()), int(ks.sum())
    H, scale = 16 if name == "large_tiles" else 2, float(d) ** -0.5
    g = torch.Generator().manual_seed(11)
    Q, K, V = (torch.randn(1, H, n, d, generator=g).to(dtype) for n in (Nq, Nk, Nk))
    kbar, vbar = (torch.randn(1, H, Ck, d, generator=g).to(torch.bfloat16).float() for _ in range(2))
    masks, bits, ptrs, cols = [], [], [], []
    for h in range(H):
        m = rng.random((Cq + 1, Ck + 1)) < density
        m[Cq], m[:, Ck] = True, True
        m &= np.outer(qs > 0, ks > 0)
        masks.append(m)
        bits.append(torch.from_numpy(mask_to_bits(m, Cq, Ck).view(np.int32)))
        ptr, col = csr_from_mask(m)
        ptrs.append(torch.from_numpy(ptr))
        cols.append(torch.from_numpy(col))
    # keys of a cluster that no query cluster of a head routes are never looked at, whatever they hold
    unseen = [b for b in range(Ck) if ks[b] and not any(m[:Cq, b].any() for m in masks) and tail == 0]
    off = np.concatenate([[0], np.cumsum(ks)])
    Kx, Vx = K.clone(), V.clone()
    if dtype == torch.float32:
        for b in unseen:
            Kx[:, :, off[b]:off[b + 1]] = float("nan")
            Vx[:, :, off[b]:off[b + 1]] = float("inf")
    offs = [torch.from_numpy(np.concatenate([[0], np.cumsum(x)]).astype(np.int32)).expand(1, H, -1).contiguous().to(dev())
            for x in (qs, ks)]
    lists = [torch.stack(x)[None].contiguous().to(dev()) for x in (bits, ptrs, cols)]
    tables = [t.to(dev()) for t in (Kx, Vx, kbar, vbar)]
    O, lse = sv.sparse_attn_comp(Q.to(dev()), *tables, *offs, *lists, scale, want_lse=True)
    # the same through a permutation of the queries, which only moves rows
    perm = torch.stack([torch.randperm(Nq, generator=g) for _ in range(H)])[None]
    tokens = torch.empty_like(Q)
    for h in range(H):
        tokens[0, h, perm[0, h]] = Q[0, h]
    O2, lse2 = sv.sparse_attn_comp(tokens.to(dev()), *tables, *offs, *lists, scale, want_lse=True,
                                   q_perm=perm.int().contiguous().to(dev()))
    two = None
    if dtype == torch.bfloat16 and d == 128:  # routed keys and centroids by themselves, merged
        two = sv.sparse_attn_comp(Q.to(dev()), *tables, *offs, *lists, scale, want_lse=True, two_stage=True)
    torch.cuda.synchronize()
    for h in sorted({0, H // 2, H - 1}):
        ref, ref_lse = _definition(Q[0, h].double(), K[0, h].double(), V[0, h].double(), kbar[0, h].double(),
                                   vbar[0, h].double(), qs, ks, masks[h], scale)
        none = torch.isinf(ref_lse)  # text rows of a head without text keys see nothing
        for out in (O, lse), two:
            if out is None:
                continue
            got, got_lse = out[0][0, h].cpu(), out[1][0, h].cpu()
            assert torch.equal(torch.isinf(got_lse), none) and not got[none].any()
            err = (got.double() - ref)[~none].norm() / ref[~none].norm()
            assert err <= TOL[dtype], f"head {h}: rel-L2 {err:.3e}"
            lse_err = (got_lse.double() - ref_lse)[~none].abs().max()
            assert lse_err <= _lse_tol(dtype, d), f"head {h}: log-sum-exp {lse_err:.3e}"
        got, got_lse = O[0, h].cpu(), lse[0, h].cpu()
        assert torch.equal(O2[0, h].cpu()[perm[0, h]], got) and torch.equal(lse2[0, h].cpu()[perm[0, h]], got_lse)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,rows", [(8, [400] * 40), (2, [70] * 40)])  # tiles of 384 rows and of 128
def test_whole_tiles_of_keys_without_weight_come_first(dtype, d, H, rows):
    """Keys whose logits are all -inf weigh nothing, also where a row meets them before any other."""
    qs, ks = np.array(rows + [3]), np.array([200, 61, 90, 7, 0])
    Cq, Ck, Nq, Nk = len(qs) - 1, len(ks) - 1, int(qs.sum()), int(ks.sum())
    g = torch.Generator().manual_seed(7)
    Q, K, V = (torch.randn(1, H, n, d, generator=g) for n in (Nq, Nk, Nk))
    Q[..., 0] = Q[..., 0].abs() + 0.5
    K[:, :, :250, 0] = -float("inf")
    Q, K, V = (x.to(dtype) for x in (Q, K, V))
    kbar, vbar = (torch.randn(1, H, Ck, d, generator=g).to(torch.bfloat16).float() for _ in range(2))
    mask = np.outer(qs > 0, ks > 0)
    mask[:Cq, 2] = False
    row_ptr, col_idx = csr_from_mask(mask)
    lists = [torch.from_numpy(x)[None, None].expand(1, H, *x.shape).contiguous().to(dev())
             for x in (mask_to_bits(mask, Cq, Ck).view(np.int32), row_ptr, col_idx)]
    offs = [torch.from_numpy(np.concatenate([[0], np.cumsum(x)]).astype(np.int32)).expand(1, H, -1).contiguous().to(dev())
            for x in (qs, ks)]
    O, lse = sv.sparse_attn_comp(*(x.to(dev()) for x in (Q, K, V, kbar, vbar)), *offs, *lists, d ** -0.5, want_lse=True)
    torch.cuda.synchronize()
    for h in (0, H - 1):
        ref, ref_lse = _definition(*(x[0, h].double() for x in (Q, K, V, kbar, vbar)), qs, ks, mask, d ** -0.5)
        got, got_lse = O[0, h].cpu().double(), lse[0, h].cpu().double()
        assert (got - ref).norm() <= TOL[dtype] * ref.norm()
        assert (got_lse - ref_lse).abs().max() <= _lse_tol(dtype, d)


@pytest.mark.parametrize("H,rows", [(8, [400] * 40), (2, [70] * 40)])  # tiles of 384 rows and of 128
def test_the_largest_weight_of_a_row_is_exact(H, rows):
    """bf16 heads of 64: the weight of a row's largest logit, here of a key in the second tile, is 1 whatever came
    before it. With equal values everywhere the output is that value to the bit: the other weights, some
    2^-8 and less, are off by 2^-9 of themselves."""
    qs, ks, d = np.array(rows + [0]), np.array([100, 41, 0]), 64
    Cq, Ck, Nq, Nk = len(qs) - 1, len(ks) - 1, int(qs.sum()), int(ks.sum())
    g = torch.Generator().manual_seed(2)
    Q, K = torch.zeros(1, H, Nq, d), torch.zeros(1, H, Nk, d)
    Q[..., 0] = 8.0 * (1.0 + 0.05 * torch.rand(1, H, Nq, generator=g))  # logits of 5.2 to 5.5 for key 90
    K[..., 0], K[:, :, 0, 0], K[:, :, 90, 0] = -60.0, 0.0, 5.1875
    V = torch.randn(1, H, 1, d, generator=g).expand(1, H, Nk, d)
    Q, K, V = (x.to(torch.bfloat16) for x in (Q, K, V))
    mask = np.outer(qs > 0, ks > 0)
    row_ptr, col_idx = csr_from_mask(mask)
    lists = [torch.from_numpy(x)[None, None].expand(1, H, *x.shape).contiguous().to(dev())
             for x in (mask_to_bits(mask, Cq, Ck).view(np.int32), row_ptr, col_idx)]
    offs = [torch.from_numpy(np.concatenate([[0], np.cumsum(x)]).astype(np.int32)).expand(1, H, -1).contiguous().to(dev())
            for x in (qs, ks)]
    means = torch.zeros(1, H, Ck, d, device=dev())
    O, lse = sv.sparse_attn_comp(*(x.to(dev()).contiguous() for x in (Q, K, V)), means, means, *offs, *lists, d ** -0.5,
                                 want_lse=True)
    torch.cuda.synchronize()
    assert torch.equal(O.cpu(), V[:, :, :1].expand_as(O))
    logits = (Q.double()[..., :1] * K.double()[..., 0][:, :, None, :]) * d ** -0.5
    assert (lse.cpu().double() - torch.logsumexp(logits, -1)).abs().max() <= 2e-5


@pytest.mark.parametrize("Nq,Cq", [(300, 3), (208000, 100)])  # keys split over 128-row tiles; tiles of 384 rows
def test_heads_of_more_than_33_million_keys(Nq, Cq):
    """bf16 heads of 64 whose K and V rows lie more than 2^32 bytes apart are reached by 64-bit addresses. The
    cluster that makes up the distance is compensated, so its rows are never read (nor initialised here)."""
    d, scale = 64, 0.125
    ks = np.array([90, 2 ** 25 + 77, 130, 64, 200, 0])
    qs = np.append(np.full(Cq, Nq // Cq), 0)
    qs[0] += Nq - qs.sum()
    Ck, Nk, off = len(ks) - 1, int(ks.sum()), np.concatenate([[0], np.cumsum(ks)])
    g = torch.Generator(device=dev()).manual_seed(4)
    K, V = (torch.empty(1, 1, Nk, d, dtype=torch.bfloat16, device=dev()) for _ in range(2))
    near = [0, 2, 3, 4]
    for b in near:
        for x in (K, V):
            x[0, 0, off[b]:off[b + 1]] = torch.randn(int(ks[b]), d, generator=g, device=dev())
    Q = torch.randn(1, 1, Nq, d, generator=g, device=dev()).to(torch.bfloat16)
    Q[..., 0] = 8.0
    kbar, vbar = (torch.randn(1, 1, Ck, d, generator=g, device=dev()).to(torch.bfloat16).float() for _ in range(2))
    kbar[0, 0, 1, 0] = -17.0  # logit about -17 + ln 2^25
    mask = np.outer(qs > 0, ks > 0)
    mask[:, 1] = False
    mask[: Cq // 2, 3] = False
    row_ptr, col_idx = csr_from_mask(mask)
    lists = [torch.from_numpy(x)[None, None].contiguous().to(dev())
             for x in (mask_to_bits(mask, Cq, Ck).view(np.int32), row_ptr, col_idx)]
    offs = [torch.from_numpy(np.concatenate([[0], np.cumsum(x)]).astype(np.int32))[None, None].contiguous().to(dev()) for x in (qs, ks)]
    O, lse = sv.sparse_attn_comp(Q, K, V, kbar, vbar, *offs, *lists, scale, want_lse=True)
    torch.cuda.synchronize()
    rows = np.unique(np.linspace(0, Nq - 1, 1500).astype(int))
    cluster = np.repeat(np.arange(Cq + 1), qs)[rows]
    q = Q[0, 0, torch.from_numpy(rows).to(dev())].double().cpu()
    parts, values = [], []
    for b in range(Ck):
        on = torch.from_numpy(mask[cluster, b])[:, None]
        c = (q @ kbar[0, 0, b].double().cpu())[:, None] * scale + float(np.log(ks[b]))
        if b == 1:
            parts.append(c)
            values.append(vbar[0, 0, 1:2].double().cpu())
            continue
        s = (q @ K[0, 0, off[b]:off[b + 1]].double().cpu().t()) * scale
        parts += [s.masked_fill(~on, -np.inf), c.masked_fill(on, -np.inf)]
        values += [V[0, 0, off[b]:off[b + 1]].double().cpu(), vbar[0, 0, b:b + 1].double().cpu()]
    logits = torch.cat(parts, 1)
    ref, ref_lse = torch.softmax(logits, 1) @ torch.cat(values), torch.logsumexp(logits, 1)
    at = torch.from_numpy(rows).to(dev())
    assert (O[0, 0, at].double().cpu() - ref).norm() <= TOL[torch.bfloat16] * ref.norm()
    assert (lse[0, 0, at].double().cpu() - ref_lse).abs().max() <= _lse_tol(torch.bfloat16, d)
