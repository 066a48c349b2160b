"""The workloads whose speed this repository is held to, through its public entry points.

A case is one call (or one whole layer) of the SVG-EAR attention hot path as a video model's
attention layer makes it: k-means of queries and keys, the cluster permutation of K and V, the
error probe with its router, the fused sparse attention, and all of them in a row. Sizes are
those of the layers this repository is built for (21 x 45 x 80 and 33 x 45 x 80 video tokens,
40 and 24 heads of 128, the paper's cluster counts, 256 text tokens), what one of eight GPUs
holds of them (5 heads), and small, odd and ragged ones; d = 64 and fp32 are the other head
size and type that the entry points take.

Tokens come from a Gaussian mixture whose component follows the token's (t, h, w) position for
four tokens in five, so that clusters are ragged and lie all over the tensor as they do in a
video model. Everything a call has in hand before it (cluster means, permuted rows, offsets,
routing masks) is made here with plain torch; cluster sums are whole numbers, so the same seed
gives the same state.
"""
import math

import torch

import paper_2603_08982_amd as sv

GPU = "cuda"
DT = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(name, what, dtype, d, heads, t, h, w, tail, cq, ck, iters=0, rho=0.25, **more):
    c = {"what": what, "dtype": dtype, "d": d, "batch": 1, "heads": heads, "t": t, "h": h, "w": w, "tail": tail,
         "cq": cq, "ck": ck, "iters": iters, "rho": rho, **more}
    return {"name": name, **c} if name else c


def listed():
    return [
        # the smallest layer call: a few hundred tokens, ragged clusters, text tokens; launches and latency
        _case("layer_small_tail", "layer", "bf16", 128, 2, 5, 9, 14, 37, 10, 30, iters=4),
        # one fp32 head of 4096 tokens: the configuration on which everything is checked in fp32
        _case("layer_tiny_f32", "layer", "f32", 64, 1, 16, 16, 16, 0, 32, 64, iters=10),
        # the benchmark's layer: 40 heads, 75,600 tokens, first denoising step (cold k-means)
        _case("layer_wan", "layer", "bf16", 128, 40, 21, 45, 80, 0, 100, 500, iters=10),
        # the largest layer, with text tokens, at the paper's cluster counts and in the middle of a
        # generation: centroids carried over from the previous denoising step, two iterations
        _case("layer_hunyuan_warm", "layer", "bf16", 128, 24, 33, 45, 80, 256, 400, 1000, iters=2, warm=True),
        # keys of a first step at the paper's cluster count, values averaged along
        _case("kmeans_keys_1000", "kmeans", "bf16", 128, 40, 21, 45, 80, 0, 300, 1000, iters=10, x2=True),
        # fp32 rows of 64, an odd number of tokens
        _case("kmeans_f32_d64", "kmeans", "f32", 64, 8, 13, 31, 45, 0, 60, 200, iters=5, x2=True),
        # K and V of the largest layer laid out by cluster
        _case("permute_hunyuan_kv", "permute", "bf16", 128, 24, 33, 45, 80, 256, 100, 500),
        # probe and router at the paper's cluster counts, one budget per head
        _case("probe_wan_c300", "probe", "bf16", 128, 40, 21, 45, 80, 0, 300, 1000),
        # what one of eight GPUs routes with adaptive row budgets (smaller cluster counts)
        _case("probe_top_p_shard", "probe", "bf16", 128, 5, 21, 45, 80, 0, 200, 500, top_p=0.8),
        # what one of eight GPUs attends to at the paper's cluster counts
        _case("attention_c300_shard", "attention", "bf16", 128, 5, 21, 45, 80, 0, 300, 1000, token_order=True),
        # heads of 64, text tokens, a shorter and smaller clip
        _case("attention_d64_tail", "attention", "bf16", 64, 24, 9, 45, 80, 77, 64, 300, token_order=True),
        # fp32 heads of 128, permuted queries in, rows put back afterwards
        _case("attention_f32_d128", "attention", "f32", 128, 8, 7, 23, 37, 0, 48, 160, token_order=False),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    what = rng.choice(["layer", "kmeans", "permute", "probe", "attention", "attention"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    d = rng.choice([128, 128, 64])
    small = dtype == "f32" and what in ("layer", "attention", "probe")
    n = log(600, 20000 if small else 119000)
    t = rng.randint(3, 33)
    w = max(2, int(math.sqrt(n / t * 16 / 9)))
    h = max(2, n // (t * w))
    n = t * h * w
    tail = rng.choice([0, 0, rng.randint(1, 256)])
    cq = max(2, min(log(8, 400), n // 12))
    ck = max(2, min(log(20, 1000), n // 6))
    per_pair = what in ("layer", "attention", "probe")  # work grows with n squared there
    most = (24 if what == "probe" or not per_pair else 14) * (118800 / n) ** (2 if per_pair else 1)
    heads = max(1, min(rng.choice([1, 2, 5, 8, 12, 24, 40]), int(most)))
    if small:
        heads = max(1, min(heads, int(24 * (9000 / n) ** 2)))
    more = {}
    if what == "probe" and rng.random() < 0.4:
        more["top_p"] = round(rng.uniform(0.3, 0.9), 2)
    if what == "layer" and rng.random() < 0.5:
        more["warm"] = True
    if what == "kmeans":
        more["x2"] = rng.random() < 0.6
    if what == "attention":
        more["token_order"] = rng.random() < 0.75
    iters = 2 if more.get("warm") else rng.choice([2, 4, 10])
    return _case("", what, dtype, d, heads, t, h, w, tail, cq, ck, iters=iters if what in ("layer", "kmeans") else 0,
                 rho=round(rng.uniform(0.05, 0.3), 3), **more)


# ------------------------------------------------------------------------------------ inputs
def _n(case):
    return case["t"] * case["h"] * case["w"] + case["tail"]


def _generator(seed):
    g = torch.Generator(device=GPU)
    g.manual_seed(int(seed))
    return g


def _qkv(case, g):
    """Q, K, V [1, heads, n, d]; a token's three rows share one component of separate centre tables."""
    H, d, nv, tail = case["heads"], case["d"], _n(case) - case["tail"], case["tail"]
    T, Hh, Ww = case["t"], case["h"], case["w"]
    comps = (4, 8, 8) if nv >= 16384 else (2, 4, 4)
    i = torch.arange(nv, device=GPU)
    cell = ((i // (Hh * Ww)) * comps[0] // T * comps[1] + (i // Ww) % Hh * comps[1] // Hh) * comps[2] + i % Ww * comps[2] // Ww
    nc = comps[0] * comps[1] * comps[2]
    stray = torch.rand(H, nv, generator=g, device=GPU) >= 0.8
    z = torch.where(stray, torch.randint(0, nc, (H, nv), generator=g, device=GPU), cell[None])
    z = torch.cat([z, torch.full((H, tail), nc, device=GPU)], 1)
    out = []
    for _ in range(3):
        mu = torch.randn(H, nc + 1, d, generator=g, device=GPU)
        x = torch.empty(1, H, nv + tail, d, dtype=DT[case["dtype"]], device=GPU)
        for k in range(H):
            x[0, k] = mu[k][z[k]] + 0.3 * torch.randn(nv + tail, d, generator=g, device=GPU)
        out.append(x)
    return out


def _start(x, c, nv, g):
    """c distinct rows of every head, fp32 [1, heads, c, d]."""
    return torch.stack([x[0, k][torch.randperm(nv, generator=g, device=GPU)[:c]].float() for k in range(x.shape[1])])[None]


def _means(x, lab, old):
    """Means of a head's rows by label; the sums are whole numbers, so their order does not matter."""
    c, d = old.shape
    total = torch.zeros(c, d, dtype=torch.int64, device=GPU).index_add_(0, lab, (x.float() * 65536.0).round().long())
    n = torch.bincount(lab, minlength=c)
    mean = (total.double() / 65536.0 / n.clamp(min=1)[:, None].double()).float()
    return torch.where((n > 0)[:, None], mean, old)


def _nearest(x, c):
    return ((c * c).sum(1)[None] - 2.0 * (x @ c.t())).argmin(1)


def _cluster(x, c0, nv, iters, x2=None):
    """Labels, centroids and, with x2, its means, all of `iters` plain Lloyd iterations of every head."""
    labels, cents, means2 = [], [], []
    for k in range(x.shape[1]):
        rows, c = x[0, k, :nv].float(), c0[0, k]
        for _ in range(iters):
            lab = _nearest(rows, c)
            c = _means(rows, lab, c)
        labels.append(lab)
        cents.append(c)
        if x2 is not None:
            means2.append(_means(x2[0, k, :nv], lab, torch.zeros_like(c)))
    return torch.stack(labels), torch.stack(cents)[None], torch.stack(means2)[None] if x2 is not None else None


def _order(labels, c, tail):
    """perm [1, heads, n] and offsets [1, heads, c + 2], int32, of rows sorted by label, text rows last."""
    H = labels.shape[0]
    full = torch.cat([labels, torch.full((H, tail), c, device=GPU)], 1)
    perm = torch.argsort(full, dim=1, stable=True)
    sizes = torch.stack([torch.bincount(r, minlength=c + 1) for r in full])
    off = torch.cat([torch.zeros(H, 1, dtype=torch.int64, device=GPU), sizes.cumsum(1)], 1)
    return perm.int()[None].contiguous(), off.int()[None].contiguous()


def _rows(x, perm):
    return torch.stack([x[0, k][perm[0, k].long()] for k in range(x.shape[1])])[None].contiguous()


def _budget(case):
    return int(case["rho"] * _n(case) ** 2)


def _route(score, qoff, koff, budget):
    """[heads, cq + 1, ck + 1] mask: text blocks, then blocks by descending score while they fit."""
    H, cq, ck = score.shape
    qs, ks = qoff[0].diff(dim=1).long(), koff[0].diff(dim=1).long()
    cost = qs[:, :, None] * ks[:, None, :]
    inner = cost[:, :cq, :ck].reshape(H, -1)
    left = budget - (cost.sum((1, 2)) - inner.sum(1))
    key = torch.where(inner > 0, score.reshape(H, -1).double(), -1.0)
    at = torch.argsort(key, dim=1, descending=True, stable=True)
    fits = (inner.gather(1, at).cumsum(1) <= left[:, None]) & (inner.gather(1, at) > 0)
    mask = torch.zeros(H, cq + 1, ck + 1, dtype=torch.bool, device=GPU)
    mask[:, :cq, :ck] = torch.zeros_like(fits).scatter_(1, at, fits).reshape(H, cq, ck)
    mask[:, cq, :] = True
    mask[:, :, ck] = True
    return mask & (cost > 0)


def _lists(mask):
    """mask_bits, row_ptr and col_idx of a mask, laid out as svgear_probe_route writes them."""
    H, R, C = mask.shape
    W = (C + 31) // 32
    words = torch.zeros(H, R, W * 32, dtype=torch.int64, device=GPU)
    words[:, :, :C] = mask
    bits = (words.reshape(H, R, W, 32) << torch.arange(32, device=GPU)).sum(3)
    bits = torch.where(bits >= 1 << 31, bits - (1 << 32), bits).int()
    ptr = torch.cat([torch.zeros(H, 1, dtype=torch.int64, device=GPU), mask.sum(2).cumsum(1)], 1).int()
    col = torch.zeros(H, R * C, dtype=torch.int32, device=GPU)
    k, r, c = mask.nonzero(as_tuple=True)
    pos = mask.reshape(H, -1).long().cumsum(1) - 1
    col[k, pos[k, r * C + c]] = c.int()
    return bits[None].contiguous(), ptr[None].contiguous(), col[None].contiguous()


def prepare(case, seed):
    g = _generator(seed)
    n, tail, cq, ck, what = _n(case), case["tail"], case["cq"], case["ck"], case["what"]
    nv = n - tail
    Q, K, V = _qkv(case, g)
    s = {"case": case, "scale": float(case["d"]) ** -0.5, "n": n}
    if what == "layer":
        cq0, ck0 = _start(Q, cq, nv, g), _start(K, ck, nv, g)
        if case.get("warm"):  # the previous step's centroids; this step's tokens have drifted
            cq0, ck0 = _cluster(Q, cq0, nv, 3)[1], _cluster(K, ck0, nv, 3)[1]
            for x in (Q, K, V):
                for k in range(x.shape[1]):
                    x[0, k] = x[0, k].float() + 0.05 * torch.randn(n, case["d"], generator=g, device=GPU)
        return {**s, "Q": Q, "K": K, "V": V, "cq0": cq0, "ck0": ck0, "budget": _budget(case)}
    if what == "kmeans":
        return {**s, "K": K, "V": V if case.get("x2") else None, "ck0": _start(K, ck, nv, g)}
    lab_k, kbar, vbar = _cluster(K, _start(K, ck, nv, g), nv, 3, V)
    if what == "permute":
        return {**s, "K": K, "V": V, "labels": lab_k.int()[None].contiguous()}
    lab_q, qbar, _ = _cluster(Q, _start(Q, cq, nv, g), nv, 3)
    perm_q, qoff = _order(lab_q, cq, tail)
    perm_k, koff = _order(lab_k, ck, tail)
    s.update(Kp=_rows(K, perm_k), Vp=_rows(V, perm_k), qbar=qbar, kbar=kbar, vbar=vbar, qoff=qoff, koff=koff,
             budget=_budget(case))
    if what == "probe":
        return s
    sizes = koff[0].diff(dim=1)[:, :ck]
    logit = (qbar[0] @ kbar[0].transpose(1, 2).contiguous()) * s["scale"]
    logit = torch.where(sizes[:, None] > 0, logit, -math.inf)
    mask = _route(torch.exp(2.0 * (logit - logit.amax(2, keepdim=True))), qoff, koff, s["budget"])
    bits, ptr, col = _lists(mask)
    s.update(mask=mask, bits=bits, ptr=ptr, col=col, perm_q=perm_q, Q=Q)
    if not case["token_order"]:
        s["Q"] = _rows(Q, perm_q)
    return s


# ------------------------------------------------------------------------------------- calls
def run(s):
    case = s["case"]
    what = case["what"]
    if what == "layer":
        cq, ck = s["cq0"].clone(), s["ck0"].clone()  # the call updates them in place
        O, _ = sv.attention_layer(s["Q"], s["K"], s["V"], cq, ck, case["iters"], s["budget"], case["tail"])
        return {"O": O, "cq": cq, "ck": ck}
    if what == "kmeans":
        ck = s["ck0"].clone()
        labels, counts, means2 = sv.kmeans(s["K"], ck, case["iters"], case["tail"], x2=s["V"])
        return {"centroids": ck, "labels": labels, "counts": counts, "means2": means2}
    if what == "permute":
        perm, offsets, (Kp, Vp) = sv.permute(s["labels"], case["ck"], [s["K"], s["V"]], case["tail"])
        return {"perm": perm, "offsets": offsets, "Kp": Kp, "Vp": Vp}
    if what == "probe":
        r = sv.probe_route(s["qbar"], s["kbar"], s["vbar"], s["Kp"], s["Vp"], s["qoff"], s["koff"], s["budget"],
                           s["scale"], top_p=case.get("top_p"))
        # the mask holds all that row_ptr, col_idx (unwritten behind its last entry) and routed_cost say
        out = {"scores": r["scores"], "mask": r["mask_bits"]}
        if "row_budget" in r:
            out["row_budget"] = r["row_budget"]
        return out
    perm = s["perm_q"] if case["token_order"] else None
    O, lse = sv.sparse_attn_comp(s["Q"], s["Kp"], s["Vp"], s["kbar"], s["vbar"], s["qoff"], s["koff"], s["bits"],
                                 s["ptr"], s["col"], s["scale"], want_lse=True, q_perm=perm)
    return {"O": O if case["token_order"] else sv.unpermute(O, s["perm_q"]), "lse": lse}


def work(case):
    H, n, d, cq, ck, tail = case["heads"], _n(case), case["d"], case["cq"], case["ck"], case["tail"]
    es = 2 if case["dtype"] == "bf16" else 4
    rows, what = H * n * d * es, case["what"]
    tables = 4.0 * H * d * (cq + 2 * ck)
    pairs = case["rho"] * float(n) ** 2 + (n - tail) * ck * 0.75  # routed, and the pseudo-keys of the rest
    attend, probe = 4.0 * H * d * pairs, 2.0 * H * n * cq * d
    assign = 2.0 * H * n * d  # for one centroid: one pass over all of them cannot be left out
    if what == "layer":
        return {"bytes": 4.0 * rows + 2.0 * tables, "flops": attend + probe + assign * (cq + ck)}
    if what == "kmeans":
        return {"bytes": rows * (2.0 if case.get("x2") else 1.0) + 4.0 * H * (n + 3 * ck * d), "flops": assign * ck}
    if what == "permute":
        return {"bytes": 4.0 * rows + 8.0 * H * n, "flops": 0.0}
    if what == "probe":
        return {"bytes": 2.0 * rows + tables + 4.0 * H * cq * ck, "flops": probe}
    return {"bytes": 4.0 * rows + tables + H * n * 8.0, "flops": attend}


def tolerance(case):
    what, bf = case["what"], case["dtype"] == "bf16"
    if what == "permute":
        return "exact"
    if what == "kmeans":  # fp32 sums of up to some thousand rows; a row between two centroids may go to either
        return {"rel": 1e-4, "max": 0.2, "differ": 1e-3}
    if what == "probe":  # sums over a cluster of squares of fp32 differences; blocks at the budget's edge may swap
        return {"rel": 5e-6, "max": 1e-3, "differ": 1e-3}
    if what == "attention":
        return {"rel": 1e-2, "max": 0.1} if bf else {"rel": 4e-6, "max": 1e-4}
    return {"rel": 1e-2, "max": 0.3} if bf else {"rel": 1e-4, "max": 1e-2}


# ------------------------------------------------------------------------- the same in 64 bits
def _kmeans64(x, c0, nv, iters, x2=None):
    labels, cents, means2 = [], [], []
    for k in range(x.shape[1]):
        rows, c = x[0, k, :nv].double(), c0[0, k].double()
        for _ in range(iters):
            lab = _nearest(rows, c)
            n = torch.bincount(lab, minlength=c.shape[0])[:, None]
            c = torch.where(n > 0, torch.zeros_like(c).index_add_(0, lab, rows) / n.clamp(min=1), c)
        labels.append(lab)
        cents.append(c)
        if x2 is not None:
            means2.append(torch.zeros_like(c).index_add_(0, lab, x2[0, k, :nv].double()) / n.clamp(min=1))
    return torch.stack(labels), torch.stack(cents)[None], torch.stack(means2)[None] if x2 is not None else None


def _scores64(qbar, kbar, vbar, Kp, Vp, koff, scale):
    """Squared error of every block per query and key, over the row's largest centroid weight."""
    out = []
    for k in range(Kp.shape[1]):
        ck = kbar.shape[2]
        sizes = koff[0, k].diff()[:ck].long()
        lab = torch.repeat_interleave(torch.arange(ck, device=GPU), sizes)
        nv = lab.numel()
        q, kb, vb = qbar[0, k].double(), kbar[0, k].double(), vbar[0, k].double()
        S = torch.where(sizes[None] > 0, (q @ kb.t()) * scale, -math.inf)
        m = S.amax(1, keepdim=True)
        W = torch.exp(S - m)
        w = torch.exp((q @ Kp[0, k, :nv].double().t()) * scale - m)
        v = Vp[0, k, :nv].double()
        off = v - vb[lab]
        gap = W[:, lab] - w
        # |W vbar - w v|^2 with v = vbar + off
        err = gap * gap * (vb * vb).sum(1)[lab] - 2.0 * gap * w * (vb[lab] * off).sum(1) + w * w * (off * off).sum(1)
        E = torch.zeros(q.shape[0], ck, dtype=torch.float64, device=GPU).index_add_(1, lab, err)
        out.append(torch.where(sizes[None] > 0, E / sizes.clamp(min=1)[None], 0.0))
    return torch.stack(out)


def _attend64(Qp, Kp, Vp, kbar, vbar, qoff, koff, mask, scale):
    """Output and log of the softmax's denominator, rows in permuted order."""
    outs, lses = [], []
    for k in range(Kp.shape[1]):
        cq, ck = mask.shape[1] - 1, mask.shape[2] - 1
        qs, ks = qoff[0, k].diff().long(), koff[0, k].diff().long()
        rows_of = torch.repeat_interleave(torch.arange(cq + 1, device=GPU), qs)
        keys_of = torch.repeat_interleave(torch.arange(ck + 1, device=GPU), ks)
        K64, V64, kb, vb = Kp[0, k].double(), Vp[0, k].double(), kbar[0, k].double(), vbar[0, k].double()
        o, l = [], []
        for r0 in range(0, Qp.shape[2], 1024):
            q, a = Qp[0, k, r0:r0 + 1024].double(), rows_of[r0:r0 + 1024]
            s = (q @ K64.t()) * scale
            s.masked_fill_(~mask[k][a][:, keys_of], -math.inf)
            c = (q @ kb.t()) * scale + torch.log(ks[:ck].double())[None]
            c.masked_fill_(mask[k][a][:, :ck] | (a == cq)[:, None], -math.inf)
            lse = torch.logaddexp(torch.logsumexp(s, 1), torch.logsumexp(c, 1))[:, None]
            o.append(torch.exp(s - lse) @ V64 + torch.exp(c - lse) @ vb)
            l.append(lse[:, 0])
        outs.append(torch.cat(o))
        lses.append(torch.cat(l))
    return torch.stack(outs)[None], torch.stack(lses)[None]


def _back(x, perm):
    return torch.empty_like(x).scatter_(2, perm.long().reshape(perm.shape + (1,) * (x.dim() - 3)).expand(x.shape), x)


def exact(case, seed):
    what, n, tail = case["what"], _n(case), case["tail"]
    if what == "permute" or (what == "layer" and case["heads"] * n > 20000):
        return None  # rows are moved as they are; a large layer's clusters take too long in 64 bits
    s = prepare(case, seed)
    nv = n - tail
    if what == "kmeans":
        _, c, c2 = _kmeans64(s["K"], s["ck0"], nv, case["iters"], s["V"])
        return {"centroids": c, "labels": None, "counts": None, "means2": c2}
    if what == "probe":
        out = {"scores": _scores64(s["qbar"], s["kbar"], s["vbar"], s["Kp"], s["Vp"], s["koff"], s["scale"])[None],
               "mask": None}
        return {**out, "row_budget": None} if "top_p" in case else out
    if what == "attention":
        Qp = _rows(s["Q"], s["perm_q"]) if case["token_order"] else s["Q"]
        O, lse = _attend64(Qp, s["Kp"], s["Vp"], s["kbar"], s["vbar"], s["qoff"], s["koff"], s["mask"], s["scale"])
        return {"O": _back(O, s["perm_q"]), "lse": _back(lse, s["perm_q"]) if case["token_order"] else lse}
    lab_q, cq, _ = _kmeans64(s["Q"], s["cq0"], nv, case["iters"])
    lab_k, ck, vbar = _kmeans64(s["K"], s["ck0"], nv, case["iters"], s["V"])
    perm_q, qoff = _order(lab_q, case["cq"], tail)
    perm_k, koff = _order(lab_k, case["ck"], tail)
    Kp, Vp = _rows(s["K"], perm_k), _rows(s["V"], perm_k)
    mask = _route(_scores64(cq, ck, vbar, Kp, Vp, koff, s["scale"]), qoff, koff, s["budget"])
    O, _ = _attend64(_rows(s["Q"], perm_q), Kp, Vp, ck, vbar, qoff, koff, mask, s["scale"])
    return {"O": _back(O, perm_q), "cq": cq, "ck": ck}
