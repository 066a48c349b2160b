"""ctypes binding of libsvgear.so: argument marshalling only.

Each function mirrors one entry point of include/svgear.h, allocates outputs and the
workspace with torch on the inputs' device, and enqueues the call on torch's current
stream. No arithmetic of the method happens here.
"""
from __future__ import annotations

import ctypes
import os
from typing import Optional, Sequence

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB = None

PROBE_PLAIN = 1
ROUTE_PER_ROW = 2
USE_GIVEN_SCORES = 4

EXPORTED_SYMBOLS = [
    "svgear_version", "svgear_last_hip_error",
    "svgear_kmeans_workspace", "svgear_kmeans", "svgear_kmeans_stepwise", "svgear_kmeans_list_threshold",
    "svgear_permute_workspace", "svgear_permute", "svgear_permute_rows",
    "svgear_permute_static_capacity", "svgear_permute_static",
    "svgear_probe_route_workspace", "svgear_probe_route", "svgear_probe_route_top_p",
    "svgear_sparse_attn_comp_workspace", "svgear_sparse_attn_comp", "svgear_sparse_attn_comp_token_order",
    "svgear_sparse_attn_two_stage_workspace", "svgear_sparse_attn_two_stage",
    "svgear_unpermute",
]

_c = ctypes
_vp, _i, _i64, _sz, _f, _u = _c.c_void_p, _c.c_int, _c.c_int64, _c.c_size_t, _c.c_float, _c.c_uint
_I64x3 = _c.c_int64 * 3


class SvgearError(RuntimeError):
    pass


def lib_path() -> str:
    return os.path.join(_HERE, "libsvgear.so")


def load_library():
    """Loads the built library; builds it first only if no built library exists."""
    global _LIB
    if _LIB is not None:
        return _LIB
    path = lib_path()
    if not os.path.exists(path):
        from .build import build

        build()
    lib = ctypes.CDLL(path)
    lib.svgear_version.restype = _i
    lib.svgear_last_hip_error.restype = _i
    lib.svgear_kmeans_workspace.restype = _sz
    lib.svgear_kmeans_workspace.argtypes = [_i, _i, _i64, _i, _i]
    lib.svgear_kmeans.restype = _i
    lib.svgear_kmeans.argtypes = [_vp, _vp, _i, _i, _i, _i64, _i64, _i, _c.POINTER(_c.c_int64), _i, _i,
                                  _vp, _vp, _vp, _vp, _vp, _sz, _vp]
    lib.svgear_kmeans_stepwise.restype = _i
    lib.svgear_kmeans_stepwise.argtypes = lib.svgear_kmeans.argtypes
    lib.svgear_permute_workspace.restype = _sz
    lib.svgear_permute_workspace.argtypes = [_i, _i, _i64, _i]
    lib.svgear_permute.restype = _i
    lib.svgear_permute.argtypes = [_vp, _i, _i, _i64, _i64, _i, _vp, _vp, _i, _c.POINTER(_vp),
                                   _c.POINTER(_I64x3), _c.POINTER(_vp), _i, _i, _vp, _sz, _vp]
    lib.svgear_permute_static_capacity.restype = _sz
    lib.svgear_permute_static_capacity.argtypes = []
    lib.svgear_permute_static.restype = _i
    lib.svgear_permute_static.argtypes = lib.svgear_permute.argtypes[:14] + [_vp]
    lib.svgear_permute_rows.restype = _i
    lib.svgear_permute_rows.argtypes = [_vp, _i, _i, _i64, _i, _c.POINTER(_vp), _c.POINTER(_I64x3), _c.POINTER(_vp),
                                        _i, _i, _vp]
    lib.svgear_probe_route_workspace.restype = _sz
    lib.svgear_probe_route_workspace.argtypes = [_i, _i, _i64, _i, _i, _i]
    lib.svgear_probe_route.restype = _i
    lib.svgear_probe_route.argtypes = [_vp, _vp, _vp, _vp, _vp, _i, _vp, _vp, _i, _i, _i64, _i64, _i, _i, _i,
                                       _i64, _f, _u, _vp, _vp, _vp, _vp, _vp, _vp, _sz, _vp]
    lib.svgear_probe_route_top_p.restype = _i
    lib.svgear_probe_route_top_p.argtypes = [_vp, _vp, _vp, _vp, _vp, _i, _vp, _vp, _i, _i, _i64, _i64, _i, _i, _i,
                                             _f, _f, _u, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _sz, _vp]
    lib.svgear_sparse_attn_comp_workspace.restype = _sz
    lib.svgear_sparse_attn_comp_workspace.argtypes = [_i, _i, _i64, _i64, _i, _i, _i]
    lib.svgear_sparse_attn_comp.restype = _i
    lib.svgear_sparse_attn_comp.argtypes = [_vp, _vp, _vp, _i, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _i, _i, _i64,
                                            _i64, _i, _i, _i, _f, _vp, _vp, _vp, _sz, _vp]
    lib.svgear_sparse_attn_comp_token_order.restype = _i
    lib.svgear_sparse_attn_comp_token_order.argtypes = [_vp, _c.POINTER(_c.c_int64), _vp, _vp, _i, _vp, _vp, _vp, _vp,
                                                        _vp, _vp, _vp, _vp, _i, _i, _i64, _i64, _i, _i, _i, _f, _vp,
                                                        _c.POINTER(_c.c_int64), _vp, _vp, _sz, _vp]
    lib.svgear_sparse_attn_two_stage_workspace.restype = _sz
    lib.svgear_sparse_attn_two_stage_workspace.argtypes = lib.svgear_sparse_attn_comp_workspace.argtypes
    lib.svgear_sparse_attn_two_stage.restype = _i
    lib.svgear_sparse_attn_two_stage.argtypes = lib.svgear_sparse_attn_comp.argtypes
    lib.svgear_unpermute.restype = _i
    lib.svgear_unpermute.argtypes = [_vp, _vp, _i, _i, _i, _i64, _i, _vp, _c.POINTER(_c.c_int64), _vp]
    _LIB = lib
    return lib


_STATUS = {-1: "invalid argument", -2: "workspace too small", -3: "HIP runtime error", -4: "unsupported"}


def _check(rc: int, what: str):
    if rc != 0:
        extra = f" (hip error {load_library().svgear_last_hip_error()})" if rc == -3 else ""
        raise SvgearError(f"{what} failed: {_STATUS.get(rc, rc)}{extra}")


def _dt(t: torch.Tensor) -> int:
    if t.dtype == torch.float32:
        return 0
    if t.dtype == torch.bfloat16:
        return 1
    raise SvgearError(f"unsupported dtype {t.dtype}")


def _need_gpu(*ts):
    for t in ts:
        if t is not None and not t.is_cuda:
            raise SvgearError("svgear needs device tensors: there is no CPU path")


def _stream() -> int:
    return torch.cuda.current_stream().cuda_stream


def _ptr(t: Optional[torch.Tensor]):
    return None if t is None else t.data_ptr()


def _strides4(t: torch.Tensor):
    assert t.dim() == 4 and t.stride(3) == 1, "expected [B,H,N,d] with contiguous d"
    return _I64x3(t.stride(0), t.stride(1), t.stride(2))


def _ws(nbytes: int, device) -> torch.Tensor:
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device=device)


def kmeans_list_threshold(min_centroids: int = 0) -> int:
    """svgear_kmeans_list_threshold: sets (>= 1) or queries (<= 0) the number of centroids from which
    the later k-means iterations use candidate lists; returns the previous value."""
    lib = load_library()
    lib.svgear_kmeans_list_threshold.restype = _i
    lib.svgear_kmeans_list_threshold.argtypes = [_i]
    return int(lib.svgear_kmeans_list_threshold(int(min_centroids)))


def kmeans(x: torch.Tensor, centroids: torch.Tensor, iters: int, n_tail: int = 0,
           x2: Optional[torch.Tensor] = None, one_launch: bool = True):
    """svgear_kmeans (one_launch=False: svgear_kmeans_stepwise, the same results with launches of its own for
    every step of a small call too). x [B,H,N,d]; centroids [B,H,C,d] fp32 (updated in place).
    Returns (labels [B,H,N-n_tail] i32, counts [B,H,C] i32, centroids2 or None)."""
    _need_gpu(x, centroids, x2)
    lib = load_library()
    B, H, N, d = x.shape
    C = centroids.shape[2]
    assert centroids.dtype == torch.float32 and centroids.is_contiguous()
    if x2 is not None:
        assert x2.shape == x.shape and x2.stride() == x.stride() and x2.dtype == x.dtype
    labels = torch.empty(B, H, N - n_tail, dtype=torch.int32, device=x.device)
    counts = torch.empty(B, H, C, dtype=torch.int32, device=x.device)
    c2 = torch.zeros(B, H, C, d, dtype=torch.float32, device=x.device) if x2 is not None else None
    ws = _ws(lib.svgear_kmeans_workspace(B, H, N, d, C), x.device)
    st = _strides4(x)
    fn = lib.svgear_kmeans if one_launch else lib.svgear_kmeans_stepwise
    rc = fn(_ptr(x), _ptr(x2), _dt(x), B, H, N, n_tail, d, st, C, iters, _ptr(centroids), _ptr(c2), _ptr(labels),
            _ptr(counts), _ptr(ws), ws.numel(), _stream())
    _check(rc, "svgear_kmeans" if one_launch else "svgear_kmeans_stepwise")
    return labels, counts, c2


def permute(labels: torch.Tensor, C: int, tensors: Sequence[torch.Tensor] = (), n_tail: int = 0,
            static_scratch: bool = False, out=None):
    """svgear_permute (static_scratch=True: svgear_permute_static, whose scratch is an array inside
    the library; with out=(perm, offsets, [dst tensors]) preallocated by the caller that call
    touches no allocator at all). Returns (perm [B,H,N] i32, offsets [B,H,C+2] i32, [permuted tensors])."""
    _need_gpu(labels, *tensors)
    lib = load_library()
    B, H, nv = labels.shape
    N = nv + n_tail
    assert labels.dtype == torch.int32 and labels.is_contiguous()
    n = len(tensors)
    d, dt = 64, 0
    if n:
        d, dt = tensors[0].shape[3], _dt(tensors[0])
        for t in tensors:
            assert t.shape == (B, H, N, d) and _dt(t) == dt
    if out is not None:
        perm, offsets, outs = out
        assert perm.shape == (B, H, N) and perm.dtype == torch.int32 and perm.is_contiguous()
        assert offsets.shape == (B, H, C + 2) and offsets.dtype == torch.int32 and offsets.is_contiguous()
        assert len(outs) == n
        for o, t in zip(outs, tensors):
            assert o.shape == t.shape and o.dtype == t.dtype and o.is_contiguous()
        _need_gpu(perm, offsets, *outs)
    else:
        perm = torch.empty(B, H, N, dtype=torch.int32, device=labels.device)
        offsets = torch.empty(B, H, C + 2, dtype=torch.int32, device=labels.device)
        outs = [torch.empty(B, H, N, d, dtype=t.dtype, device=t.device) for t in tensors]
    src = (_vp * max(n, 1))(*[t.data_ptr() for t in tensors])
    dst = (_vp * max(n, 1))(*[t.data_ptr() for t in outs])
    sst = (_I64x3 * max(n, 1))(*[_strides4(t) for t in tensors])
    if static_scratch:
        rc = lib.svgear_permute_static(_ptr(labels), B, H, N, n_tail, C, _ptr(perm), _ptr(offsets), n, src, sst, dst,
                                       dt, d, _stream())
        _check(rc, "svgear_permute_static")
        return perm, offsets, outs
    ws = _ws(lib.svgear_permute_workspace(B, H, N, C), labels.device)
    rc = lib.svgear_permute(_ptr(labels), B, H, N, n_tail, C, _ptr(perm), _ptr(offsets), n, src, sst, dst, dt, d,
                            _ptr(ws), ws.numel(), _stream())
    _check(rc, "svgear_permute")
    return perm, offsets, outs


def permute_rows(perm: torch.Tensor, tensors: Sequence[torch.Tensor]):
    """svgear_permute_rows: the tensors' rows gathered through an existing permutation."""
    _need_gpu(perm, *tensors)
    lib = load_library()
    B, H, N = perm.shape
    assert perm.dtype == torch.int32 and perm.is_contiguous() and len(tensors) >= 1
    d, dt = tensors[0].shape[3], _dt(tensors[0])
    for t in tensors:
        assert t.shape == (B, H, N, d) and _dt(t) == dt
    outs = [torch.empty(B, H, N, d, dtype=t.dtype, device=t.device) for t in tensors]
    n = len(tensors)
    src = (_vp * n)(*[t.data_ptr() for t in tensors])
    dst = (_vp * n)(*[t.data_ptr() for t in outs])
    sst = (_I64x3 * n)(*[_strides4(t) for t in tensors])
    rc = lib.svgear_permute_rows(_ptr(perm), B, H, N, n, src, sst, dst, dt, d, _stream())
    _check(rc, "svgear_permute_rows")
    return outs


def probe_route(qbar, kbar, vbar, kp, vp, q_offsets, k_offsets, budget_cost: int, scale: float,
                flags: int = 0, scores: Optional[torch.Tensor] = None, Nq: Optional[int] = None,
                top_p: Optional[float] = None):
    """svgear_probe_route, or svgear_probe_route_top_p when top_p is given (budget_cost is then
    ignored). Returns dict(scores, mask_bits, row_ptr, col_idx, routed_cost[, row_budget])."""
    _need_gpu(qbar, kbar, vbar, kp, vp, q_offsets, k_offsets, scores)
    lib = load_library()
    B, H, Cq, d = qbar.shape
    Ck = kbar.shape[2]
    Nk = kp.shape[2]
    Nq = Nk if Nq is None else int(Nq)
    dev = qbar.device
    if scores is None:
        scores = torch.empty(B, H, Cq, Ck, dtype=torch.float32, device=dev)
    assert scores.shape == (B, H, Cq, Ck) and scores.dtype == torch.float32 and scores.is_contiguous()
    W = (Ck + 1 + 31) // 32
    mask_bits = torch.empty(B, H, Cq + 1, W, dtype=torch.int32, device=dev)
    row_ptr = torch.empty(B, H, Cq + 2, dtype=torch.int32, device=dev)
    col_idx = torch.empty(B, H, (Cq + 1) * (Ck + 1), dtype=torch.int32, device=dev)
    routed_cost = torch.empty(B, H, dtype=torch.int64, device=dev)
    ws = _ws(lib.svgear_probe_route_workspace(B, H, Nk, d, Cq, Ck), dev)
    for t in (qbar, kbar, vbar, kp, vp, q_offsets, k_offsets):
        assert t.is_contiguous()
    if top_p is not None:
        row_budget = torch.empty(B, H, Cq, dtype=torch.int64, device=dev)
        rc = lib.svgear_probe_route_top_p(_ptr(qbar), _ptr(kbar), _ptr(vbar), _ptr(kp), _ptr(vp), _dt(kp),
                                          _ptr(q_offsets), _ptr(k_offsets), B, H, Nq, Nk, d, Cq, Ck, float(top_p),
                                          float(scale), int(flags), _ptr(scores), _ptr(mask_bits), _ptr(row_ptr),
                                          _ptr(col_idx), _ptr(routed_cost), _ptr(row_budget), _ptr(ws), ws.numel(),
                                          _stream())
        _check(rc, "svgear_probe_route_top_p")
        return dict(scores=scores, mask_bits=mask_bits, row_ptr=row_ptr, col_idx=col_idx, routed_cost=routed_cost,
                    row_budget=row_budget)
    rc = lib.svgear_probe_route(_ptr(qbar), _ptr(kbar), _ptr(vbar), _ptr(kp), _ptr(vp), _dt(kp), _ptr(q_offsets),
                                _ptr(k_offsets), B, H, Nq, Nk, d, Cq, Ck, int(budget_cost), float(scale),
                                int(flags), _ptr(scores), _ptr(mask_bits), _ptr(row_ptr), _ptr(col_idx),
                                _ptr(routed_cost), _ptr(ws), ws.numel(), _stream())
    _check(rc, "svgear_probe_route")
    return dict(scores=scores, mask_bits=mask_bits, row_ptr=row_ptr, col_idx=col_idx, routed_cost=routed_cost)


def sparse_attn_comp(qp, kp, vp, kbar, vbar, q_offsets, k_offsets, mask_bits, row_ptr, col_idx, scale: float,
                     want_lse: bool = False, ws: Optional[torch.Tensor] = None, two_stage: bool = False,
                     q_perm: Optional[torch.Tensor] = None, out: Optional[torch.Tensor] = None):
    """svgear_sparse_attn_comp (two_stage=True: svgear_sparse_attn_two_stage, the same result
    through separate routed / compensation passes and a merge).
    With q_perm: svgear_sparse_attn_comp_token_order: the first argument is then the UNPERMUTED
    query tensor [B,H,Nq,d] (any strides with contiguous d), and output and lse come in token
    order, written into `out` if given. Returns (output [B,H,Nq,d], lse or None)."""
    _need_gpu(qp, kp, vp, kbar, vbar, q_offsets, k_offsets, mask_bits, row_ptr, col_idx, q_perm, out)
    lib = load_library()
    assert not (two_stage and q_perm is not None)
    ws_fn = lib.svgear_sparse_attn_two_stage_workspace if two_stage else lib.svgear_sparse_attn_comp_workspace
    B, H, Nq, d = qp.shape
    Nk = kp.shape[2]
    Cq = q_offsets.shape[2] - 2
    Ck = k_offsets.shape[2] - 2
    for t in (kp, vp, kbar, vbar, q_offsets, k_offsets, mask_bits, row_ptr, col_idx):
        assert t.is_contiguous()
    lse = torch.empty(B, H, Nq, dtype=torch.float32, device=qp.device) if want_lse else None
    if ws is None:
        ws = _ws(ws_fn(B, H, Nq, Nk, d, Cq, Ck), qp.device)
    if q_perm is not None:
        assert q_perm.is_contiguous() and q_perm.dtype == torch.int32 and q_perm.shape == (B, H, Nq)
        o = torch.empty(B, H, Nq, d, dtype=qp.dtype, device=qp.device) if out is None else out
        assert o.shape == qp.shape and o.dtype == qp.dtype
        rc = lib.svgear_sparse_attn_comp_token_order(
            _ptr(qp), _strides4(qp), _ptr(kp), _ptr(vp), _dt(qp), _ptr(kbar), _ptr(vbar), _ptr(q_offsets),
            _ptr(k_offsets), _ptr(mask_bits), _ptr(row_ptr), _ptr(col_idx), _ptr(q_perm), B, H, Nq, Nk, d, Cq, Ck,
            float(scale), _ptr(o), _strides4(o), _ptr(lse), _ptr(ws), ws.numel(), _stream())
        _check(rc, "svgear_sparse_attn_comp_token_order")
        return o, lse
    assert qp.is_contiguous()
    fn = lib.svgear_sparse_attn_two_stage if two_stage else lib.svgear_sparse_attn_comp
    op = torch.empty_like(qp)
    rc = fn(_ptr(qp), _ptr(kp), _ptr(vp), _dt(qp), _ptr(kbar), _ptr(vbar), _ptr(q_offsets), _ptr(k_offsets),
            _ptr(mask_bits), _ptr(row_ptr), _ptr(col_idx), B, H, Nq, Nk, d, Cq, Ck, float(scale), _ptr(op), _ptr(lse),
            _ptr(ws), ws.numel(), _stream())
    _check(rc, "svgear_sparse_attn_two_stage" if two_stage else "svgear_sparse_attn_comp")
    return op, lse


def unpermute(op: torch.Tensor, perm: torch.Tensor, out: Optional[torch.Tensor] = None):
    """svgear_unpermute: out[b,h,perm[p]] = op[b,h,p]."""
    _need_gpu(op, perm, out)
    lib = load_library()
    B, H, N, d = op.shape
    assert op.is_contiguous() and perm.is_contiguous()
    if out is None:
        out = torch.empty_like(op)
    rc = lib.svgear_unpermute(_ptr(op), _ptr(perm), _dt(op), B, H, N, d, _ptr(out), _strides4(out), _stream())
    _check(rc, "svgear_unpermute")
    return out


_SIDE_STREAMS = {}


def run_pair(fn_side, fn_main):
    """Runs two independent library calls concurrently: fn_side on a second stream of the
    same device (default priority), fn_main on the current stream, and joins them. The
    k-means and permutation calls of Q and of K/V do not depend on each other and their small
    kernels leave CUs idle, so running the two side by side shortens the layer (measured
    14.2 -> 12.9 ms for both k-means and permutations at the Wan shape). Tensors fn_side
    returns are handed over to the current stream. Returns (fn_side(), fn_main())."""
    main = torch.cuda.current_stream()
    key = main.device_index
    side = _SIDE_STREAMS.get(key)
    if side is None:
        side = _SIDE_STREAMS[key] = torch.cuda.Stream(device=main.device)
    side.wait_stream(main)
    with torch.cuda.stream(side):
        a = fn_side()
    b = fn_main()
    main.wait_stream(side)

    def hand_over(x):
        if isinstance(x, torch.Tensor):
            x.record_stream(main)
        elif isinstance(x, (tuple, list)):
            for y in x:
                hand_over(y)

    hand_over(a)
    return a, b


def attention_layer(Q, K, V, init_q, init_k, iters: int, budget_cost: int, n_tail: int = 0, flags: int = 0,
                    scale: Optional[float] = None, overlap: bool = True, top_p: Optional[float] = None, mark=None,
                    token_order: bool = True):
    """One pass of the whole hot path over a batch of heads: k-means, permutation, probe + route,
    fused attention, un-permutation.

    token_order=True (default): Q's rows are never moved: only its permutation index is
    computed, and the attention kernel reads the queries and writes the output through it
    (svgear_sparse_attn_comp_token_order), so the "unpermute" stage is empty and the
    intermediates hold neither "Qp" nor "Op". token_order=False materialises Qp, runs
    svgear_sparse_attn_comp and svgear_unpermute.

    overlap=True uses a second stream of default priority for Q's side of the k-means and
    permutation stages (they do not depend on K's and V's; the small kernels of one stream fill
    the gaps of the other), joined before the probe, which needs the queries' offsets. (One fork and
    one join for both stages, since a pair costs the host some 40 us: 2 heads of 667 tokens take 192 us with one pair,
    231 with two; with mark, which tells the stages apart, a pair for each.)

    init_q [B,H,Cq,d], init_k [B,H,Ck,d] fp32 are the starting centroids (updated in place,
    so a caller can carry them to the next denoising step). With top_p the routing budget is
    the adaptive per-query-cluster one and budget_cost is ignored. mark(name), if given, is
    called on the current stream after each stage ("kmeans", "permute", "probe_route",
    "attention", "unpermute"). Returns (O, intermediates)."""
    B, H, N, d = Q.shape
    if scale is None:
        scale = float(d) ** -0.5
    Cq, Ck = init_q.shape[2], init_k.shape[2]
    km_q, km_k = lambda: kmeans(Q, init_q, iters, n_tail), lambda: kmeans(K, init_k, iters, n_tail, x2=V)
    pm_q = lambda lab: permute(lab, Cq, [] if token_order else [Q], n_tail)
    pm_k = lambda lab: permute(lab, Ck, [K, V], n_tail)

    def q_side():
        r = km_q()
        return r, pm_q(r[0])

    def k_side():
        r = km_k()
        return r, pm_k(r[0])

    one_pair = overlap and mark is None
    mark = mark or (lambda name: None)
    if one_pair:
        (q, q_rows), (k, k_rows) = run_pair(q_side, k_side)
    else:
        pair = run_pair if overlap else (lambda f, g: (f(), g()))
        q, k = pair(km_q, km_k)
        mark("kmeans")
        q_rows, k_rows = pair(lambda: pm_q(q[0]), lambda: pm_k(k[0]))
    (lab_q, qcnt, _), (lab_k, kcnt, vbar) = q, k
    (perm_q, qoff, q_rows), (perm_k, koff, (Kp, Vp)) = q_rows, k_rows
    mark("permute")
    r = probe_route(init_q, init_k, vbar, Kp, Vp, qoff, koff, budget_cost, scale, flags, top_p=top_p)
    mark("probe_route")
    if token_order:
        O, _ = sparse_attn_comp(Q, Kp, Vp, init_k, vbar, qoff, koff, r["mask_bits"], r["row_ptr"], r["col_idx"], scale,
                                q_perm=perm_q)
        mark("attention")
    else:
        (Qp,) = q_rows
        Op, _ = sparse_attn_comp(Qp, Kp, Vp, init_k, vbar, qoff, koff, r["mask_bits"], r["row_ptr"], r["col_idx"],
                                 scale)
        mark("attention")
        O = unpermute(Op, perm_q)
        r.update(Qp=Qp, Op=Op)
    mark("unpermute")
    r.update(lab_q=lab_q, lab_k=lab_k, qcnt=qcnt, kcnt=kcnt, qbar=init_q, kbar=init_k, vbar=vbar, perm_q=perm_q,
             perm_k=perm_k, qoff=qoff, koff=koff, Kp=Kp, Vp=Vp, O=O)
    return O, r
