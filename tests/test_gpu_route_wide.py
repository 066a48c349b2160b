"""GPU parity of the router where a head's blocks are cut and listed by many workgroups (16,384
blocks and more), on both sides of that line, from injected scores: masks, lists and costs are
whole numbers and equal the oracle's."""
import numpy as np
import pytest
import torch

import paper_2603_08982_amd as sv
from oracle import svgear_oracle as orc
from helpers import dev, to_np, bits_to_mask, full_mask, csr_from_mask

pytestmark = pytest.mark.gpu


def _scores(kind, rng, H, Cq, Ck):
    if kind == "equal":  # one digit holds every block
        return np.full((H, Cq, Ck), 0.75, np.float32)
    s = rng.lognormal(0.0, 2.0, (H, Cq, Ck)).astype(np.float32)
    if kind == "odd":  # NaN and infinity first, zeros of both signs tied, runs of equal scores
        s[rng.random(s.shape) < 0.01] = np.nan
        s[rng.random(s.shape) < 0.01] = np.inf
        s[rng.random(s.shape) < 0.2] = 0.0
        s[rng.random(s.shape) < 0.1] = -0.0
        s[rng.random(s.shape) < 0.3] = 1.0
    if kind == "close":  # equal in the leading 12 bits of the key, apart in the last
        s = (1.0 + rng.integers(0, 1 << 16, s.shape) * 2.0 ** -23).astype(np.float32)
    return s


@pytest.mark.parametrize("Cq,Ck", [(127, 129), (128, 128), (1, 8192), (300, 1000), (8, 2049), (2050, 8), (5, 3999), (5, 4000)])
@pytest.mark.parametrize("kind", ["plain", "equal", "odd", "close"])
def test_cut_and_lists_of_many_blocks(Cq, Ck, kind):
    rng = np.random.default_rng(Cq * 7 + Ck)
    H, n_tail = 2, 21
    nv = max(3 * Cq, 2 * Ck, 9000)
    N = nv + n_tail
    lab_q, lab_k = rng.integers(0, Cq, (H, nv)).astype(np.int32), rng.integers(0, Ck, (H, nv)).astype(np.int32)
    if Cq > 2:
        lab_q[lab_q == 1] = 2  # an empty query cluster
    lab_k[lab_k == Ck - 1] = 0  # an empty key cluster
    _, qoff, _ = sv.permute(torch.from_numpy(lab_q)[None].to(dev()), Cq, n_tail=n_tail)
    _, koff, _ = sv.permute(torch.from_numpy(lab_k)[None].to(dev()), Ck, n_tail=n_tail)
    scores = _scores(kind, rng, H, Cq, Ck)
    given = torch.from_numpy(scores)[None].to(dev())
    z = torch.zeros(1, H, 1, 64, device=dev())
    qbar, kbar = z.expand(1, H, Cq, 64).contiguous(), z.expand(1, H, Ck, 64).contiguous()
    Kp = torch.zeros(1, H, N, 64, dtype=torch.bfloat16, device=dev())
    for budget, flags in ((0, 0), (N * N // 4, 0), (N * N - 1, 0), (N * N, 0), (N * N // 3, sv.ROUTE_PER_ROW)):
        r = sv.probe_route(qbar, kbar, kbar, Kp, Kp, qoff, koff, budget, 0.125, flags=sv.USE_GIVEN_SCORES | flags,
                           scores=given.clone())
        torch.cuda.synchronize()
        for h in range(H):
            qs, ks = np.bincount(lab_q[h], minlength=Cq), np.bincount(lab_k[h], minlength=Ck)
            m_ref, _, _, cost_ref = orc.route(scores[h], qs, ks, budget, n_tail_q=n_tail, n_tail_k=n_tail,
                                              per_row=bool(flags))
            mask = full_mask(m_ref, Cq, Ck)
            assert np.array_equal(bits_to_mask(to_np(r["mask_bits"][0, h]), Ck), mask)
            row_ptr, col_idx = csr_from_mask(mask)
            assert np.array_equal(to_np(r["row_ptr"][0, h]), row_ptr)
            assert np.array_equal(to_np(r["col_idx"][0, h])[: row_ptr[-1]], col_idx[: row_ptr[-1]])
            assert int(r["routed_cost"][0, h]) == cost_ref
