"""GPU counting sort at the sizes where its one-workgroup form changes: tokens around multiples of the
64-token step and of the 1,024-token round, at its largest and just above, few and many labels, text
rows. Whole numbers, equal to a stable argsort."""
import numpy as np
import pytest
import torch

import paper_2603_08982_amd as sv
from helpers import dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,C", [(N, C) for C in (1, 2, 63, 1000, 1023, 1024, 2048, 2049)
                                 for N in (2, 63, 64, 65, 1023, 1024, 1025, 4096, 4097, 8191, 8192, 8193) if C < N])
def test_sort_is_the_stable_argsort(N, C):
    rng = np.random.default_rng(N + C)
    H = 3
    for n_tail in (0, 1 if N < 66 else 37):
        nv = N - n_tail
        if C > nv:
            continue
        lab = np.stack([rng.integers(0, C, nv), np.full(nv, C - 1), np.sort(rng.integers(0, max(1, C // 3), nv))[::-1]])
        x = torch.randn(1, H, N, 64, device=dev())
        perm, off, (xp,) = sv.permute(torch.from_numpy(lab.astype(np.int32))[None].to(dev()), C, [x], n_tail=n_tail)
        torch.cuda.synchronize()
        for h in range(H):
            full = np.concatenate([lab[h], np.full(n_tail, C)])
            ref = np.argsort(full, kind="stable")
            assert np.array_equal(to_np(perm[0, h]), ref)
            assert np.array_equal(to_np(off[0, h]), np.concatenate([[0], np.cumsum(np.bincount(full, minlength=C + 1))]))
            assert torch.equal(xp[0, h], x[0, h][torch.from_numpy(ref).to(dev())])


@pytest.mark.parametrize("N", [3000, 30000])
def test_tensors_move_as_if_one_after_the_other(N):
    """A destination may be where another tensor's rows lie: a chain of three moves through one spare buffer,
    and a source that an earlier move has written."""
    C, d = 50, 128
    lab = torch.randint(0, C, (1, 1, N), generator=torch.Generator().manual_seed(N), dtype=torch.int32).to(dev())
    order = torch.argsort(lab[0, 0].long(), stable=True)
    fresh = lambda: [torch.randn(1, 1, N, d, device=dev()).to(torch.bfloat16) for _ in range(3)]
    out = lambda tensors: (torch.empty(1, 1, N, dtype=torch.int32, device=dev()),
                           torch.empty(1, 1, C + 2, dtype=torch.int32, device=dev()), tensors)
    a, b, c = fresh()
    spare, want = torch.empty_like(a), [x[:, :, order].clone() for x in (a, b, c)]
    sv.permute(lab, C, [a, b, c], out=out([spare, a, b]))
    torch.cuda.synchronize()
    for got, ref in zip((spare, a, b), want):
        assert torch.equal(got, ref)
    a, b, c = fresh()
    want = [a[:, :, order].clone(), a[:, :, order][:, :, order].clone()]
    sv.permute(lab, C, [a, b], out=out([b, c]))
    torch.cuda.synchronize()
    assert torch.equal(b, want[0]) and torch.equal(c, want[1])
