"""The counting sort of heads too long for one workgroup: labels placed chunk by chunk (2,048 tokens, a wave per
quarter), against a stable sort. Integers: equal."""
import pytest
import torch

from paper_2603_08982_amd import binding

pytestmark = pytest.mark.gpu


# sizes: one token into a chunk, a quarter and whole chunks; labels: one, up to a power of two and past it, more than
# 64 KB of counters; from 3,700 on tokens are stored from their own order
@pytest.mark.parametrize("n,tail", [(8193, 0), (8704, 5), (10240, 0), (10239, 700), (12289, 1)])
@pytest.mark.parametrize("c", [1, 31, 32, 257, 1000, 3699, 3700, 5000, 8000])
@pytest.mark.parametrize("kind", ["random", "runs"])
def test_long_sorts_are_stable(n, tail, c, kind):
    gen = torch.Generator().manual_seed(n + c)
    nv = n - tail
    if kind == "random":
        labels = torch.randint(0, c, (1, 3, nv), generator=gen, dtype=torch.int32)
    else:  # runs of one label longer and shorter than a wave
        labels = ((torch.arange(nv) // 97 * 5 + torch.arange(3)[:, None]) % c).to(torch.int32)[None]
    perm, offsets, _ = binding.permute(labels.cuda(), c, (), n_tail=tail)
    full = torch.cat([labels, torch.full((1, 3, tail), c, dtype=torch.int32)], dim=2)
    want = torch.argsort(full.long(), dim=2, stable=True)
    assert torch.equal(perm.cpu().long(), want)
    counts = torch.stack([torch.bincount(full[0, h].long(), minlength=c + 1) for h in range(3)])
    assert torch.equal(offsets.cpu()[0, :, 1:].long(), counts.cumsum(1))
    assert int(offsets[0, :, 0].abs().max()) == 0
