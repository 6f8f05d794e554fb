"""GPU parity of eb_sum_partials for any column count: four elements per thread
that may span bags, a remainder of n % 4, both load depths, and buffers at any
multiple of 4 bytes.  The sources are added in order in fp32 and the mean is one
division, so the same steps in plain tensor operations give the same bits.
"""
import pytest
import torch

from paper_2512_05831_amd import eb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G,B,T,D", [(1, 1, 1, 1), (2, 3, 2, 1), (3, 5, 3, 2), (8, 7, 1, 3), (5, 6, 4, 5), (16, 33, 3, 13),
                                     (8, 64, 5, 128), (4, 700, 9, 171), (3, 300, 26, 135), (2, 1024, 8, 128), (2, 1025, 8, 128), (9, 257, 16, 255)])
@pytest.mark.parametrize("shift", [0, 1])
def test_any_columns(G, B, T, D, shift, device):
    g = torch.Generator(device=device).manual_seed(G * B + D)
    n = B * T * D
    p = torch.randn(G * n + 4, generator=g, device=device)[shift:shift + G * n].view(G, B, T * D)
    lengths = torch.randint(0, 4, (T * B,), generator=g, device=device)
    off = torch.zeros(T * B + 1, dtype=torch.int64, device=device)
    torch.cumsum(lengths, 0, out=off[1:])
    nnz = int(off[-1]) - 1  # the last bag with ids is cut by one
    want = torch.zeros(B, T * D, device=device)
    for s in range(G):
        want += p[s]
    cut = off.clamp(max=max(nnz, 0))
    L = (cut[1:] - cut[:-1]).view(T, B).t()[:, :, None].float()
    mean = torch.where(L > 0, want.view(B, T, D) / L, torch.zeros((), device=device)).reshape(B, T * D)
    for offsets, ref in ((None, want), (off, mean)):
        buf = torch.full((n + 8,), float("nan"), device=device)
        out = buf[shift:shift + n].view(B, T * D)
        eb.sum_partials(p, B, T, D, mean_offsets=offsets, nnz=max(nnz, 0), out=out)
        assert torch.equal(out, ref)
        assert torch.isnan(buf[:shift]).all() and torch.isnan(buf[shift + n:]).all()
