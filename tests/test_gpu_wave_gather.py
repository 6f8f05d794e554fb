"""GPU parity of the wave gather: a wave, or up to 16 waves, per bag.

Ragged rows are read with 16-byte loads whose last one overlaps its
neighbour, so widths sit around the 16-byte chunk, the 64-lane row and the
8-KB limit, at odd alignments of tables and output; bag lengths around the
64-id window and around the lengths at which a bag is split over waves.  The
first and last rows of every table are among the ids.  All against the oracle
within the summation bound, hit counts exactly.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import assert_parity, max_bag_len, to_device_table
from paper_2512_05831_amd import eb, workloads as wl

pytestmark = pytest.mark.gpu

ROWS, LO, HI = 3000, 100, 2900


def check(D, dtype, lengths, T, device, hint=0, itype=np.int64, weighted=False, oshift=0, tshift=0, seed=0):
    g = np.random.default_rng(seed + D)
    B = len(lengths) // T
    off = wl.offsets_from_lengths(np.asarray(lengths, dtype=np.int64))
    idx = g.integers(LO - 40, HI + 40, int(off[-1]), dtype=np.int64)
    idx[::7], idx[3::11] = HI - 1, LO  # the shard's last and first rows
    tables = [wl.table(seed, t, D, dtype, LO, HI) for t in range(T)]
    w = g.standard_normal(idx.size).astype(np.float32) if weighted else None
    dts = []
    for t in tables:
        d = to_device_table(t, dtype, device)
        big = torch.empty(d.numel() + 16, dtype=d.dtype, device=device)
        dts.append(big[tshift:tshift + d.numel()].view(d.shape).copy_(d))
    et = eb.EmbeddingBagTables(dts, rows=[ROWS] * T, shard_lo=LO, shard_hi=HI)
    W = T * D + 3  # odd row stride: output rows at any multiple of 4 bytes
    for mode in (wl.SUM,) if weighted else (wl.SUM, wl.MEAN):
        buf = torch.full((B * W + 8,), float("nan"), dtype=torch.float32, device=device)
        out = buf[oshift:oshift + B * W].view(B, W)
        hits = torch.full((B, T), -7, dtype=torch.int32, device=device)
        et.forward_ex(torch.from_numpy(idx.astype(itype)).to(device), torch.from_numpy(off.astype(itype)).to(device),
                      B, mode=mode | hint, out=out, hits=hits,
                      weights=None if w is None else torch.from_numpy(w).to(device))
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        assert np.all(np.isnan(got[:, T * D:])), "columns past the tables were written"
        assert torch.isnan(buf[:oshift]).all() and torch.isnan(buf[oshift + B * W:]).all()
        ref, ref_hits, mag = oracle.forward(tables, [ROWS] * T, D, dtype, idx, off, B, mode, LO, HI, weights=w)
        assert_parity(got[:, :T * D], ref, mag, max_bag_len(off, idx.size), dtype, hits.cpu().numpy(), ref_hits)
    et.close()


@pytest.mark.parametrize("D,dtype", [(8, wl.F16), (9, wl.F16), (15, wl.BF16), (17, wl.BF16), (5, wl.F32), (189, wl.F16),
                                     (257, wl.F32), (511, wl.F16), (513, wl.BF16), (1025, wl.F32), (4095, wl.F16)])
@pytest.mark.parametrize("hint", [0, eb.EB_HINT_STREAM_ROWS])
def test_ragged_rows(D, dtype, hint, device):
    lengths = [0, 1, 2, 31, 63, 64, 65, 127, 128, 129, 3, 200]
    check(D, dtype, lengths, 2, device, hint=hint, oshift=1, tshift=1)


@pytest.mark.parametrize("D,dtype", [(64, wl.F32), (64, wl.F16), (189, wl.F16), (300, wl.F32)])
@pytest.mark.parametrize("bags,length", [(1, 5000), (8, 95), (8, 97), (60, 400), (300, 200)])
@pytest.mark.parametrize("weighted,itype", [(False, np.int64), (True, np.int32)])
def test_split_bags(D, dtype, bags, length, weighted, itype, device):
    lengths = np.random.default_rng(bags).integers(length // 2, 2 * length, bags)
    lengths[0] = 0 if bags > 1 else length
    check(D, dtype, lengths, 1, device, weighted=weighted, itype=itype)


@pytest.mark.parametrize("D,dtype", [(64, wl.F32), (189, wl.F16), (300, wl.F32)])
@pytest.mark.parametrize("weighted,itype", [(False, np.int64), (True, np.int32)])
def test_split_bags_around_one_window(D, dtype, weighted, itype, device):
    """Bags of up to one window of 64 ids among longer ones: in a split call the
    first wave ends them alone."""
    lengths = [64, 65, 0, 63, 200, 1, 64, 128, 129, 64, 40, 300]
    check(D, dtype, lengths, 2, device, weighted=weighted, itype=itype)


@pytest.mark.parametrize("D,dtype", [(32, wl.F32), (128, wl.F32), (256, wl.BF16), (512, wl.F16), (75, wl.F16)])
def test_large_batch_of_windows(D, dtype, device):
    lengths = np.random.default_rng(D).integers(0, 130, 2 * 4200)
    check(D, dtype, lengths, 2, device)


def test_neighbouring_rows_stay_out(device):
    """Infinities and NaNs in rows no bag names reach no sum, whatever the
    loads overlap; those in named rows do."""
    D, n = 21, 64
    t = torch.full((n, D), float("nan"), dtype=torch.float16, device=device)
    t[::2] = float("inf")
    t[10], t[33] = 1.5, 6e-8  # 6e-8: subnormal in fp16
    et = eb.EmbeddingBagTables([t])
    idx = torch.tensor([10, 33, 10, 33, 0, 10], device=device)
    off = torch.tensor([0, 2, 3, 4, 4, 6], device=device)
    for w in (None, torch.ones(6, device=device)):
        out = et.forward_ex(idx, off, 5, weights=w)
        sub = t[33, 0].float()
        want = torch.stack([1.5 + sub, t[10, 0].float(), sub, torch.zeros_like(sub), torch.full_like(sub, float("inf"))])
        assert torch.equal(out, want[:, None].expand(5, D))
    et.close()
