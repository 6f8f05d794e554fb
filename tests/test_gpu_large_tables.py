"""GPU parity of the kernels that tables of 4 GB and more take, of the wave
kernel's streamed rows (tables of 2 GB and more), and of it at its address limit.

The wave kernel's row offsets are 32-bit products, so a call with a larger table
takes the team kernel (16-, 8- and 4-byte chunks; small-batch, normal and narrow
mapping; windows of every team width) or the plain kernel, as do rows of 16 bytes
to 8 KB nowhere else in small batches.  Each case states the kernel that it
reaches.  The ids name the first rows of a table, or none; dyadic values, so sums
are exact in any order.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import TORCH_DT, to_device_table
from paper_2512_05831_amd import eb, workloads as wl
from route_util import PLAIN, TEAM, WAVE, route

pytestmark = pytest.mark.gpu

LO, HI = 500, 2500
ES = {wl.F32: 4, wl.F16: 2, wl.BF16: 2}


@pytest.fixture(scope="module")
def memory(device):
    """A little over 4 GB for the first table of each case."""
    buf = torch.empty((1 << 32) + (1 << 16), dtype=torch.uint8, device=device)
    yield buf
    del buf
    torch.cuda.empty_cache()


def place(buf, table, dtype, device, rows, shift):
    """A table of `rows` rows, `shift` bytes past a 16-byte boundary, that starts with `table`."""
    D, es = table.shape[1], ES[dtype]
    if buf is None:
        buf = torch.empty(rows * D * es + 16, dtype=torch.uint8, device=device)
    t = buf[shift:shift + rows * D * es].view(TORCH_DT[dtype]).view(rows, D)
    t[:table.shape[0]] = to_device_table(table, dtype, device)
    assert t.data_ptr() % 16 == shift
    return t


# (D, dtype, table shift in bytes, output shift in floats) and the chunk bytes of the team kernel (0: plain)
SHAPES = [
    (4, wl.F32, 0, 0, 16), (16, wl.F16, 0, 0, 16), (64, wl.F16, 0, 0, 16), (96, wl.F16, 0, 0, 16),
    (128, wl.BF16, 0, 0, 16), (128, wl.F32, 0, 0, 16), (256, wl.F32, 0, 0, 16), (512, wl.F32, 0, 0, 16),
    (2048, wl.F32, 0, 0, 16),
    (100, wl.F16, 0, 0, 8), (36, wl.F16, 0, 0, 8), (128, wl.F32, 8, 0, 8), (32, wl.F32, 0, 2, 8),
    (50, wl.BF16, 0, 0, 4), (64, wl.F32, 4, 0, 4), (60, wl.F32, 0, 1, 4), (3, wl.F32, 0, 0, 4),
    (130, wl.BF16, 0, 0, 0), (189, wl.F16, 0, 0, 0), (128, wl.F16, 2, 0, 0), (257, wl.F32, 0, 0, 0),
    (4095, wl.BF16, 0, 0, 0),
]


def check(D, dtype, tshift, oshift, B, max_len, hint, big, memory, device):
    """Two tables, the first of `big` rows.  Returns the route of the calls."""
    T = 2
    g = np.random.default_rng(D + 7 * B + tshift + 100 * oshift)
    off = wl.offsets_from_lengths(g.integers(0, max_len + 1, T * B))
    idx = g.integers(LO - 200, HI, int(off[-1]), dtype=np.int64)
    idx[5::17] = 2**31 - 1 - g.integers(0, 9, idx[5::17].size)  # past the last row of both tables
    assert LO + big < 2**31 - 9
    tables = [wl.table(D, t, D, dtype, LO, HI, values="dyadic") for t in range(T)]
    et = eb.EmbeddingBagTables([place(memory, tables[0], dtype, device, big, tshift),
                                place(None, tables[1], dtype, device, HI - LO, tshift)],
                               rows=[LO + big, HI], shard_lo=LO)
    W = T * (D + 3) // 4 * 4 + 4
    cols = [0, (D + 3) // 4 * 4]
    w = (g.integers(-8, 9, idx.size) / 4.0).astype(np.float32)  # dyadic weights: exact products
    for mode, weights, itype in ((wl.SUM, None, torch.int64), (wl.MEAN, None, torch.int32), (wl.SUM, w, torch.int32)):
        buf = torch.full((B * W + 4,), float("nan"), dtype=torch.float32, device=device)
        out = buf[oshift:oshift + B * W].view(B, W)
        hits = torch.full((B, T), -7, dtype=torch.int32, device=device)
        et.forward_ex(torch.from_numpy(idx).to(device).to(itype), torch.from_numpy(off).to(device).to(itype), B,
                      mode=mode | hint, out=out, out_cols=cols, hits=hits,
                      weights=None if weights is None else torch.from_numpy(weights).to(device))
        torch.cuda.synchronize()
        got = out.cpu().numpy().astype(np.float64)
        got = np.concatenate([got[:, c:c + D] for c in cols], axis=1)
        ref, ref_hits, _ = oracle.forward(tables, [HI] * T, D, dtype, idx, off, B, mode, LO, HI, weights=weights)
        assert np.array_equal(hits.cpu().numpy(), ref_hits)
        if mode == wl.SUM:
            assert np.array_equal(got, ref)
        else:  # one division after an exact sum
            assert np.all(np.abs(got - ref) <= np.abs(ref) * 2.0 ** -24)
    et.close()
    return route(D, dtype, T, B, idx.size / (T * B), LO + big, big, hint=bool(hint), align=tshift or 16,
                 out_align=4 * oshift or 16)


@pytest.mark.parametrize("D,dtype,tshift,oshift,chunk", SHAPES)
@pytest.mark.parametrize("B,max_len", [(7, 700), (3000, 30), (20000, 10)])
@pytest.mark.parametrize("hint", [0, eb.EB_HINT_STREAM_ROWS])
def test_kernels_of_large_tables(D, dtype, tshift, oshift, chunk, B, max_len, hint, memory, device):
    rb = D * ES[dtype]
    if rb > 2048:
        B = min(B, 1000)
    r = check(D, dtype, tshift, oshift, B, max_len, hint, (1 << 32) // rb + 1, memory, device)
    assert (r.kernel, r.chunk_bytes) == (TEAM if chunk else PLAIN, chunk)
    if B == 7 or rb <= 2048:
        assert r.small_batch == (1 if chunk and B == 7 else 0)


@pytest.mark.parametrize("D,dtype", [(64, wl.F16), (35, wl.F32), (128, wl.BF16), (189, wl.F16), (128, wl.F32), (256, wl.F32),
                                     (512, wl.F32), (257, wl.F32), (701, wl.F32), (1025, wl.BF16), (1290, wl.F32),
                                     (3100, wl.F16), (3700, wl.BF16), (4095, wl.F16)])
@pytest.mark.parametrize("B,max_len", [(7, 700), (1000, 40)])
def test_streamed_rows(D, dtype, B, max_len, memory, device):
    r = check(D, dtype, 0, 0, B, max_len, eb.EB_HINT_STREAM_ROWS, (3 << 30) // (D * ES[dtype]), memory, device)
    assert (r.kernel, r.non_temporal) == (WAVE, 1)
    assert (r.split > 1) == (B == 7)


@pytest.mark.parametrize("D,dtype", [(189, wl.F16), (128, wl.F32), (8, wl.F16)])
@pytest.mark.parametrize("hint", [0, eb.EB_HINT_STREAM_ROWS])
def test_rows_at_the_address_limit(D, dtype, hint, memory, device):
    """Rows on both sides of byte 2^31 and at the end of the largest table that
    the wave kernel takes, and of the smallest that it does not."""
    rb = D * ES[dtype]
    most = (2**32 - 1) // rb
    mid = 2**31 // rb
    for rows, kernels in ((most, (WAVE,)), (most + 1, (TEAM, PLAIN))):
        table = memory[:rows * rb].view(TORCH_DT[dtype]).view(rows, D)
        named = torch.tensor([0, 1, mid - 1, mid, mid + 1, 3 * mid // 2, rows - 2, rows - 1], device=device)
        values = torch.arange(named.numel() * D, device=device).view(-1, D) % 61 / 8 - 3
        table[named] = values.to(table.dtype)
        ids = torch.cat([named, named.flip(0), named, torch.tensor([rows, -1, 2**31 + 5], device=device), named[-3:]])
        off = torch.tensor([0, 8, 9, 24, 24, 27, 30], device=device)
        assert route(D, dtype, 1, 6, 5, rows, hint=bool(hint)).kernel in kernels
        et = eb.EmbeddingBagTables([table])
        out, hits = et.forward(ids, off, 6, mode=eb.EB_SUM | hint, hits=True)
        rows_of = torch.cat([values, values.flip(0), values, torch.zeros(3, D, device=device), values[-3:]]).double()
        want = torch.stack([rows_of[a:b].sum(0) for a, b in zip(off.tolist(), off.tolist()[1:])])
        assert torch.equal(out.double(), want)
        assert hits[:, 0].tolist() == [8, 1, 15, 0, 0, 3]
        et.close()


@pytest.mark.parametrize("hint", [0, eb.EB_HINT_STREAM_ROWS])
def test_wave_bags_split_over_launches(hint, device):
    """64 tables of 18-byte rows: a launch holds 262,144 bags of each, the rest come in a second."""
    T, B, D, rows = 64, 263_000, 9, 1000
    g = np.random.default_rng(hint + 3)
    L = np.where(g.random(T * B) < 0.05, g.integers(1, 5, T * B), 0)
    off = wl.offsets_from_lengths(L)
    idx = g.integers(-2, rows + 2, int(off[-1]), dtype=np.int64)
    assert route(D, wl.F16, T, B, idx.size / (T * B), rows, hint=bool(hint)).kernel == WAVE
    tables = [wl.table(78, t, D, wl.F16, 0, rows, values="dyadic") for t in range(T)]
    et = eb.EmbeddingBagTables([to_device_table(t, wl.F16, device) for t in tables])
    out, hits = et.forward(torch.from_numpy(idx).to(device), torch.from_numpy(off).to(device), B, mode=eb.EB_SUM | hint,
                           hits=True)
    torch.cuda.synchronize()
    ref, ref_hits, _ = oracle.forward(tables, [rows] * T, D, wl.F16, idx, off, B, wl.SUM)
    assert np.array_equal(hits.cpu().numpy(), ref_hits)
    assert np.array_equal(out.cpu().numpy(), ref)
    et.close()
