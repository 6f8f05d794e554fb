"""GPU parity of eb_bucketize's two-kernel path (at most 64 destinations and
a few million ids, EB_BUCKETIZE_ONE_PASS unset) against the oracle, bit for bit:
destination counts around each owner method, workgroups of one table's bags
(255 at most) and their waves' 64-id chunks and 512-id passes, empty bags at
either end, out-of-order and overlapping offsets, short capacity, and, at its
id limits, against the other paths.
"""
import numpy as np
import pytest
import torch

import test_gpu_exchange
from paper_2512_05831_amd import eb, workloads as wl
from test_gpu_exchange import bucket_case, check_bucketize, even_bounds, run_bucketize

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def default_path(monkeypatch):
    monkeypatch.delenv("EB_BUCKETIZE_ONE_PASS", raising=False)


@pytest.mark.parametrize("G", [1, 2, 7, 8, 9, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("seed", range(4))
def test_matches_oracle(G, seed, device):
    T, B, idx, off, bounds = bucket_case(seed * 37 + G, G, uneven=(seed % 2 == 1), maxL=[40, 3, 200, 700][seed])
    check_bucketize(T, B, idx, off, bounds, device, index_dtype=np.int32 if seed == 2 else np.int64)
    if idx.size > 10:
        check_bucketize(T, B, idx, off, bounds, device, capacity=idx.size // 3)


@pytest.mark.parametrize("G", [3, 16, 40])
@pytest.mark.parametrize("T,B,length", [(1, 1, 1), (1, 1, 513), (1, 255, 8), (1, 256, 8), (2, 257, 7), (600, 2, 3),
                                        (3, 2, 5000), (1, 30_000, 2), (5, 800, 60)])
def test_group_and_pass_edges(G, T, B, length, device):
    g = np.random.default_rng(T * B + G)
    rows = [4000] * T
    for L in (np.full(T * B, length), g.integers(0, 2 * length + 1, T * B)):
        off = wl.offsets_from_lengths(L.astype(np.int64))
        check_bucketize(T, B, g.integers(-3, 4003, int(off[-1])), off, even_bounds(rows, G), device)


@pytest.mark.parametrize("tail", [1, 64, 65, 200])
@pytest.mark.parametrize("ids", [0, 63, 64, 256, 2048])
def test_empty_bags_at_the_ends(tail, ids, device):
    g = np.random.default_rng(tail + ids)
    L = np.concatenate([np.zeros(tail), [ids], np.zeros(tail)]).astype(np.int64)
    off = wl.offsets_from_lengths(np.concatenate([L, L]))
    check_bucketize(2, L.size, g.integers(0, 900, int(off[-1])), off, even_bounds([900, 900], 8), device)


@pytest.mark.parametrize("G", [2, 8, 13, 50])
@pytest.mark.parametrize("kind", ["one", "shuffled", "overlap", "outside"])
def test_disordered_offsets(G, kind, device):
    """Bags that overlap send an id once per bag, so the ids sent may exceed nnz."""
    g = np.random.default_rng(G)
    T, B = 3, 150
    off = wl.offsets_from_lengths(g.integers(0, 30, T * B))
    nnz = int(off[-1])
    if kind == "one":
        off[200] = off[203] + 5
    elif kind == "shuffled":
        off = g.permutation(off)
    elif kind == "overlap":
        off[::2] = g.integers(0, nnz // 2, off[::2].size)
        off[1::2] = nnz
    else:
        off[5], off[-1], off[100] = -7, nnz + 50, nnz + 3
    idx = g.integers(0, 5000, nnz)
    check_bucketize(T, B, idx, off, even_bounds([5000] * T, G), device, capacity=40 * nnz)
    check_bucketize(T, B, idx, off, even_bounds([5000] * T, G), device)


@pytest.mark.parametrize("itype", [torch.int64, torch.int32])
def test_more_ids_than_32_bits_before_ordered_bags(itype, device):
    """2048 bags that each send the whole batch put the ordered bags behind them
    at positions past 2^32: none of their ids may land in out_indices."""
    nnz, repeats, tail = 1 << 21, 2048, 4096
    gen = torch.Generator(device=device).manual_seed(3)
    idx = torch.randint(0, 5000, (nnz,), generator=gen, device=device).to(itype)
    step = nnz // 2 // tail
    off = torch.cat([torch.tensor([0, nnz], device=device).repeat(repeats),
                     nnz // 2 + step * torch.arange(tail + 1, device=device)])
    lengths = (off[1:] - off[:-1]).clamp(min=0)
    want = torch.cat([lengths.new_zeros(1), lengths.cumsum(0)])
    assert int(want[-1]) > 1 << 32
    bounds = torch.tensor([[0, 5000, 5000]], device=device)
    out_off, out_idx, seg = eb.bucketize(bounds, idx, off.to(itype), 1, off.numel() - 1, capacity=nnz)[:3]
    assert seg.tolist() == [0, int(want[-1]), int(want[-1])]
    assert torch.equal(out_off[0], want) and not out_off[1].any()
    assert torch.equal(out_idx[:nnz], idx)


def test_bounds_and_ids_at_the_type_limits(device):
    hi, lo = np.iinfo(np.int64).max, np.iinfo(np.int64).min
    idx = np.array([lo, -1, 0, 5, hi - 1, hi, lo + 1, 5], dtype=np.int64)
    bounds = np.array([[lo, -5, 0, 6, hi]], dtype=np.int64)
    check_bucketize(1, 3, idx, np.array([0, 3, 4, 8]), bounds, device)


@pytest.mark.parametrize("G,ids", [(8, (7 << 19) - 1), (8, 7 << 19), (20, (5 << 20) - 1), (20, 5 << 20), (40, (7 << 19) - 1)])
@pytest.mark.parametrize("itype", [torch.int64, torch.int32])
def test_id_limits_against_the_other_paths(G, ids, itype, device, monkeypatch):
    T, B, rows = 6, 9000, 1_000_000
    gen = torch.Generator(device=device).manual_seed(G)
    cuts = torch.sort(torch.randint(0, ids + 1, (T * B - 1,), generator=gen, device=device)).values
    off = torch.cat([torch.zeros(1, device=device, dtype=torch.int64), cuts,
                     torch.full((1,), ids, device=device, dtype=torch.int64)]).to(itype)
    idx = torch.randint(0, rows, (ids,), generator=gen, device=device).to(itype)
    bounds = torch.from_numpy(even_bounds([rows] * T, G)).to(device)
    got = eb.bucketize(bounds, idx, off, T, B)[:3]
    monkeypatch.setenv("EB_BUCKETIZE_ONE_PASS", "0")
    want = eb.bucketize(bounds, idx, off, T, B)[:3]
    assert all(torch.equal(a, b) for a, b in zip(got, want))


def test_graph_replays(device):
    T, B, idx, off, bounds = bucket_case(5, 8, T=4, B=200, maxL=40)
    want = run_bucketize(bounds, idx, off, T, B, device)
    d = [torch.from_numpy(np.ascontiguousarray(x)).to(device) for x in (bounds, idx, off)]
    G = 8
    out_off = torch.empty((G, T * B + 1), dtype=torch.int64, device=device)
    out_idx = torch.empty(max(1, idx.size), dtype=torch.int64, device=device)
    seg = torch.empty(G + 1, dtype=torch.int64, device=device)
    n = eb.eb_bucketize_workspace(T, B, G)
    ws = torch.empty(n, dtype=torch.uint8, device=device)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        eb.eb_bucketize(T, B, G, d[0].data_ptr(), d[1].data_ptr(), idx.size, d[2].data_ptr(), out_off.data_ptr(),
                        out_idx.data_ptr(), idx.size, seg.data_ptr(), ws.data_ptr(), n,
                        torch.cuda.current_stream(device).cuda_stream)
    for _ in range(4):
        for x in (out_off, out_idx, seg):
            x.fill_(-1)
        ws.random_(0, 256)
        graph.replay()
        torch.cuda.synchronize()
        sent = int(seg[-1])
        assert np.array_equal(out_off.cpu().numpy(), want[0]) and np.array_equal(seg.cpu().numpy(), want[2])
        assert np.array_equal(out_idx[:sent].cpu().numpy(), want[1])


@pytest.mark.parametrize("seed", range(40))
def test_random_config(seed, device):
    test_gpu_exchange.test_bucketize_random_config(seed, device)
