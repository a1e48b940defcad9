"""The row copy engine on rows that start at any multiple of 4: rows moved in
16-byte pieces (the last one overlapping the piece before it) and, below 16
bytes, in words.  Staging and the gather (cache hits, local rows and misses)
against a plain index of the shards, with the bytes around every row kept."""
import numpy as np
import pytest
import torch

from paper_2606_02916_amd import gg

pytestmark = pytest.mark.gpu

N, P = 700, 3


def placed(rows, stride, offset, dev, fill=None):
    """A (rows, stride) byte tensor `offset` bytes past a 16-byte boundary."""
    base = torch.full((rows * stride + 64,), 0xA5, dtype=torch.uint8, device=dev)
    start = (-base.data_ptr()) % 16 + offset
    t = base[start:start + rows * stride].view(rows, stride)
    if fill is not None:
        t.copy_(torch.from_numpy(fill))
    return t


@pytest.mark.parametrize("offset", [0, 4, 12])
@pytest.mark.parametrize("rb,stride", [(4, 4), (12, 20), (16, 16), (20, 20), (28, 32), (60, 60),
                                       (300, 300), (2408, 2412)])
def test_rows_at_any_word(rb, stride, offset):
    print(f"rows of {rb} bytes, stride {stride}, offset {offset}", flush=True)
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(rb + offset)
    rows = [(N - m + P - 1) // P for m in range(P)]
    host = [rng.integers(0, 256, (r, stride), dtype=np.uint8) for r in rows]
    shards = [placed(r, stride, offset, dev, h) for r, h in zip(rows, host)]
    part = gg.make_part(P, gg.PART_MOD, 0, N)
    feat = gg.make_feat(rb, shards, [stride] * P, rows)
    feature = np.empty((N, rb), dtype=np.uint8)
    for m in range(P):
        feature[m::P] = host[m][:, :rb]
    # two of every three remote nodes staged, owner by owner
    ids = np.arange(N)
    hot = np.concatenate([ids[(ids % P == m) & (ids % 5 > 1)] for m in (1, 2)]).astype(np.int32)
    off = [0, 0, int((hot % P == 1).sum()), len(hot)]
    bucket = torch.from_numpy(hot).to(dev)
    owner_off = torch.tensor(off, dtype=torch.int64, device=dev)
    cache = placed(len(hot), stride, offset, dev)
    slot_of = torch.full((N,), -1, dtype=torch.int32, device=dev)
    status = torch.zeros(1, dtype=torch.int32, device=dev)
    stats = torch.zeros(gg.STAGE_STATS_BYTES, dtype=torch.uint8, device=dev)
    ws = torch.empty(max(gg.gg_ws_stage(len(hot), P), gg.gg_ws_gather(2 * N, 2, P)),
                     dtype=torch.uint8, device=dev)
    gg.gg_stage_bulk(bucket, owner_off, len(hot), part, feat, cache, stride, len(hot), slot_of,
                     None, None, None, None, stats, status, ws)
    torch.cuda.synchronize()
    got = cache.cpu().numpy()
    assert np.array_equal(got[:, :rb], feature[hot]) and (got[:, rb:] == 0xA5).all()
    n = 2 * N - 33
    want = rng.integers(0, N, n).astype(np.int32)
    in_ids = torch.from_numpy(want).to(dev)
    bounds = torch.tensor([0, 641, n], dtype=torch.int64, device=dev)
    for flags in (0, gg.GG_GATHER_SHARED):
        out = placed(n + 3, stride, offset, dev)
        gst = torch.zeros((2, gg.GATHER_STATS_BYTES), dtype=torch.uint8, device=dev)
        gg.gg_gather_batch(in_ids, bounds.data_ptr(), 2, n + 3, part, feat, cache, stride,
                           len(hot), slot_of, out, stride, gst.data_ptr(), status, ws,
                           flags=flags)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        assert np.array_equal(got[:n, :rb], feature[want])
        assert (got[:n, rb:] == 0xA5).all() and (got[n:] == 0xA5).all()
        st = [gg.gather_stats_from_bytes(g.cpu().numpy().tobytes(), P) for g in gst]
        assert sum(s["misses"] for s in st) == int((~np.isin(want, hot) & (want % P > 0)).sum())
    assert int(status) == 0
