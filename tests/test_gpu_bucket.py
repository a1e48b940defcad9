"""Bucketing by owner where a block takes more than one span of ids, or more than
one run of the owner-order check: the second turns of their loops.  Against the
oracle's stable partition."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,kind,n,order", [
    (64, 0, 1_300_007, "shuffled"),      # 1,024 blocks: two spans of 1,024 ids each
    (64, 0, 2_500_001, "ascending"),     # three spans, the last blocks empty
    (5, 0, 1_750_003, "shuffled"),       # 1,638 blocks, two spans
    (3, 1, 2_300_001, "ascending"),      # 2,048 blocks of 1,024 ids: a second turn
    (64, 1, 2_300_001, "descent"),       # out of order in that turn only
    (1, 0, 8_400_000, "shuffled")])      # one owner: 8,192 blocks, two spans
def test_more_ids_than_one_turn(P, kind, n, order):
    print(f"{n} ids, {P} owners, kind {kind}, {order}", flush=True)
    from oracle import ggref
    from paper_2606_02916_amd import gg
    rng = np.random.default_rng(n)
    N = 9_000_001
    rs = None
    if kind == 1:                        # uneven ranges, one of them empty
        rs = [0] + sorted(rng.integers(0, N, P - 1).tolist()) + [N]
        rs[1] = 0
    ids = np.flatnonzero(rng.random(N) < (n + 4000) / N).astype(np.int32)[:n]
    assert len(ids) == n
    if order == "shuffled":
        rng.shuffle(ids)
    elif order == "descent":
        a, b = 2_097_152 + 5000, n - 3
        ids[[a, b]] = ids[[b, a]]
    part_ref = ggref.make_part(P, kind, 0, N, rs)
    want, want_off = ggref.bucket_by_owner(ids, part_ref)
    dev = torch.device("cuda:0")
    cap = n + 777
    hot = torch.zeros(cap, dtype=torch.int32, device=dev)
    hot[:n] = torch.from_numpy(ids).to(dev)
    cnt = torch.tensor([n, n], dtype=torch.int64, device=dev)
    out = torch.full((cap,), -7, dtype=torch.int32, device=dev)
    off = torch.full((P + 1,), -9, dtype=torch.int64, device=dev)
    status = torch.zeros(1, dtype=torch.int32, device=dev)
    ws = torch.full((gg.gg_ws_bucket(cap, P),), 0xFF, dtype=torch.uint8, device=dev)
    part = gg.make_part(P, kind, 0, N, rs)
    gg.gg_bucket_by_owner(hot, cnt, cap, part, out, off, status, ws)
    torch.cuda.synchronize()
    assert int(status) == 0
    assert np.array_equal(off.cpu().numpy(), want_off)
    assert np.array_equal(out[:n].cpu().numpy(), want)
    assert (out[n:] == -7).all()
