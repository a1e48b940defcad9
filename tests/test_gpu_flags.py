"""Block flags of the sampler's sets at the size where the library takes them by
itself: 64 batches over 6.4M nodes, too many LDS slices and 51 MB of sets.  With
the byte map at the last hop (the library's choice there: its marks set no
flags), and with atomics throughout.  Against the oracle."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import World

pytestmark = pytest.mark.gpu

N, W = 6_400_000, 64


@pytest.fixture(scope="module")
def inst():
    rng = np.random.default_rng(11)
    deg = rng.poisson(3.0, N)
    deg[rng.integers(0, N, 100)] = 500
    row_ptr = np.zeros(N + 1, dtype=np.int64)
    np.cumsum(deg, out=row_ptr[1:])
    # neighbours crowd into some blocks of 512 nodes and leave others empty
    col = (N * rng.random(row_ptr[-1]) ** 3).astype(np.int32)
    wl = synth.Workload("hand", N, col.shape[0], False, 64, synth.PART_MOD, 4, 1, 4, "fp32",
                        "normal", (4, 3, 2), 30, W, "perm_all", n_windows=1)
    return synth.Instance(wl, row_ptr, col, *synth.seed_batches(wl),
                          [synth.shard_features(wl, m) for m in range(4)], None)


@pytest.mark.parametrize("fields", [dict(), dict(bytemap_max_mb=-1), dict(sample_order=2),
                                    dict(sample_order=1, bytemap_max_mb=-1)])
def test_flagged_sets_match_oracle(inst, fields):
    print(f"{W} batches over {N} nodes, tuning {fields}", flush=True)
    from paper_2606_02916_amd import gg
    words = gg.gg_bits_words(N)
    assert W * words * 4 >= 48 << 20 and words > 8 * 8 * 2048      # flags, no LDS slices
    assert 30 * 5 * 4 * 3 <= words // 16 * 16                      # few entries per block
    assert W * words * 32 <= 512 << 20                             # the byte map fits
    w = World(inst, W=W, tuning=gg.make_tuning(**fields))
    sizes = np.full(W, 30)
    sizes[[0, 5, 63]] = 0, 1, 0
    so = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    seeds = np.array(inst.seeds[:so[-1]])
    seeds[so[7]:so[8]] = [0, N - 1, 511, 512, 65535, 65536] * 5    # edges of blocks and chunks
    w.run_and_compare(0, seeds=seeds, so=so, b0=0)
    w.run_and_compare(0, seeds=seeds[::-1].copy(), so=so, b0=9)    # over the first window's flags
    assert torch.cuda.is_available() and w.pipe.read_status() == 0
