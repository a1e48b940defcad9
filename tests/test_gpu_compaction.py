"""The two forms of a level's compaction on both sides of the host's choice
between them (an eighth of the nodes by the bound on a batch's entries, a 64th for
the seeds), over one chunk and several, with and without the node tiles' table.
Against the oracle."""
import numpy as np
import pytest

import synth
from tests import helpers
from tests.gpu_util import World

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [0, 2])
@pytest.mark.parametrize("n,batch", [(2048, 64), (2047, 64), (200_003, 6250), (200_003, 6251),
                                     (65_536, 1024), (65_535, 1024), (65_537, 2049)])
def test_both_forms_match_oracle(n, batch, order):
    print(f"{n} nodes, batches of {batch}, order {order}", flush=True)
    from paper_2606_02916_amd import gg
    rng = np.random.default_rng(n + batch)
    row_ptr, col = helpers.random_graph(n, 6 * n, rng) if n < 3000 else _crowded(n, rng)
    wl = synth.Workload("hand", n, col.shape[0], False, 64, synth.PART_MOD, 4, 1, 4, "fp32",
                        "normal", (3, 2), batch, 3, "perm_all", n_windows=1)
    inst = synth.Instance(wl, row_ptr, col, *synth.seed_batches(wl),
                          [synth.shard_features(wl, m) for m in range(4)], None)
    w = World(inst, W=3, tuning=gg.make_tuning(sample_order=order))
    so = np.array([0, batch, batch, batch + batch // 2], dtype=np.int64)
    w.run_and_compare(0, seeds=np.array(inst.seeds[:so[-1]]), so=so, b0=0)


def _crowded(n, rng):
    """Neighbours crowded into a few runs of words, whole words among them."""
    deg = rng.poisson(4.0, n)
    row_ptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(deg, out=row_ptr[1:])
    return row_ptr, (n * rng.random(row_ptr[-1]) ** 4).astype(np.int32)
