"""The GraphSAGE layers at the sizes where their kernels change: rows narrower
than one 16-byte load, rows that end inside a load or a pass, every number of
column tiles, layers projected first and layers gathered first, fan-outs around
the neighbour rows in flight, and rows of halves that start at odd halves.
Against the fp64 oracle, with its derived rounding bound."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import World
from tests.test_gpu_parity import _sage_layers, _sage_tolerance

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp16,dims,fanout", [
    (False, [1, 16, 1], (10, 5)), (False, [3, 17, 16], (6, 5)), (False, [4, 48, 2], (1, 32)),
    (False, [33, 16, 64], (32, 10)), (False, [63, 16], (1,)), (False, [130, 81, 100], (5, 4)),
    (False, [261, 96, 128, 5], (3, 2, 6)), (False, [300, 16, 20], (11, 10)),
    (True, [1, 16], (7,)), (True, [7, 33, 16], (5, 5)), (True, [9, 128], (10,)),
    (True, [41, 16, 7], (10, 5)), (True, [131, 112, 48], (4, 17)), (True, [515, 40], (5,))])
def test_layer_sizes(fp16, dims, fanout):
    print(f"GraphSAGE {dims}, fp16 {fp16}, fan-out {fanout}", flush=True)
    from oracle import ggref
    from paper_2606_02916_amd import SageConsumer
    inst = synth.instance("tiny")
    w = World(inst, W=3, fanout=fanout, batch=61)
    boff = np.array([0, 61, 62, 107], dtype=np.int64)
    r = w.run_and_compare(0, seeds=inst.seeds[:107], so=boff, b0=0)
    Wk, L = 3, len(fanout)
    rng = np.random.default_rng(dims[0] * 10 + len(dims))
    n = int(r["foff"][(L + 1) * Wk] - r["foff"][L * Wk])
    d = dims[0]
    es = 2 if fp16 else 4
    x = rng.standard_normal((n, d)).astype(np.float16 if fp16 else np.float32)
    layers = _sage_layers(rng, dims)
    ref, ab = ggref.sage_forward(r["fids"], r["foff"], r["nids"], r["noff"], Wk, list(fanout),
                                 x.view(np.uint8), 1 if fp16 else 0, d * es, layers)
    # rows back to back, the first one an odd number of elements into its buffer
    flat = torch.full((n * d + 9,), float("nan"), dtype=torch.float16 if fp16 else torch.float32,
                      device=w.dev)
    xd = flat[3:3 + n * d]
    xd.copy_(torch.from_numpy(x.reshape(-1)))
    lt = [(torch.from_numpy(a).to(w.dev), torch.from_numpy(b).to(w.dev),
           torch.from_numpy(c).to(w.dev), relu) for a, b, c, relu in layers]
    cons = SageConsumer(w.pipe.geo, lt, x_dtype=1 if fp16 else 0, device=w.dev)
    cons.ws.fill_(0xFF)              # NaNs wherever nothing was computed
    got = cons.forward(w.pipe.buf, Wk, xd, d * es, w.pipe.status)
    torch.cuda.synchronize()
    assert w.pipe.read_status() == 0
    got = got[:ref.shape[0]].cpu().numpy().astype(np.float64)
    err, tol = np.abs(got - ref), _sage_tolerance(layers, list(fanout), ab)
    assert np.all(err <= tol), (float(np.nanmax(err - tol)), float(np.nanmax(err)))
