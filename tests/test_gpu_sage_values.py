"""Values that the GraphSAGE layers must not lose on the way: infinities and
NaNs.  Against the fp64 oracle."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import World
from tests.test_gpu_parity import _sage_layers, _sage_tolerance

pytestmark = pytest.mark.gpu

WK = 3


def sampled(fanout):
    """Three ragged batches of the tiny graph: (world, oracle outputs, rows of
    their N_b)."""
    inst = synth.instance("tiny")
    w = World(inst, W=WK, fanout=fanout, batch=61)
    boff = np.array([0, 61, 62, 107], dtype=np.int64)
    r = w.run_and_compare(0, seeds=inst.seeds[:107], so=boff, b0=0)
    L = len(fanout)
    return w, r, int(r["foff"][(L + 1) * WK] - r["foff"][L * WK])


def oracle_forward(r, fanout, x, layers):
    from oracle import ggref
    return ggref.sage_forward(r["fids"], r["foff"], r["nids"], r["noff"], WK, list(fanout),
                              x.view(np.uint8), 1 if x.dtype == np.float16 else 0,
                              x.shape[1] * x.itemsize, layers)


def forward(w, x, layers):
    from paper_2606_02916_amd import SageConsumer
    n, d = x.shape
    fp16 = x.dtype == np.float16
    # rows back to back, the first one an odd number of elements into its buffer
    flat = torch.full((n * d + 9,), float("nan"), dtype=torch.float16 if fp16 else torch.float32,
                      device=w.dev)
    xd = flat[3:3 + n * d]
    xd.copy_(torch.from_numpy(x.reshape(-1)))
    lt = [(torch.from_numpy(a).to(w.dev), torch.from_numpy(b).to(w.dev),
           torch.from_numpy(c).to(w.dev), relu) for a, b, c, relu in layers]
    cons = SageConsumer(w.pipe.geo, lt, x_dtype=1 if fp16 else 0, device=w.dev)
    cons.ws.fill_(0xFF)              # NaNs wherever nothing was computed
    got = cons.forward(w.pipe.buf, WK, xd, d * x.itemsize, w.pipe.status)
    torch.cuda.synchronize()
    assert w.pipe.read_status() == 0
    return got.cpu().numpy()


@pytest.mark.parametrize("fp16,dims,fanout", [
    (False, [9, 12, 5], (4, 3)), (False, [300, 12, 20], (11, 10)),
    (True, [70, 41, 20, 7], (5, 3, 2)), (True, [40, 100, 3], (4, 6))])
def test_infinities_and_nans_stay_where_the_formula_puts_them(fp16, dims, fanout):
    """Features of +inf, -inf and NaN, hidden widths between whole column tiles
    (the second case projects its first layer).  Hidden units see a +inf of the
    first feature only as -inf, which ReLU makes 0, and one of the second as
    +inf in a single unit, so that outputs are finite, infinite and NaN."""
    print(f"GraphSAGE {dims} with infinities, fp16 {fp16}, fan-out {fanout}", flush=True)
    w, r, n = sampled(fanout)
    rng = np.random.default_rng(dims[1])
    x = rng.standard_normal((n, dims[0])).astype(np.float16 if fp16 else np.float32)
    layers = _sage_layers(rng, dims)
    for m in layers[0][:2]:
        m[:2] = -np.abs(m[:2]) - 0.01
        m[1, 3] *= -1
    finite = x.copy()
    hit = rng.permutation(n)
    a, b = n // 64, n // 64 + n // 128
    x[hit[:a], 0] = np.inf
    x[hit[a:b], 1] = np.inf
    x[hit[b:b + 2], 2] = -np.inf
    x[hit[b + 2:b + 4], 3] = np.nan
    ref, _ = oracle_forward(r, fanout, x, layers)
    # the magnitudes with the infinities left out bound those of every finite
    # output, to which hidden rows of -inf contribute nothing
    _, ab = oracle_forward(r, fanout, finite, layers)
    got = forward(w, x, layers)[:ref.shape[0]].astype(np.float64)
    for kind in (np.isfinite, np.isposinf, np.isneginf, np.isnan):
        assert np.array_equal(kind(got), kind(ref)), kind.__name__
        # (two layers after the infinite unit every infinity has met its opposite)
        assert kind(ref).any() or (len(dims) > 3 and kind in (np.isposinf, np.isneginf))
    ok = np.isfinite(ref)
    tol = _sage_tolerance(layers, list(fanout), ab)
    assert np.all(np.abs(got[ok] - ref[ok]) <= tol[ok])
