"""Values that the GraphSAGE layers must not lose on the way: infinities and
NaNs, digits, and the largest finite features.  Against the fp64 oracle."""
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
    (True, [70, 41, 20, 7], (5, 3, 2)), (True, [40, 100, 3], (4, 6)),
    (False, [300, 12, 100, 20, 9], (2, 3, 2, 10))])
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


def projected_first(r, fanout, x, layers):
    """The layers in fp32 by their definition's other order: every input row
    times [W_self | W_neigh], one product after the other, then the mean of the
    projected rows."""
    f32, L = np.float32, len(fanout)
    h = x.astype(f32)

    def product(w):
        acc = np.zeros((h.shape[0], w.shape[1]), dtype=f32)
        for k in range(w.shape[0]):      # a fused multiply-add per step
            acc = (acc + h[:, k:k + 1].astype(np.float64) * w[k].astype(np.float64)).astype(f32)
        return acc

    for j, (ws, wn, bias, relu) in enumerate(layers):
        lvl = L - 1 - j
        zs, zn = product(ws), product(wn)
        out = []
        for b in range(WK):
            s, above = lvl * WK + b, (lvl + 1) * WK + b
            ids = r["fids"][r["foff"][above]:r["foff"][above + 1]]
            first = r["foff"][above] - r["foff"][(lvl + 1) * WK]
            own = first + np.searchsorted(ids, r["fids"][r["foff"][s]:r["foff"][s + 1]])
            nbr = r["nids"][r["noff"][s]:r["noff"][s + 1]].reshape(len(own), fanout[lvl])
            pos = first + np.searchsorted(ids, np.maximum(nbr, 0))
            total = np.zeros((len(own), ws.shape[1]), dtype=f32)
            for t in range(fanout[lvl]):
                ok = nbr[:, t] >= 0
                total[ok] += zn[pos[ok, t]]
            inv = f32(1) / np.maximum((nbr >= 0).sum(1), 1).astype(f32)
            out.append(zs[own] + total * inv[:, None] + bias)
        h = np.concatenate(out)
        if relu:
            h = np.maximum(h, 0)
    return h


@pytest.mark.parametrize("fp16,dims,fanout", [
    (False, [16, 16, 16, 16], (10, 8, 5)), (False, [17, 77, 29], (5, 5)),
    (False, [25, 52, 34], (15, 10)), (False, [48, 48, 16], (25, 10)),
    (False, [100, 16, 47], (10, 5)), (True, [20, 124, 42], (10, 5)),
    (True, [128, 128, 64], (10, 5)), (False, [300, 40, 20], (11, 10))])
def test_no_more_rounding_error_than_projecting_first(fp16, dims, fanout):
    """Averaging rows before their product must not cost accuracy against
    averaging projected rows, whose rounding errors the mean makes smaller.
    Bound: the plain order's own error; 5% above it, as the 2-norm of the
    rounding errors of some 2,000 outputs that share hidden rows varies by a
    few percent."""
    print(f"GraphSAGE {dims}, error, fp16 {fp16}, fan-out {fanout}", flush=True)
    w, r, n = sampled(fanout)
    rng = np.random.default_rng(sum(dims))
    x = rng.standard_normal((n, dims[0])).astype(np.float16 if fp16 else np.float32)
    layers = _sage_layers(rng, dims)
    ref, _ = oracle_forward(r, fanout, x, layers)
    got = forward(w, x, layers)[:ref.shape[0]]
    err, plain = (np.linalg.norm(v.astype(np.float64) - ref) / np.linalg.norm(ref)
                  for v in (got, projected_first(r, fanout, x, layers)))
    print(f"{err:.3e}, projected first {plain:.3e}: {err / plain:.3f}", flush=True)
    assert err <= 1.05 * plain


@pytest.mark.parametrize("dims,fanout", [([12, 12, 5], (10, 5)), ([70, 64], (32,)),
                                         ([300, 12, 20], (11, 10))])
def test_means_of_huge_rows_are_finite(dims, fanout):
    """Features of one sign close to the largest float: two of them overflow,
    their mean does not."""
    print(f"GraphSAGE {dims}, huge features, fan-out {fanout}", flush=True)
    w, r, n = sampled(fanout)
    rng = np.random.default_rng(dims[0])
    x = (3.4e38 * rng.uniform(0.6, 1.0, (n, dims[0]))).astype(np.float32)
    layers = _sage_layers(rng, dims)
    layers[0] = (layers[0][0] * np.float32(2 ** -16), layers[0][1] * np.float32(2 ** -16),
                 *layers[0][2:])
    ref, ab = oracle_forward(r, fanout, x, layers)
    got = forward(w, x, layers)[:ref.shape[0]].astype(np.float64)
    assert np.isfinite(got).all()
    assert np.all(np.abs(got - ref) <= _sage_tolerance(layers, list(fanout), ab))


def test_last_level_list_is_not_read():
    """The rows of N_b are found by rank in the bit sets: the last level's id
    list may have been overwritten since the gather."""
    print("GraphSAGE without the last level's ids", flush=True)
    dims, fanout = [20, 16, 7], (6, 5)
    w, r, n = sampled(fanout)
    rng = np.random.default_rng(4)
    x = rng.standard_normal((n, dims[0])).astype(np.float32)
    layers = _sage_layers(rng, dims)
    ref, ab = oracle_forward(r, fanout, x, layers)
    w.pipe.frontier_ids[int(r["foff"][len(fanout) * WK]):] = -5
    got = forward(w, x, layers)[:ref.shape[0]].astype(np.float64)
    assert np.all(np.abs(got - ref) <= _sage_tolerance(layers, list(fanout), ab))
