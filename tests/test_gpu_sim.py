"""The simulator's accumulation over one and many events: a lane per event,
the results added in a fixed order, so the fp64 sums equal plain Python's bit
for bit."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2606_02916_amd import gg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nseg,P,local", [(1, 1, 0), (1, 64, 5), (3, 5, -1), (16, 4, 0),
                                          (64, 4, 3), (64, 64, 63)])
def test_accumulate_equals_python(nseg, P, local):
    print(f"{nseg} batches, {P} owners, local {local}", flush=True)
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(nseg * 100 + P)
    kw = {k: rng.uniform(0, s, P) for k, s in (("eps_init", 0.1), ("eps_row", 1e-4),
                                               ("lam_init", 1e-3), ("lam_row", 1e-6))}
    coeffs = gg.make_sim_coeffs(P, bw_bytes_per_s=1.1e9, row_bytes=404.0, p_idle=30.0, **kw)
    part = gg.make_part(P, gg.PART_MOD, local, 1000)
    acc = torch.zeros(gg.SIM_ACC_BYTES, dtype=torch.uint8, device=dev)
    want = gg.gg_sim_acc_t()
    for rnd in range(3):
        st = gg.gg_stage_stats_t()
        gs = (gg.gg_gather_stats_t * nseg)()
        draw = lambda: int(rng.integers(0, 100000)) * int(rng.integers(0, 2))   # noqa: E731
        for m in range(P):
            st.delta_rows[m] = draw()
            for b in range(nseg):
                gs[b].miss_rows[m] = draw() if b % 4 != 1 else 0
        for b in range(nseg):
            gs[b].hits, gs[b].misses = draw(), draw()

        def event(x):
            e, tmax, rows, owners = 0.0, 0.0, 0, 0
            for m in range(P):
                if m != local and x[m] > 0:
                    e += float(kw["eps_init"][m]) + float(kw["eps_row"][m]) * float(x[m])
                    tmax = max(tmax, float(kw["lam_init"][m]) + float(kw["lam_row"][m]) * x[m])
                    rows += x[m]
                    owners += 1
            want.t_stall += max(tmax, rows * 404.0 / 1.1e9) if rows else 0.0
            return e, rows, owners

        e, rows, owners = event(st.delta_rows)
        want.e_rebuild += e
        want.rebuild_rows += rows
        want.rebuild_events += owners
        for b in range(nseg):
            e, rows, owners = event(gs[b].miss_rows)
            want.e_miss += e
            want.miss_rows += rows
            want.miss_events += owners
            want.hits += gs[b].hits
            want.remote_rows += gs[b].hits + gs[b].misses
        want.windows += 1
        want.batches += nseg
        want.e_stall = 30.0 * want.t_stall
        want.e_phy = (want.e_rebuild + want.e_miss) + want.e_stall
        st_d = torch.from_numpy(np.frombuffer(bytes(st), dtype=np.uint8).copy()).to(dev)
        gs_d = torch.from_numpy(np.frombuffer(bytes(gs), dtype=np.uint8).copy()).to(dev)
        assert st_d.numel() == C.sizeof(st)
        gg.gg_sim_accumulate(st_d, gs_d.data_ptr(), nseg, part, coeffs, acc)
    torch.cuda.synchronize()
    got = gg.sim_acc_from_bytes(acc.cpu().numpy().tobytes())
    assert got == {name: getattr(want, name) for name in got}
