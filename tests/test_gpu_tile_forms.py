"""The forms of the bf16 and int4 tile paths and of the router logits (64-, 128- and
256-row tiles, picked by the mean rows per expert; 32 x 32 to 256 x 256 router
tiles, picked by their number) are one function: the same tokens give the same
bytes whichever form their batch takes, at the edges of every rule, and the
largest batch agrees with the fp64 oracle (max-abs / max|ref| <= 1e-2, the
bf16 bound: act and output rows rounded to bf16 once each)."""
import numpy as np
import pytest

import synth
from _gpu_helpers import device_layer, log, make_plan, oracle_compare, run_layer

pytestmark = pytest.mark.gpu

# 8 experts, top-2: T / 4 mean rows per expert; 64-row tiles up to 48 (T 192), 128-row up to 112 (T 448)
LAYER = synth.Workload("tile_forms", 38, synth.LayerShape(460, 512, 8, 2, 384, "bf16"))
# 64-row gate/up tiles up to 64 mean rows (T 256)
LAYER_Q4 = synth.Workload("tile_forms_q4", 42, synth.LayerShape(300, 512, 8, 2, 384, "q4b32"))
# ragged expert count: a partial router tile in every form
ROUTER = synth.Workload("router_forms", 39, synth.LayerShape(4100, 256, 1000, 4, 128, "bf16"),
                        prior="zipf", prior_param=1.1, tau=0.3)


@pytest.mark.parametrize("wl,sizes", [(LAYER, (460, 452, 448, 300, 196, 192, 65, 64, 33)),
                                      (LAYER_Q4, (300, 260, 257, 256, 200, 129, 65, 64))])
def test_tile_forms(wl, sizes):
    import torch  # noqa: F401  (loads its HIP runtime before the library)
    import oracle
    import paper_2608_23805_amd as msi
    li = synth.layer_inputs(wl)
    dl = device_layer(li)
    plan = make_plan(li, capacity=wl.shape.E)
    old = msi.stream_threshold()
    msi.stream_threshold(1)                 # every expert of two or more rows on the tile path
    try:
        ref = None
        for T in sizes:
            log(f"case {wl.name} T={T}")
            res = run_layer(plan, dl, T=T)
            assert res["counts"].min() >= 2
            out = res["out"].cpu().numpy()
            if ref is None:
                ref = out
                err, _, _ = oracle_compare(oracle.Oracle(), li, res, list(range(T)), 1e-2)
                log(f"{wl.name} err={err:.3e}")
            assert out.tobytes() == ref[:T].tobytes()
    finally:
        msi.stream_threshold(old)
        plan.close()


def test_router_forms():
    import torch
    import torch  # noqa: F401  (loads its HIP runtime before the library)
    import oracle
    import paper_2608_23805_amd as msi
    li = synth.layer_inputs(ROUTER, lazy=True)
    dl = device_layer(li)
    s = ROUTER.shape
    plan = make_plan(li, capacity=1, experts=[0])
    ref = None
    for T in (4100, 4096, 2049, 2048, 513, 512, 257, 33, 17):   # 256, 128, 128, 64, 64, 32 .. 32 columns
        log(f"case router_forms T={T}")
        r = msi.Routing.alloc(T, s.K, s.E)
        ws = plan.workspace(T)
        plan.route(dl.x[:T], dl.wr, dl.bias, r, ws)
        torch.cuda.synchronize()
        L = ws[:T * s.E * 4].view(torch.float32).view(T, s.E).cpu().numpy()
        idx, w = r.idx.cpu().numpy(), r.weights.cpu().numpy()
        if ref is None:
            ref = (L, idx, w)
            o = oracle.Oracle()
            exact = o.router_logits(li.x, li.wr, li.bias, s.xdtype)
            assert np.abs(L - exact).max() <= 1e-5 * np.abs(exact).max()   # fp32 sums of 256 exact products
        assert L.tobytes() == ref[0][:T].tobytes()
        assert np.array_equal(idx, ref[1][:T]) and w.tobytes() == ref[2][:T].tobytes()
    plan.close()
