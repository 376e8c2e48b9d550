"""A demanded expert without a published slot on the device-built lists (T above
the stream threshold): the attempt publishes nothing, runs none of that expert's
rows and writes nothing past the workspace (a guard as large as the permuted rows
would reach keeps its pattern, on the tile path and on the stream path, with and
without a shared expert), and the rescheduled forward agrees with the fp64 oracle
(max-abs / max|ref| <= 1e-2: act and output rows rounded to bf16 once each)."""
import dataclasses

import numpy as np
import pytest

import synth
from _gpu_helpers import device_layer, log, make_plan, oracle_compare

pytestmark = pytest.mark.gpu

GUARD = 0xA7


@pytest.mark.parametrize("shared", [True, False])
@pytest.mark.parametrize("fmt,I", [("bf16", 128), ("q4b32", 128), ("kq", 256)])
def test_unpublished_expert(fmt, I, shared):
    import torch  # loads its HIP runtime before the library
    import oracle
    import paper_2608_23805_amd as msi
    T = 48
    wl = synth.Workload("unpublished", 46, synth.LayerShape(2 * T, 256, 64, 4, I, fmt, shared=shared),
                        prior="dirichlet", prior_param=0.3, tau=1.0)
    li = synth.layer_inputs(wl)
    s = wl.shape
    la = dataclasses.replace(li, x=li.x[:T])
    lb = dataclasses.replace(li, x=li.x[T:], bias=np.ascontiguousarray(li.bias[::-1]))   # other experts are popular
    plan = make_plan(li, capacity=s.E)
    ws0 = plan.workspace(T)
    ws = torch.empty(ws0.numel() + s.K * T * s.d * 2, dtype=torch.uint8, device="cuda")
    ws[ws0.numel():] = GUARD
    r = msi.Routing.alloc(T, s.K, s.E)
    out = torch.empty((T, s.d), dtype=torch.float32, device="cuda")
    seen, fills = None, 0
    plan.set_timing(True, kinds=["permute"])           # the work-list launch (and the mix's token copies)
    for step, l in (("a fills", la), ("a, host list", la), ("b meets unpublished experts", lb), ("b again", lb)):
        log(f"case unpublished {fmt} shared={shared}: batch {step}")
        dl = device_layer(l)
        before = plan.timings()["permute"][0]
        plan.route(dl.x, dl.wr, dl.bias, r, ws)
        st = plan.forward_status(0, dl.x, r, dl.shared, out, ws, torch.cuda.current_stream(), torch.cuda.Stream())
        torch.cuda.synchronize()
        assert st == msi.MSI_OK, msi.last_error()
        assert torch.all(ws[ws0.numel():] == GUARD), "written past the workspace"
        counts = r.counts.cpu().numpy()
        if step.startswith("b meets"):
            assert plan.timings()["permute"][0] > before        # the device lists were tried first
            new = [int(e) for e in np.flatnonzero(counts) if e not in seen]
            assert plan.stats()["fills"] == fills + len(new)
            # on both paths, and with rows the shared expert's buffers do not have
            assert any(counts[e] > 16 for e in new) and any(counts[e] <= 16 for e in new)
            assert max(int(r.offsets[e]) for e in new) >= T
            res = {"idx": r.idx.cpu().numpy(), "out": out}
            err, _, _ = oracle_compare(oracle.Oracle(), lb, res, list(range(T)), 1e-2)
            log(f"unpublished err={err:.3e}")
            ref = out.cpu().numpy()
        elif step == "b again":
            assert out.cpu().numpy().tobytes() == ref.tobytes()
        else:
            seen, fills = set(np.flatnonzero(counts).tolist()), plan.stats()["fills"]
    plan.close()
