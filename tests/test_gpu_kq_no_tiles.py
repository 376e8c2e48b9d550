"""A quantized-mix batch above the stream threshold without a tile item (no shared
expert, at most 16 rows each): the scheduled and the device-built forward leave the
tokens' fp16 copy out (its place, Ys, keeps its pattern) and give the same bytes; with
a busy expert the copy is there and the outputs agree with the fp64 oracle
(max-abs / max|ref| <= 1e-2: act and output rows rounded to bf16 once each)."""
import numpy as np
import pytest

import synth
from _gpu_helpers import device_layer, log, make_plan, oracle_compare, workspace_parts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("busy", [False, True])
def test_no_tiles(busy):
    import torch  # loads its HIP runtime before the library
    import oracle
    import paper_2608_23805_amd as msi
    T = 24
    wl = synth.Workload("kq_no_tiles", 53, synth.LayerShape(T, 256, 64, 2, 256, "kq", shared=False))
    li = synth.layer_inputs(wl)
    s = wl.shape
    li.bias = np.zeros(s.E, np.float32)
    if busy:
        li.bias[5] = 100.0
    dl = device_layer(li)
    plan = make_plan(li, capacity=s.E)
    r, ws = msi.Routing.alloc(T, s.K, s.E), plan.workspace(T)
    out = torch.empty((T, s.d), dtype=torch.float32, device="cuda")
    at = workspace_parts(T, s.E, s.K, s.d, s.I, "kq")["ys"]
    ys = ws[at:at + T * s.d * 2].view(torch.int64)
    ref = None
    for again in range(3):                              # the last runs on the device-built lists
        log(f"case kq_no_tiles busy={busy} call {again}")
        ws.fill_(0x5A)
        plan.route(dl.x, dl.wr, dl.bias, r, ws)
        st = plan.forward_status(0, dl.x, r, None, out, ws, torch.cuda.current_stream(), torch.cuda.Stream())
        torch.cuda.synchronize()
        assert st == msi.MSI_OK, msi.last_error()
        assert bool((r.counts > 16).any()) == busy
        kept = ys == 0x5A5A5A5A5A5A5A5A
        assert not kept.any() if busy else kept.all()
        got = out.cpu().numpy()
        ref = got if ref is None else ref
        assert got.tobytes() == ref.tobytes()
    err, _, _ = oracle_compare(oracle.Oracle(), li, {"idx": r.idx.cpu().numpy(), "out": out}, list(range(T)), 1e-2)
    log(f"kq_no_tiles err={err:.3e}")
    plan.close()
