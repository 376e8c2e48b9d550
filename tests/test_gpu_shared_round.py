"""A forward of several rounds runs the shared expert with its first one, beside the
later rounds' fills, where nothing stands in the way: on the stream path of every
format (for the quantized mix the shared outputs' place holds the tile path's
tokens while tile items are left).  The last round's fill is held in the source;
the shared outputs are in the workspace before it is let go."""
import threading
import time

import numpy as np
import pytest

import synth
from _gpu_helpers import device_layer, log, make_plan, make_source_plan, run_layer, workspace_parts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", ["bf16", "q4b32", "kq"])
def test_shared_expert_in_the_first_round(fmt, tmp_path):
    import torch
    import paper_2608_23805_amd as msi
    T = 8
    wl = synth.Workload("shared_round", 49, synth.LayerShape(T, 256, 32, 4, 256, fmt))
    li = synth.layer_inputs(wl)
    s = wl.shape
    dl = device_layer(li)
    control = make_plan(li, capacity=s.E)
    ref = run_layer(control, dl)
    control.close()
    demanded = np.flatnonzero(ref["counts"])
    plan = make_source_plan(li, 4, str(tmp_path / "canon.bin"))
    assert len(demanded) > 8                             # several rounds; misses go in ascending order
    plan.source_fault(0, int(demanded[-1]), 0, "hold")
    r, ws = msi.Routing.alloc(T, s.K, s.E), plan.workspace(T)
    ws.fill_(0x5A)
    out = torch.empty((T, s.d), dtype=torch.float32, device="cuda")
    plan.route(dl.x, dl.wr, dl.bias, r, ws)
    torch.cuda.synchronize()
    compute, side, look = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()
    at = workspace_parts(T, s.E, s.K, s.d, s.I, fmt)["ys"]
    status = []
    log(f"case shared_round {fmt}: {len(demanded)} experts in 4 slots, the last one held")
    fwd = threading.Thread(target=lambda: status.append(
        plan.forward_status(0, dl.x, r, dl.shared, out, ws, compute, side)))
    fwd.start()
    early = False
    t0 = time.time()
    with torch.cuda.stream(look):
        while not early and time.time() - t0 < 5.0:      # (well inside the hold's own time limit)
            early = not bool((ws[at:at + T * s.d * 2].view(torch.int64) == 0x5A5A5A5A5A5A5A5A).any())
            time.sleep(0.01)
    running = fwd.is_alive()
    plan.source_release()
    fwd.join()
    torch.cuda.synchronize()
    assert status == [msi.MSI_OK], msi.last_error()
    assert running and early, "the shared expert waited for the last round"
    assert out.cpu().numpy().tobytes() == ref["out"].cpu().numpy().tobytes()
    plan.close()
