"""The stream kernels of the 4-bit formats take 16 or 32 weight rows per
wavefront by what bounds a launch's items (32 and more: the wide form): the
experts and routed rows of a decode, the largest round on the scheduled path.
Both are one function: with every expert resident a 16-token batch (40 experts,
128 rows) and its first 3 tokens (24 rows) give the same bytes, and so do the
rounds of a layer of 16 slots, at the chunk widths d leaves; the batch agrees
with the fp64 oracle (max-abs / max|ref| <= 1e-2: act and output rows rounded to
bf16 once each)."""
import numpy as np
import pytest

import synth
from _gpu_helpers import device_layer, log, make_plan, oracle_compare, run_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt,d,I", [("q4b32", 256, 128), ("q4b32", 768, 384), ("q4b32", 512, 256), ("q4b32", 1024, 512),
                                     ("kq", 256, 256), ("kq", 768, 256), ("kq", 512, 512), ("kq", 1024, 768)])
def test_stream_forms(fmt, d, I):
    import torch  # noqa: F401  (loads its HIP runtime before the library)
    import oracle
    wl = synth.Workload("stream_forms", 41, synth.LayerShape(16, d, 40, 8, I, fmt))
    li = synth.layer_inputs(wl)
    dl = device_layer(li)
    ref = None
    for slots in (40, 16):
        plan = make_plan(li, capacity=slots)
        for T in (16, 3):
            for again in range(3):              # the last of a resident layer runs on a device-built list
                log(f"case stream_forms {fmt} d={d} I={I} slots={slots} T={T} call {again}")
                res = run_layer(plan, dl, T=T)
                out = res["out"].cpu().numpy()
                if ref is None:
                    ref = out
                    # wide: one round of 32 items and more; narrow: rounds of 8 items or 24 rows
                    assert np.count_nonzero(res["counts"]) >= 32
                    err, _, _ = oracle_compare(oracle.Oracle(), li, res, list(range(T)), 1e-2)
                    log(f"stream_forms err={err:.3e}")
                assert out.tobytes() == ref[:T].tobytes()
        plan.close()
