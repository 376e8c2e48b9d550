"""The stream kernels of the 4-bit formats take 16 or 32 weight rows per
wavefront by the batch's routed rows (32 rows and more: the wide form); both
are one function: the tokens of a 7-token batch (28 rows) give the same bytes
in an 8-token one (32 rows), at the chunk widths d leaves, and the batch agrees
with the fp64 oracle (max-abs / max|ref| <= 1e-2: act and output rows rounded to
bf16 once each)."""
import pytest

import synth
from _gpu_helpers import device_layer, log, make_plan, oracle_compare, run_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt,d,I", [("q4b32", 256, 128), ("q4b32", 768, 384), ("q4b32", 512, 256), ("q4b32", 1024, 512),
                                     ("kq", 256, 256), ("kq", 768, 256), ("kq", 512, 512), ("kq", 1024, 768)])
def test_stream_forms(fmt, d, I):
    import torch  # noqa: F401  (loads its HIP runtime before the library)
    import oracle
    wl = synth.Workload("stream_forms", 41, synth.LayerShape(8, d, 12, 4, I, fmt))
    li = synth.layer_inputs(wl)
    dl = device_layer(li)
    plan = make_plan(li, capacity=12)
    outs = {}
    for T in (8, 7):
        for again in range(3):              # the last runs on a device-built list
            log(f"case stream_forms {fmt} d={d} I={I} T={T} call {again}")
            res = run_layer(plan, dl, T=T)
            out = res["out"].cpu().numpy()
            assert outs.setdefault(T, out).tobytes() == out.tobytes()
        if T == 8:
            err, _, _ = oracle_compare(oracle.Oracle(), li, res, list(range(T)), 1e-2)
            log(f"stream_forms err={err:.3e}")
    assert outs[7].tobytes() == outs[8][:7].tobytes()
    plan.close()
