"""The bf16 stream down kernel reads its act rows directly up to 8 mean rows per
expert and through LDS past that (where I is at most 768); both are one function:
the tokens of a 32-token batch (8 mean rows) give the same bytes in a 33-token
one where their experts have at most 16 rows (the stream path) or more (the tile
path) in both, at every chunk width and number of staged pieces I leaves, and the batch
agrees with the fp64 oracle (max-abs / max|ref| <= 1e-2: act and output rows
rounded to bf16 once each)."""
import pytest

import synth
from _gpu_helpers import device_layer, log, make_plan, oracle_compare, run_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,I", [(256, 128), (512, 256), (256, 384), (1024, 512), (256, 640), (512, 768), (256, 896),
                                 (256, 1024)])
def test_staged_rows(d, I):
    import torch  # noqa: F401  (loads its HIP runtime before the library)
    import oracle
    wl = synth.Workload("stream_staged", 44, synth.LayerShape(33, d, 8, 2, I, "bf16"))
    li = synth.layer_inputs(wl)
    dl = device_layer(li)
    plan = make_plan(li, capacity=8)
    outs, counts = {}, {}
    for T in (33, 32):
        for again in range(3):              # the last runs on a device-built list
            log(f"case stream_staged d={d} I={I} T={T} call {again}")
            res = run_layer(plan, dl, T=T)
            out = res["out"].cpu().numpy()
            assert outs.setdefault(T, out).tobytes() == out.tobytes()
        counts[T] = res["counts"]
        if T == 33:
            err, _, _ = oracle_compare(oracle.Oracle(), li, res, list(range(T)), 1e-2)
            log(f"stream_staged err={err:.3e}")
            ids = res["idx"]
    plan.close()
    same = (counts[32] > 16) == (counts[33] > 16)
    rows = same[ids[:32]].all(axis=1)
    assert rows.sum() >= 8 and (counts[33] <= 16).sum() >= 4
    assert outs[32][rows].tobytes() == outs[33][:32][rows].tobytes()
