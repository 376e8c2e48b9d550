"""Tile list and stream list of a resident layer in one launch: the same bytes as
the scheduled forward's separate launches (the first call of a plan), for lists
that are both there, nearly all stream (17 tokens, where the shared expert has
two 16-row groups) and nearly all tiles, at every chunk width d and I leave; and
the middle batch agrees with the fp64 oracle (max-abs / max|ref| <= 1e-2: act
and output rows rounded to bf16 once each)."""
import pytest

import synth
from _gpu_helpers import device_layer, log, make_plan, oracle_compare, run_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt,d,I", [("bf16", 256, 128), ("bf16", 512, 384), ("bf16", 1024, 256), ("bf16", 2048, 512),
                                     ("q4b32", 256, 128), ("q4b32", 512, 256), ("q4b32", 768, 384),
                                     ("q4b32", 1024, 512),
                                     ("kq", 256, 256), ("kq", 512, 512), ("kq", 1024, 768)])
def test_both_lists(fmt, d, I):
    import torch  # noqa: F401  (loads its HIP runtime before the library)
    import oracle
    wl = synth.Workload("both_lists", 43, synth.LayerShape(140, d, 12, 4, I, fmt), prior="zipf", prior_param=1.1,
                        tau=0.3)
    li = synth.layer_inputs(wl)
    dl = device_layer(li)
    seen = set()
    for T in (17, 40, 140):
        plan = make_plan(li, capacity=12)
        ref = None
        for again in range(3):
            log(f"case both_lists {fmt} d={d} I={I} T={T} call {again}")
            res = run_layer(plan, dl, T=T)
            out = res["out"].cpu().numpy()
            ref = out if ref is None else ref
            assert out.tobytes() == ref.tobytes()
        c = res["counts"]
        seen |= {(bool((c > 16).any()), bool(((c > 0) & (c <= 16)).any()))}
        if T == 40:
            err, _, _ = oracle_compare(oracle.Oracle(), li, res, list(range(0, T, 3)), 1e-2)
            log(f"both_lists err={err:.3e}")
        plan.close()
    assert (True, True) in seen
