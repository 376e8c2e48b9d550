"""The quantized mix's tile kernels at what their integer form must carry
exactly: super-blocks with a zero or changing d, the extreme k6 scales, token
rows of zeros, of very large and very small magnitude and with one dominant
element, at the edges of both tile forms (64 rows, mean rows per expert on
either side of 64).  Every row's output against the fp64 oracle on that row's
own scale (max-abs / max|ref row| <= 1e-2: act and output rows rounded to bf16
once each), and byte-identical across batch sizes, slot capacities (rounds) and
the static-scratch entry point."""
import numpy as np
import pytest

import synth
from _gpu_helpers import device_layer, log, make_plan, run_layer

pytestmark = pytest.mark.gpu

# every expert selected (K = E), so an expert's rows are the whole batch
LAYER = synth.Workload("kq_tiles", 40, synth.LayerShape(200, 512, 4, 4, 512, "kq"))


def _layer():
    li = synth.layer_inputs(LAYER)
    s = LAYER.shape
    d, I = s.d, s.I
    nib, hdr = I * d // 2, I * (d // 256) * 16
    o = li.expert(1)
    for mat, row, sb in ((0, 3, 0), (1, 5, 1), (0, 7, 0), (0, 7, 1)):      # gate / up headers: d = 0
        at = mat * (nib + hdr) + nib + (row * (d // 256) + sb) * 16
        o[at:at + 2] = 0
    at = 0 * (nib + hdr) + nib + (9 * (d // 256) + 1) * 16                  # a unit 2^12 larger than its neighbour's
    h = o[at:at + 2].view(np.float16)
    h *= np.float16(4096.0)
    wd = 2 * (nib + hdr)
    sc = wd + d * I // 2 + d * I // 4
    o[sc + 2 * (I // 16):sc + 3 * (I // 16)] = 128                          # down row 2: every scale -128
    o[sc + 4 * (I // 16):sc + 5 * (I // 16)] = 127
    dd = sc + d * I // 16 + 6 * (I // 256) * 2
    o[dd:dd + 2] = 0                                                        # down row 6, first super-block: d = 0
    x = synth.bf16_bits_to_f32(li.x)
    x[0] = 0.0
    x[1] *= 2.0 ** 30
    x[2] *= 2.0 ** -30
    x[3, 17] = 2.0 ** 14
    li.x[:] = synth.f32_to_bf16_bits(x)
    return li


def test_kq_tile_forms():
    import torch
    import oracle
    import paper_2608_23805_amd as msi
    li = _layer()
    dl = device_layer(li)
    s = LAYER.shape
    ora = oracle.Oracle().moe_layer(li.x, li.wr, li.bias, [li.expert(e) for e in range(s.E)], li.shared, s.K, s.I,
                                    s.wdtype, s.xdtype)
    den = np.abs(ora["out"]).max(axis=1)
    den[den == 0] = 1.0
    ref = None
    for cap in (s.E, 2):
        plan = make_plan(li, capacity=cap)
        for T in (200, 129, 128, 65, 64, 63, 17):
            log(f"case kq_tiles capacity={cap} T={T}")
            res = run_layer(plan, dl, T=T)
            out = res["out"].cpu().numpy()
            if ref is None:
                ref = out
                err = (np.abs(out - ora["out"]).max(axis=1) / den).max()
                log(f"kq_tiles err={err:.3e}")
                assert err <= 1e-2
            assert out.tobytes() == ref[:T].tobytes()
            static = torch.empty_like(res["out"])
            assert plan.forward_noalloc_status(0, dl.x[:T], res["routing"], dl.shared, static) == msi.MSI_OK
            torch.cuda.synchronize()
            assert static.cpu().numpy().tobytes() == out.tobytes()
        plan.close()
