"""Token rows of a wide range on the quantized mix's tile path, which holds tokens as
scaled fp16: rows whose small elements fall into fp16's subnormal range and are held
exactly there (multiples of 2^-1, down to 2^-37 of the largest element) and rows that
it cannot hold (other elements below 2^-31 of the largest, down to 2^-120), with the large element against weights that are exactly zero, so the
outputs are the small elements' alone; and a row whose act values are near the end
of binary32's range (2^113), where down's sums must not leave it.  Each row against
the fp64 oracle on its own scale (max-abs / max|ref row| <= 1e-2: act and output
rows rounded to bf16 once each), byte-identical across batch sizes (both tile
forms), slot capacities and the static-scratch entry point."""
import numpy as np
import pytest

import synth
from _gpu_helpers import device_layer, log, make_plan, run_layer

pytestmark = pytest.mark.gpu

# every expert selected (K = E), so an expert's rows are the whole batch
LAYER = synth.Workload("kq_tokens", 50, synth.LayerShape(130, 512, 4, 4, 512, "kq"))
J0, J1 = 5, 256 + 100                   # against zeros in Wg and Wu; against zeros in Wu
POWERS = (14, 20, 26, 28, 30, 34, 36, 40, 60, 120)


def _layer():
    li = synth.layer_inputs(LAYER)
    s = LAYER.shape
    d, I = s.d, s.I
    nib, hdr = I * d // 2, I * (d // 256) * 16
    for o in [li.expert(e) for e in range(s.E)] + [li.shared]:
        for mat, j in ((0, J0), (1, J0), (1, J1)):
            at = mat * (nib + hdr)
            q = o[at:at + nib].reshape(I, d // 2)
            h = o[at + nib:at + nib + hdr].reshape(I, d // 256, 16)
            q[:, j // 2] &= np.uint8(0x0F if j & 1 else 0xF0)          # code 0 ...
            sub = (j % 256) // 32
            m = h[:, j // 256, 10:16].astype(np.uint64)
            word = sum(m[:, b] << np.uint64(8 * b) for b in range(6))
            word &= ~np.uint64(63 << (6 * sub))                        # ... and a min of 0
            for b in range(6):
                h[:, j // 256, 10 + b] = (word >> np.uint64(8 * b)) & np.uint64(255)
    wr = synth.bf16_bits_to_f32(li.wr)
    wr[:, [J0, J1]] = 0.0                                              # (the routing does not see them)
    li.wr[:] = synth.f32_to_bf16_bits(wr)
    x = synth.bf16_bits_to_f32(li.x)
    x[:, [J0, J1]] = 0.0
    t = np.arange(s.T)
    coarse = (t // len(POWERS)) % 2 == 0
    x[coarse] = np.sign(x[coarse]) * (np.minimum(np.floor(np.abs(x[coarse]) * 2), 3) + 1) / 2
    x[t, J0] = 2.0 ** np.array(POWERS)[t % len(POWERS)]
    x[7::13, J0] = 0.0
    x[7::13, J1] = 2.0 ** 119
    li.x[:] = synth.f32_to_bf16_bits(x)
    return li


def test_kq_token_range():
    import torch
    import oracle
    import paper_2608_23805_amd as msi
    li = _layer()
    dl = device_layer(li)
    s = LAYER.shape
    ora = oracle.Oracle().moe_layer(li.x, li.wr, li.bias, [li.expert(e) for e in range(s.E)], li.shared, s.K, s.I,
                                    s.wdtype, s.xdtype)
    den = np.abs(ora["out"]).max(axis=1)
    assert np.all(den[7::13] > 2.0 ** 100) and np.isfinite(den).all() and den.min() > 0
    ref = None
    for cap in (s.E, 2):
        plan = make_plan(li, capacity=cap)
        for T in (130, 128, 65, 64, 17):
            for again in range(3 if cap == s.E else 1):     # the last runs on device-built lists
                log(f"case kq_tokens capacity={cap} T={T} call {again}")
                res = run_layer(plan, dl, T=T)
                out = res["out"].cpu().numpy()
                if ref is None:
                    ref = out
                    err = np.abs(out - ora["out"]).max(axis=1) / den
                    log(f"kq_tokens err={err.max():.3e} at row {int(err.argmax())}")
                    assert err.max() <= 1e-2
                assert out.tobytes() == ref[:T].tobytes()
            static = torch.empty_like(res["out"])
            assert plan.forward_noalloc_status(0, dl.x[:T], res["routing"], dl.shared, static) == msi.MSI_OK
            torch.cuda.synchronize()
            assert static.cpu().numpy().tobytes() == out.tobytes()
        plan.close()
