"""Hidden states with one element near the end of binary32's range, in int4 layers
on the stream path: the codes enter the dot products as they are, so a row stays
finite as long as its own products do (codes offset by a constant c would make
c times the element of it, and the difference of two infinities).  The element
meets codes of either sign in Wg and zeros in Wu, so act keeps the element's
size; each row against the fp64 oracle on its own scale (max-abs / max|ref row|
<= 1e-2: act and output rows rounded to bf16 once each)."""
import numpy as np
import pytest

import synth
from _gpu_helpers import device_layer, log, make_plan, run_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,I,E", [(256, 128, 12), (1024, 256, 12), (1024, 256, 40)])     # 16 weight rows, 32
def test_token_range_q4(d, I, E):
    import torch  # noqa: F401  (loads its HIP runtime before the library)
    import oracle
    wl = synth.Workload("token_range", 47, synth.LayerShape(16, d, E, 4, I, "q4b32"))
    li = synth.layer_inputs(wl)
    s = wl.shape
    x = synth.bf16_bits_to_f32(li.x)
    at = np.arange(s.T) * 13 % d                        # token t's large element
    mbytes = I * d // 2 + I * (d // 32) * 2
    for o in [li.expert(e) for e in range(s.E)] + [li.shared]:
        nib = o[mbytes:mbytes + I * d // 2].reshape(I, d // 2)
        for j in at:
            nib[:, j // 2] &= np.uint8(0x0F if j & 1 else 0xF0)
    wr = synth.bf16_bits_to_f32(li.wr)
    wr[:, at] = 0.0                                     # (the routing does not see it)
    li.wr[:] = synth.f32_to_bf16_bits(wr)
    x[np.arange(s.T), at] = 2.0 ** 121
    li.x[:] = synth.f32_to_bf16_bits(x)
    ora = oracle.Oracle().moe_layer(li.x, li.wr, li.bias, [li.expert(e) for e in range(s.E)], li.shared, s.K, s.I,
                                    s.wdtype, s.xdtype)
    den = np.abs(ora["out"]).max(axis=1)
    assert den.min() > 2.0 ** 90 and den.max() < 2.0 ** 120
    dl = device_layer(li)
    plan = make_plan(li, capacity=s.E)
    for T in (16, 7, 1):                                # (40 experts: 32 weight rows at 16 tokens)
        for again in range(3):                          # the last runs on a device-built list
            log(f"case token_range d={d} I={I} T={T} call {again}")
            out = run_layer(plan, dl, T=T)["out"].cpu().numpy()
            err = (np.abs(out - ora["out"][:T]).max(axis=1) / den[:T]).max()
            log(f"token_range err={err:.3e}")
            assert err <= 1e-2
    plan.close()
