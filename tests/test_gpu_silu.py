"""SiLU of the 4-bit formats' kernels over the range where e^-z is large: z / (1 +
e^-z) keeps its relative accuracy.  Tokens with one non-zero element and weights
that make every dot product exact (power-of-two units, no mins) leave SiLU and
one product as the only roundings in front of bf16: five units of 2^-24 in all
(expf two, the sum, the quotient and the product one each).  So an act value is
the correctly rounded one wherever the exact value is farther than that from a
rounding boundary.  (The exponential of a rounded product -z log2 e is off by up
to |z| 2^-24, and fails here.)  Stream path, both tile forms."""
import numpy as np
import pytest

import synth
from _gpu_helpers import device_layer, log, make_plan, run_layer, workspace_parts

pytestmark = pytest.mark.gpu

ERR = 5 * 2.0 ** -24


def _weights(fmt, o, I, d, e):
    """Fill Wg and Wu of expert e's object; returns z / v of each of the I rows, and u / v."""
    if fmt == "q4b32":
        n, m = I * d // 2, I * d // 2 + I * (d // 32) * 2
        s = (2.1 + 5.8 * np.arange(I) / I).astype(np.float16)
        for mat, q, sc in ((0, 0xB, s), (1, 0x1, np.full(I, 1 + e / 8, np.float16))):      # q = -5 and 1
            o[mat * m:mat * m + n] = q * 0x11
            o[mat * m + n:(mat + 1) * m] = np.repeat(sc[:, None], d // 32, 1).reshape(-1).view(np.uint8)
        return -5.0 * s.astype(np.float64), 1 + e / 8
    n, m = I * d // 2, I * d // 2 + I * (d // 256) * 16
    pairs = [(sc, q) for sc in range(1, 64) for q in range(1, 16) if 160 <= sc * q <= 640]
    pairs = [pairs[i * len(pairs) // I] for i in range(I)]
    for mat in (0, 1):
        nib, hdr = o[mat * m:mat * m + n].reshape(I, -1), o[mat * m + n:(mat + 1) * m].reshape(I, d // 256, 16)
        hdr[:] = 0
        for i, (sc, q) in enumerate(pairs):
            sc, q = (sc, q) if mat == 0 else (16 + 2 * e, 1)
            nib[i] = q * 0x11
            hdr[i, :, 0:2] = np.array([2.0 ** -4], np.float16).view(np.uint8)     # d; dmin is 0
            hdr[i, :, 4:10] = np.frombuffer(sum(sc << (6 * j) for j in range(8)).to_bytes(6, "little"), np.uint8)
    return np.array([sc * q / 16 for sc, q in pairs]), 1 + e / 8


@pytest.mark.parametrize("fmt", ["q4b32", "kq"])
def test_silu_accuracy(fmt):
    import torch
    import paper_2608_23805_amd as msi
    T, d, E, I = 128, 256, 8, 512
    wl = synth.Workload("silu", 48, synth.LayerShape(T, d, E, E, I, fmt))
    li = synth.layer_inputs(wl)
    v = (1 + np.arange(T) / 128) * (1 if fmt == "q4b32" else -1)              # every bf16 number of one binade
    x = np.zeros((T, d), np.float32)
    x[np.arange(T), np.arange(T) * 37 % d] = v
    li.x[:] = synth.f32_to_bf16_bits(x)
    exact = torch.empty((E, T, I), dtype=torch.float64)
    for e in range(E):
        zv, u = _weights(fmt, li.expert(e), I, d, e)
        z = zv[None, :] * v[:, None]
        assert -80 < z.min() and z.max() < -9
        exact[e] = torch.from_numpy(z / (1 + np.exp(-z)) * u * v[:, None])
    far = (exact * (1 + ERR)).to(torch.bfloat16) == (exact * (1 - ERR)).to(torch.bfloat16)
    dl = device_layer(li)
    plan = make_plan(li, capacity=E)
    r, ws = msi.Routing.alloc(T, E, E), plan.workspace(T)
    out = torch.empty((T, d), dtype=torch.float32, device="cuda")
    for n in (128, 48, 16):                             # rows of 128 and 64 tokens, stream path
        log(f"case silu {fmt} T={n}")
        plan.route(dl.x[:n], dl.wr, dl.bias, r, ws)
        st = plan.forward_status(0, dl.x[:n], r, dl.shared, out, ws, torch.cuda.current_stream(), torch.cuda.Stream())
        torch.cuda.synchronize()
        assert st == msi.MSI_OK
        at = workspace_parts(n, E, E, d, I, fmt)["act"]
        act = ws[at:at + n * E * I * 2].view(torch.bfloat16).view(E, n, I).cpu()
        bad = (act != exact[:, :n].to(torch.bfloat16)) & far[:, :n]
        log(f"silu {fmt} T={n}: {int(bad.sum())} of {int(far[:, :n].sum())} off the correctly rounded value")
        assert not bad.any()
    plan.close()
