"""The residual kernels at both sides of their row lengths' limits (rows of up to 2048
and 4096 columns stay in registers, longer ones are read twice) and at ragged ones,
against the oracle's step: h is the fp32 sum exactly; x is the nearest bf16 of h / rms
wherever that is farther from a rounding boundary than fp32 leaves open (the sum of
squares of up to 33 terms a thread, two reductions, quotient, root, reciprocal and
product: under 48 units of 2^-24)."""
import numpy as np
import pytest

import synth
from _gpu_helpers import log

pytestmark = pytest.mark.gpu

ERR = 48 * 2.0 ** -24


@pytest.mark.parametrize("cols", [1, 255, 257, 2047, 2048, 2049, 2304, 4096, 4097, 8200])
def test_residual_rows(cols):
    import torch
    import oracle
    import paper_2608_23805_amd as msi
    log(f"case residual_rows cols={cols}")
    o = oracle.Oracle()
    g = np.random.default_rng([52, cols])
    rows = 5
    x0 = synth.f32_to_bf16_bits(g.standard_normal((rows, cols)).astype(np.float32))
    out = (g.standard_normal((rows, cols)) * [[0.5], [2.0], [1e-3], [30.0], [0.0]]).astype(np.float32)
    h, x = torch.empty((rows, cols), device="cuda"), torch.zeros((rows, cols), dtype=torch.int16, device="cuda")

    def check(want_h):
        assert h.cpu().numpy().tobytes() == want_h.tobytes()
        hd = want_h.astype(np.float64)
        exact = torch.from_numpy(hd / np.sqrt((hd ** 2).mean(axis=1, keepdims=True) + 1e-6))
        near = (exact * (1 + ERR)).to(torch.bfloat16) != (exact * (1 - ERR)).to(torch.bfloat16)
        _, ref = o.residual_step(hd)
        got = x.cpu().numpy().view(np.uint16)
        assert np.all((got == ref) | near.numpy())
        assert near.float().mean() <= 0.01 or cols == 1

    msi.residual_init(torch.from_numpy(x0.view(np.int16)).cuda(), h, x, torch.cuda.current_stream())
    torch.cuda.synchronize()
    first = synth.bf16_bits_to_f32(x0)
    check(first)
    msi.residual_add(torch.from_numpy(out).cuda(), h, x, torch.cuda.current_stream())
    torch.cuda.synchronize()
    check(first + out)
