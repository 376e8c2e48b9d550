"""Down rows of the quantized mix's tile path against the exact sums of the act
rows they were formed from: the share of values off the correctly rounded bf16 is no
larger than that of plain fp32 arithmetic over the same codes, a 16-element sub-block
at a time (its exact partial rounded, then one FMA with its scale), which is computed
here beside it.  Both shares count a few hundred values; 1.25 times the plain one
leaves three standard deviations of either count.  Both tile forms."""
import numpy as np
import pytest

import synth
from _gpu_helpers import device_layer, log, make_plan, workspace_parts

pytestmark = pytest.mark.gpu


def _k6(o, d, I):
    """Wd's integers sc (q - 32) as sub-block scales in fp32 [d, I / 16] and codes [d, I]."""
    o = o[2 * synth.k4_matrix_nbytes(I, d):]
    a, b, c = d * I // 2, d * I // 2 + d * I // 4, d * I // 2 + d * I // 4 + d * I // 16
    low, high = o[:a].reshape(d, I // 2), o[a:b].reshape(d, I // 4)
    q = np.stack([low & 15, low >> 4], -1).reshape(d, I).astype(np.int64)
    q += 16 * np.stack([(high >> (2 * t)) & 3 for t in range(4)], -1).reshape(d, I)
    dd = o[c:c + d * (I // 256) * 2].view(np.float16).astype(np.float32).reshape(d, I // 256)
    sc = o[b:c].view(np.int8).astype(np.float32).reshape(d, I // 16)
    return np.repeat(dd, 16, 1) * sc, q - 32


@pytest.mark.parametrize("E,T", [(4, 4096), (64, 1024)])       # 4096 and 64 mean rows for each expert
def test_kq_down_sums(E, T):
    import torch
    import paper_2608_23805_amd as msi
    d, I, K = 512, 512, 4
    wl = synth.Workload("kq_down_sums", 51, synth.LayerShape(T, d, E, K, I, "kq"))
    li = synth.layer_inputs(wl)
    dl, plan = device_layer(li), make_plan(li, capacity=E)
    r, ws = msi.Routing.alloc(T, K, E), plan.workspace(T)
    out = torch.empty((T, d), dtype=torch.float32, device="cuda")
    log(f"case kq_down_sums E={E} T={T}")
    plan.route(dl.x, dl.wr, dl.bias, r, ws)
    st = plan.forward_status(0, dl.x, r, dl.shared, out, ws, torch.cuda.current_stream(), torch.cuda.Stream())
    torch.cuda.synchronize()
    assert st == msi.MSI_OK
    at = workspace_parts(T, E, K, d, I, "kq")
    act = ws[at["act"]:at["act"] + T * K * I * 2].view(torch.bfloat16).view(T * K, I)
    y = ws[at["y"]:at["y"] + T * K * d * 2].view(torch.bfloat16).view(T * K, d)
    off = r.offsets.cpu().numpy()
    n_off = n_plain = n = 0
    for e in range(E):
        lo, hi = int(off[e]), int(off[e + 1])
        if hi - lo <= 16:                                       # the stream path's
            continue
        s, q = (torch.from_numpy(v).cuda() for v in _k6(li.expert(e), d, I))
        a, w = act[lo:hi].double(), r.row_weight[lo:hi, None]
        exact = torch.zeros((hi - lo, d), dtype=torch.float64, device="cuda")
        plain = torch.zeros((hi - lo, d), dtype=torch.float32, device="cuda")
        for j in range(I // 16):
            part = a[:, 16 * j:16 * j + 16] @ q[:, 16 * j:16 * j + 16].double().t().contiguous()
            exact += part * s[:, j].double()
            plain = (part.float().double() * s[:, j].double() + plain.double()).float()
        want = (exact * w.double()).to(torch.bfloat16)
        n_off += int((y[lo:hi] != want).sum())
        n_plain += int(((plain * w).to(torch.bfloat16) != want).sum())
        n += want.numel()
    plan.close()
    log(f"kq_down_sums E={E}: {n_off} of {n} off the correctly rounded value, plain fp32 {n_plain}")
    assert n > T * K * d // 2 and n_off <= 1.25 * n_plain + 3
