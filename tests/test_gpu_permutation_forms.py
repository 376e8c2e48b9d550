"""The permutation of a routing at both sides of its forms' limits (one
workgroup with the selection's bitmask up to 256 tokens, one with running counts
up to 512, block launches above), for few and for 1024 experts and up to the
sixteen of top-16: whole numbers, equal to the definition on the host (an
expert's rows are its tokens ascending)."""
import numpy as np
import pytest

import synth
from _gpu_helpers import device_layer, log, make_plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,K", [(1024, 16), (1000, 7), (65, 10), (8, 1)])
def test_permutation_forms(E, K):
    import torch  # loads its HIP runtime before the library
    import paper_2608_23805_amd as msi
    wl = synth.Workload("permutation_forms", 45, synth.LayerShape(513, 256, E, K, 128, "bf16"), prior="zipf",
                        prior_param=1.1, tau=0.3)
    li = synth.layer_inputs(wl, lazy=True)
    dl = device_layer(li)
    plan = make_plan(li, capacity=1, experts=[0])
    for T in (513, 512, 511, 300, 257, 256):
        log(f"case permutation_forms E={E} K={K} T={T}")
        r = msi.Routing.alloc(T, K, E)
        plan.route(dl.x[:T], dl.wr, dl.bias, r, plan.workspace(T))
        torch.cuda.synchronize()
        idx, w = r.idx.cpu().numpy().reshape(-1), r.weights.cpu().numpy().reshape(-1)
        counts = np.bincount(idx, minlength=E)
        order = np.argsort(idx, kind="stable")             # by expert, then token
        inv = np.empty(T * K, np.int64)
        inv[order] = np.arange(T * K)
        dem = np.flatnonzero(counts)
        assert np.array_equal(r.counts.cpu().numpy(), counts)
        assert np.array_equal(r.offsets.cpu().numpy(), np.concatenate([[0], np.cumsum(counts)]))
        assert np.array_equal(r.demand.cpu().numpy()[:len(dem) + 1], np.concatenate([[len(dem)], dem]))
        assert np.array_equal(r.perm.cpu().numpy(), order // K)
        assert np.array_equal(r.inv.cpu().numpy().reshape(-1), inv)
        assert r.row_weight.cpu().numpy().tobytes() == w[order].tobytes()
    plan.close()
