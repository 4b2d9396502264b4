"""fp32 storage: the projections at the edges of their 32x32 and 64x64 tiles and 64-deep slabs, against the oracle, for
units cached together: K of whole slabs and not, both tile sizes, and weights that are not aligned to 16 bytes (the scalar
kernel).
fp32 sums of up to 4096 terms: 2^-24 sqrt(4096) = 4e-6 of the largest value per product, 2e-5 over a layer's four."""
import numpy as np
import pytest
import torch

import keep_synth as ks
from gpu_util import Problem, max_rel, to_np

pytestmark = pytest.mark.gpu


def _shape(hidden, ffn):
    return ks.ModelShape(2, hidden, 4, 2, 16, ffn, 97, 1.0e4, 1e-6, "f32")


@pytest.mark.parametrize("hidden,ffn,n,aligned", [(64, 96, 10, True), (80, 104, 31, True), (80, 136, 32, True),
                                                  (64, 104, 33, True), (128, 264, 65, True), (80, 104, 33, False),
                                                  (64, 4096, 513, True)])   # the last: 64x64 tiles for gate/up
def test_f32_units_match_oracle(hidden, ffn, n, aligned):
    pb = Problem(_shape(hidden, ffn), [n - 9, 9], 1, seed=n, std=0.5 / np.sqrt(hidden), bias=True)
    if not aligned:
        for w in pb.layers_d:
            for name in ks.INT4_MATS:           # the seven projections
                t = w[name]
                w[name] = torch.empty(t.numel() + 1, device="cuda")[1:].view(t.shape).copy_(t)
    ctx = pb.context(max_tokens=n + 2)
    assert not ctx.uses_mfma
    kc = torch.zeros((2, n, 2, 16), dtype=torch.float32, device="cuda")
    vc = torch.zeros_like(kc)
    ctx.precompute_groups([n - 9, 9], pb.ids[:n], kc, vc)
    torch.cuda.synchronize()
    for l in range(2):
        for g, rows in enumerate((slice(0, n - 9), slice(n - 9, n))):
            ek, ev = max_rel(to_np(kc[l][rows]), pb.kb[l][g]), max_rel(to_np(vc[l][rows]), pb.vb[l][g])
            print(n, "layer", l, "unit", g, "K %.2e V %.2e" % (ek, ev))
            assert ek < 2e-5 and ev < 2e-5
