"""Launches of 17 rows and more at the edges of the GEMM's tiles, against the oracle: units cached together through the
fused QKV epilogue of the 128x128 tiles (row counts around a wave's 32 rows and the tile's 128, launches cut along K and
not), and row counts on both sides of the line between 128x128 and 256x256 tiles.  bf16 storage bounds the error: 2e-2 of
the largest value, as for the other bf16 launches."""
import numpy as np
import pytest
import torch

import keep_synth as ks
from gpu_util import Problem, max_rel, to_np

pytestmark = pytest.mark.gpu

# K = 512 (8 slices: two pieces) and 1152 (18: four pieces); an odd number of tile columns, one key / value head
CUT = ks.ModelShape(2, 512, 4, 2, 128, 1152, 211, 1.0e6, 1e-6, "bf16")
ODD = ks.ModelShape(2, 640, 3, 1, 128, 320, 211, 1.0e6, 1e-6, "bf16")
# gate/up: 64 tile columns x 32 K slices x 2 tile rows, which the large tiles take from 410 rows on
LINE = ks.ModelShape(2, 2048, 2, 1, 128, 8192, 211, 1.0e6, 1e-6, "bf16")


@pytest.mark.parametrize("shape,n", [(s, n) for s in (CUT, ODD) for n in (17, 31, 32, 33, 64, 65, 127, 128, 129, 161)] +
                         [(LINE, 409), (LINE, 410)],
                         ids=lambda v: str(v) if isinstance(v, int) else "h%d" % v.hidden)
def test_units_match_oracle(shape, n):
    pb = Problem(shape, [n - 9, 9], 1, seed=n, std=0.5 / np.sqrt(shape.hidden), bias=True)
    ctx = pb.context(max_tokens=n + 2)
    assert ctx.uses_mfma
    L = shape.n_layers
    kc = torch.zeros((L, n, shape.n_kv_heads, shape.head_dim), dtype=torch.bfloat16, device="cuda")
    vc = torch.zeros_like(kc)
    ctx.precompute_groups([n - 9, 9], pb.ids[:n], kc, vc)       # (the oracle made the same units' caches for the problem)
    torch.cuda.synchronize()
    for l in range(L):
        for g, rows in enumerate((slice(0, n - 9), slice(n - 9, n))):
            ek, ev = max_rel(to_np(kc[l][rows]), pb.kb[l][g]), max_rel(to_np(vc[l][rows]), pb.vb[l][g])
            print(n, "layer", l, "unit", g, "K %.2e V %.2e" % (ek, ev))
            assert ek < 2e-2 and ev < 2e-2
