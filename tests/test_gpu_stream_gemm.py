"""8 to 128 rows, the weight-streaming kernel with a ring of stages: row counts around its three forms (32, 64, 128 rows)
and where the narrow projections are cut along K (8, 17, 33, 64), widths that give a workgroup part of a tile of columns,
several tile widths for gate/up, more than one tile per workgroup, and columns that straddle heads and q, k and v.  bf16
storage bounds the error: 2e-2 of the largest value, as for the other bf16 launches."""
import numpy as np
import pytest
import torch

import keep_synth as ks
from gpu_util import Problem, max_rel, to_np
from layer_probe import LayerProbe

pytestmark = pytest.mark.gpu


def _shape(hidden, heads, kv, ffn):
    return ks.ModelShape(2, hidden, heads, kv, 128, ffn, 211, 1.0e6, 1e-6, "bf16")


# K = 1024 (the shortest ring) and 1152; 5 and 6 gate/up pairs per workgroup; pairs across heads
NARROW = [(_shape(1024, 8, 2, 1152), n) for n in (17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 96, 127, 128, 129)] + \
         [(_shape(1152, 9, 3, 1408), n) for n in (17, 48, 64, 100)]
# gate/up pairs per workgroup: 33 and 64 (four tiles of gate, four of up), 65 and 80 (five), 81 (seven, or two rounds)
WIDE = [(_shape(1024, 8, 1, ffn), n) for ffn in (8320, 16384, 16512, 20480, 20608) for n in (20, 50, 100)]


# up to 16 rows, where a shape is wide enough: gate/up and QKV from 8 rows on, O and down from 13
FEW = [(_shape(5120, 40, 8, 5376), n) for n in (10, 12, 13, 16)]

# cuts along K: 2048 and 2176 (splits of 8 and 9 slices) around 33 and 64 rows; from 8 rows on with K = 8192, 4 splits of 16
# columns and 8 of 32; 80 columns, and 160 with 8 splits; 192 columns (the widest tile)
CUT = [(_shape(2048, 16, 2, 2176), n) for n in (32, 33, 64, 65, 128)] + \
      [(_shape(1024, 8, 1, 8192), n) for n in (10, 16, 17, 64, 65, 127)] + \
      [(_shape(5120, 40, 8, 8192), n) for n in (17, 64, 100)] + [(_shape(2048, 64, 16, 2176), n) for n in (40, 64)]


@pytest.mark.parametrize("shape,n", NARROW + WIDE + FEW + CUT, ids=lambda v: str(v) if isinstance(v, int) else "h%d_f%d" % (v.hidden, v.ffn_dim))
def test_units_match_oracle(shape, n):
    pb = Problem(shape, [n - 9, 9], 1, seed=n, std=0.5 / np.sqrt(shape.hidden), bias=True)
    ctx = pb.context(max_tokens=n + 2)
    assert ctx.uses_mfma
    L = shape.n_layers
    kc = torch.zeros((L, n, shape.n_kv_heads, shape.head_dim), dtype=torch.bfloat16, device="cuda")
    vc = torch.zeros_like(kc)
    ctx.precompute_groups([n - 9, 9], pb.ids[:n], kc, vc)
    torch.cuda.synchronize()
    for l in range(L):
        for g, rows in enumerate((slice(0, n - 9), slice(n - 9, n))):
            ek, ev = max_rel(to_np(kc[l][rows]), pb.kb[l][g]), max_rel(to_np(vc[l][rows]), pb.vb[l][g])
            print(n, "layer", l, "unit", g, "K %.2e V %.2e" % (ek, ev))
            assert ek < 2e-2 and ev < 2e-2


# the same forms and edges, every projection of a layer for itself; and layers too wide for the oracle: weight rows a multiple
# of 4 KB apart, where the workgroups start at different slices (gate/up at 2048, 4096, 6144; down 16384 x 6144 and QKV
# 8192 x 10240, cut), the widest gate/up tiles (96 and 108 pairs of a workgroup) and, past 64 rows, two rounds of them
BY_SHAPE = {}
for _s, _n in NARROW + WIDE + FEW + CUT:
    BY_SHAPE.setdefault((_s.hidden, _s.n_q_heads, _s.n_kv_heads, _s.ffn_dim), []).append(_n)
BY_SHAPE[2048, 16, 4, 8192] = [8, 17, 32, 33, 64, 100, 128]
BY_SHAPE[4096, 8, 2, 14336] = [8, 13, 16, 17, 48, 64, 65, 128]
BY_SHAPE[4096, 2, 1, 24576] = [16, 17, 64, 65]
BY_SHAPE[5120, 4, 1, 27648] = [16, 17, 64, 65, 128]
BY_SHAPE[6144, 4, 1, 16384] = [8, 16, 17, 64, 65]
BY_SHAPE[8192, 64, 8, 1024] = [8, 17, 33, 64, 65]


@pytest.mark.parametrize("shape", BY_SHAPE, ids=lambda v: "h%d_q%d_f%d" % (v[0], v[1], v[3]))
def test_projections(shape):
    hidden, heads, kv, ffn = shape
    rows = sorted(set(BY_SHAPE[shape]))
    probe = LayerProbe(ks.ModelShape(1, hidden, heads, kv, 128, ffn, 211, 1.0e6, 1e-6, "bf16"), rows[-1], seed=ffn)
    for n in rows:
        probe.check(n)
