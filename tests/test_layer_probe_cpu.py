"""What the comparison by blocks sees: faults of a tile's size, planted in the 64-bit reference, against its tolerance."""
import pytest
import torch

import keep_synth as ks
import layer_probe as lp

SHAPES = [ks.ModelShape(1, 1024, 8, 2, 128, 8192, 97, 1.0e6, 1e-6, "bf16"),
          ks.ModelShape(1, 2048, 16, 2, 128, 2176, 97, 1.0e6, 1e-6, "bf16"),
          ks.ModelShape(1, 512, 4, 1, 128, 27648, 97, 1.0e6, 1e-6, "bf16")]


@pytest.mark.parametrize("s", SHAPES, ids=lambda s: "h%d_f%d" % (s.hidden, s.ffn_dim))
def test_faults_of_a_tile_exceed_the_tolerance(s):
    n = 33
    w = {k: t.to(torch.float64) for k, t in lp.weights(s, 1, "cpu").items()}
    g = torch.Generator().manual_seed(2)
    x = 0.02 * torch.randn((n, s.hidden), generator=g, dtype=torch.float64)
    o = torch.randn((n, s.q_dim), generator=g, dtype=torch.float64)
    pos = torch.arange(3, 3 + n)
    q, k, v = lp.qkv(s, w, x, pos)
    kc, vc = (torch.cat([torch.randn((3,) + t.shape[1:], generator=g, dtype=t.dtype), t]) for t in (k, v))
    parts = {"wq": lambda w: lp.attention(s, lp.qkv(s, w, x, pos)[0], kc, vc, pos), "wk": lambda w: lp.qkv(s, w, x, pos)[1],
             "wv": lambda w: lp.qkv(s, w, x, pos)[2], "wo": lambda w: torch.mm(o, w["wo"].T)}
    parts.update({name: lambda w: lp.ffn(s, w, x) for name in ("wgate", "wup", "wdown")})
    for name, part in parts.items():
        ref = part(w)
        # what storing to bfloat16 alone costs, and 256 values' scatter around it
        assert lp.block_err(ref.to(torch.bfloat16), ref) < 0.4 * lp.TOL
        rows, depth = w[name].shape
        for what, cut in (("16 columns", (slice(rows - 16, rows), slice(None))), ("a slice of K", (slice(None), slice(depth - 64, depth)))):
            bad = dict(w)
            bad[name] = w[name].clone()
            bad[name][cut] = 0.0
            e = lp.block_err(part(bad), ref)
            print(name, what, "%.3f" % e)
            assert e > 2 * (lp.ATTENTION_TOL if name == "wq" else lp.TOL), (name, what)
    # one stale 32-deep product of one tile
    ref, stale = torch.mm(o, w["wo"].T), torch.mm(o[:16, :32], w["wo"][:16, :32].T)
    bad = ref.clone()
    bad[:16, :16] -= stale
    assert lp.block_err(bad, ref) > 2 * lp.TOL
