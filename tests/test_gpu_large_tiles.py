"""The 256x256 tiles of the GEMM at the edges of a last tile's rows: more and fewer than 64, 128 and 192 of them, one, and
none missing: every projection of a layer for itself, where its tiles are whole and where they are cut along K (the fused
QKV epilogue, the residual add and SwiGLU run inside the kernel in the one case, behind it in the other), and units
with positions of their own, whose single passes go through other kernels; there both sides round to bf16 at every step:
2e-2 of the largest value."""
import numpy as np
import pytest
import torch

import keep_synth as ks
from gpu_util import Problem, max_rel, to_np
from layer_probe import LayerProbe

pytestmark = pytest.mark.gpu

# 2304 rows and more: ten rows of tiles x (10, 8, 32 and 8 columns of tiles) x 32 K slices
SHAPE = ks.ModelShape(2, 2048, 16, 2, 128, 4096, 211, 1.0e6, 1e-6, "bf16")


@pytest.fixture(scope="module")
def problem():
    pb = Problem(SHAPE, [2], 1, std=0.5 / np.sqrt(2048), bias=True, random_cache=True)
    return pb, pb.context(max_tokens=2560)


@pytest.mark.parametrize("n", [2305, 2367, 2368, 2369, 2432, 2433, 2496, 2497, 2560])
def test_units_in_one_pass_match_single_units(problem, n):
    pb, ctx = problem
    rng = np.random.default_rng(n)
    lens = [300] * 7
    lens.append(n - sum(lens))
    ids = rng.integers(0, SHAPE.vocab, size=n).astype(np.int32)

    def cache(rows):
        k = torch.zeros((2, rows, 2, 128), dtype=torch.bfloat16, device="cuda")
        return k, torch.zeros_like(k)

    kc, vc = cache(n)
    ctx.precompute_groups(lens, ids, kc, vc)
    again = cache(n)
    ctx.precompute_groups(lens, ids, *again)
    torch.cuda.synchronize()
    assert torch.equal(kc, again[0]) and torch.equal(vc, again[1])
    for first, count in ((0, 300), (n - lens[-1], lens[-1])):
        k1, v1 = cache(count)
        ctx.precompute_group(ids[first:first + count], k1, v1)
        torch.cuda.synchronize()
        for l in range(2):
            ek = max_rel(to_np(kc[l, first:first + count]), to_np(k1[l]))
            ev = max_rel(to_np(vc[l, first:first + count]), to_np(v1[l]))
            print(n, "layer", l, "rows", first, count, "K %.2e V %.2e" % (ek, ev))
            assert ek < 2e-2 and ev < 2e-2


def test_hidden_rows_at_an_odd_address():
    """The residual of the output projection at an address that is no multiple of 4 bytes (3000 rows: large tiles otherwise)."""
    pb = Problem(ks.ModelShape(1, 2048, 16, 2, 128, 1024, 211, 1.0e6, 1e-6, "bf16"), [2950], 50, std=0.5 / np.sqrt(2048),
                 random_cache=True)
    ctx, pr = pb.context(), pb.prompt()
    x = torch.randn((3000, 2048), generator=torch.Generator().manual_seed(1)).to(torch.bfloat16).cuda()
    odd = torch.empty(x.numel() + 1, dtype=x.dtype, device="cuda")[1:].view(x.shape).copy_(x)
    outs = []
    for rows in (x, odd):
        out = torch.empty_like(x)
        kc, vc = pb.empty_cache()
        ctx.recompute_layer(pr, 0, [0], rows, out, kc[0], vc[0])
        torch.cuda.synchronize()
        outs.append(to_np(out) - to_np(x))
    assert np.isfinite(outs[0]).all() and max_rel(outs[1], outs[0]) < 2e-2


EDGES = [2304 + e for e in (1, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256)]


def _cuts(rows, columns, k):
    """Pieces along K of the last tiles of an XCD's share (1: whole), as the launch plans them."""
    per_xcd = -(-(-(-rows // 256) * (columns // 256)) // 8)
    rem = per_xcd % 32
    return max(1, min(16, 32 // rem, k // 64 // 4)) if rem else 1


# whole tiles: 13 columns of tiles for QKV, O and down (17 tiles per XCD: a second piece would not fit its 32 CUs); gate/up has
# whole tiles and one per XCD that is cut.  Cut ones: 12, 10 and 10 columns of tiles.
@pytest.mark.parametrize("heads,hidden,ffn,cuts", [(22, 3328, 3328, (1, 1, 13, 1)), (20, 2560, 4096, (2, 2, 4, 2))],
                         ids=["whole", "cut"])
def test_projections(heads, hidden, ffn, cuts):
    shape = ks.ModelShape(1, hidden, heads, 2, 128, ffn, 211, 1.0e6, 1e-6, "bf16")
    probe = LayerProbe(shape, EDGES[-1], seed=hidden)
    for n in EDGES:
        plan = tuple(_cuts(n, c, k) for c, k in ((shape.q_dim + 2 * shape.kv_dim, hidden), (hidden, shape.q_dim),
                                                 (2 * ffn, hidden), (hidden, ffn)))
        assert plan == cuts
        probe.check(n)
