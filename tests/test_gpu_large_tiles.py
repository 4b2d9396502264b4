"""The 256x256 tiles of the GEMM at the edges of a last tile's rows: more and fewer than 64, 128 and 192 of them, one, and
none missing, through all four projections of a layer (the fused QKV epilogue with biases and unit-local positions, the
residual add, SwiGLU) and the next layer's keys and values.  The same units cached one by one go through other kernels,
which the oracle checks at their sizes; both round to bf16 at every step: 2e-2 of the largest value."""
import numpy as np
import pytest
import torch

import keep_synth as ks
from gpu_util import Problem, max_rel, to_np

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
