"""Attention and scores of the generic family at every kind of head width (one instance per multiple of 16, up to 256; from
144 on without the next key tile in registers), query rows per KV head that do not fill a tile of 16, and key ranges
shorter and longer than the eight waves' tiles, against the oracle: fp32 1e-4, bf16 2e-2 of the largest value."""
import numpy as np
import pytest
import torch

import keep_synth as ks
from gpu_util import Problem, layer_state_err, max_rel, to_np
from oracle import keep_oracle as ko

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dh,heads,kv,storage", [(16, 4, 4, "f32"), (32, 7, 1, "f32"), (48, 6, 2, "f32"), (80, 3, 3, "f32"),
                                                 (96, 4, 2, "bf16"), (112, 2, 2, "f32"), (128, 5, 1, "f32"),
                                                 (144, 2, 1, "f32"), (208, 3, 1, "bf16"), (224, 2, 1, "f32"),
                                                 (256, 2, 2, "f32")])
def test_layer(dh, heads, kv, storage):
    tol = 1e-4 if storage == "f32" else 2e-2
    shape = ks.ModelShape(1, 64, heads, kv, dh, 96, 97, 1.0e4, 1e-6, storage)
    glen, lq = [1, 15, 16, 17, 130, 3], 5
    pb = Problem(shape, glen, lq, seed=dh, std=0.1, bias=True)
    ctx, pr = pb.context(), pb.prompt()
    for groups in (list(range(len(glen))), [1, 4], []):
        n_rows = pr.n_rows(groups)
        x_t = ks.make_random_rows(n_rows, shape.hidden, storage, seed=dh + len(groups))
        kh, vh = pb.oracle_joined_cache(0)
        probe = {}
        xo, lse, S_ref = ko.selective_layer(pb.sh, pb.layers[0], ks.to_numpy_f64(x_t), groups, glen, lq, kh, vh, probe=probe)
        kc, vc = pb.empty_cache(1)
        x_out = torch.empty_like(x_t, device="cuda")
        ctx.recompute_layer(pr, 0, groups, x_t.cuda(), x_out, kc[0], vc[0])
        eo, el = layer_state_err(ctx, n_rows, probe, lse)
        assert eo < tol and el < tol, (groups, eo, el)
        assert max_rel(to_np(x_out), xo) < tol
        if groups:
            _, _, S = ctx.score_groups(pr, 0, groups, 0.5, 2)
            assert np.abs(S - S_ref).max() <= tol * S_ref.max()


@pytest.mark.parametrize("glen,lq,heads", [([70, 1], 20, 4), ([33], 1, 7), ([4] * 256, 5, 3), ([5, 2] * 120, 40, 6)],
                         ids=["long", "one", "short", "ragged"])
def test_scores(glen, lq, heads):
    """Few long memories, whose rows mostly lie in the block they would look at, and so many short ones that a block is one
    wave's (4096 pairs of 16 rows and a block)."""
    shape = ks.ModelShape(1, 64, heads, 1, 32, 96, 97, 1.0e4, 1e-6, "f32")
    pb = Problem(shape, glen, lq, seed=lq, std=0.1, bias=True, random_cache=True)
    ctx, pr = pb.context(), pb.prompt()
    for groups in (list(range(len(glen))), [0], list(range(0, len(glen), 2))):
        n_rows = pr.n_rows(groups)
        x_t = ks.make_random_rows(n_rows, shape.hidden, "f32", seed=len(groups))
        kh, vh = pb.oracle_joined_cache(0)
        _, _, want = ko.selective_layer(pb.sh, pb.layers[0], ks.to_numpy_f64(x_t), groups, glen, lq, kh, vh)
        kc, vc = pb.empty_cache(1)
        ctx.recompute_layer(pr, 0, groups, x_t.cuda(), torch.empty_like(x_t, device="cuda"), kc[0], vc[0])
        _, _, S = ctx.score_groups(pr, 0, groups, 0.5, 2)
        assert np.abs(S - want).max() <= 1e-4 * want.max()


@pytest.mark.parametrize("dh,storage", [(16, "f32"), (96, "bf16"), (112, "f32"), (256, "f32")])
def test_values_that_are_not_finite_reach_the_rows_that_see_them(dh, storage):
    """Rows of two memories and the instruction share a tile of 16 query rows; the memory between them, which is not
    recomputed, holds infinities and a NaN in one key's V.  The rows in front of it are as without them, bit for bit, and so
    is every other dimension behind it."""
    shape = ks.ModelShape(1, 64, 2, 2, dh, 96, 97, 1.0e4, 1e-6, storage)
    pb = Problem(shape, [5, 20, 6], 4, seed=dh, std=0.1, bias=True)
    x = ks.make_random_rows(15, shape.hidden, storage, seed=dh).cuda()
    plant = {0: float("inf"), 3: float("-inf"), dh - 1: float("nan")}
    outs, states = [], []
    for values in ({}, plant):
        for d, value in values.items():
            pb.vb_d[0][1][3, 1, d] = value
        ctx, pr = pb.context(kernel_path=1), pb.prompt()
        assert not ctx.uses_mfma
        kc, vc = pb.empty_cache(1)
        x_out = torch.empty_like(x)
        ctx.recompute_layer(pr, 0, [0, 2], x, x_out, kc[0], vc[0])
        outs.append(to_np(x_out))
        states.append(ctx.read_layer_state(0, 15).astype(np.float64).reshape(15, 2, dh))
    assert np.isfinite(outs[0]).all()
    assert np.array_equal(outs[1][:5], outs[0][:5])
    want = states[0].copy()
    for d, value in plant.items():
        want[5:, 1, d] = value
    assert np.array_equal(states[1], want, equal_nan=True)


@pytest.mark.parametrize("dh,storage", [(16, "f32"), (144, "bf16")])
def test_units_do_not_see_each_other(dh, storage):
    """Units cached in one pass, several in a tile of query rows: one whose token has no finite embedding leaves the others'
    keys and values as they are, bit for bit."""
    shape = ks.ModelShape(2, 64, 2, 1, dh, 96, 97, 1.0e4, 1e-6, storage)
    lens = [3, 4, 9, 2]
    pb = Problem(shape, lens, 1, seed=3, std=0.1, bias=True)
    ids = np.arange(sum(lens), dtype=np.int32)
    rows = []
    for bad in (False, True):
        if bad:
            pb.embed_d[4] = float("nan")            # the second token of the second unit
        ctx = pb.context(kernel_path=1)
        k, v = (torch.zeros((2, sum(lens), 1, dh), dtype=pb.embed_d.dtype, device="cuda") for _ in range(2))
        ctx.precompute_groups(lens, ids, k, v)
        torch.cuda.synchronize()
        rows.append((to_np(k), to_np(v)))
    others = [r for r in range(sum(lens)) if not 4 <= r < 7]
    for clean, got in zip(*rows):
        assert np.isfinite(clean).all() and np.array_equal(got[:, others], clean[:, others])
        assert np.isnan(got[1, 4:7]).all()          # the token and those behind it in its unit
