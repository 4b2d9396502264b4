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
