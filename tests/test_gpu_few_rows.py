"""Launches of up to 16 rows (the weight-streaming projections) at the edges of their tiles, against the oracle: a unit
cached on its own and one decoded token, for row counts around the limit and for widths that leave waves without a
step (K < 512), a step more on some waves than on others, and part-filled tiles of weight rows."""
import numpy as np
import pytest
import torch

import keep_synth as ks
from oracle import keep_oracle as ko
from gpu_util import Problem, max_rel, to_np
from test_gpu_decode import head_weights
from test_gpu_int4 import Int4Problem

pytestmark = pytest.mark.gpu

# 7 query heads on 1 KV head, K = 448 (7 steps for 8 waves), FFN 1344 (21 steps); and K = 8256 (129 steps, a row of
# activations beyond the two vectors a thread keeps in registers) with tiles of 9 units
NARROW = ks.ModelShape(2, 448, 7, 1, 128, 1344, 1031, 1.0e6, 1e-6, "bf16")
WIDE = ks.ModelShape(2, 8256, 2, 1, 128, 320, 211, 1.0e6, 1e-6, "bf16")
# an FFN wide enough that workgroups own tiles of 17 units (two MFMA tiles, and on the 4-bit form rows of two storage
# blocks) and more than one of them, and so many heads that a QKV tile holds 16 column pairs; and the same for the output
# and down projections
FAN = ks.ModelShape(2, 512, 28, 4, 128, 8320, 211, 1.0e6, 1e-6, "bf16")
# wide enough for the ring of stages from 8 rows on, which takes no weights at odd addresses
RING = ks.ModelShape(2, 5120, 40, 8, 128, 5376, 211, 1.0e6, 1e-6, "bf16")
WIDE4 = ks.ModelShape(2, 8320, 2, 1, 128, 384, 211, 1.0e6, 1e-6, "bf16")


def _odd(t):
    """The same matrix at an address that is no multiple of 4 bytes."""
    return torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")[1:].view(t.shape).copy_(t)


@pytest.mark.parametrize("shape,n,aligned", [(s, n, True) for s in (NARROW, WIDE) for n in (1, 2, 15, 16, 17)] +
                         [(FAN, n, True) for n in (1, 2, 9, 16)] + [(FAN, n, False) for n in (1, 9)] + [(RING, n, False) for n in (10, 16)],
                         ids=lambda v: "h%d" % v.hidden if isinstance(v, ks.ModelShape) else str(v))
def test_few_rows_match_oracle(shape, n, aligned):
    pb = Problem(shape, [n], 1, seed=n, std=0.5 / np.sqrt(shape.hidden), bias=True)
    if not aligned:
        for w in pb.layers_d:
            for name in ks.INT4_MATS:           # the seven projections
                w[name] = _odd(w[name])
    ctx = pb.context(max_tokens=n + 2)
    assert ctx.uses_mfma
    L = shape.n_layers
    kc = torch.zeros((L, n + 1, shape.n_kv_heads, shape.head_dim), dtype=torch.bfloat16, device="cuda")
    vc = torch.zeros_like(kc)
    k1, v1 = kc[:, :n].contiguous(), vc[:, :n].contiguous()
    ctx.precompute_group(pb.ids[:n], k1, v1)
    torch.cuda.synchronize()
    for l in range(L):      # (the oracle made the same unit's caches for the problem)
        ek, ev = max_rel(to_np(k1[l]), pb.kb[l][0]), max_rel(to_np(v1[l]), pb.vb[l][0])
        print(n, "layer", l, "K %.2e V %.2e" % (ek, ev))
        assert ek < 2e-2 and ev < 2e-2

    # one token decoded behind the unit, on the oracle's caches
    for l in range(L):
        kc[l, :n], vc[l, :n] = pb.kb_t[l][0].cuda(), pb.vb_t[l][0].cuda()
    fn, lm = head_weights(shape)
    x = torch.randn(shape.hidden, generator=torch.Generator().manual_seed(n)).to(torch.bfloat16)
    lg = torch.empty((2, shape.vocab), dtype=torch.float32, device="cuda")
    toks = ctx.decode(fn.cuda(), lm.cuda() if aligned else _odd(lm), x.cuda(), kc, vc, n, 2, logits_out=lg)
    pad = lambda rows: [np.concatenate([r[0], np.zeros((1,) + r[0].shape[1:])]) for r in rows]
    kr, vr = pad(pb.kb), pad(pb.vb)
    _, ref = ko.greedy_decode(pb.sh, pb.layers, pb.embed, ks.to_numpy_f64(fn), ks.to_numpy_f64(lm), ks.to_numpy_f64(x),
                              kr, vr, n, 2, forced_tokens=toks)
    for t in range(2):
        e = max_rel(to_np(lg)[t], ref[t])
        print(n, "token", t, "logits %.2e" % e)
        assert e < 2e-2
    for l in range(L):
        assert max_rel(to_np(kc[l, n]), kr[l][n]) < 2e-2 and max_rel(to_np(vc[l, n]), vr[l][n]) < 2e-2


@pytest.mark.parametrize("shape", [FAN, WIDE4], ids=lambda v: "h%d" % v.hidden)
@pytest.mark.parametrize("n", [1, 2, 9, 16, 17])
def test_few_rows_int4_match_oracle(shape, n):
    """The same on the 4-bit form of the projections (17 rows: the kernel behind the line)."""
    pb = Int4Problem(shape, std=0.5 / np.sqrt(shape.hidden), seed=n)
    L = shape.n_layers
    ids = ks.make_token_ids(n, shape.vocab, n)
    ctx = pb.context(n + 2, 1)
    k, v = (torch.zeros((L, n, shape.n_kv_heads, shape.head_dim), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    ctx.precompute_group(ids, k, v)
    kb, vb = ko.precompute_group_caches(pb.sh, pb.layers, pb.embed, ids, [n])
    for l in range(L):
        ek, ev = max_rel(to_np(k[l]), kb[l][0]), max_rel(to_np(v[l]), vb[l][0])
        print(n, "layer", l, "K %.2e V %.2e" % (ek, ev))
        assert ek < 2e-2 and ev < 2e-2
    # one token decoded behind the unit
    x = torch.randn(shape.hidden, generator=torch.Generator().manual_seed(n)).to(torch.bfloat16)
    kc, vc = (torch.cat([t, torch.zeros_like(t[:, :1])], dim=1) for t in (k, v))
    kr, vr = ([to_np(t[l]) for l in range(L)] for t in (kc, vc))
    lg = torch.empty((2, shape.vocab), dtype=torch.float32, device="cuda")
    toks = ctx.decode(pb.fn_t.cuda(), pb.lm_t.cuda(), x.cuda(), kc, vc, n, 2, logits_out=lg)
    _, ref = ko.greedy_decode(pb.sh, pb.layers, pb.embed, ks.to_numpy_f64(pb.fn_t), ks.to_numpy_f64(pb.lm_t),
                              ks.to_numpy_f64(x), kr, vr, n, 2, forced_tokens=toks)
    for t in range(2):
        assert max_rel(to_np(lg)[t], ref[t]) < 2e-2
    for l in range(L):
        assert max_rel(to_np(kc[l, n]), kr[l][n]) < 2e-2 and max_rel(to_np(vc[l, n]), vr[l][n]) < 2e-2


@pytest.mark.parametrize("form", ["bf16", "int4"])
@pytest.mark.parametrize("hidden", [76800, 76928])
def test_longest_row_in_lds_and_longer(form, hidden):
    """One decoded token at the longest row of activations that fits LDS and at the next longer one, with a vocabulary
    that fills no last tile."""
    shape = ks.ModelShape(1, hidden, 1, 1, 128, 128, 97, 1.0e6, 1e-6, "bf16")
    std = 0.5 / np.sqrt(hidden)
    if form == "int4":
        pb = Int4Problem(shape, std=std)
        ctx, fn, lm = pb.context(4, 1), pb.fn_t, pb.lm_t
    else:
        pb = Problem(shape, [2], 1, std=std)
        ctx = pb.context(max_tokens=4)
        fn, lm = head_weights(shape)
    g = torch.Generator().manual_seed(2)
    x = torch.randn(hidden, generator=g).to(torch.bfloat16)
    kc, vc = (torch.randn((1, 4, 1, 128), generator=g).to(torch.bfloat16).cuda() for _ in range(2))
    kr, vr = [to_np(kc[0])], [to_np(vc[0])]
    lg = torch.full((2, shape.vocab), float("nan"), dtype=torch.float32, device="cuda")
    toks = ctx.decode(fn.cuda(), lm.cuda(), x.cuda(), kc, vc, 2, 2, logits_out=lg)
    _, ref = ko.greedy_decode(pb.sh, pb.layers, pb.embed, ks.to_numpy_f64(fn), ks.to_numpy_f64(lm), ks.to_numpy_f64(x),
                              kr, vr, 2, 2, forced_tokens=toks)
    for t in range(2):
        assert max_rel(to_np(lg)[t], ref[t]) < 2e-2
    assert max_rel(to_np(kc[0, 2]), kr[0][2]) < 2e-2 and max_rel(to_np(vc[0, 2]), vr[0][2]) < 2e-2
