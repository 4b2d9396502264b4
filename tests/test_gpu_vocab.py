"""The vocabulary projection and the greedy choice at vocabularies of real size: past the 32768 logits that the choice's
workgroups cover in one step and the 262144 of one trip of its loop, against the oracle; and its rules: among equal
largest logits the lowest id, wherever the others lie, and a NaN only where there is nothing else."""
import numpy as np
import pytest
import torch

import keep_synth as ks
from oracle import keep_oracle as ko
from gpu_util import Problem, max_rel, to_np

pytestmark = pytest.mark.gpu

SHAPES = {"bf16": ks.ModelShape(1, 64, 1, 1, 128, 64, 300007, 1.0e6, 1e-6, "bf16"),
          "f32": ks.ModelShape(1, 64, 4, 2, 16, 64, 300007, 1.0e6, 1e-6, "f32")}


class Head:
    """A context and a hidden row whose first token depends on the vocabulary projection alone."""

    def __init__(self, storage):
        self.shape = SHAPES[storage]
        self.pb = Problem(self.shape, [4], 1, seed=3)
        self.ctx = self.pb.context(max_tokens=8)
        g = torch.Generator().manual_seed(5)
        dt = ks.torch_dtype(storage)
        self.fn = (1.0 + 0.1 * torch.randn(self.shape.hidden, generator=g)).to(dt)
        self.x = torch.randn(self.shape.hidden, generator=g).to(dt)
        self.lm = (0.05 * torch.randn(self.shape.vocab, self.shape.hidden, generator=g)).to(dt)
        self.kc = torch.zeros((1, 8, self.shape.n_kv_heads, self.shape.head_dim), dtype=dt, device="cuda")

    def first(self, lm):
        """(token, its logits) for the first rows of a vocabulary projection"""
        full = torch.zeros((self.shape.vocab, self.shape.hidden), dtype=lm.dtype)
        full[:lm.shape[0]] = lm
        lg = torch.full((1, self.shape.vocab), float("nan"), dtype=torch.float32, device="cuda")
        tok = self.ctx.decode(self.fn.cuda(), full.cuda(), self.x.cuda(), self.kc, self.kc.clone(), 4, 1, logits_out=lg)
        return tok[0], lg[0].cpu().numpy()


@pytest.fixture(scope="module", params=["bf16", "f32"])
def head(request):
    return Head(request.param)


def test_logits_match_oracle(head):
    tok, lg = head.first(head.lm)
    ref = ko.lm_logits(head.pb.sh, ks.to_numpy_f64(head.fn), ks.to_numpy_f64(head.lm), ks.to_numpy_f64(head.x)[None])[0]
    # bf16: the normalised row is stored with 2^-9 relative error; fp32: sums of 64 terms
    assert max_rel(lg, ref) < (2.0 ** -8 if head.shape.storage == "bf16" else 1e-5)
    assert tok == int(np.argmax(lg))


# (twins of the largest logit: neighbours, other workgroups, other steps of a workgroup, other trips of its loop, the ends)
@pytest.mark.parametrize("ids", [(0, 1), (7, 263), (255, 256), (300, 300 + 32768), (32767, 32768), (70000, 70001, 299),
                                 (262143, 262144), (5, 5 + 262144), (300006, 0), (300006,), (300005, 131072, 262150)])
def test_lowest_id_among_equal_logits(head, ids):
    lm = head.lm.clone()
    n = ko.lm_logits(head.pb.sh, ks.to_numpy_f64(head.fn), np.eye(head.shape.hidden), ks.to_numpy_f64(head.x)[None])[0]
    for i in ids:
        lm[i] = torch.from_numpy(n).to(lm.dtype)        # the normalised row itself: its logit is about 64
    tok, lg = head.first(lm)
    assert len({float(lg[i]) for i in ids}) == 1 and float(lg[ids[0]]) == float(lg.max())
    assert tok == min(ids)


def test_zero_logits_and_nan(head):
    assert head.first(torch.zeros_like(head.lm))[0] == 0
    lm = head.lm.clone()
    for i in (0, 17, 40000, 299999):
        lm[i] = float("nan")
    tok, lg = head.first(lm)
    assert np.isnan(lg[[0, 17, 40000, 299999]]).all() and tok == int(np.nanargmax(lg))
    tok, lg = head.first(torch.full_like(head.lm, float("nan")))
    assert np.isnan(lg).all() and tok == 0
