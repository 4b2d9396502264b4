"""One layer of keep_recompute_layer, projection by projection, against plain torch in 64 bits on the same device.

A whole layer's output hides its parts: the residual stream is several times what a projection adds to it, and a wrong tile
of 16 columns or a lost slice of K is a few percent of one projection.  Here the hidden rows are small beside the updates,
the layer runs once without its FFN (wdown = 0) and once without its attention's output (wo = 0), and every product is
compared in blocks of 16 x 16 values, the tiles the matrix instructions write.

Tolerance: every value has gone through at most six roundings to bfloat16 on its way from the compared product's inputs,
each 2^-9 / sqrt(3) of a value on average (2-norm), together 2.8e-3 (and half as much again behind
SwiGLU, which multiplies two of them); a block of 256 values scatters little around that, a block at the edge, of 16 values,
up to twice it.  What a test must see is larger: 16 columns of 27 648 in front of the down
projection are 2.4e-2 of its outputs, a stale 32-deep product of 864 is 3.4e-2 of its block.  The attention is looked at for
the queries' sake alone (16 wrong columns change it by 0.4): what a score of order one, or of several, adds to each weight's
rounding is allowed for with four times as much."""
import torch

import keep_synth as ks

TOL, ATTENTION_TOL = 1e-2, 4e-2
PAST = 3            # cached rows in front of the recomputed ones


def rmsnorm(x, w, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * w


def rotate(x, pos, theta):
    half = x.shape[-1] // 2
    freq = theta ** (-2.0 * torch.arange(half, device=x.device, dtype=x.dtype) / x.shape[-1])
    ang = pos.to(x.dtype)[:, None] * freq
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    return torch.cat([x[..., :half] * c - x[..., half:] * s, x[..., half:] * c + x[..., :half] * s], -1)


def qkv(s, w, x, pos):
    h = rmsnorm(x, w["ln1"], s.rms_eps)
    q, k, v = (torch.mm(h, w[m].T).add_(w[b]).view(len(x), -1, s.head_dim) for m, b in (("wq", "bq"), ("wk", "bk"), ("wv", "bv")))
    return rotate(q, pos, s.rope_theta), rotate(k, pos, s.rope_theta), v


def attention(s, q, k, v, pos):
    o = torch.empty_like(q)
    hidden = torch.arange(len(k), device=q.device)[None] > pos[:, None]
    for h in range(s.n_q_heads):
        kv = h // (s.n_q_heads // s.n_kv_heads)
        sc = torch.mm(q[:, h], k[:, kv].T.contiguous()) / s.head_dim ** 0.5
        o[:, h] = torch.mm(torch.softmax(sc.masked_fill_(hidden, -float("inf")), -1), v[:, kv].contiguous())
    return o


def ffn(s, w, x):
    h = rmsnorm(x, w["ln2"], s.rms_eps)
    g = torch.mm(h, w["wgate"].T)
    return torch.mm(g * torch.sigmoid(g) * torch.mm(h, w["wup"].T), w["wdown"].T)


def block_err(got, ref):
    """Largest 2-norm of the difference over a block of 16 x 16 values, over the block's own or, where that is small, half of
    what a block has on average (at the edges, where a block may hold 16 values, all of it)."""
    got, ref = (t.reshape(len(t), -1).to(torch.float64) for t in (got, ref))
    pad = (0, -ref.shape[1] % 16, 0, -ref.shape[0] % 16)

    def blocks(t):
        t = torch.nn.functional.pad(t, pad)
        return t.view(t.shape[0] // 16, 16, t.shape[1] // 16, 16).sum((1, 3))

    size = blocks(torch.ones_like(ref))
    floor = (ref * ref).mean() * size * torch.where(size == 256, 0.25, 1.0)
    e = (blocks((got - ref) ** 2) / torch.maximum(blocks(ref * ref), floor)).max()
    return float(e.sqrt())


def weights(s, seed, device):
    g = torch.Generator(device=device).manual_seed(seed)
    w = {}
    for name, size in ks.layer_weight_shapes(s).items():
        t = torch.randn(size, generator=g, device=device)
        # (queries four times as large: scores of order one)
        t = 1 + 0.1 * t if name.startswith("ln") else t * ((2.0 if name == "wq" else 0.5) / size[1] ** 0.5)
        w[name] = t.to(torch.bfloat16)
    for name, size in (("bq", s.q_dim), ("bk", s.kv_dim), ("bv", s.kv_dim)):
        w[name] = (0.1 * torch.randn(size, generator=g, device=device)).to(torch.bfloat16)
    return w


class LayerProbe:
    """One context of a one-layer model; check(n) runs the layer on n rows behind a short cached memory."""

    def __init__(self, shape, max_rows, seed=0):
        from paper_2602_23592_amd import KeepContext
        self.s, self.w = shape, weights(shape, seed, "cuda")
        self.embed = torch.zeros((shape.vocab, shape.hidden), dtype=torch.bfloat16, device="cuda")
        self.ctx = KeepContext(shape, [self.w], self.embed, max_rows + PAST, 1)
        assert self.ctx.uses_mfma

    def _layer(self, prompt, x, n, without):
        s, kept = self.s, self.w[without].clone()
        self.w[without].zero_()
        k, v = (torch.zeros((n + PAST, s.n_kv_heads, s.head_dim), dtype=torch.bfloat16, device="cuda") for _ in range(2))
        out = torch.full_like(x, float("nan"))
        self.ctx.recompute_layer(prompt, 0, [], x, out, k, v)
        o = torch.from_numpy(self.ctx.read_layer_state(0, n)).cuda()
        self.w[without].copy_(kept)
        return out, k, v, o

    def check(self, n):
        from paper_2602_23592_amd import KeepPrompt
        s = self.s
        g = torch.Generator(device="cuda").manual_seed(n)
        x = (0.02 * torch.randn((n, s.hidden), generator=g, device="cuda")).to(torch.bfloat16)
        past = [torch.randn((PAST, s.n_kv_heads, s.head_dim), generator=g, device="cuda").to(torch.bfloat16) for _ in range(2)]
        prompt = KeepPrompt([PAST], n, ks.make_token_ids(n + PAST, s.vocab, n), [[past[0]]], [[past[1]]], 1)
        w = {name: t.to(torch.float64) for name, t in self.w.items()}
        x64, pos = x.to(torch.float64), torch.arange(PAST, PAST + n, device="cuda")

        out, k, v, o = self._layer(prompt, x, n, "wdown")
        q_ref, k_ref, v_ref = qkv(s, w, x64, pos)
        errs = {"k": block_err(k[PAST:], k_ref), "v": block_err(v[PAST:], v_ref)}
        errs["attention"] = block_err(o, attention(s, q_ref, k.to(torch.float64), v.to(torch.float64), pos))
        errs["o"] = block_err(out.to(torch.float64) - x64, torch.mm(o.to(torch.float64).view(n, -1), w["wo"].T))
        out = self._layer(prompt, x, n, "wo")[0]
        errs["ffn"] = block_err(out.to(torch.float64) - x64, ffn(s, w, x64))
        print(n, " ".join("%s %.1e" % e for e in errs.items()), flush=True)
        assert all(e < (ATTENTION_TOL if part == "attention" else TOL) for part, e in errs.items()), (n, errs)
