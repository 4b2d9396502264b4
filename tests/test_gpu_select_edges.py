"""The selection at the edges of its parts, bit-exact against the oracle: candidate counts around the sort's powers of
two, the row totals' blocks (16 rows, 256 columns, 32 additions) and the walk's chunks of 64; lengths that make the
token walk pass over single memories, over most of a chunk, and over whole chunks; ties and negative zeros."""
import numpy as np
import pytest

import keep_synth as ks
from oracle import keep_oracle as ko
from gpu_util import Problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    shape = ks.ModelShape(2, 64, 4, 2, 16, 96, 97, 1.0e4, 1e-6, "f32")
    return Problem(shape, [4] * 8, 2, seed=2, random_cache=True).context(max_groups=2100)


@pytest.mark.parametrize("m", [1, 2, 3, 15, 16, 31, 33, 63, 64, 65, 127, 129, 255, 256, 257, 511, 513, 1023, 1024, 1025,
                               2047, 2049])
def test_selection_edges(ctx, m):
    rng = np.random.default_rng(m)
    groups = list(range(m))
    for lens in ("short", "mixed", "one_long"):
        glen = rng.integers(1, 4, size=m) if lens == "short" else np.exp(rng.uniform(0, 7, size=m)).astype(int) + 1
        if lens == "one_long":
            glen[:] = 5
            glen[rng.integers(0, m)] = 100000
        glen = [int(v) for v in glen]
        S = np.tril(rng.random((m + 1, m)), -1).astype(np.float32)
        if lens == "short":                     # ties, a memory nothing attends to, rows without mass
            S = (np.round(S * 4) / 4).astype(np.float32)
            S[:, m // 2] = -0.0
            S[m // 3] = 0.0
        for mode in (0, 1):
            for hops, ratio in ((1, 0.3), (3, 0.05), (4, 0.6)):
                want, runs = ko.select_multihop(S, groups, glen, ratio, hops, mode)
                got, got_runs = ctx.select_groups(S, groups, glen, ratio, hops, mode)
                assert got == want and got_runs == runs, (m, lens, mode, hops)


@pytest.mark.parametrize("m", [1, 2, 4, 9, 17, 40, 62, 63, 64])
def test_few_candidates(ctx, m):
    """Around the line below which one wave selects alone, through both entry points, with the query as a source of the
    propagation and without."""
    import torch
    from paper_2602_23592_amd import binding as kb
    rng = np.random.default_rng(100 + m)
    G = m + 3
    for trial in range(6):
        glen = [int(v) for v in (rng.integers(1, 90, size=G) if trial % 2 else np.exp(rng.uniform(0, 7, size=G)).astype(int) + 1)]
        groups = sorted(int(v) for v in rng.choice(G, size=m, replace=False))
        S = np.tril(rng.random((m + 1, m)), -1).astype(np.float32)
        if trial >= 4:                          # ties, rows without mass, a query that attends to nothing
            S = (np.round(S * 3) / 3).astype(np.float32)
            S[m] = 0.0 if trial == 5 else S[m]
        for sources in (kb.KEEP_SOURCES_QUERY_AND_SET, kb.KEEP_SOURCES_SET_ONLY):
            ctx.set_option(kb.KEEP_OPT_PROPAGATION_SOURCES, sources)
            for mode in (kb.KEEP_BUDGET_GROUP_COUNT, kb.KEEP_BUDGET_TOKENS):
                for hops, ratio in ((1, 0.3), (2, 0.5), (4, 0.15), (9, 0.7), (3, 1.0), (3, 0.0)):
                    want = ko.select_multihop(S, groups, glen, ratio, hops, mode, sources == kb.KEEP_SOURCES_SET_ONLY)
                    assert ctx.select_groups(S, groups, glen, ratio, hops, mode) == want, (m, trial, sources, mode, hops)
                    res = torch.full((m + 3,), -7, dtype=torch.int32, device="cuda")
                    kb.select_groups_static(torch.from_numpy(S).cuda(), torch.tensor(groups, dtype=torch.int32, device="cuda"),
                                            torch.tensor(glen, dtype=torch.int32, device="cuda"), sum(glen), ratio, hops,
                                            mode, sources, res)
                    out = res.cpu().tolist()
                    assert (out[2:2 + out[0]], out[1]) == want and out[m + 2] == -7, (m, trial, sources, mode, hops)
    ctx.set_option(kb.KEEP_OPT_PROPAGATION_SOURCES, kb.KEEP_SOURCES_QUERY_AND_SET)


@pytest.mark.parametrize("m", [9, 63, 64, 300])
def test_an_infinite_score(ctx, m):
    """An infinite score makes its candidate's importance inf / inf and every other one zero.  No importance is greater
    than a NaN, so the count budget takes the candidate beside the others' first k (ties by index); the token walk comes
    to it last."""
    rng = np.random.default_rng(m)
    glen = [int(v) for v in rng.integers(1, 9, size=m)]
    for b in (0, m // 2, m - 1):
        S = np.tril(rng.random((m + 1, m)), -1).astype(np.float32)
        S[m, b] = np.inf
        others = [i for i in range(m) if i != b]
        for ratio in (0.1, 0.6):
            got, _ = ctx.select_groups(S, list(range(m)), glen, ratio, 1, 0)
            assert got == sorted(others[:ko.budget_count(ratio, m, m)] + [b]), (m, b, ratio)
            left, want = ko.budget_tokens(ratio, sum(glen)), []
            for i in others + [b]:
                if glen[i] <= left:
                    want.append(i)
                    left -= glen[i]
            assert ctx.select_groups(S, list(range(m)), glen, ratio, 1, 1)[0] == sorted(want), (m, b, ratio)


def test_most_candidates():
    """4096 candidates through the entry point that allocates nothing, 6000 through a context: the most either takes."""
    import torch
    from paper_2602_23592_amd import binding as kb
    shape = ks.ModelShape(2, 64, 4, 2, 16, 96, 97, 1.0e4, 1e-6, "f32")
    big = Problem(shape, [4] * 8, 2, seed=2, random_cache=True).context(max_groups=6000)
    for m, mode in ((4096, 1), (6000, 0)):
        rng = np.random.default_rng(m)
        glen = [int(v) for v in rng.integers(1, 200, size=m)]
        S = np.tril(rng.random((m + 1, m), dtype=np.float32), -1)
        want = ko.select_multihop(S, list(range(m)), glen, 0.2, 2, mode)
        print(m, len(want[0]), "kept", flush=True)
        assert big.select_groups(S, list(range(m)), glen, 0.2, 2, mode) == want
        if m == 4096:
            res = torch.zeros(m + 2, dtype=torch.int32, device="cuda")
            ids, lens = (torch.tensor(v, dtype=torch.int32, device="cuda") for v in (list(range(m)), glen))
            kb.select_groups_static(torch.from_numpy(S).cuda(), ids, lens, sum(glen), 0.2, 2, mode, 0, res)
            out = res.cpu().tolist()
            assert (out[2:2 + out[0]], out[1]) == want
