"""The selection over several launches (many candidates), bit-exact against the oracle around the line where it begins:
sets of more and fewer members than a block of the propagation (112 rows), of one member, sets that repeat before the last
selection, both budgets and both propagation readings, through both entry points; and as many selections as a caller may
ask for, on sets that repeat before and behind the point where one workgroup goes on alone."""
import numpy as np
import pytest
import torch

import keep_synth as ks
from gpu_util import Problem
from oracle import keep_oracle as ko
from paper_2602_23592_amd import binding as kb

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    shape = ks.ModelShape(2, 64, 4, 2, 16, 96, 97, 1.0e4, 1e-6, "f32")
    return Problem(shape, [4] * 8, 2, seed=2, random_cache=True).context(max_groups=1700)


@pytest.mark.parametrize("m", [899, 900, 961, 1601])
@pytest.mark.parametrize("kind", ["random", "ties", "settled"])
def test_selection(ctx, m, kind):
    rng = np.random.default_rng(m)
    glen = [int(v) for v in rng.integers(1, 200, size=m)]
    groups = list(range(m))
    S = np.tril(rng.random((m + 1, m)) * np.exp(rng.standard_normal(m)), -1).astype(np.float32)
    if kind == "ties":
        S = (np.round(S * 2) / 2).astype(np.float32)
        S[m // 3] = 0.0
    elif kind == "settled":                   # memories ignore each other: the second selection repeats the first
        S[:m] = 0.0
    d = [torch.tensor(v, dtype=dt, device="cuda") for v, dt in ((S, torch.float32), (groups, torch.int32), (glen, torch.int32))]
    for sources in (kb.KEEP_SOURCES_QUERY_AND_SET, kb.KEEP_SOURCES_SET_ONLY):
        ctx.set_option(kb.KEEP_OPT_PROPAGATION_SOURCES, sources)
        for mode, ratio, hops in ((0, 1.5 / m, 3), (0, 0.125, 2), (0, 0.3, 4), (1, 0.1, 3), (1, 0.55, 2), (0, 0.2, 1)):
            want, runs = ko.select_multihop(S, groups, glen, ratio, hops, mode, drop_query=sources == kb.KEEP_SOURCES_SET_ONLY)
            got, got_runs = ctx.select_groups(S, groups, glen, ratio, hops, mode)
            assert got == want and got_runs == runs, (mode, ratio, hops, sources)
            res = torch.full((m + 2,), -1, dtype=torch.int32, device="cuda")
            kb.select_groups_static(*d, int(sum(glen)), ratio, hops, mode, sources, res)
            r = res.cpu().numpy()
            assert r[0] == len(want) and r[1] == runs and r[2:2 + r[0]].tolist() == want, (mode, ratio, hops, sources)
    ctx.set_option(kb.KEEP_OPT_PROPAGATION_SOURCES, kb.KEEP_SOURCES_QUERY_AND_SET)


def _chain(m, last):
    """Memory a speaks of a + 1 alone, the three from `last` on of each other in turn: a set of three moves on by one memory
    per selection and repeats when it has reached the three."""
    S = np.zeros((m + 1, m), np.float32)
    S[m] = 1e-3
    S[m, :3] = 2e-3
    S[np.arange(m - 1), np.arange(1, m)] = 1.0
    S[last + 2] = 0.0
    S[last + 2, last] = 1.0
    return S


@pytest.mark.parametrize("m", [900, 2048, 3000])
@pytest.mark.parametrize("last", [0, 4, 6, 7, 12, 30])
def test_fixed_point(ctx, m, last):
    """Large `hops` ask for the set that repeats: it is found after last + 2 selections, whatever they are."""
    S, groups, glen = _chain(m, last), list(range(m)), [2] * m
    d = [torch.tensor(v, dtype=dt, device="cuda") for v, dt in ((S, torch.float32), (groups, torch.int32), (glen, torch.int32))]
    for hops in (1, last + 1, last + 2, last + 3, 100000, 2 ** 31 - 1):
        want, runs = [min(hops - 1, last) + i for i in range(3)], min(hops, last + 2)
        if m == 900:
            assert (want, runs) == ko.select_multihop(S, groups, glen, 3 / m, min(hops, last + 3), 0)
        for mode, ratio in ((0, 3 / m), (1, 6 / (2 * m))):          # three memories, or their six tokens
            if m <= 1700:
                got, got_runs = ctx.select_groups(S, groups, glen, ratio, hops, mode)
                assert got == want and got_runs == runs, (hops, mode)
            res = torch.full((m + 2,), -1, dtype=torch.int32, device="cuda")
            kb.select_groups_static(*d, 2 * m, ratio, hops, mode, kb.KEEP_SOURCES_QUERY_AND_SET, res)
            r = res.cpu().numpy()
            assert r[0] == 3 and r[1] == runs and r[2:5].tolist() == want, (hops, mode)


def test_fixed_point_in_a_graph(ctx):
    """A captured call with a large `hops` holds few launches, and a replay finds what an eager call finds."""
    m = 1000
    groups = torch.arange(m, dtype=torch.int32, device="cuda")
    glen = torch.full((m,), 2, dtype=torch.int32, device="cuda")
    S = torch.zeros((m + 1, m), device="cuda")
    res = torch.full((m + 2,), -1, dtype=torch.int32, device="cuda")
    call = lambda stream: kb.select_groups_static(S, groups, glen, 2 * m, 3 / m, 2 ** 31 - 1, 0, kb.KEEP_SOURCES_QUERY_AND_SET,
                                                  res, stream)
    stream = torch.cuda.Stream()
    S.copy_(torch.from_numpy(_chain(m, 3)))
    call(stream)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        call(stream)
    for last in (2, 20, 0, 7):
        S.copy_(torch.from_numpy(_chain(m, last)))
        res.fill_(-1)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert res[:5].tolist() == [3, last + 2, last, last + 1, last + 2]
