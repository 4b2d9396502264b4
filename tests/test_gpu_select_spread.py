"""The selection over several launches (many candidates), bit-exact against the oracle around the line where it begins:
sets of more and fewer members than a block of the propagation (112 rows), of one member, sets that repeat before the last
selection, both budgets and both propagation readings, through both entry points."""
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
