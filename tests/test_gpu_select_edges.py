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
