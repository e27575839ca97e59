"""BFS level steps whose frontier is spread over the grid in virtual blocks of
fewer than 256 entries: levels equal the oracle for frontiers around the sizes
where the block halves, at every granularity, with a participant threshold,
with and without counters (which keep full blocks)."""
import numpy as np
import pytest

import oracle
from paper_2201_02789_amd import graphgen as gg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2201_02789_amd import dpo  # noqa: E402


def _fan(parents):
    """Directed: one root, `parents` vertices of degrees 0 to 144 (every 97th
    of degree 1200), whose targets overlap; slots just above the frontier."""
    i = np.arange(parents)
    deg = np.where(i % 97 == 0, 1200, i % 37 * 4)
    src = np.repeat(i, deg)
    j = np.arange(len(src)) - np.repeat(np.cumsum(deg) - deg, deg)
    targets = 2 * parents + 9
    dst = 1 + parents + (src * 5 + j * 131) % targets
    e = np.concatenate([np.stack([np.zeros_like(i), 1 + i], 1), np.stack([1 + src, dst], 1)])
    return gg.from_edges(1 + parents + targets, e, symmetric=False)


OPTS = [dpo.Options(threshold=16, coarsen=1, child_block=64, agg=a, agg_threshold=t, claim_hint=h)
        for a, t, h in ((dpo.DPO_AGG_NONE, 0, dpo.DPO_HINT_OFF), (dpo.DPO_AGG_WAVE, 3, dpo.DPO_HINT_OFF),
                        (dpo.DPO_AGG_WAVE, 0, dpo.DPO_HINT_ON), (dpo.DPO_AGG_BLOCK, 4, dpo.DPO_HINT_OFF),
                        (dpo.DPO_AGG_MULTIBLOCK, 0, dpo.DPO_HINT_OFF),
                        (dpo.DPO_AGG_MULTIBLOCK, 0, dpo.DPO_HINT_ON), (dpo.DPO_AGG_GRID, 0, dpo.DPO_HINT_OFF))]
OPTS += [dpo.Options(threshold=100000, serial_wave=s) for s in (0, 1)] + [dpo.Options.flat()]


@pytest.mark.parametrize("parents", [511, 2047, 4097, 8191, 8193, 16384, 16385, 32769, 65537])
def test_spread_frontiers_match_oracle(parents):
    g = _fan(parents)
    dg = dpo.DeviceGraph.from_host(g)
    want = oracle.bfs(g, 0)[0]
    out = torch.empty(g.n, dtype=torch.int32, device="cuda")
    for o in OPTS:
        print(parents, o.label(), flush=True)
        ws = dpo.alloc_workspace(dg, o)
        ws.fill_(0xA5)
        for stats in (False, True):  # with counters: blocks of 256
            out.fill_(-7)
            dpo.dpo_bfs(dg, 0, o, out, ws, stats=stats)
            assert np.array_equal(out.cpu().numpy(), want), (o.label(), stats)
