"""A BFS engine that is never idle while its running queries are by turns much work
(replays with bottom-up nodes) and little (without): every result equals the
oracle's, on a symmetric arena and on a directed one."""
import numpy as np
import pytest

import oracle
from paper_2201_02789_amd import graphgen as gg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2201_02789_amd import dpo  # noqa: E402


def _one_way(g, seed):
    s = np.repeat(np.arange(g.n), g.degrees())
    keep = ((s < g.col_idx) == (((np.minimum(s, g.col_idx) * 31 + np.maximum(s, g.col_idx) + seed) % 7) < 4))
    rp = np.concatenate([[0], np.cumsum(np.bincount(s[keep], minlength=g.n))]).astype(np.int32)
    return gg.Graph(rp, g.col_idx[keep])


@pytest.mark.parametrize("directed", [False, True])
@pytest.mark.parametrize("steps", [1, 3])
def test_bursts_among_a_trickle(directed, steps):
    gs = [gg.rmat(16, 24, 5, perm_seed=6), gg.rmat(15, 24, 7, perm_seed=8), gg.rmat(10, 10, 1, perm_seed=2),
          gg.path_graph(400)]
    if directed:
        gs = [_one_way(g, k) for k, g in enumerate(gs[:3])] + gs[3:]
    ar, vbase = gg.pack_arena(gs)
    eng = dpo.Engine(dpo.DeviceArena(ar, vbase), "bfs", [dpo.Options(steps_per_replay=steps)], max_queries=64,
                     max_slots=1 << 21)
    rng = np.random.default_rng(9)
    # the path, at hundreds of levels, keeps the engine from becoming idle
    plan = [[3]] + [[0] * 10 + [1] * 8] + [[2]] * 12 + [[3, 0]] * 3 + [[0] * 14] + [[2, 3]] * 4 + [[1] * 20]
    outs, done = {}, set()
    for _ in range(20000):
        for k in (plan.pop(0) if plan else []):
            s = int(rng.choice(np.flatnonzero(gs[k].degrees()))) if k != 3 else 0
            t = torch.full((gs[k].n,), -9, dtype=torch.int32, device="cuda")
            outs[eng.submit(k, s, t)] = (k, s, t)
        rest = eng.step()
        done.update(eng.poll())
        if not plan and rest == (0, 0):
            break
    assert done == set(outs)
    for k, s, t in outs.values():
        assert np.array_equal(t.cpu().numpy(), oracle.bfs(gs[k], s)[0]), (k, s)
    eng.close()
