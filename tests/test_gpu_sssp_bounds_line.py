"""SSSP bound bytes around the slot count from which they are kept, and in a
serving engine, whose queries take over the slots (and bytes) of earlier ones."""
import numpy as np
import pytest

import oracle
from paper_2201_02789_amd import graphgen as gg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2201_02789_amd import dpo  # noqa: E402

LINE = 3 << 19


@pytest.mark.parametrize("n", [LINE - 32, LINE - 31, LINE + 1])
@pytest.mark.parametrize("top", [20, 256, 1 << 27])
def test_distances_match_oracle(n, top):
    g = gg.erdos_renyi(n, 2 * n, 5)
    g = gg.Graph(g.row_ptr, g.col_idx, np.random.default_rng(7).integers(0, top, g.m).astype(np.uint32))
    want = oracle.dijkstra(g, 3)
    dg = dpo.DeviceGraph.from_host(g)
    for o in (dpo.Options(claim_hint=dpo.DPO_HINT_ON, split_min=0),
              dpo.Options(claim_hint=dpo.DPO_HINT_ON, threshold=4, agg=dpo.DPO_AGG_WAVE)):
        print(n, top, o.label(), flush=True)
        ws = dpo.alloc_workspace(dg, o)
        ws.fill_(0)  # bytes that rule everything out, unless the call sets them
        out = torch.full((n,), -7, dtype=torch.int32, device="cuda")
        dpo.dpo_sssp(dg, 3, o, out, ws)
        assert np.array_equal(dpo.as_uint32(out), want), o.label()


@pytest.mark.parametrize("steps", [1, 4])
def test_engine_queries_reuse_slots(steps):
    rng = np.random.default_rng(4)
    gs = []
    for k, (scale, top) in enumerate([(12, 3), (12, 1 << 20), (13, 256), (11, 1 << 27), (13, 2)]):
        g = gg.rmat(scale, 14, k, perm_seed=k + 5)
        gs.append(gg.Graph(g.row_ptr, g.col_idx, rng.integers(0, top, g.m).astype(np.uint32)))
    ar, vbase = gg.pack_arena(gs)
    da = dpo.DeviceArena(ar, vbase)
    opts = dpo.Options(steps_per_replay=steps, threshold=32, coarsen=1, split_min=2048)
    probe = dpo.Engine(da, "sssp", [opts], max_queries=4, max_slots=LINE)
    ws = torch.zeros(probe.ws.numel(), dtype=torch.uint8, device="cuda")
    probe.close()
    # four at a time, always in the pool's first slots
    eng = dpo.Engine(da, "sssp", [opts], max_queries=4, max_slots=LINE, workspace=ws)
    outs, done = {}, set()
    for i in range(40):
        k = int(rng.integers(len(gs)))
        s = int(gg.sample_sources(gs[k], 1, i)[0])
        t = torch.full((gs[k].n,), -9, dtype=torch.int32, device="cuda")
        outs[eng.submit(k, s, t)] = (k, s, t)
    for _ in range(20000):
        rest = eng.step()
        done.update(eng.poll())
        if rest == (0, 0):
            break
    assert done == set(outs)
    for k, s, t in outs.values():
        assert np.array_equal(dpo.as_uint32(t), oracle.dijkstra(gs[k], s)), (k, s)
    eng.close()
