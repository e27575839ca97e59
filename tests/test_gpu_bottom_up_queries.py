"""Batches and serving engines whose queries go bottom-up on their wide levels:
every query equals the oracle, on symmetric arenas and on arenas where one
graph misses symmetry by one entry, with queries at different points of their
traversals, repeated queries and graphs too small to qualify."""
import numpy as np
import pytest

import oracle
from paper_2201_02789_amd import graphgen as gg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2201_02789_amd import dpo  # noqa: E402


def _graphs(broken):
    """Skewed, uniform, tiny, long and partly isolated graphs; `broken`: one
    directed entry of the third is missing."""
    gs = [gg.rmat(16, 16, 1, perm_seed=2), gg.rmat(9, 8, 3, perm_seed=4), gg.rmat(14, 30, 5, perm_seed=6),
          gg.erdos_renyi(20011, 300000, 7), gg.path_graph(260), gg.complete_graph(300),
          gg.from_edges(75, [(1, 2), (2, 3)])]
    if broken:
        g = gs[2]
        rp, col = g.row_ptr.copy(), np.delete(g.col_idx, g.m // 3)
        rp[rp > g.m // 3] -= 1
        gs[2] = gg.Graph(rp, col)
    return gs


@pytest.fixture(scope="module", params=[False, True], ids=["symmetric", "one-missing"])
def arena(request):
    gs = _graphs(request.param)
    ar, vbase = gg.pack_arena(gs)
    rng = np.random.default_rng(3)
    qs = []
    for _ in range(9):
        qs += [(k, int(rng.choice(np.flatnonzero(g.degrees())))) for k, g in enumerate(gs)]
    qs += [qs[0], qs[2]]
    return gs, dpo.DeviceArena(ar, vbase), qs, [oracle.bfs(gs[k], s)[0] for k, s in qs]


BOPTS = [dict(), dict(threshold=32, coarsen=1, child_block=128), dict(steps_per_replay=2, split_min=0),
         dict(agg=dpo.DPO_AGG_WAVE, threshold=8), dict(agg=dpo.DPO_AGG_BLOCK, split_min=1 << 30),
         dict(claim_hint=dpo.DPO_HINT_OFF)]


@pytest.mark.parametrize("o", BOPTS, ids=str)
def test_batch(arena, o):
    gs, da, qs, wants = arena
    opts = dpo.Options(**o)
    tot, slot0 = dpo.dpo_batch_slots(da, qs)
    ws = torch.full((dpo.dpo_batch_workspace_bytes(da, qs, opts),), 0xC3, dtype=torch.uint8, device="cuda")
    for _ in range(2):
        out = torch.full((tot,), -7, dtype=torch.int32, device="cuda")
        print("batch", o, flush=True)
        dpo.dpo_bfs_batch(da, qs, [opts], out, ws)
        host = out.cpu().numpy()
        for i, (k, s) in enumerate(qs):
            assert np.array_equal(host[slot0[i]:slot0[i] + gs[k].n], wants[i]), (i, k, s)
            assert (host[slot0[i] + gs[k].n:slot0[i + 1]] == -7).all()


@pytest.mark.parametrize("o", [dict(steps_per_replay=1), dict(steps_per_replay=2, threshold=32, coarsen=1),
                               dict(steps_per_replay=4, split_min=0)], ids=str)
def test_engine(arena, o):
    gs, da, qs, wants = arena
    eng = dpo.Engine(da, "bfs", [dpo.Options(**o)], max_queries=6, max_slots=130 * 1024,
                     workspace=None)
    for _ in range(2):  # idle in between
        outs, done, todo = {}, set(), list(zip(qs, wants))
        for _ in range(20000):
            for (k, s), want in todo[:2]:
                t = torch.full((gs[k].n,), -9, dtype=torch.int32, device="cuda")
                outs[eng.submit(k, s, t)] = (t, want, k, s)
            todo = todo[2:]
            running, waiting = eng.step()
            done.update(eng.poll())
            if not todo and running == 0 and waiting == 0:
                break
        done.update(eng.poll())
        assert done == set(outs)
        for t, want, k, s in outs.values():
            assert np.array_equal(t.cpu().numpy(), want), (o, k, s)
    eng.close()


def test_an_entry_that_leaves_its_graph_is_reported():
    """A symmetric pair of entries between two graphs of an arena."""
    gs = [gg.rmat(14, 16, 1, perm_seed=2), gg.rmat(14, 16, 8, perm_seed=9)]
    ar, vbase = gg.pack_arena(gs)
    u, v = gg.max_degree_vertex(gs[0]), int(vbase[1]) + gg.max_degree_vertex(gs[1])
    rp, col = ar.row_ptr.astype(np.int64), ar.col_idx
    for a, b in ((u, v), (v, u)):
        col = np.insert(col, rp[a + 1], b)
        rp[a + 1:] += 1
    da = dpo.DeviceArena(gg.Graph(rp.astype(np.int32), col.astype(np.int32)), vbase)
    qs = [(0, u), (1, 5), (0, 7)] * 20
    opts = dpo.Options()
    tot, _ = dpo.dpo_batch_slots(da, qs)
    out = torch.empty(tot, dtype=torch.int32, device="cuda")
    ws = torch.empty(dpo.dpo_batch_workspace_bytes(da, qs, opts), dtype=torch.uint8, device="cuda")
    with pytest.raises(dpo.DpoError) as e:
        dpo.dpo_bfs_batch(da, qs, [opts], out, ws)
    assert e.value.status == dpo.DPO_ERR_ARG


def test_engine_results_of_every_size_reach_unaligned_outputs():
    """Queries that finish together, of sizes around the copy's chunk (4,096
    slots), into outputs 4 bytes past a 16-byte boundary; nothing is written
    past their ends."""
    sizes = [1, 2, 63, 4095, 4096, 4097, 8193]
    gs = [gg.path_graph(2) if n == 2 else gg.star_graph(n) if n > 2 else gg.from_edges(1, []) for n in sizes]
    ar, vbase = gg.pack_arena(gs)
    da = dpo.DeviceArena(ar, vbase)
    eng = dpo.Engine(da, "bfs", [dpo.Options()], max_queries=16, max_slots=1 << 16)
    outs = []
    for k, n in enumerate(sizes):
        buf = torch.full((n + 9,), -5, dtype=torch.int32, device="cuda")
        outs.append(buf)
        eng.submit(k, n - 1, buf[1:n + 1])
    for _ in range(100):
        if eng.step() == (0, 0):
            break
    assert len(eng.poll()) == len(sizes)
    for k, n in enumerate(sizes):
        host = outs[k].cpu().numpy()
        assert np.array_equal(host[1:n + 1], oracle.bfs(gs[k], n - 1)[0]), n
        assert host[0] == -5 and (host[n + 1:] == -5).all(), n
    eng.close()
