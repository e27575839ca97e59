"""Single traversals without counters, the calls that run consecutive narrow
levels in one workgroup: results equal the oracle where that path begins, ends
and hands over (frontiers around what LDS holds, levels around its edge limit,
traversals longer than one launch's levels, bitmaps too large for LDS), with
found bytes and with the two shared copies, with a workspace and without."""
import numpy as np
import pytest

import oracle
from paper_2201_02789_amd import graphgen as gg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2201_02789_amd import dpo  # noqa: E402


def _stars(leaves, chain):
    """A path of `chain` vertices into a hub with `leaves` leaves, each leaf
    with one more vertex behind it."""
    hub = chain
    e = [(i, i + 1) for i in range(chain)]
    e += [(hub, hub + 1 + i) for i in range(leaves)]
    e += [(hub + 1 + i, hub + 1 + leaves + i) for i in range(leaves)]
    return gg.from_edges(hub + 1 + 2 * leaves, e)


GRAPHS = [
    ("one", lambda: gg.from_edges(1, []), 0),
    ("isolated", lambda: gg.from_edges(9, [(1, 2)]), 4),
    ("path", lambda: gg.path_graph(9001), 0),          # more levels than one launch runs
    ("cycle", lambda: gg.cycle_graph(1001), 7),
    ("complete", lambda: gg.complete_graph(300), 3),   # 89,700 edges: wide at level 1
    ("stars-7700", lambda: _stars(7700, 3), 0),
    ("stars-8191", lambda: _stars(8191, 2), 0),
    ("stars-8192", lambda: _stars(8192, 2), 0),
    ("stars-8193", lambda: _stars(8193, 2), 0),
    ("stars-8191-1", lambda: _stars(4095, 1), 0),
    ("stars-8193-1", lambda: _stars(4097, 1), 0),
    ("stars-131071", lambda: _stars(131071, 1), 0),
    ("stars-131073", lambda: _stars(131073, 1), 0),
    ("road", lambda: gg.road_like(150, 170, 3), 11),
    ("grid", lambda: gg.grid_graph(300, 211), 0),
    ("rmat16", lambda: gg.rmat(16, 16, 16, perm_seed=24), 5),
    ("er", lambda: gg.erdos_renyi(50001, 60000, 4), 1),
    ("no-lds-bitmap", lambda: gg.erdos_renyi(790001, 850000, 5), 3),
]
OPTS = [dpo.Options(), dpo.Options(threshold=16, coarsen=1, split_min=0, claim_hint=dpo.DPO_HINT_ON),
        dpo.Options(threshold=16, coarsen=1, split_min=2000, claim_hint=dpo.DPO_HINT_OFF),
        dpo.Options(threshold=0, agg=dpo.DPO_AGG_WAVE, claim_hint=dpo.DPO_HINT_ON)]


@pytest.mark.parametrize("name,make,src", GRAPHS, ids=[g[0] for g in GRAPHS])
def test_narrow_levels_match_oracle(name, make, src):
    g = gg.add_weights(make(), 9)
    dg = dpo.DeviceGraph.from_host(g)
    want, dwant = oracle.bfs(g, src)[0], oracle.dijkstra(g, src)
    for opts in OPTS:
        ws = dpo.alloc_workspace(dg, opts)
        ws.fill_(0xA5)
        print(name, opts.label(), flush=True)
        out = torch.full((g.n,), -7, dtype=torch.int32, device="cuda")
        for _ in range(2):
            dpo.dpo_bfs(dg, src, opts, out, ws)
            assert np.array_equal(out.cpu().numpy(), want), (name, opts.label())
            dpo.dpo_sssp(dg, src, opts, out, ws)
            assert np.array_equal(dpo.as_uint32(out), dwant), (name, opts.label())
        if dpo.dpo_workspace_bytes(dg, opts) <= dpo.NOALLOC_SCRATCH_BYTES:
            out.fill_(-7)
            dpo.dpo_bfs_noalloc(dg, src, opts, out)
            assert np.array_equal(out.cpu().numpy(), want), (name, opts.label())


def test_vertex_id_out_of_range_is_reported():
    """A neighbour id past n on a narrow level and on a wide one: the call
    reports it and the next call is unaffected."""
    for leaves in (100, 80000):
        g = _stars(leaves, 1)
        bad = gg.Graph(g.row_ptr, g.col_idx.copy(), np.ones(g.m, dtype=np.uint32))
        bad.col_idx[bad.row_ptr[1 + leaves // 2 + 1]] = g.n + 5
        for opts in (dpo.Options(), dpo.Options(claim_hint=dpo.DPO_HINT_ON)):
            db, dg = dpo.DeviceGraph.from_host(bad), dpo.DeviceGraph.from_host(g)
            out = torch.empty(g.n, dtype=torch.int32, device="cuda")
            ws = dpo.alloc_workspace(dg, opts)
            for call in (dpo.dpo_bfs, dpo.dpo_sssp):
                with pytest.raises(dpo.DpoError) as e:
                    call(db, 0, opts, out, ws)
                assert e.value.status == dpo.DPO_ERR_ARG
            dpo.dpo_bfs(dg, 0, opts, out, ws)
            assert np.array_equal(out.cpu().numpy(), oracle.bfs(g, 0)[0])
