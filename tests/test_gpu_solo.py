"""SSSP on small graphs, in one workgroup: results equal the oracle where that
path begins and ends (vertex and edge limits), with frontiers past what LDS
holds, rows of every length and large weights; and batches of small weighted
graphs."""
import numpy as np
import pytest

import oracle
from paper_2201_02789_amd import graphgen as gg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2201_02789_amd import dpo  # noqa: E402

GRAPHS = [
    ("one", lambda: gg.from_edges(1, []), 0),
    ("isolated", lambda: gg.from_edges(9, [(1, 2)]), 4),
    ("path", lambda: gg.path_graph(3000), 7),
    ("star-16384", lambda: gg.star_graph(16384), 5),   # a frontier several times what LDS holds
    ("star-16385", lambda: gg.star_graph(16385), 0),   # one vertex too many
    ("grid", lambda: gg.grid_graph(127, 129), 11),
    ("road", lambda: gg.road_like(100, 90, 3), 4041),
    ("rmat13", lambda: gg.rmat(13, 16, 13, perm_seed=4), 5),
    ("rmat14", lambda: gg.rmat(14, 30, 14, perm_seed=4), 6),
    ("er-64", lambda: gg.erdos_renyi(9001, 16 * 9001, 4), 1),
    ("complete-512", lambda: gg.complete_graph(512), 3),  # 261,632 entries
    ("complete-513", lambda: gg.complete_graph(513), 3),  # 262,656: past the limit
]
OPTS = [dpo.Options(), dpo.Options(threshold=16, coarsen=1, claim_hint=dpo.DPO_HINT_ON),
        dpo.Options(threshold=0, agg=dpo.DPO_AGG_WAVE, claim_hint=dpo.DPO_HINT_OFF)]


@pytest.mark.parametrize("name,make,src", GRAPHS, ids=[g[0] for g in GRAPHS])
def test_single(name, make, src):
    g = gg.add_weights(make(), 9)
    # heavier: sums of a few edges pass 2^31; still below 2^32 - 1 on these paths
    heavy = gg.Graph(g.row_ptr, g.col_idx, g.weights * np.uint32(5001))
    for h in (g, heavy):
        dg = dpo.DeviceGraph.from_host(h)
        want = oracle.dijkstra(h, src)
        for opts in OPTS:
            print(name, opts.label(), flush=True)
            ws = dpo.alloc_workspace(dg, opts)
            ws.fill_(0xA5)
            out = torch.full((g.n,), -7, dtype=torch.int32, device="cuda")
            for _ in range(2):
                dpo.dpo_sssp(dg, src, opts, out, ws)
                assert np.array_equal(dpo.as_uint32(out), want), (name, opts.label())


WEIGHTS = {"equal": lambda r, m: np.full(m, 7), "zeros": lambda r, m: r.integers(0, 2, m) * 9,
           "octets": lambda r, m: r.integers(1, 256, m), "skewed": lambda r, m: 1 << r.integers(0, 28, m),
           # three edges stay below 2^32 - 1, 1.5 times two do not
           "heavy": lambda r, m: r.integers(1300000000, 1400000000, m)}


@pytest.mark.parametrize("weights", WEIGHTS)
@pytest.mark.parametrize("leaves,hubs", [(15018, 3), (15019, 3), (8191, 6), (16378, 6), (16377, 7), (5000, 9)])
def test_bound_moves(leaves, hubs, weights):
    """Every leaf at every hub: around the entries from which a bound is kept,
    bounds that let one vertex or all of them through, more than LDS holds."""
    e = np.stack(np.meshgrid(np.arange(hubs), hubs + np.arange(leaves)), -1).reshape(-1, 2)
    g = gg.from_edges(hubs + leaves, e)
    w = WEIGHTS[weights](np.random.default_rng(leaves), g.m).astype(np.uint32)
    g = gg.Graph(g.row_ptr, g.col_idx, w)  # not the same both ways
    dg = dpo.DeviceGraph.from_host(g)
    o = dpo.Options()
    ws = dpo.alloc_workspace(dg, o)
    for src in (0, hubs + 1):
        print(leaves, hubs, weights, src, flush=True)
        ws.fill_(0xA5)
        out = torch.full((g.n,), -7, dtype=torch.int32, device="cuda")
        dpo.dpo_sssp(dg, src, o, out, ws)
        assert np.array_equal(dpo.as_uint32(out), oracle.dijkstra(g, src)), src


def test_batch():
    gs = [gg.rmat(9, 8, 3, perm_seed=4), gg.rmat(13, 16, 5, perm_seed=6), gg.road_like(60, 70, 2),
          gg.star_graph(9000), gg.path_graph(400), gg.from_edges(75, [(1, 2), (2, 3)]),
          gg.complete_graph(600)]
    gs = [gg.add_weights(g, 31 + i) for i, g in enumerate(gs)]
    ar, vbase = gg.pack_arena(gs)
    da = dpo.DeviceArena(ar, vbase)
    rng = np.random.default_rng(5)
    qs = [(k, int(rng.choice(np.flatnonzero(g.degrees())))) for _ in range(3) for k, g in enumerate(gs)]
    wants = [oracle.dijkstra(gs[k], s) for k, s in qs]
    for opts in OPTS:
        tot, slot0 = dpo.dpo_batch_slots(da, qs)
        ws = torch.full((dpo.dpo_batch_workspace_bytes(da, qs, opts),), 0xC3, dtype=torch.uint8, device="cuda")
        for _ in range(2):
            out = torch.full((tot,), -7, dtype=torch.int32, device="cuda")
            print("batch", opts.label(), flush=True)
            dpo.dpo_sssp_batch(da, qs, [opts], out, ws)
            host = out.cpu().numpy()
            for i, (k, s) in enumerate(qs):
                assert np.array_equal(host[slot0[i]:slot0[i] + gs[k].n].view(np.uint32), wants[i]), (i, k, s)
                assert (host[slot0[i] + gs[k].n:slot0[i + 1]] == -7).all()


def test_vertex_id_out_of_range_is_reported():
    g = gg.add_weights(gg.grid_graph(40, 40), 3)
    for at in (g.row_ptr[700], g.row_ptr[0]):
        bad = gg.Graph(g.row_ptr, g.col_idx.copy(), g.weights)
        bad.col_idx[at] = g.n + 3
        out = torch.empty(g.n, dtype=torch.int32, device="cuda")
        dg = dpo.DeviceGraph.from_host(bad)
        with pytest.raises(dpo.DpoError) as e:
            dpo.dpo_sssp(dg, 0, dpo.Options(), out, dpo.alloc_workspace(dg, dpo.Options()))
        assert e.value.status == dpo.DPO_ERR_ARG
