"""Row pointers that are not a CSR's, as every path takes them: a row that would
launch and lies past the m entries is DPO_ERR_CAPACITY and is not read; a row
that ends before it starts has no entries.  (The arrays are longer than m says, so
nothing here lies outside them.)"""
import numpy as np
import pytest

import oracle
from paper_2201_02789_amd import graphgen as gg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2201_02789_amd import dpo  # noqa: E402

T = 128


def _hub_last(n, deg):
    """A path over all vertices but the last, which has `deg` of them as
    neighbours: a hub whose row is the last one."""
    u = np.arange(n - 2)
    return gg.add_weights(gg.from_edges(n, [*zip(u, u + 1), *((n - 1, k) for k in range(deg))]), 3)


def _calls(dg, opts, out):
    ws = dpo.alloc_workspace(dg, opts)
    return {"bfs": lambda s: dpo.dpo_bfs(dg, s, opts, out, ws),
            "noalloc": lambda s: dpo.dpo_bfs_noalloc(dg, s, opts, out),
            "sssp": lambda s: dpo.dpo_sssp(dg, s, opts, out, ws)}


# solo SSSP; near-far SSSP
@pytest.mark.parametrize("n,deg", [(700, 400), (30000, 500)])
@pytest.mark.parametrize("call", ["bfs", "noalloc", "sssp"])
@pytest.mark.parametrize("hint", [dpo.DPO_HINT_AUTO, dpo.DPO_HINT_ON])
def test_a_launching_row_past_the_entries_is_an_error(n, deg, call, hint):
    g = _hub_last(n, deg)
    dg = dpo.DeviceGraph.from_host(g)
    out = torch.empty(n, dtype=torch.int32, device="cuda")
    opts = dpo.Options(threshold=T, claim_hint=hint)
    want = {"sssp": oracle.dijkstra(g, 3).view(np.int32)}.get(call, oracle.bfs(g, 3)[0])
    _calls(dg, opts, out)[call](3)
    assert np.array_equal(out.cpu().numpy(), want)
    dg.m -= deg // 2  # the hub's row ends past the entries
    with pytest.raises(dpo.DpoError) as e:
        _calls(dg, opts, out)[call](3)
    assert e.value.status == dpo.DPO_ERR_CAPACITY
    # a row below the threshold is read as it stands
    opts = dpo.Options(threshold=deg + 1, claim_hint=hint)
    _calls(dg, opts, out)[call](3)
    assert np.array_equal(out.cpu().numpy(), want)


@pytest.mark.parametrize("n", [600, 30000])
@pytest.mark.parametrize("call", ["bfs", "noalloc", "sssp"])
def test_a_row_that_ends_before_it_starts_has_no_entries(n, call):
    """Vertex z, a neighbour of the source beside others, with such a row; the
    vertex before it has no edges."""
    z = n // 2
    e = [(0, 1), (0, 2), (0, z), (1, 3), (2, 4), (2, 5)] + [(k, k + 1) for k in range(5, z - 2)]
    e += [(4, k) for k in range(z + 1, z + 40)]
    g = gg.add_weights(gg.from_edges(n, e), 5)
    rp = g.row_ptr.copy()
    assert rp[z - 1] == rp[z] and rp[z + 1] == rp[z] + 1
    empty = np.delete(np.stack([np.repeat(np.arange(n), g.degrees()), g.col_idx]), rp[z], axis=1)
    w = np.delete(g.weights, rp[z])
    ref = gg.Graph(np.concatenate([[0], np.cumsum(np.bincount(empty[0], minlength=n))]).astype(np.int32),
                   empty[1].astype(np.int32), w)
    rp[z] += 7  # the row of z: [x + 7, x + 1)
    dg = dpo.DeviceGraph.from_host(gg.Graph(rp, g.col_idx, g.weights))
    out = torch.empty(n, dtype=torch.int32, device="cuda")
    want = oracle.dijkstra(ref, 0).view(np.int32) if call == "sssp" else oracle.bfs(ref, 0)[0]
    _calls(dg, dpo.Options(threshold=T), out)[call](0)
    assert np.array_equal(out.cpu().numpy(), want)


def test_rows_past_the_entries_leave_a_graph_top_down():
    """Entries past m: the part within m is symmetric, so only the row pointers'
    end tells that a bottom-up level would read on."""
    g = gg.rmat(14, 24, 7, perm_seed=3)
    n = g.n + 200  # 200 more vertices, a row of 150 entries past m each
    rp = np.concatenate([g.row_ptr, g.m + 150 * (1 + np.arange(200))]).astype(np.int32)
    col = np.concatenate([g.col_idx, np.zeros(150 * 200, np.int32)]).astype(np.int32)
    dg = dpo.DeviceGraph.from_host(gg.Graph(rp, col))
    dg.m = g.m
    out = torch.empty(n, dtype=torch.int32, device="cuda")
    s = gg.max_degree_vertex(g)
    want = np.concatenate([oracle.bfs(g, s)[0], np.full(200, -1, np.int32)])
    for name, f in _calls(dg, dpo.Options(threshold=T, claim_hint=dpo.DPO_HINT_ON), out).items():
        if name != "sssp":
            f(s)
            assert np.array_equal(out.cpu().numpy(), want), name
