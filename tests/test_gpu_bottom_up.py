"""Wide BFS levels of single traversals: bottom-up on graphs found symmetric,
top-down on all others.  Levels equal the oracle's on symmetric graphs and on
graphs that miss symmetry by as little as one entry, with and without a
workspace of the caller's."""
import numpy as np
import pytest

import oracle
from paper_2201_02789_amd import graphgen as gg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2201_02789_amd import dpo  # noqa: E402


def _csr(n, src, dst, seed):
    """CSR of directed entries as given (duplicates and loops kept), rows in
    random order inside."""
    p = np.random.default_rng(seed).permutation(src.size)
    src, dst = src[p], dst[p]
    o = np.argsort(src, kind="stable")
    rp = np.concatenate([[0], np.cumsum(np.bincount(src, minlength=n))]).astype(np.int32)
    return gg.Graph(rp, dst[o].astype(np.int32))


def _entries(g):
    return np.repeat(np.arange(g.n), g.degrees()).astype(np.int64), g.col_idx.astype(np.int64)


def _rmat():
    return gg.rmat(15, 24, 7, perm_seed=3)


def _without(k):
    """The R-MAT graph without k of its directed entries (0: symmetric)."""
    def make():
        s, d = _entries(_rmat())
        keep = np.ones(s.size, dtype=bool)
        keep[np.random.default_rng(k).choice(s.size, k, replace=False)] = False
        return _csr(1 << 15, s[keep], d[keep], 1)
    return make


def _doubled(both):
    """Every seventh entry twice; its reverse too if `both`."""
    def make():
        s, d = _entries(_rmat())
        pick = (np.minimum(s, d) * 31 + np.maximum(s, d)) % 7 == 0
        if not both:
            pick &= s < d
        return _csr(1 << 15, np.concatenate([s, s[pick]]), np.concatenate([d, d[pick]]), 2)
    return make


def _loops():
    s, d = _entries(_rmat())
    v = np.arange(0, 1 << 15, 3)
    return _csr(1 << 15, np.concatenate([s, v]), np.concatenate([d, v]), 3)


def _one_way():
    s, d = _entries(_rmat())
    keep = s < d
    return _csr(1 << 15, s[keep], d[keep], 4)


def _far_hub():
    """Beside the R-MAT graph a star of 70,000 leaves that no search reaches."""
    s, d = _entries(_rmat())
    h = 1 << 15
    leaf = h + 1 + np.arange(70000)
    hub = np.full(leaf.size, h)
    return _csr(h + 1 + leaf.size, np.concatenate([s, hub, leaf]), np.concatenate([d, leaf, hub]), 5)


GRAPHS = [("symmetric", _without(0)), ("one-missing", _without(1)), ("five-missing", _without(5)),
          ("doubled", _doubled(True)), ("doubled-one-way", _doubled(False)), ("loops", _loops),
          ("one-way", _one_way), ("far-hub", _far_hub),
          ("er-dense", lambda: gg.erdos_renyi(20001, 640000, 6)),
          ("er-odd", lambda: gg.erdos_renyi(200033, 2000000, 8)),
          ("complete", lambda: gg.complete_graph(700)),
          ("rmat18", lambda: gg.rmat(18, 16, 9, perm_seed=2))]


@pytest.mark.parametrize("name,make", GRAPHS, ids=[g[0] for g in GRAPHS])
def test_wide_levels_match_oracle(name, make):
    g = make()
    dg = dpo.DeviceGraph.from_host(g)
    srcs = [int(s) for s in gg.sample_sources(g, 3, 4)] + [gg.max_degree_vertex(g)]
    for opts in (dpo.Options(claim_hint=dpo.DPO_HINT_ON),
                 dpo.Options(threshold=64, coarsen=1, child_block=128, dyn_share=25, split_min=0,
                             claim_hint=dpo.DPO_HINT_ON)):
        ws = dpo.alloc_workspace(dg, opts)
        ws.fill_(0x5A)
        out = torch.full((g.n,), -7, dtype=torch.int32, device="cuda")
        for s in srcs:
            print(name, opts.label(), s, flush=True)
            want = oracle.bfs(g, s)[0]
            dpo.dpo_bfs(dg, s, opts, out, ws)
            assert np.array_equal(out.cpu().numpy(), want), (name, opts.label(), s)
            out.fill_(-7)
            dpo.dpo_bfs_noalloc(dg, s, opts, out)
            assert np.array_equal(out.cpu().numpy(), want), (name, opts.label(), s)


def test_id_out_of_range_in_an_unreached_row_is_no_error():
    """An entry past n in a row that no search reaches did not matter before
    wide levels read every row, and does not now; in a reached row the call
    reports it."""
    s, d = _entries(_rmat())
    n = (1 << 15) + 2
    for row, fails in ((n - 1, False), (int(s[0]), True)):
        g = _csr(n, np.append(s, row), np.append(d, n + 9), 6)
        dg = dpo.DeviceGraph.from_host(g)
        opts = dpo.Options()
        out = torch.empty(n, dtype=torch.int32, device="cuda")
        ws = dpo.alloc_workspace(dg, opts)
        src = gg.max_degree_vertex(g)
        if fails:
            with pytest.raises(dpo.DpoError) as e:
                dpo.dpo_bfs(dg, src, opts, out, ws)
            assert e.value.status == dpo.DPO_ERR_ARG
        else:
            dpo.dpo_bfs(dg, src, opts, out, ws)
            keep = gg.Graph(g.row_ptr.copy(), g.col_idx[:-1].copy())
            keep.row_ptr[-1] -= 1
            assert np.array_equal(out.cpu().numpy(), oracle.bfs(keep, src)[0])
