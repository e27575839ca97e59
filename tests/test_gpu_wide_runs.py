"""Runs of wide BFS levels, launched several steps at a time: levels equal the
oracle's where the run ends inside such a part (in narrow levels, in the last
level or in a bottom-up one), on local and shuffled ids, directed and not."""
import numpy as np
import pytest

import oracle
from paper_2201_02789_amd import graphgen as gg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2201_02789_amd import dpo  # noqa: E402


def _layers(widths, deg, seed, shuffle=False, one_way=False):
    """Layers of the given widths; each vertex has `deg` neighbours in the next."""
    rng = np.random.default_rng(seed)
    at = np.concatenate([[0], np.cumsum(widths)])
    u = np.concatenate([np.repeat(np.arange(at[k], at[k + 1]), deg) for k in range(len(widths) - 1)])
    v = np.concatenate([rng.integers(at[k + 1], at[k + 2], widths[k] * deg) for k in range(len(widths) - 1)])
    # every vertex of a layer has a parent
    lone = np.concatenate([np.arange(at[k + 1], at[k + 2]) for k in range(len(widths) - 1)])
    par = np.concatenate([rng.integers(at[k], at[k + 1], widths[k + 1]) for k in range(len(widths) - 1)])
    u, v = np.concatenate([u, par]), np.concatenate([v, lone])
    n = int(at[-1])
    if shuffle:
        p = rng.permutation(n)
        u, v = p[u], p[v]
        first = int(p[0])
    else:
        first = 0
    src, dst = (u, v) if one_way else (np.concatenate([u, v]), np.concatenate([v, u]))
    o = np.lexsort((dst, src))
    rp = np.concatenate([[0], np.cumsum(np.bincount(src, minlength=n))]).astype(np.int32)
    return gg.Graph(rp, dst[o].astype(np.int32)), first


W = 9000  # past the narrow kernel's frontier
SHAPES = [("wide-to-the-end", [1] + [W] * 14, 2), ("wide-narrow-wide", [1] + [W] * 9 + [5] * 40 + [W] * 12 + [3] * 3, 2),
          ("dense", [1] + [W] * 8, 9), ("growing", [1, 40, 1000] + [W] * 3 + [60000] * 2 + [W] * 7, 6)]


@pytest.mark.parametrize("shuffle,one_way", [(False, False), (True, False), (True, True)])
@pytest.mark.parametrize("name,widths,deg", SHAPES, ids=[s[0] for s in SHAPES])
def test_levels_match_oracle(name, widths, deg, shuffle, one_way):
    g, s = _layers(widths, deg, 5, shuffle, one_way)
    want = oracle.bfs(g, s)[0]
    dg = dpo.DeviceGraph.from_host(g)
    out = torch.empty(g.n, dtype=torch.int32, device="cuda")
    for o in (dict(), dict(split_min=1024, child_block=128, threshold=8, coarsen=1),
              dict(claim_hint=dpo.DPO_HINT_ON, steps_per_replay=2), dict(claim_hint=dpo.DPO_HINT_OFF, split_min=0)):
        opts = dpo.Options(**o)
        ws = dpo.alloc_workspace(dg, opts)
        ws.fill_(0x5A)
        print(name, o, flush=True)
        for call in (lambda: dpo.dpo_bfs(dg, s, opts, out, ws), lambda: dpo.dpo_bfs_noalloc(dg, s, opts, out)):
            out.fill_(-7)
            call()
            assert np.array_equal(out.cpu().numpy(), want), (name, o)


def test_queries_over_layers():
    """A batch and an engine with enough work for bottom-up queries, of which some go
    bottom-up near their end, some on their wide levels and some, beside what they
    never reach, not at all."""
    gs = [_layers([1] + [4000] * 12, 9, 1)[0], _layers([1, 500] + [6000] * 8, 9, 2, shuffle=True)[0],
          gg.rmat(14, 24, 7, perm_seed=3), gg.pack_arena([gg.rmat(13, 24, k, perm_seed=k) for k in range(4)])[0]]
    ar, vbase = gg.pack_arena(gs)
    da = dpo.DeviceArena(ar, vbase)
    rng = np.random.default_rng(6)
    qs = [(k, int(rng.choice(np.flatnonzero(gs[k].degrees())))) for k in (0, 1, 2, 3) * 14]
    want = [oracle.bfs(gs[k], s)[0] for k, s in qs]
    for o in (dict(), dict(threshold=16, coarsen=1, steps_per_replay=3)):
        opts = dpo.Options(**o)
        tot, slot0 = dpo.dpo_batch_slots(da, qs)
        out = torch.full((tot,), -7, dtype=torch.int32, device="cuda")
        ws = torch.full((dpo.dpo_batch_workspace_bytes(da, qs, opts),), 0xC3, dtype=torch.uint8, device="cuda")
        dpo.dpo_bfs_batch(da, qs, [opts], out, ws)
        host = out.cpu().numpy()
        for i, (k, s) in enumerate(qs):
            assert np.array_equal(host[slot0[i]:slot0[i] + gs[k].n], want[i]), (o, i)
        eng = dpo.Engine(da, "bfs", [opts], max_queries=64, max_slots=1 << 22)
        outs = [torch.full((gs[k].n,), -9, dtype=torch.int32, device="cuda") for k, _ in qs]
        for (k, s), t in zip(qs, outs):
            eng.submit(k, s, t)
        for _ in range(2000):
            if eng.step() == (0, 0):
                break
        assert len(eng.poll()) == len(qs)
        for w, t in zip(want, outs):
            assert np.array_equal(t.cpu().numpy(), w), o
        eng.close()


@pytest.mark.parametrize("parts", [2, 5])
@pytest.mark.parametrize("o", [dict(split_min=2048, child_block=128, threshold=64, coarsen=1), dict()], ids=str)
def test_beside_what_the_search_never_reaches(parts, o):
    """Several graphs in one CSR, isolated vertices among them: bottom-up levels would
    read the rows of the others."""
    gs = [gg.rmat(15, 20, k, perm_seed=k + 3) for k in range(parts)]
    ar, vbase = gg.pack_arena(gs)
    dg = dpo.DeviceGraph.from_host(ar)
    opts = dpo.Options(**o)
    ws = dpo.alloc_workspace(dg, opts)
    out = torch.full((ar.n,), -7, dtype=torch.int32, device="cuda")
    for s in [int(vbase[k]) + gg.max_degree_vertex(gs[k]) for k in range(parts)] + [int(np.flatnonzero(ar.degrees() == 0)[0])]:
        dpo.dpo_bfs(dg, s, opts, out, ws)
        assert np.array_equal(out.cpu().numpy(), oracle.bfs(ar, s)[0]), s
