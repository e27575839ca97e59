"""Engine results for memory that a kernel on the engine's device does not store
to word by word: an address off a word's boundary, pinned host memory, beside
ordinary device arrays in the same step."""
import numpy as np
import pytest

import oracle
from paper_2201_02789_amd import graphgen as gg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2201_02789_amd import dpo  # noqa: E402


@pytest.mark.parametrize("kind", ["bfs", "sssp"])
def test_results_reach_any_memory(kind):
    gs = [gg.add_weights(gg.rmat(s, 8, 40 + s, perm_seed=s), s) for s in (9, 10, 12)]
    ar, vbase = gg.pack_arena(gs)
    da = dpo.DeviceArena(ar, vbase)
    eng = dpo.Engine(da, kind, [dpo.Options()], max_queries=8, max_slots=1 << 14)
    want = [oracle.bfs(g, 3)[0] if kind == "bfs" else oracle.dijkstra(g, 3) for g in gs]
    odd = torch.full((gs[0].n * 4 + 8,), 5, dtype=torch.uint8, device="cuda")
    pinned = torch.full((gs[1].n + 2,), -5, dtype=torch.int32, pin_memory=True)
    plain = torch.full((gs[2].n + 2,), -5, dtype=torch.int32, device="cuda")
    eng.submit(0, 3, odd[3:])
    eng.submit(1, 3, pinned)
    eng.submit(2, 3, plain)
    done = []
    for _ in range(1000):
        rest = eng.step()
        done += eng.poll()
        if rest == (0, 0):
            break
    assert len(done) == 3
    got = [odd.cpu().numpy()[3:3 + 4 * gs[0].n].copy().view(want[0].dtype),
           pinned.numpy()[:gs[1].n].copy().view(want[1].dtype), plain.cpu().numpy()[:gs[2].n].view(want[2].dtype)]
    for k in range(3):
        assert np.array_equal(got[k], want[k]), k
    host = odd.cpu().numpy()
    assert (host[:3] == 5).all() and (host[3 + 4 * gs[0].n:] == 5).all()
    assert (pinned[gs[1].n:] == -5).all() and (plain[gs[2].n:] == -5).all()
    eng.close()
