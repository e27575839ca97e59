"""SSSP with a byte per vertex that rules most sums out before the distance is
read (many slots): distances equal the oracle for weights of all sizes, around
the slot count from which the bytes are kept."""
import numpy as np
import pytest

import oracle
from paper_2201_02789_amd import graphgen as gg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2201_02789_amd import dpo  # noqa: E402

KINDS = {"small": lambda r, m: r.integers(1, 20, m), "octets": lambda r, m: r.integers(1, 256, m),
         "zeros": lambda r, m: r.integers(0, 2, m) * r.integers(0, 70000, m),
         "wide": lambda r, m: r.integers(0, 1 << 27, m),
         "steps": lambda r, m: (1 << r.integers(0, 31, m)) + r.integers(-1, 2, m)}


@pytest.mark.parametrize("n", [(1 << 20) - 32, (1 << 20) - 31, (1 << 20) + 1])
@pytest.mark.parametrize("kind", KINDS)
def test_distances_match_oracle(n, kind):
    g = gg.erdos_renyi(n, 2 * n, 5)
    w = KINDS[kind](np.random.default_rng(7), g.m).astype(np.uint32)
    g = gg.Graph(g.row_ptr, g.col_idx, w)
    want = oracle.dijkstra(g, 3)
    dg = dpo.DeviceGraph.from_host(g)
    for o in (dpo.Options(claim_hint=dpo.DPO_HINT_ON, split_min=0),
              dpo.Options(claim_hint=dpo.DPO_HINT_ON, threshold=4, agg=dpo.DPO_AGG_WAVE),
              dpo.Options(claim_hint=dpo.DPO_HINT_ON, mode=dpo.DPO_MODE_FLAT)):
        print(n, kind, o.label(), flush=True)
        ws = dpo.alloc_workspace(dg, o)
        ws.fill_(0)  # bytes that rule everything out, unless the call sets them
        out = torch.full((n,), -7, dtype=torch.int32, device="cuda")
        dpo.dpo_sssp(dg, 3, o, out, ws)
        assert np.array_equal(dpo.as_uint32(out), want), o.label()
