"""The gather of large launches: a unit's first rows by the work-group that selected it, the others by
the copy launch, at the edges between the two."""
import pytest
import torch

import synth
from test_gpu_parity import _check_evict, _evict, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("longest,budget,short", [
    (16384, 1.0, 0),     # first 1024 rows, then blocks of 128
    (16384, 1.0, 500),   # ... with capacities below the counts
    (20000, 1.0, 0),     # streamed units: first 1152 rows
    (7000, 0.29, 0),     # capacity just past 2 x 1024 rows
    (7000, 0.25, 0),     # ... within them: one launch
    (16384, 0.4, 0),
])
def test_gather_split_between_launches(longest, budget, short):
    _say("evict gather longest=%d budget=%s short=%d" % (longest, budget, short))
    edges = [0, 1, 1023, 1024, 1025, 1151, 1152, 1153, 1279, 1281, 2047, 2048, 2049, 2176, 3001]
    lengths = [16] * 760 + [n for n in edges if n <= longest] + [longest, longest - 1]
    K, V, seq_off = synth.make_cache(lengths, seed=3, device="cuda")
    sc = 0.5 + torch.rand(K.shape[0], generator=torch.Generator(device="cuda").manual_seed(4), device="cuda")
    cap = None
    if budget == 1.0:  # every row is retained: the copy is K and V themselves, up to the capacity
        cap = [0]
        for n in lengths:
            cap.append(cap[-1] + max(n - short, 0) + (0 if short else 3))
    out = _evict(K, V, seq_off, sc, lengths, cap_off_host=cap, budget_frac=budget, pi_min=0.01, seed=9)
    if budget < 1.0:
        _check_evict(lengths, K, V, seq_off, sc, out, budget=budget, pi_min=0.01, seed=9)
        return
    torch.cuda.synchronize()
    so, co = seq_off.tolist(), cap
    for u in range(760 - 4, len(lengths)):
        n = min(lengths[u], co[u + 1] - co[u])
        assert int(out.count[u]) == lengths[u]
        assert torch.equal(out.Kc[co[u]:co[u] + n], K[so[u]:so[u] + n]), (u, lengths[u])
        assert torch.equal(out.Vc[co[u]:co[u] + n], V[so[u]:so[u] + n]), (u, lengths[u])
