"""Which kernels a call launches, on both sides of the lines of the dispatch (timed with the library's own
record): the eviction's gather as a launch of its own or by the selection."""
import pytest
import torch

from test_gpu_parity import _say

pytestmark = pytest.mark.gpu


def _launches(names, call):
    import paper_2607_21475_amd as ebd

    ebd.ebd_timing_enable(True)
    try:
        for k in names:
            ebd.ebd_timing_read(k)
        call()
        torch.cuda.synchronize()
        return tuple(ebd.ebd_timing_read(k)[1] for k in names)
    finally:
        ebd.ebd_timing_enable(False)


@pytest.mark.parametrize("units,n,budget,design,copies", [
    (8, 1024, 0.05, 0, 0),      # a few rows: gathered by the selection
    (8, 2048, 0.05, 0, 1),      # two waves per unit, then the copy
    (64, 4096, 0.10, 0, 1),     # 640 rows: worth a copy launch for 64 units
    (181, 4096, 0.10, 0, 0),    # ... not for 181
    (255, 16384, 0.10, 0, 0),
    (300, 4096, 0.25, 0, 1),
    (300, 4096, 0.10, 0, 0),    # few rows: gathered whole
    (300, 16384, 0.25, 0, 1),
    (600, 8192, 0.10, 0, 0),
    (600, 8192, 0.25, 0, 1),    # the selection gathers a share, the copy the rest
    (330, 16400, 0.10, 0, 0),   # streamed units past those of the segment kernels
    (330, 16400, 0.10, 1, 0),
    (300, 16400, 0.25, 2, 1),
])
def test_evict_gather_launches(units, n, budget, design, copies):
    _say("evict launches units=%d n=%d budget=%s design=%d" % (units, n, budget, design))
    import paper_2607_21475_amd as ebd
    from paper_2607_21475_amd import cache

    # every unit reads the same rows of one cache: only the launches are looked at
    g = torch.Generator(device="cuda").manual_seed(1)
    K, V = (torch.randn((n, 128), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    sc = torch.rand(n, generator=g, device="cuda")
    lengths = [n] + [0] * (units - 1)
    cap = cache.plan_capacity(lengths, budget, 4, 64)
    rc_rows = cap[-1]
    so = torch.tensor([0] + [n] * units, dtype=torch.int64, device="cuda")
    co = torch.tensor(cap, dtype=torch.int64, device="cuda")
    Kc, Vc = (torch.empty((rc_rows, 128), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    pic, idx = torch.empty(rc_rows, device="cuda"), torch.empty(rc_rows, dtype=torch.int32, device="cuda")
    cnt, st = (torch.empty(units, dtype=torch.int32, device="cuda") for _ in range(2))
    p = ebd.evict_params(units, n, cap[1], so, co, budget_frac=budget, design=design, seed=3)
    ws = ebd.workspace(ebd.ebd_workspace_size(ebd.EBD_WS_EVICT, p))
    got = _launches(("evict_select", "evict_copy"),
                    lambda: ebd.ebd_evict(p, sc, K, V, Kc, Vc, pic, idx, cnt, st, ws))
    assert got == (1, copies)
