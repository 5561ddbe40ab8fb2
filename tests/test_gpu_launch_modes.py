"""Which kernels a call launches, on both sides of the lines of the dispatch (timed with the library's own
record): the eviction's gather as a launch of its own or by the selection, and attention with or without
records for a finalize."""
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
    (512, 65600, 0.10, 2, 1),   # long units, few rows: copied up to 512 units
    (513, 65700, 0.10, 2, 0),   # gathered whole
    (513, 131072, 0.10, 2, 1),  # ... up to three shares
])
def test_evict_gather_launches(units, n, budget, design, copies):
    _say("evict launches units=%d n=%d budget=%s design=%d" % (units, n, budget, design))
    import paper_2607_21475_amd as ebd
    from paper_2607_21475_amd import cache

    # one unit holds rows, the others are empty: only the launches are looked at
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


@pytest.mark.parametrize("units,n,G,finalizes", [
    (129, 4000, 4, 0),      # waves that share a unit
    (129, 4200, 4, 1),      # 129 to 180 units past 4096 rows: parts with records
    (180, 4200, 8, 1),
    (181, 4200, 4, 0),
    (256, 12000, 4, 0),
    (256, 13000, 4, 1),     # 181 to 256 past 12288 rows
    (256, 13000, 8, 0),     # ... of up to four heads
    (257, 1000, 4, 0),      # 257 to 383 of five or six splits: records
    (257, 1300, 4, 1),
    (383, 1300, 4, 1),
    (384, 1300, 4, 0),
    (512, 30000, 4, 0),
    (512, 33000, 4, 1),     # the longest
    (513, 16000, 4, 0),
    (513, 17000, 4, 1),
    (1535, 13400, 8, 0),    # eight waves, whose LDS fits where that of four does not
    (1536, 9000, 8, 0),
    (1536, 17000, 1, 1),
])
def test_attend_launches(units, n, G, finalizes):
    _say("attend launches units=%d n=%d G=%d" % (units, n, G))
    import paper_2607_21475_amd as ebd

    # every unit is empty: only the launches are looked at
    off = torch.zeros(units + 1, dtype=torch.int64, device="cuda")
    cnt = torch.zeros(units, dtype=torch.int32, device="cuda")
    K, V = (torch.zeros((16, 128), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    q, pi = torch.zeros((units, G, 128), dtype=torch.bfloat16, device="cuda"), torch.zeros(16, device="cuda")
    y, vhat, lse = torch.empty((units, G, 128), device="cuda"), *torch.empty((2, units, G), device="cuda")
    p = ebd.attend_params(units, G, n, off)
    ws = ebd.workspace(ebd.ebd_workspace_size(ebd.EBD_WS_ATTEND, p))
    got = _launches(("attend_split", "attend_finalize"),
                    lambda: ebd.ebd_attend_certify(p, q, K, V, pi, cnt, y, vhat, lse, ws))
    assert got == (1, finalizes)
    assert not y.any() and torch.all(torch.isneginf(lse))
