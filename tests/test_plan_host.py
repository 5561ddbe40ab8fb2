"""CPU checks of what a launch plan shows on the host: the sampler's workspace, which only launches of few
long units need."""
import pytest


@pytest.mark.parametrize("units,n,budget,segments", [
    (1, 16384, 0.25, False),
    (1, 16385, 0.25, True),
    (32, 131072, 0.10, True),
    (192, 16385, 0.10, True),     # the most units of any long ones, at any budget
    (192, 16385, 0.25, True),
    (193, 16385, 0.25, False),
    (193, 65536, 0.10, False),
    (193, 77200, 0.10, True),     # ... of units of at least 400 tokens for every unit of the launch
    (320, 131072, 0.10, True),
    (321, 131072, 0.10, False),
    (512, 20000, 0.10, False),
    (767, 16385, 0.05, False),
    (2, (1 << 21) + 1, 0.10, False),
])
def test_evict_workspace_of_long_units(units, n, budget, segments):
    import paper_2607_21475_amd as ebd
    from paper_2607_21475_amd import cache

    p = ebd.ebd_evict_params()
    p.num_units, p.head_dim, p.max_rows = units, 128, n
    p.max_capacity = cache.unit_capacity(n, budget, 68)
    p.seq_off = p.cap_off = 0x100000  # not read
    p.n_sink, p.n_recent, p.budget_frac, p.pi_min = 4, 64, budget, 0.01
    size = ebd.ebd_workspace_size(ebd.EBD_WS_EVICT, p)
    assert (size > 256) == segments
    if segments:
        assert size >= units * 65536
    p.design = ebd.EBD_DESIGN_TOPK
    assert ebd.ebd_workspace_size(ebd.EBD_WS_EVICT, p) == 256
