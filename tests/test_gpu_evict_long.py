"""GPU parity of the sampler on long units of small launches, selected by segments (evict_long), and
the work-group per unit that the same call falls back to with the smallest workspace: against the
oracle, and against each other bit for bit."""
import numpy as np
import pytest
import torch

import synth
from test_gpu_parity import _check_evict, _evict, _np, _say

pytestmark = pytest.mark.gpu


def _scores(kind, rows, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    if kind == "pareto":
        return synth.pareto_scores(rows, seed=seed, device="cuda")
    if kind == "lognormal":
        return torch.exp(2.0 * torch.randn(rows, generator=g, device="cuda"))
    if kind == "flat":  # every score in one bin: more around the thresholds than the list holds
        return 1.0 + 0.01 * torch.rand(rows, generator=g, device="cuda")
    if kind == "equal":
        return torch.full((rows,), 0.25, device="cuda")
    if kind == "sparse":  # mostly zeros, tiny and huge values, some denormal
        s = torch.rand(rows, generator=g, device="cuda")
        e = torch.randint(-145, 120, (rows,), generator=g, device="cuda").float()
        return torch.where(s < 0.9, torch.zeros_like(s), torch.ldexp(s, e))
    if kind == "wide":  # spread evenly over 40 octaves: scores around both thresholds however far apart
        return torch.exp2(-40.0 * torch.rand(rows, generator=g, device="cuda"))
    s = torch.rand(rows, generator=g, device="cuda")  # "bad": a few values read as zero
    s[7], s[rows // 2], s[rows - 3] = float("nan"), -1.0, float("inf")
    return s


@pytest.mark.parametrize("lengths,kind,budget,eps,mode", [
    ([16385, 4095, 4096, 4097, 0, 1, 60, 68, 69], "lognormal", 0.25, 0.01, 0),  # segment edges
    ([131072] * 2, "pareto", 0.10, 0.005, 0),
    ([20001, 30003, 17002], "lognormal", 0.05, 0.01, 0),     # units off the 16-byte grid
    ([40000], "flat", 0.25, 0.01, 0),
    ([40000], "equal", 0.30, 0.01, 0),
    ([33333] * 3, "sparse", 0.04, 1e-6, 0),
    ([20000] * 2, "sparse", 0.5, 0.01, 0),                    # nothing to evict among the positive
    ([20000] * 2, "lognormal", 0.005, 0.01, 0),               # the floor exceeds the budget
    ([20000] * 2, "bad", 0.25, 0.01, 0),
    ([20000] * 2, "lognormal", 0.25, 0.01, 1),                # lambda = m / sum s
    ([20000], "lognormal", 0.6, 0.9, 0),                      # thresholds in neighbouring bins
    ([17000] * 40, "pareto", 0.5, 0.01, 0),
    ([60000, 131072], "wide", 0.05, 1e-6, 0),                 # thresholds 20 octaves apart
])
def test_evict_long_parity(lengths, kind, budget, eps, mode):
    _say("evict long lengths=%s %s budget=%s" % (lengths[:4], kind, budget))
    import paper_2607_21475_amd as ebd
    from paper_2607_21475_amd import cache

    K, V, seq_off = synth.make_cache(lengths, seed=5, device="cuda")
    sc = _scores(kind, K.shape[0], seed=6)
    kw = dict(budget_frac=budget, pi_min=eps, pi_mode=mode, seed=9)
    cap = cache.plan_capacity(lengths, 1.0 if mode or kind == "sparse" else budget, 4, 64, pi_min=eps)
    out = _evict(K, V, seq_off, sc, lengths, cap_off_host=cap, **kw)
    p = ebd.evict_params(len(lengths), max(lengths), out.max_cap, seq_off, out.cap_off, 4, 64, budget,
                         None, eps, mode, 9)
    assert ebd.ebd_workspace_size(ebd.EBD_WS_EVICT, p) > 256
    _check_evict(lengths, K, V, seq_off, sc, out, budget=budget, pi_min=eps, seed=9, pi_mode=mode)
    # again: the same bits, whatever order the scores around the thresholds were collected in
    again = _evict(K, V, seq_off, sc, lengths, cap_off_host=cap, **kw)
    off = _np(out.cap_off)
    for k in ("count", "status", "lam", "pi_full"):
        assert torch.equal(getattr(out, k), getattr(again, k)), k
    for u in range(len(lengths)):
        sl = slice(off[u], off[u] + int(out.count[u]))
        for k in ("Kc", "Vc", "pic", "idxc"):
            assert torch.equal(getattr(out, k)[sl], getattr(again, k)[sl]), (u, k)
    # the same call with a 256-byte workspace: a work-group per unit
    ref = {k: torch.zeros_like(getattr(out, k)) for k in ("Kc", "Vc", "pic", "idxc", "count", "status", "lam")}
    pf = torch.zeros_like(out.pi_full)
    ebd.ebd_evict(p, sc, K, V, ref["Kc"], ref["Vc"], ref["pic"], ref["idxc"], ref["count"], ref["status"],
                  ebd.workspace(256), lambda_out=ref["lam"], pi_full=pf)
    torch.cuda.synchronize()
    # the two sum the scores in another order: lambda agrees to an ulp or two of fp32
    assert torch.equal(out.status, ref["status"])
    lam, rlam = _np(out.lam).astype(np.float64), _np(ref["lam"]).astype(np.float64)
    with np.errstate(invalid="ignore"):  # +inf where nothing is evicted
        same = (lam == rlam) | (np.abs(lam - rlam) <= 3e-7 * np.abs(rlam))
    assert np.all(same), (lam, rlam)
    equal = [u for u in np.nonzero(lam == rlam)[0] if lengths[u] > 0]
    assert equal  # the orders of summation differ far below an ulp of fp32: some unit has the same bits
    for u in equal:
        n = int(ref["count"][u])
        assert n == int(out.count[u])
        for k in ("Kc", "Vc", "pic", "idxc"):
            assert torch.equal(getattr(out, k)[off[u]:off[u] + n], ref[k][off[u]:off[u] + n]), (u, k)


def test_evict_long_layout_overflow_and_replay():
    """A unit longer than max_rows is flagged and left alone, one whose rows exceed its capacity keeps
    the first ones, rows past the count stay untouched, and a captured call replays the same."""
    _say("evict long layout")
    import paper_2607_21475_amd as ebd

    lengths = [20000, 30000, 18000]
    K, V, seq_off = synth.make_cache(lengths, seed=5, device="cuda")
    sc = _scores("lognormal", K.shape[0], 8)
    caps = [0, 6000, 14000, 15000]  # 5000, 7500 and 4500 rows are expected
    cap_off = torch.tensor(caps, dtype=torch.int64, device="cuda")
    o = dict(Kc=torch.full((15000, 128), 7.0, dtype=torch.bfloat16, device="cuda"),
             Vc=torch.full((15000, 128), 7.0, dtype=torch.bfloat16, device="cuda"),
             pic=torch.full((15000,), 7.0, device="cuda"),
             idxc=torch.full((15000,), 7, dtype=torch.int32, device="cuda"))
    count = torch.full((3,), -1, dtype=torch.int32, device="cuda")
    st = torch.full((3,), -1, dtype=torch.int32, device="cuda")
    lam = torch.zeros(3, device="cuda")
    p = ebd.evict_params(3, 20000, 8000, seq_off, cap_off, budget_frac=0.25, seed=4)
    ws = ebd.workspace(ebd.ebd_workspace_size(ebd.EBD_WS_EVICT, p))

    def call():
        ebd.ebd_evict(p, sc, K, V, o["Kc"], o["Vc"], o["pic"], o["idxc"], count, st, ws, lambda_out=lam)

    call()
    torch.cuda.synchronize()
    assert st.tolist() == [0, 16, 1] and int(count[1]) == 0 and float(lam[1]) == 0.0
    n0 = int(count[0])
    assert 4000 < n0 <= 6000 and int(count[2]) > 1000
    for k, v in o.items():
        assert torch.all(v[n0:14000] == 7), k
    first = {k: v.clone() for k, v in o.items()}
    i2 = o["idxc"][14000:].long()
    assert torch.all(i2[1:] > i2[:-1])
    assert torch.equal(o["Vc"][14000:], V[50000 + i2]) and torch.equal(o["Kc"][14000:], K[50000 + i2])
    g = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            call()
    first.update(count=count.clone(), status=st.clone(), lam=lam.clone())
    for _ in range(3):  # over sentinels everywhere: what the call wrote is written again, the rest is left
        for v in o.values():
            v.fill_(7)
        count.fill_(-1), st.fill_(-1), lam.fill_(7.0)
        ws.fill_(255)
        g.replay()
        torch.cuda.synchronize()
        for k, v in dict(o, count=count, status=st, lam=lam).items():
            assert torch.equal(v, first[k]), k
