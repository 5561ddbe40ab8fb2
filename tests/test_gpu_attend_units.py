"""GPU parity of certified attention where the library cuts the launch itself: a work-group of
several waves per unit (8, 4 or 2 of them), long units of small launches in several parts whose records a second kernel combines, and one wave per unit in large launches.
The oracle and the bars are those of test_gpu_parity."""
import numpy as np
import pytest
import torch

import oracle
from helpers import bf16_to_f64
from test_gpu_parity import _bits, _cert_floor, _np, _say

pytestmark = pytest.mark.gpu


def _units(sizes, G, seed, dominant=0):
    """Retained caches of the given sizes, pi in (0.05, 1] with 68 certain rows, and queries.  With
    `dominant`, that many rows of each unit, spread over it, are drawn at pi = 1e-6 with keys along
    head 0's query, each 4 (base-2) above the one before: every wave and part sees a pivot, and
    all but the last are added back."""
    from paper_2607_21475_amd import cache

    g = torch.Generator(device="cuda").manual_seed(seed)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    rows = max(int(off[-1]), 1)
    bf = dict(generator=g, device="cuda", dtype=torch.bfloat16)
    K, V = torch.randn((rows, 128), **bf), torch.randn((rows, 128), **bf)
    q = torch.randn((len(sizes), G, 128), **bf)
    pi = torch.rand(rows, generator=g, device="cuda") * 0.95 + 0.05
    for u, n in enumerate(sizes[:64]):
        pi[off[u]:off[u] + min(n, 68)] = 1.0
        d = q[u, 0].float() / torch.linalg.norm(q[u, 0].float())
        for i in range(dominant if n > 100 else 0):
            j = off[u] + 70 + (n - 71) * i // dominant
            K[j] = (d * (4.0 * np.log(2) * i * 128 ** 0.5 / float(torch.linalg.norm(q[u, 0].float())))).to(torch.bfloat16)
            pi[j] = 1e-6
    rc = cache.RetainedCache(
        Kc=K, Vc=V, pic=pi, idxc=torch.zeros(rows, dtype=torch.int32, device="cuda"),
        count=torch.tensor(sizes, dtype=torch.int32, device="cuda"),
        status=torch.zeros(len(sizes), dtype=torch.int32, device="cuda"),
        cap_off=torch.from_numpy(off).cuda(), max_cap=max(max(sizes), 1))
    return rc, q


@pytest.mark.parametrize("sizes,G,dominant", [
    ([1], 1, 0),                                   # one row
    ([15, 16, 17, 0, 31, 32, 33, 255, 256, 257], 4, 0),   # tiles and waves with nothing to do
    ([2000, 3584, 129, 0, 3583], 1, 0),            # parts, the last of them short or empty
    ([3584, 700, 127], 8, 2),
    ([3585, 40, 0, 1500, 3000], 4, 0),             # one tile more
    ([13100] * 4, 4, 6),                           # parts with pivots added back in each
    ([13100, 6000, 97], 7, 6),
    ([9000] * 3, 8, 0),
    ([40000], 2, 9),                               # the most parts
    ([5000, 4999], 12, 3),                         # two head blocks
    ([70000, 1], 1, 0),
    ([3700] * 200, 4, 0),                          # more units than would leave room for parts
    ([600 + 7 * (u % 50) for u in range(300)], 4, 2),     # four waves per unit
    ([300 + 5 * (u % 50) for u in range(600)], 7, 0),     # a wave per unit
    ([1100] * 520 + [0] * 3, 8, 0),
    ([64 + u % 40 for u in range(1540)], 4, 0),    # a wave per unit
    ([2700] * 1536, 8, 0),                         # ... whose LDS would not hold it: four waves
])
def test_attend_library_plans(sizes, G, dominant):
    _say("attend plans units=%d longest=%d G=%d dominant=%d" % (len(sizes), max(sizes), G, dominant))
    from paper_2607_21475_amd import cache

    rc, q = _units(sizes, G, seed=len(sizes) + G, dominant=dominant)
    res = cache.attend_certify(rc, q)
    again = cache.attend_certify(rc, q)
    torch.cuda.synchronize()
    assert not _np(res["status"]).any()
    for k in ("y", "vhat", "lse", "b", "r"):  # a fixed order of sums
        assert torch.equal(res[k], again[k]), k
    off = _np(rc.cap_off)
    pick = sorted(set(np.linspace(0, len(sizes) - 1, 10).astype(int)) | {int(np.argmin(sizes))})
    for u in pick:
        sl = slice(int(off[u]), int(off[u]) + sizes[u])
        y = _np(res["y"][u]).astype(np.float64)
        if sizes[u] == 0:
            assert not y.any() and np.all(np.isneginf(_np(res["lse"][u])))
            continue
        ref = oracle.attend_certify(_bits(q[u]), _bits(rc.Kc[sl]), _bits(rc.Vc[sl]), _np(rc.pic[sl]))
        nrm = np.linalg.norm(ref["y"], axis=1)
        assert np.all(np.linalg.norm(y - ref["y"], axis=1) <= 1e-4 * nrm), u
        for key in ("vhat", "b", "r"):
            got, want = _np(res[key][u]).astype(np.float64), ref[key]
            assert np.all(np.abs(got - want) <= 1e-3 * np.maximum(np.abs(want), _cert_floor(key, nrm))), (u, key, got, want)
    if dominant:  # the last dominant row does dominate: yhat is its value to a few per cent
        u = int(np.argmax(sizes))
        j = int(off[u]) + 70 + (sizes[u] - 71) * (dominant - 1) // dominant
        v = bf16_to_f64(_bits(rc.Vc[j:j + 1]))[0]
        y = _np(res["y"][u, 0]).astype(np.float64)
        assert np.linalg.norm(y - v) < 0.2 * np.linalg.norm(v)


@pytest.mark.parametrize("sizes,G,dominant", [
    ([5000, 4097, 100, 0] + [16] * 146, 7, 3),      # 129 to 199 units: three parts of four waves
    ([5000, 4097, 100, 0] + [16] * 146, 6, 0),
    ([13000, 12400, 4400, 300] + [16] * 206, 4, 5),  # ... or four; 200 to 256 longer ones too
    ([17000, 8500] + [16] * 254, 8, 9),
    ([1400, 300] + [16] * 298, 4, 2),               # 257 to 383: five one-wave splits
    ([1400, 300] + [16] * 382, 4, 2),               # four waves from 384 on
    ([3000, 2999, 17] + [40] * 530, 4, 4),          # ... also of more than 512 units
    ([1900, 700] + [40] * 511, 8, 2),
    ([13400, 9000] + [16] * 520, 8, 3),             # eight: the LDS of four would be too much
    ([3000, 1600] + [40] * 900, 1, 3),              # two waves each, all of them resident
    ([2400, 1600] + [40] * 770, 2, 3),
    ([3500, 1200] + [40] * 960, 4, 3),
    ([2500, 1200] + [40] * 960, 4, 3),              # four
    ([1900, 1300] + [40] * 900, 8, 2),              # a wave per unit
    ([33000, 100] + [16] * 300, 2, 9),              # the longest: one-wave splits
    ([16500, 100] + [16] * 520, 3, 9),
    ([9000, 5000, 300] + [16] * 24600, 1, 6),       # two waves each of the most units
])
def test_attend_library_plans_of_many_units(sizes, G, dominant):
    """The plans of more than 128 units, on both sides of their lines; the host knows the longest unit only,
    so the others are short."""
    test_attend_library_plans(sizes, G, dominant)


@pytest.mark.parametrize("sizes,G", [([13100] * 2, 4), ([600] * 5, 7)])
def test_attend_library_plans_without_offset(sizes, G):
    """The uncorrected pass over the same plans: y and ln N of the plain retained softmax, the
    certificate unchanged."""
    from paper_2607_21475_amd import cache

    _say("attend plans without offset %s G=%d" % (sizes, G))
    rc, q = _units(sizes, G, seed=3)
    ref, res = cache.attend_certify(rc, q), cache.attend_certify(rc, q, offset=False)
    torch.cuda.synchronize()
    for k in ("vhat", "b", "r"):
        assert torch.equal(ref[k], res[k]), k
    off = _np(rc.cap_off)
    for u, n in enumerate(sizes):
        k = rc.Kc[off[u]:off[u] + n].double()
        lg = q[u].double() @ k.T.contiguous() / 128 ** 0.5
        y = torch.softmax(lg, 1) @ rc.Vc[off[u]:off[u] + n].double()
        assert torch.linalg.norm(res["y"][u].double() - y) <= 1e-4 * torch.linalg.norm(y)
        assert torch.all((res["lse"][u].double() - torch.logsumexp(lg, 1)).abs() <= 1e-4)


@pytest.mark.parametrize("units,n,split", [(4, 200, 0), (4, 9000, 0), (1540, 100, 0), (6, 400, 16), (6, 400, 64)])
def test_negative_counts_are_empty_units(units, n, split):
    """A unit whose count is negative holds no rows in every launch mode (waves sharing a unit, parts,
    a wave per unit, one-wave records, the caller's splits in one work-group): empty outputs, and no
    block contributions."""
    import paper_2607_21475_amd as ebd
    from paper_2607_21475_amd import cache

    _say("attend negative counts units=%d n=%d split=%d" % (units, n, split))
    rc, q = _units([n] * units, 4, seed=units)
    want = cache.attend_certify(rc, q, split_rows=split)
    rc.count[1::2] = torch.tensor([-1, -(2 ** 31)], dtype=torch.int32, device="cuda").repeat(units)[:units // 2]
    p = ebd.attend_params(units, 4, rc.max_cap, rc.cap_off, split)
    res = {k: torch.full_like(v, 7) for k, v in want.items() if k != "ws"}
    ebd.ebd_attend_certify(p, q, rc.Kc, rc.Vc, rc.pic, rc.count, res["y"], res["vhat"], res["lse"], want["ws"],
                           brange=res["b"], radius=res["r"], status=res["status"])
    blocks = torch.full((units, 8), 7.0, device="cuda")
    ebd.ebd_block_contributions(units, 4, 8, rc.max_cap, rc.cap_off, q, rc.Kc, rc.Vc, rc.pic, rc.idxc, rc.count,
                                res["y"], res["lse"], blocks)
    torch.cuda.synchronize()
    for k in ("y", "vhat", "lse", "b", "r"):
        assert torch.equal(res[k][0::2], want[k][0::2]), k
    for k in ("y", "vhat", "b", "r", "status"):
        assert not res[k][1::2].any(), k
    assert torch.all(torch.isneginf(res["lse"][1::2]))
    assert not blocks[1::2].any() and torch.all(blocks[0::2, 0] > 0)
