"""Units cut into records: the lengths where the library begins to cut, and the finalize with its
records in LDS or, past what that holds, read from the workspace."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_attend_units import _units
from test_gpu_parity import _bits, _cert_floor, _np, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes,G,dominant,split", [
    ([1535, 1536, 1537, 769, 0, 15], 4, 2, 0),     # two parts of eight waves from 1536 rows
    ([1552] * 128, 1, 0, 0),
    ([2304, 2303, 100], 8, 6, 0),                  # ... three
    ([160, 144, 17], 2, 1, 16),                    # one-wave records, in LDS
    ([1720, 900, 1], 3, 6, 16),                    # ... 108 of them: the most that LDS holds
    ([1824, 1760, 1], 3, 6, 16),                   # ... 114: read from the workspace
])
def test_attend_records(sizes, G, dominant, split):
    _say("attend records sizes=%s G=%d split=%d" % (sizes[:6], G, split))
    from paper_2607_21475_amd import cache

    rc, q = _units(sizes, G, seed=7 + G, dominant=dominant)
    res = cache.attend_certify(rc, q, split_rows=split)
    torch.cuda.synchronize()
    assert not _np(res["status"]).any()
    off = _np(rc.cap_off)
    for u in range(min(len(sizes), 6)):
        sl = slice(int(off[u]), int(off[u]) + sizes[u])
        y = _np(res["y"][u]).astype(np.float64)
        if sizes[u] == 0:
            assert not y.any() and np.all(np.isneginf(_np(res["lse"][u])))
            continue
        ref = oracle.attend_certify(_bits(q[u]), _bits(rc.Kc[sl]), _bits(rc.Vc[sl]), _np(rc.pic[sl]))
        nrm = np.linalg.norm(ref["y"], axis=1)
        # the bars of test_gpu_attend_units: fp32 sums of exact products against fp64
        assert np.all(np.linalg.norm(y - ref["y"], axis=1) <= 1e-4 * nrm), u
        for key in ("vhat", "b", "r"):
            got, want = _np(res[key][u]).astype(np.float64), ref[key]
            assert np.all(np.abs(got - want) <= 1e-3 * np.maximum(np.abs(want), _cert_floor(key, nrm))), (u, key)
