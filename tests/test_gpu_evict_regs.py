"""The register kernels of the sampler, which large launches of units up to 6144 tokens take: every
variant (2, 4, 8 and 12 groups of 4 tokens per thread) at its edges, in every design, against the oracle."""
import pytest
import torch

import oracle
import synth
from test_gpu_parity import _check_evict, _evict, _np, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("design", [oracle.DESIGN_POISSON, oracle.DESIGN_SYSTEMATIC, oracle.DESIGN_TOPK,
                                    oracle.DESIGN_UNIFORM])
@pytest.mark.parametrize("longest", [1024, 1025, 2048, 2049, 4096, 4097, 6144])
def test_evict_register_kernels(longest, design):
    _say("evict registers longest=%d design=%d" % (longest, design))
    lengths = [16] * 765 + [0, 1, 69, 511, longest - 1, longest // 2 + 1, longest]
    K, V, seq_off = synth.make_cache(lengths, seed=3, device="cuda")
    sc = torch.exp(torch.randn(K.shape[0], generator=torch.Generator(device="cuda").manual_seed(4), device="cuda"))
    kw = dict(budget_frac=0.3, seed=9, design=design)
    out, again = (_evict(K, V, seq_off, sc, lengths, **kw) for _ in range(2))
    _check_evict(lengths, K, V, seq_off, sc, out, budget=0.3, seed=9, design=design)
    off, cnt = _np(out.cap_off), _np(out.count)
    for k in ("count", "status", "lam", "pi_full"):
        assert torch.equal(getattr(out, k), getattr(again, k)), k
    for u in range(760, len(lengths)):
        rows = slice(int(off[u]), int(off[u] + min(cnt[u], off[u + 1] - off[u])))
        for k in ("Kc", "Vc", "pic", "idxc"):
            assert torch.equal(getattr(out, k)[rows], getattr(again, k)[rows]), (u, k)
