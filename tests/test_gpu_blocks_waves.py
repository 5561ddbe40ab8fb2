"""GPU parity of the block contributions where several waves share a unit: row counts around whole
tiles and waves, bins that leave room for fewer waves, positions in no order, appended rows, and
launches of many units (fewer waves each).  The bar is that of test_gpu_finegrain."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes,G,nb,block_rows", [
    ([1, 15, 16, 17, 0, 127, 128, 129, 400], 4, 96, 64),
    ([2000, 513], 7, 8192, 4),        # bins for two waves
    ([3000, 40], 1, 4096, 64),        # ... for four
    ([900, 700], 12, 64, 64),         # two head blocks
    ([700] * 3, 8, 1, 1 << 30),       # one block of everything
    ([100 + u % 60 for u in range(700)], 2, 64, 64),    # two waves per unit
    ([60 + u % 30 for u in range(2100)], 4, 64, 64),
    ([100 + u % 90 for u in range(256)], 3, 64, 64),    # six waves per unit, the most of so short ones
    ([100 + u % 90 for u in range(257)], 3, 64, 64),    # four from here
    ([100 + u % 90 for u in range(512)], 5, 2048, 1),   # ... to here
    ([100 + u % 90 for u in range(513)], 5, 8192, 1),   # a wave per unit, the most blocks
    ([512, 130] + [40] * 1022, 4, 4096, 1),             # four of up to 1024 long units
    ([511, 130] + [40] * 600, 7, 64, 16),               # three
    ([512, 130] + [40] * 700, 2, 4097, 1),              # a wave per unit
    ([20 + u % 30 for u in range(1030)], 1, 16, 4),
    ([20 + u % 30 for u in range(1030)], 3, 16, 4),
    ([20 + u % 30 for u in range(1030)], 6, 16, 4),
    ([20 + u % 30 for u in range(1030)], 8, 16, 4),
])
def test_block_contributions_over_waves(sizes, G, nb, block_rows):
    print("block contributions over waves: %d units, longest %d, G=%d, %d blocks" % (len(sizes), max(sizes), G, nb), flush=True)
    import paper_2607_21475_amd as ebd
    from paper_2607_21475_amd import cache

    g = torch.Generator(device="cuda").manual_seed(len(sizes) + G)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    rows, U = int(off[-1]), len(sizes)
    bf = dict(generator=g, device="cuda", dtype=torch.bfloat16)
    K, V, q = torch.randn((rows, 128), **bf), torch.randn((rows, 128), **bf), torch.randn((U, G, 128), **bf)
    pi = (torch.rand(rows, generator=g, device="cuda") * 1.2 + 0.02).clamp(max=1.0)
    # positions in no order, some past the last block, some appended (-1)
    top = min(nb * block_rows * 21 // 20, 2 ** 31 - 1)
    idx = torch.randint(-1, top, (rows,), generator=g, device="cuda").to(torch.int32)
    rc = cache.RetainedCache(Kc=K, Vc=V, pic=pi, idxc=idx, max_cap=max(sizes),
                             count=torch.tensor(sizes, dtype=torch.int32, device="cuda"),
                             status=torch.zeros(U, dtype=torch.int32, device="cuda"),
                             cap_off=torch.from_numpy(off).cuda())
    res = cache.attend_certify(rc, q)
    outs = []
    for _ in range(2):
        blocks = torch.full((U, nb), float("nan"), device="cuda")
        ebd.ebd_block_contributions(U, G, nb, rc.max_cap, rc.cap_off, q, K, V, pi, idx, rc.count,
                                    res["y"], res["lse"], blocks, block_rows=block_rows)
        outs.append(blocks)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1])  # each wave's bins are its own, summed in order
    got = outs[0].cpu().numpy().astype(np.float64)
    bits = synth.bf16_bits
    for u in sorted(set(np.linspace(0, U - 1, 12).astype(int))):
        sl = slice(int(off[u]), int(off[u + 1]))
        ref = oracle.block_contributions(bits(q[u]), bits(K[sl]), bits(V[sl]), pi[sl].cpu().numpy(),
                                         idx[sl].cpu().numpy(), res["y"][u].cpu().numpy().astype(np.float64),
                                         res["lse"][u].cpu().numpy().astype(np.float64), nb, block_rows)
        tol = 1e-3 * np.abs(ref) + 1e-7 * max(ref.max(initial=0.0), 1e-30)
        assert np.all(np.abs(got[u] - ref) <= tol), u
