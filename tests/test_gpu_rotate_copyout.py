"""rotate_pack's copy-out against the separate rotation and pack (the same values,
so the same bytes): tiles inside one sample, tiles over several samples, slots
of 2, 4 and more dims at every alignment, and slots past the capacity."""
import pytest
import torch

import paper_2608_18410_amd as rs

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("dh,G", [(64, 32), (64, 16), (64, 8), (128, 32), (128, 16), (128, 8), (128, 1)])
@pytest.mark.parametrize("B,T", [(1, 1), (2, 15), (3, 16), (9, 7), (2, 33), (3, 177), (2, 600)])
@pytest.mark.parametrize("cut", [0, 1, 2, 37])
def test_copy_out(dh, G, B, T, cut):
    H = 8
    g = torch.Generator(device=DEV).manual_seed(T * 100 + G + cut)
    v = torch.randn((B, T, H, dh), generator=g, device=DEV).bfloat16()
    R = (torch.randn((H, dh, dh), generator=g, device=DEV) * dh ** -0.5).bfloat16()
    kept = torch.rand((B, T, G), generator=g, device=DEV) < 0.6
    kept[:, ::5] = False
    kept[:, 1::4] = True
    mask = (kept.long() << torch.arange(G, device=DEV)).sum(-1).to(torch.uint32)
    cap = max(1, int(kept.sum((1, 2)).max()) - cut)
    print(f"copy-out dh={dh} G={G} B={B} T={T} cap={cap}", flush=True)
    outs = []
    for fused in (True, False):
        off = torch.full((B, T + 1), -1, dtype=torch.int32, device=DEV)
        Vp = torch.full((B, H, cap, dh // G), 7.0, dtype=torch.bfloat16, device=DEV)
        if fused:
            rs.rotate_pack(v, R, mask, G, cap, out=(off, Vp))
        else:
            rs.pack_kv(rs.rotate_values(v, R), mask, G, cap, out=(off, Vp))
        outs.append((off, Vp))
    torch.cuda.synchronize()
    assert torch.equal(outs[0][0], outs[1][0])
    assert torch.equal(outs[0][1].view(torch.int16), outs[1][1].view(torch.int16))
