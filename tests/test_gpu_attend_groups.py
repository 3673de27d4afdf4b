"""Attention with two groups of waves per workgroup (at most 256 workgroups,
384 keys or more at dh = 128, 256 at dh = 64) against float64, at the edges of that rule and of the
tiles, over packed groups of every load width and over plain values."""
import math

import pytest
import torch

import paper_2608_18410_amd as rs

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("dh,G", [(64, 32), (64, 16), (64, 4), (128, 32), (128, 8), (128, 0)])
@pytest.mark.parametrize("B,H,Tq,T", [(1, 4, 8, 127), (1, 4, 8, 128), (1, 8, 56, 129), (2, 8, 70, 255), (1, 8, 64, 256),
                                      (2, 8, 65, 257), (4, 8, 57, 305), (32, 8, 5, 385), (33, 8, 5, 385), (1, 8, 20, 383),
                                      (1, 8, 20, 384), (1, 8, 3, 1023)])
def test_attend_groups(dh, G, B, H, Tq, T):
    g = torch.Generator(device=DEV).manual_seed(T + dh + G)
    rn = lambda *s: torch.randn(s, generator=g, device=DEV).bfloat16()  # noqa: E731
    q, k, v = rn(B, Tq, H, dh), rn(B, T, H, dh), rn(B, T, H, dh)
    q[:, :, 0] *= 8                       # peaked softmax: the two groups' maxima differ
    # tokens of the second group's tiles out of reach: scores of -inf for queries above 0 there
    tk = 32 if dh == 128 else 64
    hole = (torch.arange(T, device=DEV) // tk % 2) == 1
    q[0, :, 1, 0] = 1.0
    k[0, hole, 1, 0] = -math.inf
    print(f"attend groups dh={dh} G={G} B={B} H={H} Tq={Tq} T={T}", flush=True)
    if G == 0:
        got = rs.attend_values(q, k, v.transpose(1, 2).contiguous(), out_dtype=torch.float32)
        u = v.double().transpose(1, 2)
    else:
        R = torch.linalg.qr(torch.randn((H, dh, dh), generator=g, device=DEV))[0].bfloat16().contiguous()
        kept = torch.rand((B, T, G), generator=g, device=DEV) < 0.6
        mask = (kept.long() << torch.arange(G, device=DEV)).sum(-1).to(torch.uint32)
        off, Vp = rs.rotate_pack(v, R, mask, G, T * G)
        got = rs.attend(q, k, mask, off, Vp, R, G, out_dtype=torch.float32)
        # the cache as stored, back in place
        z = torch.zeros((B, H, T * G, dh // G), dtype=torch.float64, device=DEV)
        for b in range(B):
            n = int(kept[b].sum())
            z[b][:, kept[b].reshape(-1)] = Vp[b, :, :n].double()
        u = torch.matmul(z.reshape(B, H, T, dh), R.double().transpose(1, 2))
    s = torch.matmul(q.double().transpose(1, 2), k.double().permute(0, 2, 3, 1)) / math.sqrt(dh)
    want = torch.matmul(torch.softmax(s, -1), u).transpose(1, 2)
    # bf16 probabilities and, before the rotation back, bf16 sums: 2^-9 of each
    # in norm, with head room for their largest values
    err = (got.double() - want).abs().max() / want.abs().max()
    assert err < 1e-2, err
