"""Attention over short and long prefixes, in few and many workgroups, against
float64 at the edges of the tiles of keys (32 at dh = 128, 64 at dh = 64), over
packed groups of every load width and over plain values, and the bits of a
prefix against those it has in a batch."""
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
    q[:, :, 0] *= 8                       # peaked softmax: the tiles' maxima differ
    # every other tile out of reach: scores of -inf for queries above 0 there
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


@pytest.mark.parametrize("dh,G,T", [(128, 8, 700), (128, 0, 700), (64, 16, 561), (64, 0, 300), (128, 32, 177)])
def test_bits_do_not_depend_on_the_batch(dh, G, T):
    """A prefix attended to in a large call has the bits it has by itself and
    in a micro-batch."""
    B, H, Tq = 40, 8, 5
    g = torch.Generator(device=DEV).manual_seed(T + dh + G)
    rn = lambda *s: torch.randn(s, generator=g, device=DEV).bfloat16()  # noqa: E731
    q, k = rn(B, Tq, H, dh) * 2, rn(B, T, H, dh)
    if G == 0:
        V = rn(B, H, T, dh)
        call = lambda b0, b1: rs.attend_values(q[b0:b1], k[b0:b1], V[b0:b1], out_dtype=torch.float32)  # noqa: E731
    else:
        R = torch.linalg.qr(torch.randn((H, dh, dh), generator=g, device=DEV))[0].bfloat16().contiguous()
        mask = torch.randint(0, 2 ** G, (B, T), generator=g, device=DEV).to(torch.uint32)
        off, Vp = rs.rotate_pack(rn(B, T, H, dh), R, mask, G, T * G)
        call = lambda b0, b1: rs.attend(q[b0:b1], k[b0:b1], mask[b0:b1], off[b0:b1], Vp[b0:b1], R, G,  # noqa: E731
                                        out_dtype=torch.float32)
    print(f"attend batch independence dh={dh} G={G} T={T}", flush=True)
    whole = call(0, B)
    for b0, b1 in ((0, 1), (7, 9), (8, 40), (39, 40)):
        assert torch.equal(call(b0, b1), whole[b0:b1]), (b0, b1)
