"""The full-width products at the edges of their tiles: 64 rows per group in the
rotation; 64 or (more than 1536 tokens) 256 routed tokens per values tile, whose
stages of 64 dims skip the groups that no row of the tile keeps; 64 and 128 rows
staged through registers where an operand is off 16-byte boundaries; and slots
past the cache's capacity."""
import pytest
import torch

import paper_2608_18410_amd as rs

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("H,S,B,T,keep", [
    (1, 1, 1, 1, 0.5),      # one group of one head, one token: two stages in all
    (8, 8, 1, 16, 0.5),     # two stages per group, a quarter of a tile
    (8, 4, 1, 63, 0.3),     # four stages per group, just under a tile of rows
    (6, 6, 3, 43, 0.7),     # two rows past two values tiles; group count not a multiple of 8
    (24, 8, 2, 65, 0.4),    # groups of 384 dims: six stages
    (8, 1, 2, 70, 0.5),     # one group: its routed tokens keep nothing
    (16, 2, 2, 64, 0.5),    # groups of 1024 dims, exactly two tiles of tokens
    (32, 32, 2, 33, 0.06),  # most groups with a few rows
    (32, 32, 1, 130, 0.9),  # nearly dense
])
@pytest.mark.parametrize("short", [False, True])
def test_full_products(H, S, B, T, keep, short):
    g = torch.Generator(device=DEV).manual_seed(1000 * H + 10 * S + T)
    dv, ds = H * 128, H * 128 // S
    v = torch.randn((B, T, H, 128), generator=g, device=DEV).bfloat16()
    R = (torch.randn((dv, dv), generator=g, device=DEV) * dv ** -0.5).bfloat16()
    kept = torch.rand((B, T, S), generator=g, device=DEV) < keep
    kept[:, T // 2] = True          # a value-space token per sample
    mask = (kept.long() << torch.arange(S, device=DEV)).sum(-1).to(torch.uint32)
    n = kept.sum((1, 2))
    cap = max(1, int(n.max()) - 2) if short else T * S
    print(f"full products H={H} S={S} B={B} T={T} cap={cap}", flush=True)
    off = torch.zeros((B, T + 1), dtype=torch.int32, device=DEV)
    Vp = torch.zeros((B, cap, ds), dtype=torch.bfloat16, device=DEV)
    rs.full_rotate_pack(v, rs.full_transpose(R), mask, S, cap, out=(off, Vp))
    Vh = rs.full_values(R, mask, off, Vp, S, H)
    torch.cuda.synchronize()

    full = kept.all(-1)
    v64, R64 = v.reshape(B, T, dv).double(), R.double()
    z = torch.where(full[..., None], v64, v64 @ R64).reshape(B, T, S, ds)
    want_off = torch.cat((torch.zeros((B, 1), device=DEV), kept.sum(-1).cumsum(1)), 1).int()
    assert torch.equal(off, want_off)
    for b in range(B):
        zb = z[b][kept[b]]
        m = min(cap, zb.shape[0])
        # one rounding to bf16 (2^-9 of the value) and f32 sums of dv products
        # (at most dv 2^-24 of their magnitudes' sum, which is below sqrt(dv) here)
        d = (Vp[b, :m].double() - zb[:m]).abs()
        assert (d <= 2.0 ** -8 * zb[:m].abs() + dv ** 1.5 * 2.0 ** -24).all()
        assert (Vp[b, m:] == 0).all()
        # the values step from the cache as stored (slots past it read as zero)
        zc = torch.zeros((T * S, ds), dtype=torch.float64, device=DEV)
        where = kept[b].reshape(-1).nonzero()[:m, 0]
        zc[where] = Vp[b, :m].double()
        zc = zc.reshape(T, dv)
        want = torch.where(full[b][:, None], zc, zc @ R64.T).reshape(T, H, 128).transpose(0, 1)
        d = (Vh[b].double() - want).abs()
        assert (d <= 2.0 ** -8 * want.abs() + dv ** 1.5 * 2.0 ** -24).all()


def _masks(B, T, S, routed, g, keep=0.5):
    """Masks of B samples with routed[b] routed tokens anywhere (each keeping a
    share of the groups, not all), the others keeping all."""
    kept = torch.rand((B, T, S), generator=g, device=DEV) < keep
    kept[..., 0] &= ~kept.all(-1)
    for b in range(B):
        order = torch.randperm(T, generator=g, device=DEV)
        kept[b, order[routed[b]:]] = True
    return kept, (kept.long() << torch.arange(S, device=DEV)).sum(-1).to(torch.uint32)


@pytest.mark.parametrize("H,S,B,T,total,keep,short", [
    (8, 8, 33, 65, 0, 0.5, False),       # no routed token: every tile returns
    (8, 8, 33, 65, 1, 0.5, False),
    (8, 8, 33, 65, 255, 0.5, False),     # a row short of a tile
    (8, 8, 33, 65, 256, 0.5, False),
    (8, 8, 33, 65, 257, 0.5, True),      # a tile of one row; slots past the capacity
    (8, 1, 33, 65, 600, 0.5, False),     # one group: the routed tokens keep nothing, no stage runs
    (8, 2, 25, 65, 900, 0.5, True),      # groups of 512 dims
    (16, 16, 20, 81, 1500, 0.02, False),  # tiles whose rows keep few groups: most stages skipped
    (6, 6, 300, 7, 2000, 0.9, False),    # many short samples, column tiles not a multiple of 8
])
def test_many_rows_match_single_samples_and_float64(H, S, B, T, total, keep, short):
    """More than 1536 tokens: values in 256-row tiles with copying waves, bit for
    bit what calls of one sample (64-row tiles) give, and within rounding of
    float64."""
    assert B * T > 1536
    g = torch.Generator(device=DEV).manual_seed(total + S)
    dv, ds = H * 128, H * 128 // S
    r = torch.randperm(B * T, generator=g, device=DEV)[:total] // T
    routed = torch.bincount(r, minlength=B).tolist()
    kept, mask = _masks(B, T, S, routed, g, keep)
    assert int((~kept.all(-1)).sum()) == total
    v = torch.randn((B, T, H, 128), generator=g, device=DEV).bfloat16()
    R = (torch.randn((dv, dv), generator=g, device=DEV) * dv ** -0.5).bfloat16()
    Rt = rs.full_transpose(R)
    cap = max(1, int(kept.sum((1, 2)).max()) - 2) if short else T * S
    new = lambda n: (torch.zeros((n, T + 1), dtype=torch.int32, device=DEV),  # noqa: E731
                     torch.zeros((n, cap, ds), dtype=torch.bfloat16, device=DEV))
    print(f"full products H={H} S={S} B={B} T={T} routed={total} cap={cap}", flush=True)
    off, Vp = rs.full_rotate_pack(v, Rt, mask, S, cap, out=new(B))
    Vh = rs.full_values(R, mask, off, Vp, S, H)
    full, R64 = kept.all(-1), R.double()
    for b in range(B):
        if b < 4 or b % 29 == 0:
            o1, p1 = rs.full_rotate_pack(v[b:b + 1], Rt, mask[b:b + 1], S, cap, out=new(1))
            assert torch.equal(o1[0], off[b]) and torch.equal(p1[0], Vp[b])
            assert torch.equal(rs.full_values(R, mask[b:b + 1], o1, p1, S, H)[0], Vh[b]), b
        # the cache as stored (slots past it read as zero), one rounding to bf16 and
        # float32 sums of dv products
        m = min(cap, int(off[b, -1]))
        zc = torch.zeros((T * S, ds), dtype=torch.float64, device=DEV)
        zc[kept[b].reshape(-1).nonzero()[:m, 0]] = Vp[b, :m].double()
        zc = zc.reshape(T, dv)
        want = torch.where(full[b][:, None], zc, zc @ R64.T).reshape(T, H, 128).transpose(0, 1)
        assert ((Vh[b].double() - want).abs() <= 2.0 ** -8 * want.abs() + dv ** 1.5 * 2.0 ** -24).all(), b


def _off16(t, shift=4):
    """The same values at an address 8 (or 2 shift) bytes off a 16-byte boundary."""
    buf = torch.empty(t.numel() + 8, dtype=t.dtype, device=t.device)
    out = buf[shift:shift + t.numel()].view(t.shape)
    out.copy_(t)
    assert out.data_ptr() % 16 == 2 * shift
    return out


def test_full_products_off_16_byte_boundaries():
    H, S, B, T = 8, 4, 2, 70
    g = torch.Generator(device=DEV).manual_seed(5)
    v = torch.randn((B, T, H, 128), generator=g, device=DEV).bfloat16()
    R = (torch.randn((H * 128, H * 128), generator=g, device=DEV) * 0.03).bfloat16()
    kept = torch.rand((B, T, S), generator=g, device=DEV) < 0.5
    mask = (kept.long() << torch.arange(S, device=DEV)).sum(-1).to(torch.uint32)
    Rt = rs.full_transpose(R)
    out = lambda: (torch.zeros((B, T + 1), dtype=torch.int32, device=DEV),  # noqa: E731
                   torch.zeros((B, T * S, H * 128 // S), dtype=torch.bfloat16, device=DEV))
    off, Vp = rs.full_rotate_pack(v, Rt, mask, S, T * S, out=out())
    Vh = rs.full_values(R, mask, off, Vp, S, H)
    for a, b in ((_off16(v), Rt), (v, _off16(Rt))):
        print("full products: operand 8 bytes off", flush=True)
        off2, Vp2 = rs.full_rotate_pack(a, b, mask, S, T * S, out=out())
        assert torch.equal(off2, off) and torch.equal(Vp2, Vp)
    for a, b in ((_off16(R), Vp), (R, _off16(Vp))):
        assert torch.equal(rs.full_values(a, mask, off, b, S, H), Vh)


@pytest.mark.parametrize("H,S,B,T,keep,short", [(1, 1, 1, 1, 0.5, False), (8, 1, 3, 43, 0.5, False), (8, 8, 2, 64, 0.4, True),
                                                (32, 32, 5, 77, 0.1, False), (6, 6, 3, 129, 0.0, False)])
@pytest.mark.parametrize("shift", [1, 4])
def test_register_staging_gives_the_bits_of_the_dma(H, S, B, T, keep, short, shift):
    """64-row rotation and 128-row values tiles staged through registers, at
    their edges: partial last tiles, two stages in all, no stage at all."""
    g = torch.Generator(device=DEV).manual_seed(10 * H + T)
    v = torch.randn((B, T, H, 128), generator=g, device=DEV).bfloat16()
    R = (torch.randn((H * 128, H * 128), generator=g, device=DEV) * 0.03).bfloat16()
    kept = torch.rand((B, T, S), generator=g, device=DEV) < keep
    mask = (kept.long() << torch.arange(S, device=DEV)).sum(-1).to(torch.uint32)
    cap = max(1, int(kept.sum((1, 2)).max()) - 2) if short else T * S
    Rt = rs.full_transpose(R)
    out = lambda: (torch.zeros((B, T + 1), dtype=torch.int32, device=DEV),  # noqa: E731
                   torch.zeros((B, cap, H * 128 // S), dtype=torch.bfloat16, device=DEV))
    print(f"register staging H={H} S={S} B={B} T={T} cap={cap} shift={shift}", flush=True)
    off, Vp = rs.full_rotate_pack(v, Rt, mask, S, cap, out=out())
    Vh = rs.full_values(R, mask, off, Vp, S, H)
    for a, b in ((_off16(v, shift), Rt), (v, _off16(Rt, shift))):
        off2, Vp2 = rs.full_rotate_pack(a, b, mask, S, cap, out=out())
        assert torch.equal(off2, off) and torch.equal(Vp2, Vp)
    for a, b in ((_off16(R, shift), Vp), (R, _off16(Vp, shift))):
        assert torch.equal(rs.full_values(a, mask, off, b, S, H), Vh)
