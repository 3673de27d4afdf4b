"""The float32 matrix-core rotation and attention against the float64 oracle at
the edges of their 16-token tiles, waves and runs."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2608_18410_amd as rs
import synth
from tests._gpu_util import DEV, host, max_rel, put, put_mask, synth_pack_inputs

pytestmark = pytest.mark.gpu

# float32 sums of up to T + 2 dh products; the repository's float32 bar is 1e-4
# of the largest value, rounding alone stays below 64 * 2^-24 = 4e-6
TOL = 4e-6


def _case(B, T, Tq, H, dh, G, seed):
    w = synth.workload(1).replace(B=B, H=H, dh=dh, G=G, n_vis=T, n_lang=0, n_prop=0, Tq=Tq, k_vis=max(1, G // 2), seed=seed)
    rng = np.random.default_rng(seed)
    R = np.stack([synth.haar_orthogonal(rng, dh) for _ in range(H)]).astype(np.float32)
    v = rng.standard_normal((B, T, H, dh)).astype(np.float32)
    _, mask = synth_pack_inputs(w, B)
    mask[:, :: 5] = 0                      # tokens that keep no group
    mask[:, 1:: 7] = (1 << G) - 1          # and tokens that keep all
    return rng, R, v, mask


@pytest.mark.parametrize("B,T,H,dh,G", [(1, 1, 1, 64, 1), (1, 15, 4, 64, 32), (3, 17, 4, 128, 32), (2, 64, 3, 128, 1),
                                        (5, 129, 8, 128, 8), (33, 130, 16, 64, 4), (40, 130, 8, 128, 16)])
def test_rotate_f32(B, T, H, dh, G):
    rng, R, v, mask = _case(B, T, 1, H, dh, G, T + dh)
    z_ref = O.rotate(v, R)
    print(f"rotate f32 B={B} T={T} H={H} dh={dh} G={G}", flush=True)
    z = rs.rotate_values(put(v, torch.float32), put(R, torch.float32))
    cap = int(O.popcount(mask).sum(1).max()) + 3
    Vp = torch.full((B, H, cap, dh // G), 7.0, device=DEV)
    off = torch.full((B, T + 1), -1, dtype=torch.int32, device=DEV)
    rs.rotate_pack(put(v, torch.float32), put(R, torch.float32), put_mask(mask), G, cap, out=(off, Vp))
    torch.cuda.synchronize()
    assert max_rel(host(z), z_ref) <= TOL
    o_ref, p_ref = O.pack(host(z).astype(np.float64), mask, G, cap)
    assert np.array_equal(host(off), o_ref)
    got = host(Vp)
    for b in range(B):   # the rotation's own bits at the packed slots, later slots untouched
        n = o_ref[b, T]
        assert np.array_equal(got[b, :, :n], p_ref[b, :, :n].astype(np.float32))
        assert np.all(got[b, :, n:] == 7.0)
    short = max(1, cap // 2)
    Vs = torch.full((B, H, short, dh // G), 7.0, device=DEV)
    rs.rotate_pack(put(v, torch.float32), put(R, torch.float32), put_mask(mask), G, short, out=(off, Vs))
    torch.cuda.synchronize()
    assert torch.equal(Vs, Vp[:, :, :short])      # slots past the capacity are dropped
    assert np.array_equal(host(off), o_ref)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("B,T,Tq,H,dh,G,scale", [(1, 1, 1, 1, 64, 8, 0.0), (1, 16, 17, 3, 64, 32, 0.0),
                                                 (2, 63, 16, 4, 128, 4, 0.0), (2, 64, 17, 4, 64, 8, 0.0), (2, 64, 2, 8, 128, 16, 0.0), (3, 65, 33, 8, 128, 32, -0.3),
                                                 (1, 200, 5, 8, 128, 1, 0.5), (2, 129, 70, 5, 64, 2, 0.0)])
def test_attend_f32(B, T, Tq, H, dh, G, scale, causal):
    Tq = T if causal else Tq
    rng, R, v, mask = _case(B, T, Tq, H, dh, G, T + G)
    q = rng.standard_normal((B, Tq, H, dh)).astype(np.float32)
    k = rng.standard_normal((B, T, H, dh)).astype(np.float32)
    cap = max(1, int(O.popcount(mask).sum(1).max()))
    off, Vp = O.pack(O.rotate(v, R).astype(np.float32).astype(np.float64), mask, G, cap)
    print(f"attend f32 B={B} T={T} Tq={Tq} H={H} dh={dh} G={G} scale={scale} causal={causal}", flush=True)
    args = (put(q, torch.float32), put(k, torch.float32), put_mask(mask),
            torch.from_numpy(off.astype(np.int32)).to(DEV), put(Vp, torch.float32), put(R, torch.float32), G)
    got = (rs.attend_causal if causal else rs.attend)(*args, scale=scale)
    torch.cuda.synchronize()
    ref = (O.attend_packed_causal if causal else O.attend_packed)(q, k, mask, off, Vp, R, G, scale or None)
    assert max_rel(host(got), ref) <= TOL


@pytest.mark.parametrize("dh,G,T,t", [(64, 8, 40, 21), (64, 32, 33, 0), (128, 8, 47, 15), (128, 32, 16, 14), (128, 1, 90, 80)])
@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan")])
def test_causal_f32_nonfinite_value_reaches_its_own_queries_only(dh, G, T, t, bad):
    """An Inf or NaN cached for token t leaves the queries before t as they are
    (bit for bit) and reaches every query from t on."""
    H, ds, dim = 3, dh // G, dh - 3
    g = torch.Generator(device=DEV).manual_seed(T)
    rn = lambda *s: torch.randn(s, generator=g, device=DEV)  # noqa: E731
    R = torch.linalg.qr(rn(H, dh, dh))[0].contiguous()
    mask = torch.full((1, T), (1 << G) - 1, dtype=torch.int64, device=DEV).to(torch.uint32)
    q, k = rn(1, T, H, dh), rn(1, T, H, dh)
    off, Vp = rs.rotate_pack(rn(1, T, H, dh), R, mask, G, T * G)
    clean = rs.attend_causal(q, k, mask, off, Vp, R, G)
    Vp[0, 1, t * G + dim // ds, dim % ds] = bad
    print(f"causal f32 {bad} at token {t} of {T}, dh={dh} G={G}", flush=True)
    got = rs.attend_causal(q, k, mask, off, Vp, R, G)
    assert torch.equal(got[:, :t], clean[:, :t]) and torch.equal(got[:, :, ::2], clean[:, :, ::2])
    want = (R[1, :, dim] * bad).expand(T - t, dh)   # R_h of that dim's multiple
    assert torch.equal(got[0, t:, 1].nan_to_num(7.0, 8.0, 9.0), want.nan_to_num(7.0, 8.0, 9.0))
