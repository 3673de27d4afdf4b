"""The two-kernel router (products split over tiles and slices of the hidden
size, then a finishing kernel) against the float64 oracle at the edges of its
tiles, row blocks, stages and alignment rules, and against the allocation-free
call, which runs the same sums over ranges of samples."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2608_18410_amd as rs
import synth
from tests._gpu_util import DEV, host, host_mask, put, put_u8, tdtype

pytestmark = pytest.mark.gpu

# float32 sums of d terms of unit variance: rounding grows like sqrt(d) * 2^-24,
# 4e-6 of the largest score at d = 4096; four times that
TOL = 1.6e-5


def _weights(w, kind, rng):
    d, G, C, de, Hr = w.d, w.G, w.C, w.d_e, w.Hr
    n = lambda *s, f: synth.round_to(rng.standard_normal(s) * f ** -0.5, w.dtype)  # noqa: E731
    if kind == "mlp2":
        fin = 2 * d + de
        return dict(W_r=n(C, d, f=d), b_r=n(C, f=d), E=n(C, de, f=1), W1=n(Hr, fin, f=fin), b1=n(Hr, f=fin),
                    W2=n(G, Hr, f=Hr), b2=n(G, f=Hr))
    return dict(W_tok=n(G, d, f=d), b_tok=n(G, f=d), W_r=n(C, d, f=d), b_r=n(C, f=d), W_role=n(G, C, f=C),
                W_lang=n(G, d, f=d), b_lang=n(G, f=d))


def _router(kind, wt, dt):
    make = rs.Router.mlp2 if kind == "mlp2" else rs.Router.additive
    return make(**{k: put(v, dt) for k, v in wt.items()})


def _outs(B, T, G):
    return {"mask": torch.full((B, T), -1, dtype=torch.int32, device=DEV),
            "idx": torch.full((B, T, G), 7, dtype=torch.uint8, device=DEV),
            "count": torch.full((B, T), 9, dtype=torch.uint8, device=DEV),
            "scores": torch.full((B, T, G), float("nan"), dtype=torch.float32, device=DEV)}


@pytest.mark.parametrize("dtype,kind,B,n_vis,n_lang,d,Hr,G,C,de,shift", [
    ("bf16", "mlp2", 1, 1, 0, 64, 128, 8, 4, 8, 0),         # one token, no language tokens
    ("bf16", "mlp2", 1, 40, 24, 4096, 128, 8, 8, 128, 0),   # exactly one tile
    ("bf16", "mlp2", 5, 8, 5, 1024, 128, 32, 16, 64, 0),    # 65 tokens, a tile over five samples
    ("bf16", "mlp2", 3, 50, 14, 712, 17, 5, 17, 8, 0),      # ragged columns, rows and roles
    ("bf16", "mlp2", 2, 33, 7, 640, 300, 16, 3, 16, 0),     # several row chunks
    ("bf16", "mlp2", 2, 33, 7, 100, 20, 7, 3, 6, 0),        # unaligned rows
    ("bf16", "mlp2", 2, 33, 7, 512, 128, 8, 8, 64, 1),      # unaligned hidden states
    ("bf16", "mlp2", 2, 70, 9, 1001, 128, 8, 8, 64, 0),     # rows of a whole number of stages and nine columns
    ("bf16", "mlp2", 1, 70, 9, 71, 33, 5, 17, 3, 3),        # rows that end in seven columns
    ("bf16", "additive", 2, 100, 9, 131, 0, 16, 6, 0, 1),   # three columns
    ("f32", "mlp2", 2, 60, 9, 1003, 128, 8, 8, 64, 1),      # float32: three columns
    ("f32", "additive", 1, 70, 9, 33, 0, 17, 3, 0, 3),      # one column in a stage of its own
    ("bf16", "mlp2", 30, 130, 20, 512, 128, 8, 8, 64, 0),   # past the two-kernel range: one-kernel forms
    ("bf16", "mlp2", 20, 130, 30, 1024, 128, 16, 8, 64, 0),  # so many, split-K
    ("bf16", "mlp2", 30, 130, 20, 512, 128, 8, 8, 64, 1),   # so many, unaligned hidden states
    ("bf16", "mlp2", 30, 130, 20, 512, 128, 8, 8, 4, 0),    # so many, unaligned rows of W1
    ("bf16", "additive", 2, 120, 9, 4096, 0, 16, 6, 0, 0),
    ("bf16", "additive", 3, 40, 9, 520, 0, 32, 40, 0, 0),   # five row blocks
    ("bf16", "additive", 1, 17, 0, 33, 0, 1, 1, 0, 0),      # one group, odd hidden size
    ("bf16", "additive", 300, 50, 14, 64, 0, 8, 4, 0, 0),   # many tiles, one slice
    ("f32", "mlp2", 2, 100, 29, 1000, 128, 8, 8, 124, 0),   # column blocks of 256: ragged
    ("f32", "mlp2", 2, 13, 4, 257, 40, 9, 5, 3, 0),         # unaligned rows
    ("f32", "mlp2", 300, 80, 20, 64, 128, 8, 4, 8, 0),      # more tiles than one launch holds
    ("f32", "additive", 2, 61, 3, 2048, 0, 16, 6, 0, 0),
])
def test_route_tiles(dtype, kind, B, n_vis, n_lang, d, Hr, G, C, de, shift):
    rng = np.random.default_rng(d + G)
    k = tuple(int(x) for x in rng.integers(0, G + 1, 2)) + (G, G)
    w = synth.workload(2).replace(B=B, dtype=dtype, d=d, Hr=Hr, G=G, C=C, d_e=de, n_vis=n_vis, n_lang=n_lang, n_prop=0)
    wt = _weights(w, kind, rng)
    router = _router(kind, wt, tdtype(w))
    hv = synth.round_to(rng.standard_normal((B, w.T, d)), dtype)
    types = np.broadcast_to(w.types(), (B, w.T)).copy()
    types[:, rng.permutation(w.T)] = types.copy()  # language tokens anywhere in the prefix
    buf = torch.empty(hv.size + shift, dtype=tdtype(w), device=DEV)
    h = buf[shift:].view(hv.shape).copy_(put(hv, tdtype(w)))
    budget = rs.make_budget(rs.TOPK, k)
    print(f"route tiles {dtype} {kind} B={B} T={w.T} d={d} Hr={Hr} G={G} C={C} shift={shift}", flush=True)
    a = rs.route(put_u8(types), budget, G, h=h, router=router, out=_outs(B, w.T, G))
    torch.cuda.synchronize()
    if kind == "mlp2":
        ref = O.router_mlp2(hv, types, *(wt[n] for n in ("W_r", "b_r", "E", "W1", "b1", "W2", "b2")))
    else:
        ref = O.router_additive(hv, types, *(wt[n] for n in ("W_tok", "b_tok", "W_r", "b_r", "W_role", "W_lang", "b_lang")),
                                0.1, 0.1)
    got = host(a["scores"])
    assert float(np.max(np.abs(got - ref)) / np.max(np.abs(ref))) <= TOL
    # the selection, exactly, on the scores that the call gave
    want = O.select_groups(got, O.group_budget(got, types, O.TOPK, k, G))
    idx, cnt = O.mask_to_idx(want, G)
    assert np.array_equal(host_mask(a["mask"]), want)
    assert np.array_equal(host(a["idx"]), idx) and np.array_equal(host(a["count"]), cnt)
    b = rs.route_noalloc(put_u8(types), budget, G, h=h, router=router, out=_outs(B, w.T, G))
    torch.cuda.synchronize()
    for n in ("mask", "idx", "count"):
        assert torch.equal(a[n], b[n])
    assert np.array_equal(got.view(np.uint32), host(b["scores"]).view(np.uint32))


def test_route_noalloc_ranges_of_samples():
    # 400 samples at d = 4096: the pooled states alone take most of the
    # allocation-free call's array, so it runs ranges of samples, in the same bits
    B, T, d, G = 400, 2, 4096, 16
    w = synth.workload(2).replace(B=B, dtype="f32", d=d, G=G, C=6, n_vis=1, n_lang=1, n_prop=0)
    router = _router("additive", _weights(w, "additive", np.random.default_rng(1)), torch.float32)
    h = torch.randn((B, T, d), generator=torch.Generator(device=DEV).manual_seed(1), device=DEV)
    types = put_u8(np.broadcast_to(w.types(), (B, T)).copy())
    budget = rs.make_budget(rs.THRESHOLD, tau=0.0, kmin=1, kmax=G)
    print("route_noalloc over ranges of samples", flush=True)
    a = rs.route(types, budget, G, h=h, router=router, out=_outs(B, T, G))
    b = rs.route_noalloc(types, budget, G, h=h, router=router, out=_outs(B, T, G))
    torch.cuda.synchronize()
    for n in ("mask", "idx", "count", "scores"):
        assert torch.equal(a[n], b[n])


@pytest.mark.parametrize("B,n_vis,n_lang,d,G,C", [(20, 128, 48, 4096, 8, 8),   # split-K form
                                                  (40, 60, 21, 1024, 16, 6),   # split-K form, three samples a tile
                                                  (20, 128, 48, 896, 8, 8),    # split-K form, shortest hidden size
                                                 (20, 128, 48, 640, 16, 8),   # single kernel, ragged column blocks
                                                 (16, 200, 48, 512, 32, 16),  # 32 groups
                                                  (80, 30, 12, 768, 8, 5),     # short prefixes, ragged column blocks
                                                  (80, 30, 12, 64, 8, 1)])     # one stage of the hidden size
def test_scores_do_not_depend_on_the_batch(B, n_vis, n_lang, d, G, C):
    """One call over many prefixes (one-kernel router forms) gives the bits of
    calls over a few of them (two-kernel form), and of the no-alloc call."""
    w = synth.workload(2).replace(B=B, d=d, G=G, C=C, d_e=64 if C * 64 <= d else 8, n_vis=n_vis, n_lang=n_lang, n_prop=0)
    router = _router("mlp2", _weights(w, "mlp2", np.random.default_rng(d)), torch.bfloat16)
    h = torch.randn((B, w.T, d), generator=torch.Generator(device=DEV).manual_seed(d), device=DEV).bfloat16()
    types = put_u8(np.broadcast_to(w.types(), (B, w.T)).copy())
    budget = rs.make_budget(rs.TOPK, (G // 2, G // 2, G, G))
    pri = torch.ones(C, dtype=torch.bfloat16, device=DEV)
    print(f"batch independence B={B} T={w.T} d={d} G={G} C={C}", flush=True)
    a = rs.route(types, budget, G, h=h, router=router)
    pa = rs.route_allocate(types, (1, 1, G, G), G, h, router, pri)["priority"]
    n = rs.route_noalloc(types, budget, G, h=h, router=router, out=_outs(B, w.T, G))
    for b0 in range(0, B, 9):
        b1 = min(B, b0 + 9)
        b = rs.route(types[b0:b1], budget, G, h=h[b0:b1], router=router)
        pb = rs.route_allocate(types[b0:b1], (1, 1, G, G), G, h[b0:b1], router, pri)["priority"]
        torch.cuda.synchronize()
        for name in ("mask", "idx", "count", "scores"):
            assert torch.equal(a[name][b0:b1], b[name]) and torch.equal(n[name][b0:b1], b[name]), name
        assert torch.equal(pa[b0:b1], pb)


@pytest.mark.parametrize("what,de", [("h", 64), ("W1", 64), ("W_r", 64), ("E", 64), ("", 4)])
def test_scores_do_not_depend_on_the_batch_off_16_bytes(what, de):
    """The same with one operand off 16-byte boundaries: every number of tokens
    takes the form that loads it through registers."""
    B, G, C, d = 40, 8, 8, 1024
    w = synth.workload(2).replace(B=B, d=d, G=G, C=C, d_e=de, n_vis=100, n_lang=20, n_prop=0)

    def put_off(a, shift):
        return torch.empty(a.size + shift, dtype=torch.bfloat16, device=DEV)[shift:].view(a.shape).copy_(put(a, torch.bfloat16))

    wt = _weights(w, "mlp2", np.random.default_rng(d))
    router = rs.Router.mlp2(**{k: put_off(v, 3 if k == what else 0) for k, v in wt.items()})
    h = put_off(synth.round_to(np.random.default_rng(1).standard_normal((B, w.T, d)), "bf16"), 1 if what == "h" else 0)
    types = put_u8(np.broadcast_to(w.types(), (B, w.T)).copy())
    budget = rs.make_budget(rs.TOPK, (G // 2, G // 2, G, G))
    print(f"batch independence, {what or 'rows'} off 16 bytes, d_e={de}", flush=True)
    a = rs.route(types, budget, G, h=h, router=router)
    n = rs.route_noalloc(types, budget, G, h=h, router=router, out=_outs(B, w.T, G))
    for b0, b1 in ((0, 9), (9, 30), (39, 40)):
        b = rs.route(types[b0:b1], budget, G, h=h[b0:b1], router=router)
        torch.cuda.synchronize()
        for name in ("mask", "idx", "count", "scores"):
            assert torch.equal(a[name][b0:b1], b[name]) and torch.equal(n[name][b0:b1], b[name]), name


@pytest.mark.parametrize("polls", [None, "0"])
@pytest.mark.parametrize("B,T,G", [(33, 96, 8),     # every tile is one whole sample
                                   (32, 97, 8),     # tiles straddle samples
                                   (49, 64, 8),     # tiles over three samples
                                   (38, 81, 16),    # the full-width prefix
                                   (16, 200, 16),   # 16 groups, ragged last tile
                                   (9, 349, 32)])   # 32 groups
def test_split_k_matches_single_kernel_past_the_two_kernel_range(B, T, G, polls, monkeypatch):
    """The split-K form (more than 3072 tokens, a hidden size above 768) against
    the single kernel, which the allocation-free call runs: the same bits, also
    on a second call on the same workspace, whether the halves of a tile share
    its epilogue or the first leaves it to the other."""
    if polls is not None:
        monkeypatch.setenv("ROLESUB_SK_POLLS", polls)
    d, C = 1024, 8
    w = synth.workload(2).replace(B=B, d=d, G=G, C=C, d_e=64, n_vis=T - 20, n_lang=20, n_prop=0)
    router = _router("mlp2", _weights(w, "mlp2", np.random.default_rng(T)), torch.bfloat16)
    h = torch.randn((B, T, d), generator=torch.Generator(device=DEV).manual_seed(T), device=DEV).bfloat16()
    types = put_u8(np.broadcast_to(w.types(), (B, T)).copy())
    budget = rs.make_budget(rs.TOPK, (G // 2, G // 2, G, G))
    ws = torch.empty(rs.route_workspace_size(B, T, G, d, router), dtype=torch.uint8, device=DEV)
    print(f"split-K router vs single kernel: B={B} T={T} G={G} polls={polls}", flush=True)
    a = rs.route(types, budget, G, h=h, router=router, workspace=ws, out=_outs(B, T, G))
    a2 = rs.route(types, budget, G, h=h, router=router, workspace=ws, out=_outs(B, T, G))
    b = rs.route_noalloc(types, budget, G, h=h, router=router, out=_outs(B, T, G))
    torch.cuda.synchronize()
    for r in (a2, b):
        for name in ("mask", "idx", "count", "scores"):
            assert torch.equal(r[name], a[name]), name
    assert bool(torch.isfinite(a["scores"]).all())


@pytest.mark.parametrize("B,T", [(300, 1), (330, 2), (230, 12), (250, 12)])
def test_route_noalloc_of_many_short_samples(B, T):
    """Samples whose pooled states leave the array room for the products of all
    tokens (300 x 1: two-kernel form) or not (the single kernel): the bits of the
    call on a workspace, which runs the two-kernel form."""
    d, G, C = 4096, 8, 8
    w = synth.workload(2).replace(B=B, d=d, G=G, C=C, d_e=64, n_vis=T - T // 3, n_lang=T // 3, n_prop=0)
    router = _router("mlp2", _weights(w, "mlp2", np.random.default_rng(B)), torch.bfloat16)
    h = torch.randn((B, T, d), generator=torch.Generator(device=DEV).manual_seed(B), device=DEV).bfloat16()
    types = put_u8(np.broadcast_to(w.types(), (B, T)).copy())
    budget = rs.make_budget(rs.TOPK, (4, 6, G, G))
    print(f"route_noalloc, {B} samples of {T}", flush=True)
    a = rs.route(types, budget, G, h=h, router=router, out=_outs(B, T, G))
    b = rs.route_noalloc(types, budget, G, h=h, router=router, out=_outs(B, T, G))
    torch.cuda.synchronize()
    for n in ("mask", "idx", "count", "scores"):
        assert torch.equal(a[n], b[n])
