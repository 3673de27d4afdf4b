"""Token retention at the edges of its two forms (192 tokens), its chunks of 256 tokens and of the keys kept in
registers (1024), with ties, NaN, infinities, both zeros and denormals: the
kept indices are those of a stable descending sort."""
import numpy as np
import pytest
import torch

import paper_2608_18410_amd as rs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 3, 64, 65, 191, 192, 193, 255, 256, 257, 1023, 1024, 1025, 1400, 8192])
@pytest.mark.parametrize("kind", ["gauss", "ties", "special", "equal"])
def test_retain_edges(n, kind):
    r = np.random.default_rng(n)
    B, pad = 3, 5                                        # a segment before and after the tested one
    N = n + 2 * pad
    x = r.standard_normal((B, N)).astype(np.float32)
    if kind == "ties":
        x = np.round(x * 2).astype(np.float32) / 2       # many equal keys, both zeros
    elif kind == "special":
        x = r.choice(np.array([np.nan, np.inf, -np.inf, 0.0, -0.0, 1e-45, -1e-45, 3.4e38, -3.4e38, 1.0], np.float32), (B, N))
    elif kind == "equal":
        x[:] = 0.25
    for keep in sorted({0, 1, n // 3, n - 1, n}):
        print(f"retain n={n} {kind} keep={keep}", flush=True)
        got = rs.retain_tokens(torch.from_numpy(x).cuda(), [pad, n, pad], [pad, keep, 0]).cpu().numpy()
        seg = x[:, pad:pad + n]
        # NaN below every number; a stable sort leaves equal keys in index order
        key = np.where(np.isnan(seg), -np.inf, seg).astype(np.float64)
        key[np.isneginf(seg)] = -1e300
        order = np.argsort(-key, axis=1, kind="stable")[:, :keep]
        want = np.concatenate((np.tile(np.arange(pad), (B, 1)), np.sort(order, axis=1) + pad), axis=1)
        assert np.array_equal(got, want)
