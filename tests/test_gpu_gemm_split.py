"""The fp32 products on the bf16 matrix cores (three bf16 parts per value, six
products), through the layer calls of the C ABI with the identity as the
graph's matrix, so that the forward is H W, dW = H^T dZ, dH = dZ W^T.

Bounds.  A product's dropped terms are below 3 * 2^-25 |a b|, and each of the
at most 12 additions per 16 values of K, and of the additions of K parts,
rounds by at most 2^-24 of a partial sum, itself at most |A||B|; hence
|error| <= (12 ceil(K/16) + 1100) 2^-24 |A||B| elementwise for any input.
Random signs keep the normwise error orders below that: 2e-6 is held too, the
level of a plain fp32 product.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available()
    from paper_2102_10424_amd import gist as G
    return torch, G, G.Context(0)


def _layer(env, H, W, dZ):
    torch, G, ctx = env
    n, si = H.shape
    so = W.shape[1]
    rp = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    one = torch.ones(n, device="cuda")
    A = G.csr_dev(n, n, rp, rp, one)
    d = G.layer_desc(G.GIST_LAYER_GCN, G.GIST_ACT_NONE, n, si, so, order=G.GIST_ORDER_AGG_FIRST)
    ws = torch.empty(max(*G.gist_layer_workspace_size(d), 1), dtype=torch.uint8, device="cuda")
    agg, out = torch.empty_like(H), torch.full((n, so), 7.0, device="cuda")
    dW, dH = torch.full_like(W, 7.0), torch.full_like(H, 7.0)
    G.gist_gcn_layer_fwd(ctx, d, A, H, W, agg, out, ws)
    G.gist_gcn_layer_bwd(ctx, d, A, None, H, agg, out, W, dZ, dW, dH, ws)
    torch.cuda.synchronize()
    return out, dW, dH


def _check(torch, got, A, B, what):
    """got against A B in fp64."""
    A, B = A.double(), B.double()
    exact = A @ B
    K = A.shape[1]
    bound = (12 * ((K + 15) // 16) + 1100) * 2.0 ** -24 * (A.abs() @ B.abs())
    err = (got.double() - exact).abs()
    assert bool((err <= bound).all()), (what, float((err - bound).max()))
    rel = float(err.norm() / exact.norm())
    print(f"{what}: K={K} rel {rel:.2e}", flush=True)
    assert rel < 2e-6, (what, rel)


# edges of the 64 / 128 tiles and of the 16 / 64 K steps, odd and even strides, a
# K beyond 4,096 (parts of alternating sign), a long reduction (the 256 tile and
# every load width: test_gpu_gemm_variants)
SHAPES = [(1, 1, 1), (63, 64, 65), (65, 63, 64), (129, 15, 130), (127, 130, 47), (255, 602, 66),
          (257, 256, 258), (1030, 8, 1030), (300, 4500, 40), (40, 17, 4500), (70001, 20, 33),
          (1630, 1024, 4096), (3100, 602, 1023)]


@pytest.mark.parametrize("n,si,so", SHAPES)
def test_products_fp32_level(env, n, si, so):
    torch = env[0]
    print(f"n={n} si={si} so={so}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n + si + so)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")   # noqa: E731
    H, W, dZ = r(n, si), r(si, so) * 0.05, r(n, so)
    out, dW, dH = _layer(env, H, W, dZ)
    _check(torch, out, H, W, "forward")
    _check(torch, dW, H.t(), dZ, "dW")
    _check(torch, dH, dZ, W.t(), "dH")


@pytest.mark.parametrize("n,si,so", [(70, 40, 50), (700, 1100, 600), (1630, 512, 4096)])
def test_nonfinite_and_extreme_values(env, n, si, so):
    """Inf, NaN and values that round to Inf in bf16 give what fp32 arithmetic gives,
    in their own row only; the other rows keep fp32 accuracy."""
    torch = env[0]
    g = torch.Generator(device="cuda").manual_seed(3)
    H = torch.randn(n, si, generator=g, device="cuda")
    W = torch.rand(si, so, generator=g, device="cuda") * 0.01 + 0.001   # positive: Inf stays Inf
    dZ = torch.randn(n, so, generator=g, device="cuda")
    H[3, 5], H[9, 0], H[20, 7], H[31, 2], H[32, 1] = (float("inf"), float("nan"), -float("inf"),
                                                      3.4e38, -3.39e38)
    H[40, 3], H[40, 4] = float("inf"), -float("inf")
    out, _, _ = _layer(env, H, W, dZ)
    assert bool(torch.isposinf(out[3]).all()) and bool(torch.isneginf(out[20]).all())
    assert bool(torch.isnan(out[9]).all()) and bool(torch.isnan(out[40]).all())
    keep = torch.ones(n, dtype=torch.bool, device="cuda")
    keep[[3, 9, 20, 40]] = False
    exact = H[keep].double() @ W.double()
    rel = ((out[keep].double() - exact).norm(dim=1) / exact.norm(dim=1)).max()
    assert float(rel) < 2e-6, float(rel)


@pytest.mark.parametrize("scale", [1e-30, 1e-18, 1e18])
def test_small_and_large_magnitudes(env, scale):
    torch = env[0]
    g = torch.Generator(device="cuda").manual_seed(4)
    H = torch.randn(200, 300, generator=g, device="cuda") * scale
    W, dZ = torch.randn(300, 150, generator=g, device="cuda"), torch.randn(200, 150, generator=g, device="cuda")
    out, dW, _ = _layer(env, H, W, dZ)
    for got, a, b in ((out, H, W), (dW, H.t(), dZ)):
        exact = a.double() @ b.double()
        assert float((got.double() - exact).norm() / exact.norm()) < 2e-6


def test_long_reduction_has_no_bias(env):
    """The unit's sums round toward minus infinity on average; parts of alternating sign
    cancel it: the mean error over a long reduction stays far below its spread."""
    torch = env[0]
    g = torch.Generator(device="cuda").manual_seed(5)
    H = torch.randn(400000, 64, generator=g, device="cuda")
    dZ = torch.randn(400000, 64, generator=g, device="cuda")
    W = torch.randn(64, 64, generator=g, device="cuda")
    _, dW, _ = _layer(env, H, W, dZ)
    err = dW.double() - H.double().t() @ dZ.double()
    # 4,096 independent errors of equal spread: the mean of unbiased ones exceeds 6 standard
    # errors (6 / 64 of the spread) with probability 2e-9
    assert abs(float(err.mean())) < 6.0 / 64 * float(err.std()) + 1e-12
    exact = H.double().t() @ dZ.double()
    assert float(err.norm() / exact.norm()) < 2e-6


def test_strides_beyond_32_bit_tiles(env):
    """A row stride of 2^22 floats: 255 rows of it pass 32-bit offsets."""
    torch = env[0]
    s = 1 << 22
    g = torch.Generator(device="cuda").manual_seed(6)
    H = torch.randn(3, s, generator=g, device="cuda")
    W, dZ = torch.randn(s, 2, generator=g, device="cuda"), torch.randn(3, 2, generator=g, device="cuda")
    out, dW, dH = _layer(env, H, W, dZ)
    _check(torch, dW, H.t(), dZ, "dW")
    _check(torch, dH, dZ, W.t(), "dH")
    exact = H.double() @ W.double()
    assert float((out.double() - exact).norm() / exact.norm()) < 2e-6
