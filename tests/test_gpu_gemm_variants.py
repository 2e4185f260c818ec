"""Every instantiation of the dense product kernels, through the layer calls.

The graph's matrix is diagonal with powers of two, so the aggregations are exact and every product
has a plain fp64 reference; with bf16 inputs the reference rounds the operands first (nearest
even), so that both types are held to fp32 level: one lost or doubled value of K, or one wrong
element of 4,096 x 4,096, is at least 100 times the bound.

Each case names the kernels that its products take (the library's profiler reports them): the
operands' orientations, the tile and the floats per load of each.  All 72 are in the table: KK,
KR, RR; 256, 128 and 64 wide tiles; 16-, 8- and 4-byte loads, mixed ones for the small kernels;
and for every tile and type whole and cut tiles with each store (ReLU, SGD step, mask, the
two outputs of a GraphSAGE input gradient), groups, and GraphSAGE's concatenation off and on
the tile and K step.  A rounding bound: each of the at most 2 K / 16 + 512 additions to a sum rounds
by an rms of 0.42 2^-24 of it, 6e-7 of the result at K = 8,192; 2e-6 is asked for.
"""

import pytest

pytestmark = pytest.mark.gpu

CASES = [
    # kind, n, s_in, s_out, groups, bf16 inputs, floats W and dZ lie past a 16-byte boundary, fused SGD, kernels
    ("gcn", 1304, 20, 3168, 3, 0, 0, 0, 1, "KK_64x64_v44 KR_256x256_v44 RR_64x64_v44"),
    ("sage", 2, 3008, 4, 1, 0, 0, 2, 1, "KK_64x64_v22 KR_64x64_v44 RR_64x64_v22"),
    ("sage", 3, 93, 4289, 3, 0, 0, 0, 0, "KK_64x64_v11 KR_64x64_v11 RR_128x128_v11"),
    ("sage", 91, 2744, 2432, 1, 0, 0, 0, 0, "KK_128x128_v44 KR_128x128_v44 RR_256x256_v44"),
    ("sage", 98, 1274, 2491, 2, 0, 0, 2, 1, "KK_128x128_v11 KR_128x128_v11 RR_256x256_v11"),
    ("sage", 400, 3840, 3840, 1, 0, 2, 0, 0, "KK_128x128_v22 KR_128x128_v22 RR_256x256_v44"),
    ("sage", 555, 64, 8, 1, 0, 0, 1, 0, "KK_64x64_v14 KR_64x64_v44 RR_64x64_v41"),
    ("sage", 718, 4236, 2, 1, 0, 0, 1, 0, "KK_128x128_v11 KR_64x64_v22 RR_64x64_v41"),
    ("sage", 1274, 1724, 3766, 2, 0, 0, 0, 0, "KK_128x128_v22 KR_256x256_v22 RR_256x256_v22"),
    ("sage", 1686, 64, 2554, 2, 0, 2, 0, 0, "KK_64x64_v22 KR_128x128_v22 RR_64x64_v22"),
    ("sage", 1784, 1342, 5, 3, 0, 0, 1, 1, "KK_256x256_v11 KR_64x64_v11 RR_64x64_v11"),
    ("sage", 2407, 256, 1672, 3, 0, 2, 1, 1, "KK_128x128_v11 KR_256x256_v22 RR_128x128_v11"),
    ("sage", 3196, 3584, 2478, 1, 0, 1, 2, 1, "KK_128x128_v11 KR_256x256_v11 RR_256x256_v22"),
    ("sage", 3778, 3422, 1210, 1, 0, 0, 1, 0, "KK_256x256_v11 KR_256x256_v22 RR_128x128_v11"),
    ("sage", 3840, 3840, 400, 1, 0, 2, 0, 1, "KK_256x256_v22 KR_128x128_v22 RR_128x128_v44"),
    ("sage", 4034, 4, 1136, 3, 0, 1, 0, 1, "KK_64x64_v41 KR_256x256_v11 RR_64x64_v44"),
    ("sage", 4260, 126, 746, 2, 0, 0, 0, 1, "KK_128x128_v22 KR_128x128_v22 RR_128x128_v22"),
    ("xform", 2, 484, 2160, 3, 0, 1, 0, 1, "KK_64x64_v41 KR_64x64_v41 RR_128x128_v44"),
    ("xform", 552, 3, 16, 2, 0, 0, 2, 0, "KK_64x64_v44 KR_64x64_v14 RR_64x64_v14"),
    ("xform", 1374, 2494, 3, 1, 0, 0, 0, 0, "KK_128x128_v11 KR_64x64_v11 RR_64x64_v11"),
    ("xform", 1672, 3210, 2536, 3, 0, 2, 0, 0, "KK_256x256_v22 KR_256x256_v22 RR_256x256_v22"),
    ("xform", 1972, 3856, 4, 2, 0, 0, 0, 1, "KK_256x256_v44 KR_64x64_v44 RR_64x64_v44"),
    ("xform", 3340, 102, 1280, 3, 0, 0, 0, 0, "KK_128x128_v44 KR_256x256_v22 RR_128x128_v22"),
    ("sage", 5, 4, 3, 1, 1, 1, 1, 0, "KK_64x64_v11 KR_64x64_v41 RR_64x64_v41"),
    ("sage", 18, 64, 4, 1, 1, 0, 1, 0, "KK_64x64_v14 KR_64x64_v44 RR_64x64_v41"),
    ("sage", 334, 270, 4091, 3, 1, 0, 0, 1, "KK_128x128_v11 KR_128x128_v11 RR_256x256_v11"),
    ("sage", 346, 1792, 1708, 1, 1, 2, 0, 1, "KK_128x128_v22 KR_128x128_v22 RR_128x128_v44"),
    ("sage", 470, 1937, 4, 2, 1, 0, 1, 0, "KK_128x128_v14 KR_64x64_v14 RR_64x64_v11"),
    ("sage", 609, 3840, 3840, 1, 1, 2, 0, 0, "KK_256x256_v22 KR_256x256_v22 RR_256x256_v44"),
    ("sage", 1256, 668, 4, 2, 1, 0, 0, 0, "KK_128x128_v44 KR_64x64_v44 RR_64x64_v44"),
    ("sage", 1865, 2520, 247, 1, 1, 2, 0, 1, "KK_256x256_v11 KR_128x128_v41 RR_128x128_v41"),
    ("sage", 2472, 2426, 898, 1, 1, 2, 2, 0, "KK_256x256_v22 KR_256x256_v22 RR_256x256_v22"),
    ("sage", 2488, 4, 3776, 3, 1, 0, 2, 0, "KK_64x64_v22 KR_256x256_v44 RR_128x128_v22"),
    ("sage", 2870, 64, 589, 2, 1, 1, 1, 0, "KK_64x64_v11 KR_128x128_v41 RR_64x64_v41"),
    ("sage", 3568, 1728, 10, 1, 1, 0, 0, 1, "KK_256x256_v22 KR_64x64_v22 RR_64x64_v22"),
    ("sage", 3832, 64, 3636, 2, 1, 0, 0, 1, "KK_128x128_v44 KR_256x256_v44 RR_64x64_v44"),
    ("sage", 3840, 3840, 609, 1, 1, 0, 0, 1, "KK_256x256_v11 KR_256x256_v11 RR_256x256_v11"),
    ("xform", 10, 2378, 2436, 2, 1, 1, 1, 0, "KK_64x64_v41 KR_64x64_v11 RR_256x256_v22"),
    ("xform", 14, 3, 16, 1, 1, 0, 0, 1, "KK_64x64_v44 KR_64x64_v14 RR_64x64_v14"),
    ("xform", 214, 3599, 398, 3, 1, 0, 0, 1, "KK_128x128_v22 KR_64x64_v11 RR_128x128_v11"),
    ("xform", 1692, 3116, 652, 3, 1, 1, 2, 0, "KK_256x256_v11 KR_128x128_v41 RR_128x128_v44"),
    ("xform", 1718, 3, 3044, 1, 1, 0, 0, 1, "KK_64x64_v44 KR_128x128_v14 RR_64x64_v14"),
    ("xform", 2748, 3848, 448, 1, 1, 0, 0, 1, "KK_256x256_v44 KR_128x128_v44 RR_128x128_v44"),
    ("xform", 3840, 401, 3840, 1, 1, 1, 0, 0, "KK_128x128_v41 KR_256x256_v11 RR_128x128_v14"),
]


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available()
    from paper_2102_10424_amd import gist as G
    return torch, G, G.Context(0)


def test_the_table_has_every_kernel():
    want = set()
    for o in ("KK", "KR", "RR"):
        want |= {f"f32_{o}_{t}_v{v}" for t in ("256x256", "128x128", "64x64") for v in ("44", "22", "11")}
        want |= {f"bf16_{o}_{t}_v{v}" for t in ("256x256", "128x128", "64x64") for v in ("44", "22", "11")}
        want |= {f"{t}_v{v}".replace("#", o) for t in ("f32_#_64x64", "bf16_#_128x128", "bf16_#_64x64")
                 for v in ("41", "14")}
    have = {f"{'bf16' if c[5] else 'f32'}_{k}" for c in CASES for k in c[9].split()}
    assert have == want


@pytest.mark.parametrize("kind,n,si,so,groups,bf16,ow,oz,sgd,kernels", CASES)
def test_products(env, kind, n, si, so, groups, bf16, ow, oz, sgd, kernels):
    torch, G, ctx = env
    print(kind, n, si, so, groups, "bf16" if bf16 else "f32", kernels, flush=True)
    g = torch.Generator(device="cuda").manual_seed(n + si + so)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")   # noqa: E731

    def past(t, k):
        b = torch.empty(t.numel() + k, device="cuda")
        b[k:].copy_(t.reshape(-1))
        return b[k:].view(t.shape)
    sage = kind == "sage"
    rows = 2 * si if sage else si
    H, W, dZ = r(n, groups * si), past(r(groups, rows, so) * 0.05, ow), past(r(n, groups * so), oz)
    d = torch.pow(2.0, torch.randint(-2, 3, (n, 1), generator=g, device="cuda").float())
    rp = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    dv = d.reshape(-1).contiguous()
    A = G.csr_dev(n, n, rp, rp, dv)
    desc = [G.layer_desc(G.GIST_LAYER_SAGE_MEAN if sage else G.GIST_LAYER_GCN, G.GIST_ACT_RELU, n, si, so, bf16,
                         order=G.GIST_ORDER_XFORM_FIRST if kind == "xform" else G.GIST_ORDER_AGG_FIRST,
                         groups=groups, flags=f)
            for f in (0, G.GIST_LAYER_DZ_IN | G.GIST_LAYER_MASK_DH)]
    need = max(*G.gist_layer_workspace_size(desc[0]), *G.gist_layer_workspace_size(desc[1]), 1)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    agg, out, dH = torch.empty_like(H), torch.full((n, groups * so), 7.0, device="cuda"), torch.full_like(H, 7.0)
    W0, dW, lr = W.clone(), torch.full_like(W, 7.0), 0.5
    G.gist_profile_begin(ctx)
    G.gist_gcn_layer_fwd(ctx, desc[0], A, H, W, agg, out, ws)
    if sgd:
        G.gist_gcn_layer_bwd_sgd(ctx, desc[1], A, A, H, agg, None, W, dZ, lr, dH, ws)
    else:
        G.gist_gcn_layer_bwd(ctx, desc[1], A, A, H, agg, None, W, dZ, dW, dH, ws)
    names = set(G.gist_profile_read(ctx)[0])
    G.gist_profile_end(ctx)
    want = {f"gemm_{'bf16' if bf16 else 'f32'}_{k}" for k in kernels.split()}
    assert want <= names, (want - names, names)

    def check(what, got, exact, size=None, bound=2e-6):
        rel = float((got.double() - exact).norm() / (exact if size is None else size).norm())
        assert rel < bound, (what, rel)
    op = lambda t: (t.bfloat16() if bf16 else t).double()   # noqa: E731
    for k in range(groups):
        h, z = H[:, k * si:(k + 1) * si], dZ[:, k * so:(k + 1) * so]
        w, dd = op(W0[k]), d.double()
        if kind == "xform":
            y, x, t = dd * (op(h) @ w), op(h), op(d * z)
            p = t @ w.t()
        else:
            x = torch.cat([op(h), op(d * h)], 1) if sage else op(d * h)
            y, t = x @ w, op(z)
            p = t @ w.t()
            p = p[:, :si] + dd * p[:, si:] if sage else dd * p
        check("forward", out[:, k * so:(k + 1) * so], torch.relu(y), y)
        gw = x.t() @ t
        if sgd:   # one rounding of the updated weight beside the gradient's
            check("W", W[k], W0[k].double() - lr * gw, lr * gw, 3e-6)
        else:
            check("dW", dW[k], gw)
        check("dH", dH[:, k * si:(k + 1) * si], torch.where(h > 0, p, torch.zeros_like(p)), p)
