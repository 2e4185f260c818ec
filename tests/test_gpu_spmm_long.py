"""Aggregation with hub rows: rows longer than 128 entries are summed in 16 parts, shared by the
waves of a block (wide features) or the lane groups of a wave (narrow ones).

The sum of a row of k entries in any order has error <= (k + 1) 2^-24 sum |a||x|."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

LENS = [127, 128, 129, 0, 300, 1, 1025, 2500]   # the first rows; the rest have 0 to 6 entries


def _matrix(n, seed):
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, 7, n)
    place = rng.permutation(n)[:len(LENS)] if seed % 2 else np.arange(len(LENS))
    lens[place] = LENS
    rows = [np.sort(rng.choice(n, size=k, replace=False)) for k in lens]
    col = np.concatenate(rows).astype(np.int32)
    rp = np.zeros(n + 1, np.int32)
    rp[1:] = np.cumsum(lens)
    return rp, col, rng.standard_normal(len(col)).astype(np.float32), lens


@pytest.mark.parametrize("width", [1, 3, 8, 17, 64, 100, 130, 256, 602])
@pytest.mark.parametrize("n,seed", [(2501, 0), (4000, 1), (2507, 2)])
def test_hub_rows(width, n, seed):
    import torch
    from paper_2102_10424_amd import gist as G
    print(f"n={n} width={width} seed={seed}", flush=True)
    rp, col, val, lens = _matrix(n, seed)
    assert len(col) <= 16 * n
    d = [torch.from_numpy(x).cuda() for x in (rp, col, val)]
    A = G.csr_dev(n, len(col), *d)
    g = torch.Generator(device="cuda").manual_seed(seed)
    H = torch.randn(n, width, generator=g, device="cuda")
    W = torch.randn(width, 5, generator=g, device="cuda")
    desc = G.layer_desc(G.GIST_LAYER_GCN, G.GIST_ACT_NONE, n, width, 5, order=G.GIST_ORDER_AGG_FIRST)
    ws = torch.empty(max(*G.gist_layer_workspace_size(desc), 1), dtype=torch.uint8, device="cuda")
    agg, out = torch.full_like(H, 7.0), torch.empty(n, 5, device="cuda")
    G.gist_gcn_layer_fwd(G.Context(0), desc, A, H, W, agg, out, ws)
    S = torch.sparse_csr_tensor(d[0].long(), d[1].long(), d[2].double(), (n, n))
    T = torch.sparse_csr_tensor(d[0].long(), d[1].long(), d[2].abs().double(), (n, n))
    k = torch.from_numpy(lens).cuda().double()[:, None] + 1
    err = (agg.double() - S @ H.double()).abs()
    assert bool((err <= k * 2.0 ** -24 * (T @ H.abs().double()) + 1e-30).all())


def test_infinities_stay_in_their_rows():
    """The padded gathers of a short batch repeat the row's last entry and are not added: an
    infinite neighbour gives exactly an infinite sum, not NaN."""
    import torch
    from paper_2102_10424_amd import gist as G
    n = 300
    for width in (3, 64, 200):
        rp = torch.arange(n + 1, dtype=torch.int32, device="cuda")
        col = torch.arange(n, dtype=torch.int32, device="cuda")
        val = torch.full((n,), 0.5, device="cuda")
        H = torch.ones(n, width, device="cuda")
        H[7], H[8] = float("inf"), -float("inf")
        desc = G.layer_desc(G.GIST_LAYER_GCN, G.GIST_ACT_NONE, n, width, 5, order=G.GIST_ORDER_AGG_FIRST)
        ws = torch.empty(max(*G.gist_layer_workspace_size(desc), 1), dtype=torch.uint8, device="cuda")
        agg, out = torch.empty_like(H), torch.empty(n, 5, device="cuda")
        W = torch.ones(width, 5, device="cuda")
        G.gist_gcn_layer_fwd(G.Context(0), desc, G.csr_dev(n, n, rp, col, val), H, W, agg, out, ws)
        assert torch.equal(agg, H * 0.5)


def _many_hubs(n, seed):
    """Long rows next to each other and scattered: several of them share a block, a wave and a
    wave's lane groups, whether a block's rows are neighbours or lie apart; the last rows are
    long too (a partly filled block)."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, 3, n)
    lens[:40] = rng.integers(100, 420, 40)
    lens[rng.permutation(np.arange(40, n))[:90]] = rng.integers(129, 200, 90)
    lens[-3:] = 257, 1, 130
    rows = [np.sort(rng.choice(n, size=k, replace=False)) for k in lens]
    rp = np.zeros(n + 1, np.int32)
    rp[1:] = np.cumsum(lens)
    return rp, np.concatenate(rows).astype(np.int32), rng.standard_normal(int(rp[-1])).astype(np.float32), lens


def _dev(G, n, m, pad=1):
    """The matrix on the GPU with room for ``pad`` times its entries, and the tensors it points to."""
    import torch
    rp, col, val, _ = m
    cap = pad * len(col)
    c, v = torch.zeros(cap, dtype=torch.int32, device="cuda"), torch.zeros(cap, device="cuda")
    c[:len(col)], v[:len(col)] = torch.from_numpy(col).cuda(), torch.from_numpy(val).cuda()
    r = torch.from_numpy(rp).cuda()
    return G.csr_dev(n, cap, r, c, v), (r, c, v)


def _off(t, k):
    """A copy of t that starts k floats past a 16-byte boundary."""
    import torch
    b = torch.empty(t.numel() + k, device="cuda")
    v = b[k:].view(t.shape)
    v.copy_(t)
    return v


@pytest.mark.parametrize("width", [4, 17, 34, 64, 100, 256, 300])
@pytest.mark.parametrize("n", [2507, 700])
def test_sum_order_depends_on_the_row_alone(width, n):
    """The same entries give the same bits however many the descriptor has room for (below and
    beyond 16 per row: rows apart or together), at every alignment of the features (16-, 8- and
    4-byte loads), and as columns of a wider matrix; and the sums are right."""
    import torch
    from paper_2102_10424_amd import gist as G
    print(f"n={n} width={width}", flush=True)
    m = _many_hubs(n, n)
    g = torch.Generator(device="cuda").manual_seed(n + width)
    H = torch.randn(n, width, generator=g, device="cuda")
    Hw = torch.randn(n, 3 * width + 1, generator=g, device="cuda")
    Hw[:, width:2 * width] = H
    ctx = G.Context(0)

    def agg(H, pad):
        w = H.shape[1]
        A, keep = _dev(G, n, m, pad)
        W = torch.zeros(w, 1, device="cuda")
        d = G.layer_desc(G.GIST_LAYER_GCN, G.GIST_ACT_NONE, n, w, 1, order=G.GIST_ORDER_AGG_FIRST)
        ws = torch.empty(max(*G.gist_layer_workspace_size(d), 1), dtype=torch.uint8, device="cuda")
        out, z = torch.full_like(H, 7.0), torch.empty(n, 1, device="cuda")
        G.gist_gcn_layer_fwd(ctx, d, A, H, W, out, z, ws)
        torch.cuda.synchronize()
        del keep
        return out
    first = agg(H, 1)
    rp, col, val = (torch.from_numpy(x).cuda() for x in m[:3])
    S = torch.sparse_csr_tensor(rp.long(), col.long(), val.double(), (n, n))
    T = torch.sparse_csr_tensor(rp.long(), col.long(), val.abs().double(), (n, n))
    k = torch.from_numpy(m[3]).cuda().double()[:, None] + 1
    err = (first.double() - S @ H.double()).abs()
    assert bool((err <= k * 2.0 ** -24 * (T @ H.abs().double()) + 1e-30).all())
    for pad in (1, 40):
        for off in (0, 1, 2):
            assert torch.equal(agg(_off(H, off), pad), first), (pad, off)
    assert torch.equal(agg(Hw, 1)[:, width:2 * width], first)


@pytest.mark.parametrize("kind", ["gcn", "sage"])
@pytest.mark.parametrize("off", [0, 1, 2])
@pytest.mark.parametrize("si,so", [(64, 96), (20, 40), (256, 300)])
def test_masked_gradient_of_hub_rows(kind, off, si, so):
    """GIST_LAYER_MASK_DH on hub rows (with SAGE's Add): bitwise the plain call's dH with the
    entries whose H <= 0 set to zero, also where H's alignment allows narrower loads only than the
    plain call's operands; and within rounding of the exact gradient."""
    import torch
    from paper_2102_10424_amd import gist as G
    n = 2507
    print(f"{kind} off={off} {si}x{so}", flush=True)
    m = _many_hubs(n, 5)
    AT, keep = _dev(G, n, m)
    g = torch.Generator(device="cuda").manual_seed(9)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")   # noqa: E731
    sage = kind == "sage"
    H, W, dZ, a = _off(r(n, si), off), r(2 * si if sage else si, so), r(n, so), r(n, si)
    out = []
    for flags in (0, G.GIST_LAYER_MASK_DH):
        d = G.layer_desc(G.GIST_LAYER_SAGE_MEAN if sage else G.GIST_LAYER_GCN, G.GIST_ACT_NONE, n, si, so,
                         order=G.GIST_ORDER_AGG_FIRST, flags=flags)
        ws = torch.empty(max(*G.gist_layer_workspace_size(d), 1), dtype=torch.uint8, device="cuda")
        dW, dH = torch.empty_like(W), torch.full((n, si), 7.0, device="cuda")
        G.gist_gcn_layer_bwd(G.Context(0), d, AT, AT, H, a, None, W, dZ, dW, dH, ws)
        torch.cuda.synchronize()
        out.append(dH)
    plain, masked = out
    assert torch.equal(masked, torch.where(H > 0, plain, torch.zeros_like(plain)))
    S, T = (torch.sparse_csr_tensor(keep[0].long(), keep[1].long(), v.double(), (n, n))
            for v in (keep[2], keep[2].abs()))
    Wn, Ws = (W[si:].double(), W[:si].double()) if sage else (W.double(), None)
    z = dZ.double()
    exact, size = S @ (z @ Wn.t()), T @ (z.abs() @ Wn.abs().t())
    if sage:
        exact, size = exact + z @ Ws.t(), size + z.abs() @ Ws.abs().t()
    # a row's sum of at most 420 terms, each a product's sum of so terms with the bound of a plain fp32 one
    bound = (422 + so) * 2.0 ** -24 * size
    assert bool(((plain.double() - exact).abs() <= bound).all())


def test_relu_of_hub_rows():
    """The forward of a transform-first layer: ReLU in the aggregation's store."""
    import torch
    from paper_2102_10424_amd import gist as G
    n, si = 2507, 30
    m = _many_hubs(n, 6)
    A, keep = _dev(G, n, m)
    g = torch.Generator(device="cuda").manual_seed(10)
    S, T = (torch.sparse_csr_tensor(keep[0].long(), keep[1].long(), v.double(), (n, n))
            for v in (keep[2], keep[2].abs()))
    for so in (7, 64, 260):
        H, W = (torch.randn(*s, generator=g, device="cuda") for s in ((n, si), (si, so)))
        d = G.layer_desc(G.GIST_LAYER_GCN, G.GIST_ACT_RELU, n, si, so, order=G.GIST_ORDER_XFORM_FIRST)
        ws = torch.empty(max(*G.gist_layer_workspace_size(d), 1), dtype=torch.uint8, device="cuda")
        out = torch.empty(n, so, device="cuda")
        G.gist_gcn_layer_fwd(G.Context(0), d, A, H, W, None, out, ws)
        t = H.double() @ W.double()
        bound = (422 + si) * 2.0 ** -24 * (T @ (H.abs().double() @ W.abs().double()))
        assert bool(((out.double() - torch.relu(S @ t)).abs() <= bound).all()), so
