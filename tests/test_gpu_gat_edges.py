"""GPU parity of the graph attention layer at the edges of its kernels'
ranges: feature widths around the register-kept row of the edge gradient (4,
one group, a group and a remainder, 1,024 the widest kept, 1,028 beyond), odd
widths (scalar loads), rows beyond the 512 kept entries, both activations; and
every entry of the mirror map is written, also where the pattern has none."""

import numpy as np
import pytest

from gpu_util import FP32_TOL, csr_to_dev, log, relerr, to_dev, to_host
from test_gpu_gat import G, _run, ctx  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gname,so,act", [
    ("er300", 4, 1), ("er300", 60, 0), ("er300", 64, 1), ("er300", 68, 1), ("er300", 1024, 1),
    ("er300", 1028, 0), ("hub1000", 61, 1), ("hub1000", 132, 1), ("hub1000", 1024, 0),
    ("hub1000", 1028, 1)])
def test_gat_widths_and_rows(G, ctx, gname, so, act):  # noqa: F811
    # a result is a chain of at most 4 sums of up to 1,729 fp32 terms, so its
    # rounding is near 4 sqrt(1,729) 2^-24 = 1e-5 of the terms' size; FP32_TOL
    # (1e-4) leaves a factor of ten for cancellation
    log(f"gat {gname} {so} act={act}")
    got, want = _run(G, ctx, gname, 24, so, act, "f32")
    for k in want:
        assert relerr(got[k], want[k]) <= FP32_TOL, k


def test_mirror_map_fully_written(G, ctx):  # noqa: F811
    """A pattern without mirrors: what the workspace held before (two fills,
    each a valid entry) does not reach the results."""
    import torch
    n, si, so = 70, 8, 12
    rows = [[i] if i % 3 else sorted({i, (i + 5) % n, (i + 9) % n}) for i in range(n)]
    rp = np.cumsum([0] + [len(r) for r in rows]).astype(np.int32)
    col = np.concatenate(rows).astype(np.int32)
    nnz = len(col)
    rng = np.random.default_rng(1)
    r = lambda *s: to_dev(rng.standard_normal(s).astype(np.float32))   # noqa: E731
    H, W, a1, a2, dHo = r(n, si), r(si, so), r(so), r(so), r(n, so)
    A, _keep = csr_to_dev({"n": n, "nnz": nnz, "rowptr": rp, "col": col, "val": np.ones(nnz)})
    desc = G.gat_desc(n, nnz, si, so, 1, G.GIST_DTYPE_F32, 0.2)
    out = []
    for fill in (0, 1):
        ws = torch.full((max(G.gist_gat_workspace_size(desc)) // 4 + 1,), fill, dtype=torch.int32,
                        device="cuda").view(torch.uint8)
        P, Ho, alpha = (torch.empty(n, so, device="cuda"), torch.empty(n, so, device="cuda"),
                        torch.empty(nnz, device="cuda"))
        g = [torch.empty(si, so, device="cuda"), torch.empty(so, device="cuda"),
             torch.empty(so, device="cuda"), torch.empty(n, si, device="cuda")]
        G.gist_gat_layer_fwd(ctx, desc, A, H, W, a1, a2, P, alpha, Ho, ws)
        ws.view(torch.int32).fill_(fill)
        G.gist_gat_layer_bwd(ctx, desc, A, H, P, alpha, Ho, W, a1, a2, dHo, *g, ws)
        out.append([to_host(t) for t in g])
    for x, y in zip(*out):
        assert np.array_equal(x, y) and np.isfinite(x).all()


def test_rows_beyond_one_grid(G, ctx):  # noqa: F811
    """2^25 + 1 rows: the mirror map no longer fits the scores' launch.  Self
    loops only, so alpha = 1, dP = dZ, dW = H^T dZ, dH = dZ W^T."""
    import torch
    n, s = 2 ** 25 + 1, 4
    log(f"gat n={n} s={s}")
    g = torch.Generator(device="cuda").manual_seed(3)
    r = lambda *d: torch.randn(d, generator=g, device="cuda")   # noqa: E731
    H, W, a1, a2, dHo = r(n, s), r(s, s), r(s), r(s), r(n, s)
    val = torch.ones(n, device="cuda")
    rp, col = (torch.arange(k, dtype=torch.int32, device="cuda") for k in (n + 1, n))
    A = G.csr_dev(n, n, rp, col, val)
    desc = G.gat_desc(n, n, s, s, 0, G.GIST_DTYPE_F32, 0.2)
    ws = torch.full((max(G.gist_gat_workspace_size(desc)),), 255, dtype=torch.uint8, device="cuda")
    P, Ho, alpha = torch.empty(n, s, device="cuda"), torch.empty(n, s, device="cuda"), torch.empty(n, device="cuda")
    dW, d1, d2, dH = torch.empty(s, s, device="cuda"), torch.empty(s, device="cuda"), torch.empty(
        s, device="cuda"), torch.empty(n, s, device="cuda")
    G.gist_gat_layer_fwd(ctx, desc, A, H, W, a1, a2, P, alpha, Ho, ws)
    G.gist_gat_layer_bwd(ctx, desc, A, H, P, alpha, Ho, W, a1, a2, dHo, dW, d1, d2, dH, ws)
    # dW sums n fp32 terms of size 1 to about sqrt(n): partial sums of up to 4,096
    # terms, then n / 4,096 = 8,192 of them, round by at most 8,192 2^-24 = 5e-4 and,
    # the errors being random, near sqrt(8,192) 2^-24 = 5e-6 of the sums' size
    assert relerr(to_host(dW), to_host(H.double().T @ dHo.double())) <= FP32_TOL
    assert relerr(to_host(dH), to_host((dHo.double() @ W.double().T).float())) <= FP32_TOL
