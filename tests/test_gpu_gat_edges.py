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
