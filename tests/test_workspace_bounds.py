"""The layers' workspace beyond the tensors they need (dZ, dP): partial sums of the dense products,
at most 256 MiB whatever the sizes.  No GPU needed: the plan is host arithmetic."""

import pytest

from paper_2102_10424_amd import gist as G

PART = 256 << 20


def _align(x):
    return (x + 255) // 256 * 256


@pytest.mark.parametrize("dtype", [G.GIST_DTYPE_F32, G.GIST_DTYPE_BF16_IN])
@pytest.mark.parametrize("kind,n,si,so,groups", [
    (G.GIST_LAYER_SAGE_MEAN, 232965, 4096, 4096, 1),
    (G.GIST_LAYER_SAGE_MEAN, 2450000, 4096, 4096, 1),
    (G.GIST_LAYER_GCN, 2450000, 512, 512, 1),
    (G.GIST_LAYER_GCN, 2450000, 2048, 2100, 4),
    (G.GIST_LAYER_GCN, 2450000, 256, 256, 1),
    (G.GIST_LAYER_GCN, 1630, 8192, 8200, 1),
    (G.GIST_LAYER_GCN, 64, 1 << 23, 1 << 23, 1)])
def test_partial_sums_are_bounded(kind, n, si, so, groups, dtype):
    d = G.layer_desc(kind, G.GIST_ACT_NONE, n, si, so, dtype, order=G.GIST_ORDER_AGG_FIRST, groups=groups)
    fwd, bwd = G.gist_layer_workspace_size(d)
    tmp = 4 * n * si * groups
    assert fwd <= PART, fwd
    assert bwd <= _align(tmp) + PART, bwd - tmp
