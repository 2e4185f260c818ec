"""GPU parity of the fp32 products over many nodes.

The layer entry points give each dense product of eq. (2) and its backward
pass a tile (256, 128 or 64 wide) and a schedule by shape: whole tiles where
there are many, tiles cut in K where there are few and K is long (a weight
gradient reduced over the nodes), the parts summed by a second kernel.
The cases below have 4,000 to 20,011 nodes, one, 47, 64, 65 or 1,024 output
columns, and whole and ragged K, and compare the forward and backward outputs
with the fp64 oracle within 1e-4, the ReLU decisions of the backward taken
from the oracle's forward values (as in ``test_gpu_layers``).
"""

import pytest

from gist_synth.graphs import erdos_renyi

from gpu_util import FP32_TOL, log, relerr
from test_gpu_layers import run_layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    from paper_2102_10424_amd import gist
    return gist


@pytest.fixture(scope="module")
def ctx(G):
    return G.Context(0)


GRAPHS = {}


def graph(n):
    """A sparse graph on n nodes (about five neighbours each), built once."""
    if n not in GRAPHS:
        GRAPHS[n] = erdos_renyi(n, 5 * n // 2, seed=n, clusters=4)
    return GRAPHS[n]


CASES = [
    # graph nodes, s_in, s_out, order (0 auto, 1 aggregate first, 2 transform first), what it reaches
    (20011, 512, 64, 1, "forward 313 whole 64 x 64 tiles; dW 8 tiles in 79 parts over ragged K = 20011"),
    (20011, 300, 1, 1, "N = 1: one column of a 64 x 64 tile; dW 5 tiles in 105 parts"),
    (20011, 300, 65, 1, "N = 65: a second tile with one column; dW 10 tiles in 63 parts"),
    (4000, 200, 47, 2, "transform first: XW (47 columns), Abar^T dZ then dW cut over 4000"),
    (20000, 1024, 1024, 1, "128 x 128 tiles: forward and dH whole, dW 64 tiles cut in K"),
    (20011, 1040, 1024, 1, "the same with ragged tile rows and K: dW 72 tiles over 20011"),
]


@pytest.mark.parametrize("case", CASES, ids=[f"n{c[0]}-{c[1]}x{c[2]}-o{c[3]}" for c in CASES])
def test_gemm_schedule_boundaries(G, ctx, case):
    n, s_in, s_out, order, what = case
    log(f"gemm schedules n={n} {s_in}x{s_out} order={order}: {what}")
    got, want = run_layer(G, ctx, "gcn", graph(n), s_in, s_out, G.GIST_ACT_RELU, order,
                          G.GIST_DTYPE_F32)
    for k in want:
        if k == "agg" and order == 2:
            continue  # transform-first does not form Abar H
        e = relerr(got[k], want[k])
        log(f"  {k}: {e:.3e}")
        assert e <= FP32_TOL, (k, e)
