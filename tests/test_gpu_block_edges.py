"""The block kernels at the edges of their tiles, in every shape and with every number of
steps per launch that the planner picks (block_geoms.py).  Van der Waals: bitwise the
one-wavefront row sweep.  Binary: bitwise the same steps launched one by one, and the
population storage to rounding (2e-6, as the other tests of the two storages)."""
import numpy as np
import pytest

from block_geoms import EDGES
from test_gpu_block_steps import _run

pytestmark = pytest.mark.gpu

CASES = [(m, *e[1:]) for e in EDGES for m in e[0]]


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0911_0459_amd import lbcap
    return lbcap


@pytest.mark.parametrize("m,shape,K,column,g", CASES, ids=[f"{m}-shape{s}-K{K}-{c}-{g[0]}x{g[1]}" for m, s, K, c, g in CASES])
def test_tiles_at_their_edges(L, m, shape, K, column, g):
    model = {"b": "binary", "v": "vdw"}[m]
    n = 3 * K + 2   # whole launches, a remainder and (binary) a last step
    print(f"block edges {model} {g} K={K}", flush=True)
    tiles = _run(L, model, g, None, [n], 0.0)
    if m == "v":
        ref = _run(L, model, g, dict(schedule=3), [n], 0.0)
    else:
        ref = _run(L, model, g, None, [1] * n, 0.0)
        pop = _run(L, model, g, dict(schedule=4), [n], 0.0)
        assert max(float(np.abs(x - y).max()) for x, y in zip(tiles, pop)) <= 2e-6
    for x, y in zip(tiles, ref):
        assert np.array_equal(x, y)
