"""Several steps per launch in tiles (schedule 4 van der Waals, schedule 6 binary)
at the sizes where the tiles change form: channels that fit a region between their
walls, by one row not, and in three tiles; lattices smaller than a region; columns
that end one past a tile; lattices large enough for the 64-column tiles.

Van der Waals: bitwise the one-wavefront row sweep (schedule 3), whose arithmetic it
shares.  Binary: bitwise the same steps launched one by one, and the population
storage to rounding (2e-6, as the other tests of the two storages)."""
import numpy as np
import pytest

from paper_0911_0459_amd import inputs as I

pytestmark = pytest.mark.gpu

GEOMS = {
    "walls_fit": (90, 40, 0, 90, 30, 4),        # one tile from wall to wall
    "walls_one_more": (90, 40, 0, 90, 31, 4),   # two
    "three_high": (140, 90, 30, 100, 76, 6),
    "thin_walls": (64, 24, 20, 40, 22, 1),      # one wall row, periodic images behind it
    "smaller_than_a_region": (11, 9, 0, 0, 0, 0),
    "narrow_channel": (3, 22, 0, 3, 20, 1),
    "one_past": (273, 33, 129, 100, 9, 11),
    "columns64": (2600, 560, 500, 1900, 440, 50),
}


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0911_0459_amd import lbcap
    return lbcap


def _run(L, model, g, cfg, calls, force):
    kw = dict(I.VDW_CONSTS, nu_l=0.13, wall_grad=-0.1) if model == "vdw" else dict(I.BIN_CONSTS, nu_l=0.4, nu_g=0.1,
                                                                                  wall_grad=-0.2)
    liquid, gas = (4.5, 2.6) if model == "vdw" else (1.0, -1.0)
    rng = np.random.default_rng(7)
    q = np.where(np.arange(g[0]) < 0.45 * g[0], liquid, gas) + 1e-3 * rng.uniform(-1, 1, (g[1], g[0]))
    lat = L.Lattice(L.make_params(model, force_x=force, **kw), L.make_geometry(*g), q)
    if cfg:
        lat.set_launch_config(**dict(lat.launch_config().asdict(), **cfg))
    for n in calls:
        lat.step(n)
    out = lat.moments()
    assert np.all(np.isfinite(out[0]))
    lat.close()
    return out


@pytest.mark.parametrize("fp64,force", [(0, 0.0), (1, 1e-5)])
@pytest.mark.parametrize("name", list(GEOMS))
def test_vdw_tiles_are_the_row_sweep(L, name, fp64, force):
    g = GEOMS[name]
    ref = _run(L, "vdw", g, dict(schedule=3, fp64_arith=fp64), [23], force)
    for calls in ([23], [1, 5, 17]):
        print(f"block vdw {name} {calls}", flush=True)
        for x, y in zip(ref, _run(L, "vdw", g, dict(fp64_arith=fp64), calls, force)):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("fp64,force", [(0, 0.0), (1, 1e-5)])
@pytest.mark.parametrize("name", list(GEOMS))
def test_binary_tiles_do_not_depend_on_the_grouping(L, name, fp64, force):
    g = GEOMS[name]
    ref = _run(L, "binary", g, dict(fp64_arith=fp64), [1] * 13, force)
    for calls in ([13], [2, 11]):
        print(f"block binary {name} {calls}", flush=True)
        for x, y in zip(ref, _run(L, "binary", g, dict(fp64_arith=fp64), calls, force)):
            assert np.array_equal(x, y)
    pop = _run(L, "binary", g, dict(schedule=4, fp64_arith=fp64), [13], force)
    assert max(float(np.abs(x - y).max()) for x, y in zip(ref, pop)) <= 2e-6


def test_fields_through_several_pinned_chunks(L):
    """Host fields pass through pinned memory half a buffer (32768 nodes) at a time: a
    lattice of three halves and a bit reads the same as on the device."""
    import torch
    g = (700, 153, 100, 400, 90, 30)
    rng = np.random.default_rng(3)
    q = np.where(np.arange(g[0]) < 300, 1.0, -1.0) + 1e-3 * rng.uniform(-1, 1, (g[1], g[0]))
    lat = L.Lattice(L.make_params("binary", nu_l=0.4, nu_g=0.1, wall_grad=-0.2, **I.BIN_CONSTS), L.make_geometry(*g), q)
    lat.step(30)
    dev = [torch.full((g[1], g[0]), float("nan"), device="cuda") for _ in range(4)]
    lat.moments_device(*dev)
    host = lat.moments()
    torch.cuda.synchronize()
    for x, y in zip(host, dev):
        assert np.array_equal(x, y.cpu().numpy().astype(np.float64))
    lat.step(1)
    again = lat.moments()
    assert all(np.all(np.isfinite(x)) for x in again) and not np.array_equal(again[1], host[1])
    lat.close()
