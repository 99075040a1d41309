"""Single steps of large contexts (4 million fluid nodes binary, 1.5 million van der
Waals) go by the row sweep, several steps by the tiles: the fields do not depend on
which, bitwise."""
import numpy as np
import pytest

from paper_0911_0459_amd import inputs as I

pytestmark = pytest.mark.gpu

GEOMS = {"vdw": (2011, 1009, 517, 1203, 871, 55), "binary": (2903, 1711, 701, 1402, 1407, 133)}


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0911_0459_amd import lbcap
    return lbcap


@pytest.mark.parametrize("fp64,force", [(0, 0.0), (1, 1e-5), (0, 1e-5)])
@pytest.mark.parametrize("model", list(GEOMS))
def test_rows_and_tiles_step_alike(L, model, fp64, force):
    g = GEOMS[model]
    vdw = model == "vdw"
    kw = dict(I.VDW_CONSTS, nu_l=0.13, wall_grad=-0.1) if vdw else dict(I.BIN_CONSTS, nu_l=0.4, nu_g=0.1, wall_grad=-0.2)
    liquid, gas = (4.5, 2.6) if vdw else (1.0, -1.0)
    rng = np.random.default_rng(7)
    q = np.where(np.arange(g[0]) < 0.45 * g[0], liquid, gas) + 1e-3 * rng.uniform(-1, 1, (g[1], g[0]))
    out = []
    for calls in ([13], [1] * 13, [2, 1, 5, 3, 2]):
        print(f"single steps {model} fp64={fp64} force={force} {calls}", flush=True)
        lat = L.Lattice(L.make_params(model, force_x=force, **kw), L.make_geometry(*g), q)
        assert lat.fluid_nodes > (1500000 if vdw else 4000000)
        lat.set_launch_config(**dict(lat.launch_config().asdict(), fp64_arith=fp64))
        for n in calls:
            lat.step(n)
        out.append(lat.moments())
        lat.close()
    assert np.all(np.isfinite(out[0][0]))
    for other in out[1:]:
        for x, y in zip(out[0], other):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("chunk", [0, 4, 5, 12, 16])
@pytest.mark.parametrize("model", list(GEOMS))
def test_row_sweep_of_single_steps_does_not_depend_on_the_chunking(L, model, chunk):
    """The row sweep behind the single steps takes its chunks from the launch
    configuration; with van der Waals it also ends odd calls of schedule 5."""
    g = GEOMS[model]
    vdw = model == "vdw"
    kw = dict(I.VDW_CONSTS, nu_l=0.13, wall_grad=-0.1) if vdw else dict(I.BIN_CONSTS, nu_l=0.4, nu_g=0.1, wall_grad=-0.2)
    q = np.where(np.arange(g[0]) < 0.45 * g[0], *((4.5, 2.6) if vdw else (1.0, -1.0))) + np.zeros((g[1], 1))
    out = []
    for cfg, calls in ((dict(), [5]), (dict(chunk_rows=chunk), [1] * 5), (dict(schedule=5, chunk_rows=chunk), [1, 3, 1])):
        if cfg.get("schedule") == 5 and not vdw:
            continue
        print(f"chunks {model} {cfg} {calls}", flush=True)
        lat = L.Lattice(L.make_params(model, **kw), L.make_geometry(*g), q)
        lat.set_launch_config(**dict(lat.launch_config().asdict(), **cfg))
        for n in calls:
            lat.step(n)
        out.append(lat.moments())
        lat.close()
    for other in out[1:]:
        for x, y in zip(out[0], other):
            assert np.array_equal(x, y)
