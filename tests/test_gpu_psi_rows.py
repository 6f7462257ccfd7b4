"""Stream function and vortex calls on lattices of about 64 rows, up to which a
thread of k_psi takes one row and from which it takes eight, against the
oracle, for both wall schemes and storage types."""
import numpy as np
import pytest

from cavity_inputs import U_LID, random_fields
from oracle import monitors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32s"])
@pytest.mark.parametrize("wall", ["bounce-back", "nee"])
@pytest.mark.parametrize("nx,ny", [(8, 63), (40, 64), (9, 65), (130, 33)])
def test_psi_and_vortices(dtype, wall, nx, ny):
    from paper_2211_05009_amd import lbm
    c = lbm.Cavity(nx, ny, re=10.0, u_lid=U_LID, dtype=dtype, wall=wall)
    drho, ux, uy = random_fields(nx, ny, seed=nx + ny)
    c.init_fields(1.0 + drho, ux, uy)
    _, u, _ = c.moments()
    psi = c.stream_function()
    want = monitors.stream_function_nodes(u) if wall == "nee" else monitors.stream_function(u)
    # ny terms of at most 0.05, each sum's rounding at most ny ulps of it
    assert np.max(np.abs(psi - want)) <= ny * 2.0 ** -52 * 0.05 * ny
    flat = np.argmax(psi)
    ext = c.vortex_extrema()
    assert (ext[0].iy, ext[0].ix, ext[0].psi) == (flat // nx, flat % nx, psi.max())
    got, n = c.vortex_centres(0.0)
    sites = monitors.vortex_centres(psi, 0.0)
    assert n == len(sites) and [(v.psi, v.ix, v.iy) for v in got] == [
        (psi[v.iy, v.ix], v.ix, v.iy) for v in got]
    inner = psi[1:-1, 1:-1]
    around = [psi[1 + dy:ny - 1 + dy, 1 + dx:nx - 1 + dx]
              for dy in (-1, 0, 1) for dx in (-1, 0, 1) if dy or dx]
    top = np.all([inner > a for a in around], axis=0)
    low = np.all([inner < a for a in around], axis=0)
    assert n == int(top.sum() + low.sum())
    c.close()
