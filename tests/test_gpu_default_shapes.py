"""The shape a new handle starts with, on lattices at the edges of the rules
that choose it, against the one-step shape 0: the same populations, bit for
bit."""
import numpy as np
import pytest

from cavity_inputs import U_LID

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lbm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2211_05009_amd import lbm as m
    return m


@pytest.mark.parametrize("dtype,box,shape", [
    ("f64", (89, 89, 89), 4), ("f64", (88, 90, 88), 1),          # about 0.7 M sites
    ("f64", (64, 48, 64), 3), ("f64", (64, 48, 65), 1),          # 512 tiles and more
    ("f64", (2, 66, 4), 1), ("f32s", (2, 66, 4), 1),             # thinner than a tile
    ("f32s", (107, 107, 106), 4), ("f32s", (107, 106, 105), 3),  # about 1.2 M sites
    ("f32s", (13, 8, 4), 3), ("f32s", (12, 8, 4), 1),            # 40 % of a tile
])
def test_box(lbm, dtype, box, shape):
    nx, ny, nz = box
    rng = np.random.default_rng(nx)
    w = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)
    f = w[:, None, None, None] + rng.uniform(-4e-3, 4e-3, (19, nz, ny, nx))
    c = lbm.Cube(nx, ny, nz, re=2.0 * nx, u_lid=U_LID, dtype=dtype)
    assert c.get_option(lbm.LBM_OPT_STEP_VARIANT) == shape
    got = []
    for v in (shape, 0):
        c.set_option(lbm.LBM_OPT_STEP_VARIANT, v)
        c.set_populations(f)
        c.step(7)
        got.append(c.get_populations())
    assert np.array_equal(got[0], got[1])
    c.close()


@pytest.mark.parametrize("dtype,nx,ny,shape", [
    ("f32s", 2, 2, 29), ("f64", 200, 200, 29), ("f32s", 201, 200, 30),   # 640 tiles of 8 x 8
    ("f64", 384, 256, 30), ("f64", 385, 256, 31), ("f32s", 384, 272, 31),  # 256 of 24 x 16
    ("f64", 500, 256, 31), ("f64", 513, 256, 32),                        # 256 of 32 x 16
    ("f32s", 384, 448, 30), ("f32s", 385, 448, 24),                      # 448 of 24 x 16
    ("f32s", 512, 512, 24), ("f32s", 513, 512, 31),                      # 256 of 32 x 32
    ("f32s", 768, 513, 22),                                              # 768 of 32 x 16
    ("f32s", 1750, 1715, 18), ("f64", 1750, 1715, 26),                   # 3 M sites
])
def test_cavity(lbm, dtype, nx, ny, shape):
    rng = np.random.default_rng(nx)
    w = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)
    f = w[:, None, None] + rng.uniform(-4e-3, 4e-3, (9, ny, nx))
    c = lbm.Cavity(nx, ny, tau=0.56, u_lid=U_LID, dtype=dtype)
    assert c.get_option(lbm.LBM_OPT_STEP_VARIANT) == shape
    got = []
    for v in (shape, 0):
        c.set_option(lbm.LBM_OPT_STEP_VARIANT, v)
        c.set_populations(f)
        c.step(117)
        got.append((c.get_populations(), c.residual()[0]))
    assert np.array_equal(got[0][0], got[1][0])
    assert abs(got[0][1] - got[1][1]) <= 1e-12 * got[1][1]
    c.close()


@pytest.mark.parametrize("dtype", ["f64", "f32s"])
@pytest.mark.parametrize("nx,ny,tile", [
    (3, 3, (8, 8)), (160, 160, (8, 8)), (161, 160, (16, 16)),      # 400 tiles of 8 x 8
    (256, 256, (16, 16)), (257, 256, (24, 16)),                    # 256 of 16 x 16
    (385, 256, (32, 16)), (513, 256, (24, 16)),                    # 256 of 24 x 16, 32 x 16
    (385, 449, None), (513, 513, None), (768, 529, None),          # by storage type
])
def test_nee(lbm, dtype, nx, ny, tile):
    if tile is None:
        tile = (32, 16) if dtype == "f64" or nx == 513 else (32, 32)
    rng = np.random.default_rng(nx)
    w = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)
    f = w[:, None, None] + rng.uniform(-4e-3, 4e-3, (9, ny, nx))
    c = lbm.Cavity(nx, ny, re=2.0 * nx, u_lid=U_LID, dtype=dtype, wall="nee")
    assert c.get_option(lbm.LBM_OPT_STEP_VARIANT) == 6
    assert (c.get_option(lbm.LBM_OPT_TILE_X), c.get_option(lbm.LBM_OPT_TILE_Y)) == tile
    got = []
    for v in (6, 0):
        c.set_option(lbm.LBM_OPT_STEP_VARIANT, v)
        c.set_populations(f)
        c.step(117)
        got.append(c.get_populations())
    assert np.array_equal(got[0], got[1])
    c.close()
