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
