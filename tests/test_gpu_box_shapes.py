"""The shape a new box starts with, on boxes where the two-step shapes' tiles
are badly filled or their last round of blocks nearly empty: the one-step
shape, which measured faster there; and on the other side of each line.  The
populations equal those of shape 0 bit for bit."""
import numpy as np
import pytest

from cavity_inputs import U_LID

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,box,shape", [
    # FP32 below 1.2 M sites, more than one round of 256 tiles of 32 x 8 x 4
    ("f32s", (361, 281, 5), 1), ("f32s", (160, 771, 9), 1),     # 1.30, 1.34 times
    ("f32s", (510, 120, 9), 1), ("f32s", (200, 200, 10), 1),    # 1.20, 1.08
    ("f32s", (228, 12, 242), 1), ("f32s", (300, 50, 50), 1),    # 1.15, 1.02
    ("f32s", (180, 33, 33), 1), ("f32s", (66, 66, 66), 3),
    ("f32s", (256, 64, 16), 3), ("f32s", (100, 100, 100), 3),
    # FP32 just above it
    ("f32s", (350, 9, 391), 1), ("f32s", (374, 242, 14), 1),    # 1.20, 1.13
    ("f32s", (700, 700, 3), 1), ("f32s", (374, 242, 16), 4),
    ("f32s", (199, 17, 385), 1), ("f32s", (31, 92, 789), 4),    # 1.17
    # FP64 two rounds of 16 x 6 x 4 tiles; just above 0.7 M sites
    ("f64", (391, 13, 16), 1), ("f64", (479, 13, 18), 1),       # 1.19, 1.11
    ("f64", (256, 57, 11), 1), ("f64", (48, 48, 48), 3),        # 1.07
    ("f64", (757, 13, 101), 1), ("f64", (341, 6, 461), 4),      # 1.04
])
def test_thin_boxes(dtype, box, shape):
    from paper_2211_05009_amd import lbm
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
        c.step(3)
        got.append(c.get_populations())
    assert np.array_equal(got[0], got[1])
    c.close()
