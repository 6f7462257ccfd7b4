"""The series classifier's lag tiles and sample chunks against the oracle
(oracle/flowstate.py): windows and lag counts around the tiles of 64 and 768
lags and the chunks of 512 and 1024 samples, in both forms of the kernel."""
import math

import numpy as np
import pytest

from oracle import flowstate as F

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,lags,copies", [
    (9, (1, 0), 1),              # the fewest lags: three
    (8, (1, 6), 1),              # the lag range capped at n - 2
    (194, (1, 0), 1),            # 64 lags: one narrow tile
    (197, (1, 0), 1),            # 65 lags
    (577, (64, 200), 2),         # a chunk and a tile, off the grid
    (2304, (1, 768), 260),       # one wide tile, full
    (2307, (1, 769), 260),       # one lag more
    (1100, (1, 1098), 190),      # lags up to the window's end
    (3072, (1000, 1010), 1),     # three chunks of 1024, few lags
])
def test_tiles_and_chunks(n, lags, copies):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2211_05009_amd import lbm
    k = np.arange(n, dtype=np.float64)
    rng = np.random.default_rng(n)
    base = [0.02 * np.sin(2 * np.pi * k / max(5.5, n / 37.3)) + 0.01,
            rng.normal(size=n),
            1e-3 * k,
            np.full(n, 0.25),
            np.sin(2 * np.pi * k / 20) + np.sin(2 * np.pi * k * 1.618 / 20)]
    dev = torch.tensor(np.stack(base * copies), dtype=torch.float64, device="cuda")
    got = lbm.lbm_classify_series(dev, 1e-7, 0.02, *lags)
    for c in (0, copies - 1):
        for g, u in zip(got[5 * c:5 * c + 5], base):
            w = F.classify(u, 1e-7, 0.02, min_lag=lags[0], max_lag=lags[1] or None)
            assert (g["state"], g["lag"]) == (w["state"], w["lag"])
            # sums of n terms in another order: n ulps of relative error at most,
            # and the square root of a difference of D values of order 1
            for key in ("amplitude", "mean", "std", "period", "cycle"):
                assert math.isclose(g[key], w[key], rel_tol=1e-9, abs_tol=1e-14), key
            for key in ("mismatch", "cycle_mismatch"):
                assert g[key] == w[key] or abs(g[key] - w[key]) <= 1e-7, key
