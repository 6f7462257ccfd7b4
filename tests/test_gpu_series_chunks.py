"""The wide form of the series classifier's lag kernel at the ends of its
sample chunks (960 samples, summed in groups of 24) and in its later tiles (768
lags each), against the oracle (oracle/flowstate.py): the samples of the
shortest lag are one chunk, two, or a group, give or take one, and the first
return of some series lies in the second or third tile, so that its lag,
period and mismatch come from there."""
import math

import numpy as np
import pytest

from oracle import flowstate as F

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,lags,copies", [
    (961, (1, 958), 36), (960, (1, 957), 36), (962, (1, 959), 36),     # 960 samples, 959, 961
    (1060, (100, 940), 40),                                            # 960 again
    (1200, (1, 1100), 30), (1201, (1, 1100), 30), (1202, (1, 1100), 30),   # 1199, 1200, 1201
    (1920, (1, 1700), 20), (1921, (1, 1700), 20), (1922, (1, 1700), 20),   # 1919, 1920, 1921
])
def test_chunk_ends_and_later_tiles(n, lags, copies):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2211_05009_amd import lbm
    k = np.arange(n, dtype=np.float64)
    rng = np.random.default_rng(n)
    late = 0.85 * lags[1] if lags[1] < 1600 else 1583.25     # past 768, past 1536
    assert late > 768 and (lags[1] < 1600 or late > 1536)
    base = [0.02 * np.sin(2 * np.pi * k / late) + 0.01,
            np.cos(2 * np.pi * k / 781.5) + 0.2 * np.cos(4 * np.pi * k / 781.5),
            np.sin(2 * np.pi * k / 790) + 0.05 * rng.normal(size=n),
            rng.normal(size=n),
            1e-3 * k,
            np.sin(2 * np.pi * k / 37.3)]
    # the wide form is taken from 3073 narrow wavefronts (64 lags of a series) on
    assert 6 * copies * math.ceil((lags[1] - lags[0] + 1) / 64) > 3072
    dev = torch.tensor(np.stack(base * copies), dtype=torch.float64, device="cuda")
    got = lbm.lbm_classify_series(dev, 1e-7, 0.02, *lags)
    want = [F.classify(u, 1e-7, 0.02, min_lag=lags[0], max_lag=lags[1]) for u in base]
    assert want[0]["lag"] > 768 and want[1]["lag"] > 768
    for c in (0, copies - 1):
        for g, w in zip(got[6 * c:6 * c + 6], want):
            assert (g["state"], g["lag"]) == (w["state"], w["lag"])
            # sums of n terms in another order: n ulps of relative error at most,
            # and the square root of a difference of D values of order 1
            for key in ("amplitude", "mean", "std", "period", "cycle"):
                assert math.isclose(g[key], w[key], rel_tol=1e-9, abs_tol=1e-14), key
            for key in ("mismatch", "cycle_mismatch"):
                assert g[key] == w[key] or abs(g[key] - w[key]) <= 1e-7, key
