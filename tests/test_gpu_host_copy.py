"""GPU tests of the staged device-to-host copies (csrc/host_copy.hip): results
from 4 MB on go through pinned buffers and several threads, in 512 KB chunks,
from 16 MB on in 4 MB ones.

The same bytes have to arrive as by the device entry point or by a read of
every site, whatever the size of the last chunk, for fresh, unaligned,
written-to and pinned destinations, and with some outputs left out.
"""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _device_moments(torch, c, ny, nx):
    d = [torch.empty((ny, nx), dtype=torch.float64, device="cuda") for _ in range(3)]
    c.moments_device(*d)
    return [x.cpu().numpy() for x in d]


# 3 fields of 8 nx ny bytes: just below and above 4 MB and 16 MB, ragged chunks
@pytest.mark.parametrize("nx,ny", [(419, 417), (419, 418), (500, 500), (700, 998),
                                   (700, 1000), (1023, 1025), (1500, 1111)])
def test_moments_match_the_device_entry_point(nx, ny):
    import torch
    from paper_2211_05009_amd import lbm
    c = lbm.Cavity(nx, ny, 1000.0)
    c.step(20)
    ref = _device_moments(torch, c, ny, nx)
    for _ in range(2):
        for a, b in zip(c.moments(), ref):
            assert np.array_equal(a, b)
    c.close()


@pytest.mark.parametrize("kind", ["unaligned", "pinned", "left out"])
def test_destinations(kind):
    import ctypes

    import torch
    from paper_2211_05009_amd import lbm
    nx, ny = 1300, 1100
    n = nx * ny
    c = lbm.Cavity(nx, ny, 1000.0)
    c.step(20)
    ref = _device_moments(torch, c, ny, nx)
    raw = torch.zeros(3 * n + 1, dtype=torch.float64, pin_memory=kind == "pinned").numpy()
    outs = [raw[1 + k * n:1 + (k + 1) * n] for k in range(3)]
    ptr = [ctypes.c_void_p(o.ctypes.data) for o in outs]
    if kind == "left out":
        ptr[1] = None
    assert lbm._lib.lbm_moments(c.h, *ptr) == 0
    for k in range(3):
        want = np.zeros(n) if ptr[k] is None else ref[k].ravel()
        assert np.array_equal(outs[k], want)
    assert raw[0] == 0.0
    c.close()


def test_box_and_populations_and_two_threads():
    from paper_2211_05009_amd import lbm
    cubes = [lbm.Cube(96, 96, 96, 1000.0), lbm.Cube(96, 96, 96, 400.0)]
    for c in cubes:
        c.step(20)
    got = [None, None]

    def read(k):
        got[k] = (cubes[k].moments(), cubes[k].get_populations())

    threads = [threading.Thread(target=read, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k in range(2):   # 28 MB of fields, 134 MB of populations
        (rho, ux, uy, uz), f = got[k]
        f = f.reshape((19,) + rho.shape)
        assert np.allclose(f.sum(axis=0), rho, rtol=0, atol=1e-13)
        again = cubes[k].get_populations().reshape(f.shape)
        assert np.array_equal(f, again)
        cubes[k].close()
