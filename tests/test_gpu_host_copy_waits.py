"""A large read behind a long queue of the caller's own work: its helper
threads sleep until the data comes, so the process uses the CPU time of a
waiting thread or two, not of every helper."""
import time

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(500, 500), (1500, 1111)])   # 6 MB, 40 MB
def test_helpers_sleep_until_the_data_comes(nx, ny):
    import torch
    from paper_2211_05009_amd import lbm
    stream = torch.cuda.Stream()
    c = lbm.Cavity(nx, ny, 1000.0)
    c.set_stream(stream)
    c.step(20)
    c.moments()
    a = torch.ones((8192, 8192), device="cuda", dtype=torch.bfloat16)
    with torch.cuda.stream(stream):
        b = a @ a
        torch.cuda.synchronize()
        for _ in range(500):                 # about half a second
            torch.matmul(a, a, out=b)
    wall, cpu = time.perf_counter(), time.process_time()
    c.moments()
    wall, cpu = time.perf_counter() - wall, time.process_time() - cpu
    assert wall > 0.2
    # one thread may poll for the stream and the runtime may keep another one
    # busy; four to eight helpers would come on top
    assert cpu < 2.5 * wall
    c.close()
